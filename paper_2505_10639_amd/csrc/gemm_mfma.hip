// Dense modal contractions of one plan on the matrix cores: the kernels and
// their launchers (bodies and operand layout in contract_mfma.h).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "contract_mfma.h"
#include "internal.h"
#include "schedule.h"

namespace mfbd {
namespace {

using contract::floatx4;

template <int MT, int RT, int W, int CS, int DEPTH>
__global__ __launch_bounds__(64 * W) void k_grad_mfma(int R, int J, int C, int zc, int M, int bp,
                                                      const uint4* __restrict__ Zs,
                                                      const float* __restrict__ gphi,
                                                      float* __restrict__ grad,
                                                      float* __restrict__ part) {
  contract::grad_block<MT, RT, W, CS, DEPTH>(blockIdx.x, blockIdx.y, gridDim.y, MT, R, J, C, zc, M, bp,
                                      Zs, gphi, grad, part);
}

template <int CS>
__global__ __launch_bounds__(1024) void k_grad_rows(int mt, int R, int J, int C, int zc, int M,
                                                    int bp, const uint4* __restrict__ Zs,
                                                    const float* __restrict__ gphi,
                                                    float* __restrict__ grad,
                                                    float* __restrict__ part) {
  contract::grad_rows_block<1, CS>(blockIdx.x, blockIdx.y, gridDim.y, mt, R, J, C, zc, M, bp, Zs,
                                    gphi, grad, part);
}

// grid (basis x groups of four pixel tiles, column groups)
template <int CT>
__global__ __launch_bounds__(256) void k_phase_few(int R, int J, int C, int zc, int M, int Mq,
                                                   int bp, const uint4* __restrict__ ZsT,
                                                   const float* __restrict__ theta,
                                                   const float* __restrict__ alpha,
                                                   float* __restrict__ phi) {
  const int groups = bp / 64, c = blockIdx.x / groups;
  contract::phase_few_wave<CT>(c, blockIdx.x % groups * 4 + (threadIdx.x >> 6), blockIdx.y, R, J,
                               C, zc, M, Mq, bp, ZsT, theta, alpha, phi);
}

template <int CT, int W>
__global__ __launch_bounds__(64 * W) void k_phase_mfma(int tpb, int R, int J, int C, int zc,
                                                    int M, int Mq, int bp,
                                                    const uint4* __restrict__ ZsT,
                                                    const float* __restrict__ theta,
                                                    const float* __restrict__ alpha,
                                                    float* __restrict__ phi) {
  contract::phase_block<CT, W>(blockIdx.x, blockIdx.y, tpb, R, J, C, zc, M, Mq, bp, ZsT, theta,
                               alpha, phi);
}

// Dynamic LDS beyond the default 64 KB needs the kernel's attribute.
hipError_t allow_lds(const void* kernel, size_t bytes) {
  if (bytes <= 65536) return hipSuccess;
  return hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

// grad = 2 pi (part[0] + part[1] + ... + part[splits-1]), in that order;
// the blocks past the gradient's (`cblocks`) sum the per-patch loss when the
// call asks for it (ls.P > 0), saving that sum a launch of its own.
__global__ __launch_bounds__(256) void k_grad_combine(long n, int splits, int cblocks,
                                                      const float* __restrict__ part,
                                                      float* __restrict__ grad, LossSum ls) {
  if ((int)blockIdx.x >= cblocks) {
    const int p = ((int)blockIdx.x - cblocks) * 256 + threadIdx.x;
    if (p < ls.P) loss_sum_patch(p, ls.nper, ls.active, ls.loss_part, ls.loss);
    return;
  }
  const long i = (long)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  float v = part[i];
  for (int s = 1; s < splits; ++s) v += part[(size_t)s * n + i];
  grad[i] = 6.283185307179586f * v;
}

template <int MT, int RT, int W, int CS, int DEPTH = 1>
hipError_t launch_grad_k(const Dims& d, int zc, int splits, const uint4* Zs, const float* gphi,
                         float* grad, float* part, hipStream_t s) {
  const int R = d.P * d.J, rows = 16 * RT * W;
  const size_t lds = contract::grad_lds_bytes(MT);
  const hipError_t e =
      allow_lds(reinterpret_cast<const void*>(&k_grad_mfma<MT, RT, W, CS, DEPTH>), lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((k_grad_mfma<MT, RT, W, CS, DEPTH>), dim3((R + rows - 1) / rows, splits),
                     dim3(64 * W), lds, s, R, d.J, d.C, zc, d.M, d.bandpix(), Zs, gphi, grad,
                     part);
  return hipGetLastError();
}

// Whether the accumulators of MT mode tiles leave registers for two chunks in
// flight.  Beyond, the two-chunk instances spill up to 100 registers (at 16
// tiles of separate bases none, and still lose): 3072 rows of 64 x 64, one
// basis: 29 us against 35 at 224 modes, 30 against 42 at 240, 34 against 35 at
// 256; three channels 35 against 39, 36 against 44, 38 against 51; two bases 39
// against 47 at 240, 40 against 42 at 256, but at 224 39 against 38.
template <int MT, int CS>
constexpr bool kTwoChunksFit = MT <= (CS == 1 ? 14 : 13);

template <int MT, int CS>
hipError_t launch_grad_cs(const Dims& d, int zc, int splits, const uint4* Zs, const float* gphi,
                          float* grad, float* part, hipStream_t s) {
  if (d.grad_waves == 8) return launch_grad_k<MT, 2, 8, CS>(d, zc, splits, Zs, gphi, grad, part, s);
  switch (grad_row_tiles_of(d)) {
    case 3: return launch_grad_k<MT, 3, 4, CS>(d, zc, splits, Zs, gphi, grad, part, s);
    default: {
      // at most one block per CU: 133 us with two chunks of loads in flight
      // against 160 with one at 3072 rows x 150 modes of four 128 x 128 bases;
      // with more blocks the registers cost occupancy (11 532 rows x 66 modes
      // at 64 x 64: 34.5 against 32.4)
      if constexpr (kTwoChunksFit<MT, CS>) {
        const long blocks = ((long)d.P * d.J + 127) / 128 * splits;
        if (blocks <= kCus)
          return launch_grad_k<MT, 2, 4, CS, 2>(d, zc, splits, Zs, gphi, grad, part, s);
      }
      return launch_grad_k<MT, 2, 4, CS>(d, zc, splits, Zs, gphi, grad, part, s);
    }
  }
}

template <int MT>
hipError_t launch_grad_t(const Dims& d, int splits, const uint4* Zs, const float* gphi,
                         float* grad, float* part, hipStream_t s) {
  const int zc = d.zc > 0 ? d.zc : d.C;
  if (zc == d.C) return launch_grad_cs<MT, 1>(d, zc, splits, Zs, gphi, grad, part, s);
  if (d.C == 2) return launch_grad_cs<MT, 2>(d, zc, splits, Zs, gphi, grad, part, s);
  return launch_grad_cs<MT, 0>(d, zc, splits, Zs, gphi, grad, part, s);
}

}  // namespace

hipError_t launch_grad(const Dims& d, const uint4* Zs, const float* gphi, float* grad,
                       float* part, hipStream_t s, const LossSum* ls) {
  const int mt = (d.M + 15) / 16;
  const int splits = grad_splits_of(d);
  hipError_t e;
  if (grad_few_rows(d)) {
    const int R = d.P * d.J, zc = d.zc > 0 ? d.zc : d.C;
    auto* kernel = zc == d.C ? &k_grad_rows<1> : &k_grad_rows<0>;
    hipLaunchKernelGGL(kernel, dim3((R + 15) / 16, splits), dim3(64 * mt), 0, s, mt, R, d.J, d.C,
                       zc, d.M, d.bandpix(), Zs, gphi, grad, part);
    e = hipGetLastError();
  } else switch (mt) {
#define MFBD_CASE(n) \
  case n: e = launch_grad_t<n>(d, splits, Zs, gphi, grad, part, s); break;
    MFBD_CASE(1) MFBD_CASE(2) MFBD_CASE(3) MFBD_CASE(4) MFBD_CASE(5) MFBD_CASE(6)
    MFBD_CASE(7) MFBD_CASE(8) MFBD_CASE(9) MFBD_CASE(10) MFBD_CASE(11) MFBD_CASE(12)
    MFBD_CASE(13) MFBD_CASE(14) MFBD_CASE(15) MFBD_CASE(16)
#undef MFBD_CASE
    default: return hipErrorInvalidValue;
  }
  if (e != hipSuccess) return e;
  if (splits > 1) {
    const long n = (long)d.P * d.J * d.M;
    const int cblocks = (int)((n + 255) / 256);
    const LossSum none{0, 0, nullptr, nullptr, nullptr};
    const LossSum& l = ls ? *ls : none;
    hipLaunchKernelGGL(k_grad_combine, dim3((unsigned)(cblocks + (l.P + 255) / 256)), dim3(256),
                       0, s, n, splits, cblocks, part, grad, l);
    return hipGetLastError();
  }
  if (ls) return launch_loss_sum(*ls, s);
  return hipGetLastError();
}

// A block takes a quarter of the band's pixel tiles, fewer where that leaves
// CUs idle (at least one per wave): 16.4 against 28 us at 441 columns x 77 modes
// (128 x 128, three bases); going on to 512 blocks and more cost up to a
// quarter at the larger sizes, where every block stages its coefficients anew.
template <int CT, int W>
hipError_t launch_phase_ct(const Dims& d, const float* alpha, const uint4* ZsT, int Mq,
                           const float* thetat, float* phi, hipStream_t s) {
  const int R = d.P * d.J, zc = d.zc > 0 ? d.zc : d.C;
  const int cols = (R + 16 * CT - 1) / (16 * CT), tiles = d.bandpix() / 16;
  int tpb = tiles / 4;
  while (tpb > W && (long)zc * cols * ((tiles + tpb - 1) / tpb) < kCus) tpb = std::max(tpb / 2, W);
  const dim3 grid(zc * ((tiles + tpb - 1) / tpb), cols);
  const size_t lds = contract::phase_lds_bytes(CT, Mq);
  const hipError_t e = allow_lds(reinterpret_cast<const void*>(&k_phase_mfma<CT, W>), lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((k_phase_mfma<CT, W>), grid, dim3(64 * W), lds, s, tpb, R, d.J, d.C, zc, d.M,
                     Mq, d.bandpix(), ZsT, thetat, alpha, phi);
  return hipGetLastError();
}

hipError_t launch_phase(const Dims& d, const float* alpha, const uint4* ZsT, int Mq,
                        const float* thetat, float* phi, hipStream_t s) {
  const int R = d.P * d.J;
  const PhaseShape shape = phase_shape_of(d, Mq);
  if (shape.few) {
    const int zc = d.zc > 0 ? d.zc : d.C;
    hipLaunchKernelGGL(k_phase_few<1>, dim3(zc * (d.bandpix() / 64), (R + 15) / 16), dim3(256), 0,
                       s, R, d.J, d.C, zc, d.M, Mq, d.bandpix(), ZsT, thetat, alpha, phi);
    return hipGetLastError();
  }
  if (shape.ct == 8) return launch_phase_ct<8, 16>(d, alpha, ZsT, Mq, thetat, phi, s);
  if (shape.ct == 2) return launch_phase_ct<2, 8>(d, alpha, ZsT, Mq, thetat, phi, s);
  return launch_phase_ct<4, 8>(d, alpha, ZsT, Mq, thetat, phi, s);
}

}  // namespace mfbd
