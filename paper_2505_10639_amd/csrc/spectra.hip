// Power spectrum of a restored (mosaicked) image and its average over
// 30-degree sectors along the +-45 degree directions, as a function of the
// radial frequency (Sect. "Results": averaging over all angles would pick up
// the power that the periodic continuation of the field puts on the axes).
//
//   P(u) = |DFT(w (x - mean))|^2 on the L x L grid, L a power of two;
//   bin k = round(|u|), u in (-L/2, L/2]; sector: 30..60 degrees from the
//   axes in every quadrant.  Both decisions are integer tests:
//   (2k-1)^2 <= 4|u|^2 < (2k+1)^2 and u_x^2 <= 3 u_y^2, u_y^2 <= 3 u_x^2.
//
// The 2-D transform is two passes of radix-2 Stockham FFTs of whole rows
// (natural order, twiddles from sincospi), each pass writing its output
// transposed.  Every sum runs in a fixed order.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "internal.h"
#include "momfbd.h"

namespace mfbd {
namespace {

// The image mean in two passes: kMeanBlocks contiguous chunks, each summed
// by one block (strided per thread, then a tree), and the chunk sums by one
// block; every sum in a fixed order.
constexpr int kMeanBlocks = 256;
__device__ __forceinline__ double block_sum256(double v, double* red) {
  const int t = threadIdx.x;
  red[t] = v;
  __syncthreads();
  for (int h = 128; h > 0; h >>= 1) {
    if (t < h) red[t] += red[t + h];
    __syncthreads();
  }
  return red[0];
}

__global__ __launch_bounds__(256) void k_mean_part(long n, const float* __restrict__ x,
                                                   double* __restrict__ part) {
  __shared__ double red[256];
  const long chunk = (n + kMeanBlocks - 1) / kMeanBlocks;
  const long lo = (long)blockIdx.x * chunk, hi = lo + chunk < n ? lo + chunk : n;
  double s = 0.0;
  long i = lo + threadIdx.x;
  for (; i + 7 * 256 < hi; i += 8 * 256) {   // eight loads in flight, added in order
    float v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = x[i + e * 256];
#pragma unroll
    for (int e = 0; e < 8; ++e) s += (double)v[e];
  }
  for (; i < hi; i += 256) s += (double)x[i];
  const double tot = block_sum256(s, red);
  if (threadIdx.x == 0) part[blockIdx.x] = tot;
}

// The mean from the chunk sums, by every wave for itself: the tree of
// block_sum256 over them, its first two levels on a lane's own four.
__device__ __forceinline__ float mean_of(long n, const double* __restrict__ part) {
  static_assert(kMeanBlocks == 256, "four chunks per lane");
  const int lane = threadIdx.x & 63;
  double v = (part[lane] + part[lane + 128]) + (part[lane + 64] + part[lane + 192]);
  for (int h = 32; h > 0; h >>= 1) v += __shfl_xor(v, h);
  return (float)(v / (double)n);
}

// A block transforms fft_rows(L) rows, eight points per thread: thread j of a
// row's L / 8 holds the points j + q L / 8.
__host__ __device__ constexpr int fft_rows(int L) { return L >= 4096 ? 2 : L >= 1024 ? 4 : 8; }
// One free slot after every eight points: the merged stages write eight points
// apart.
__host__ __device__ constexpr int fft_slot(int i) { return i + (i >> 3); }
// Row pitch in LDS: the rows of a column lie in different banks.
__host__ __device__ constexpr int fft_pitch(int L) { return fft_slot(L) + 32 / fft_rows(L); }

__device__ __forceinline__ void butterfly(float2& v0, float2& u, float2 w) {
  const float x = fmaf(u.x, w.x, -(u.y * w.y)), y = fmaf(u.y, w.x, u.x * w.y);
  u = make_float2(v0.x - x, v0.y - y);
  v0 = make_float2(v0.x + x, v0.y + y);
}

// S radix-2 stages from length 2^n on, merged in registers: the stages' pairs
// are a thread's own points (q apart 4, 2, 1), and point `q` of `v` ends at
// bits of q in the order the stages put them.  tw[t] = exp(-2 pi i t / L).
template <int S>
__device__ __forceinline__ void fft_stages(float2 (&v)[8], int j, int lg, int n,
                                           const float2* tw, float2* row) {
  constexpr int R = 1 << S, ITEMS = 8 / R;
#pragma unroll
  for (int it = 0; it < ITEMS; ++it) {
    const int jj = j + it * (1 << (lg - 3));
    const int r = jj & ((1 << n) - 1);
    // point m of the item is v[it + m ITEMS]; after stage s its leading bits
    // index the sums (0) and differences (1) taken so far
#pragma unroll
    for (int s = 0; s < S; ++s) {
      const int gap = R >> (s + 1);
#pragma unroll
      for (int m = 0; m < R; ++m) {
        if (m & gap) continue;
        int c = 0;   // sum/difference bits of the earlier stages, first stage lowest
#pragma unroll
        for (int e = 0; e < s; ++e) c |= ((m >> (S - 1 - e)) & 1) << e;
        const int rs = r + (c << n);   // the stage's residue, below 2^(n+s)
        butterfly(v[it + m * ITEMS], v[it + (m + gap) * ITEMS],
                  tw[fft_slot(rs << (lg - 1 - n - s))]);
      }
    }
    const int d = ((jj >> n) << (n + S)) + r;
#pragma unroll
    for (int m = 0; m < R; ++m) {
      int c = 0;
#pragma unroll
      for (int e = 0; e < S; ++e) c |= ((m >> (S - 1 - e)) & 1) << e;
      row[fft_slot(d + (c << n))] = v[it + m * ITEMS];
    }
  }
}

// FFT of length L = 2^lg of fft_rows(L) rows per block, written transposed
// (out[c][row]).  First pass: real input w (x - mean); second pass: complex
// input, output |X|^2.  Three radix-2 stages run in registers between two
// barriers, with the operations and twiddles of single stages; the twiddles
// are computed once per block, and a block's rows make runs of 32 bytes of
// every output line, whose neighbours are written on the same XCD.  At 1024 x
// 1024 the passes take 9.5 and 8.5 us; with one row per block, a barrier
// and a sincospi per stage and element-wise scattered stores they took 22 and
// 20, latency of the ten stages and the stores.
template <bool FIRST>
__global__ __launch_bounds__(1024) void k_fft_rows(int lg, const float* __restrict__ x,
                                                   const float* __restrict__ win,
                                                   const double* __restrict__ mean_part,
                                                   const float2* __restrict__ cin,
                                                   float2* __restrict__ cout,
                                                   float* __restrict__ pout) {
  extern __shared__ float2 buf[];
  const int L = 1 << lg, rows = fft_rows(L), eighth = L / 8;
  const int t = threadIdx.x, nb = gridDim.x;
  const int blk = nb % 8 == 0 ? blockIdx.x % 8 * (nb / 8) + blockIdx.x / 8 : blockIdx.x;
  float2* tw = buf + rows * fft_pitch(L);
  for (int i = t; i < L / 2; i += blockDim.x) {
    float sn, cs;
    sincospif(-(float)i / (float)(L / 2), &sn, &cs);
    tw[fft_slot(i)] = make_float2(cs, sn);
  }
  const bool on = t < rows * eighth;   // a block has 64 threads at least
  const int rr = t >> (lg - 3), j = t & (eighth - 1);
  float2* row = buf + rr * fft_pitch(L);
  float2 v[8];
  const float m = FIRST ? mean_of((long)L * L, mean_part) : 0.f;
  const long g = (long)(blk * rows + rr) * L + j;
  if (on) {
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      if (FIRST) {
        const float w = win ? win[g + q * eighth] : 1.f;
        v[q] = make_float2(w * (x[g + q * eighth] - m), 0.f);
      } else {
        v[q] = cin[g + q * eighth];
      }
    }
  }
  __syncthreads();
  int n = 0;
  for (; n + 3 <= lg; n += 3) {
    if (n > 0) {
      if (on)
#pragma unroll
        for (int q = 0; q < 8; ++q) v[q] = row[fft_slot(j + q * eighth)];
      __syncthreads();
    }
    if (on) fft_stages<3>(v, j, lg, n, tw, row);
    __syncthreads();
  }
  if (n < lg) {
    if (on)
#pragma unroll
      for (int q = 0; q < 8; ++q) v[q] = row[fft_slot(j + q * eighth)];
    __syncthreads();
    if (on) {
      if (lg - n == 2)
        fft_stages<2>(v, j, lg, n, tw, row);
      else
        fft_stages<1>(v, j, lg, n, tw, row);
    }
    __syncthreads();
  }
  for (int i = t; i < rows * L; i += blockDim.x) {
    const int c = i / rows, r = i % rows;
    const float2 z = buf[r * fft_pitch(L) + fft_slot(c)];
    const long o = (long)c * L + blk * rows + r;
    if (FIRST)
      cout[o] = z;
    else
      pout[o] = fmaf(z.x, z.x, z.y * z.y);
  }
}

// One block per bin: per row u_y the sum and count of P over the sector members
// of the bin, then those over the rows (strided per thread, then a tree).  The
// 350 thousand members of a 1024 x 1024 image are read where they lie: 8.9 us;
// row sums of all bins in memory and a second launch over them took 19.
__global__ __launch_bounds__(256) void k_sector_bins(int L, const float* __restrict__ P,
                                                     double* __restrict__ out,
                                                     int* __restrict__ counts) {
  __shared__ double red[256];
  __shared__ long redc[256];
  const int k = blockIdx.x, t = threadIdx.x;
  // bin k holds (2k-1)^2 <= 4|u|^2 < (2k+1)^2 (bin 0: u = 0 only)
  const long lo2 = k == 0 ? 0 : (2L * k - 1) * (2L * k - 1), hi2 = (2L * k + 1) * (2L * k + 1);
  double sum = 0.0;
  long c = 0;
  for (int y = t; y < L; y += 256) {
    const long uy = y > L / 2 ? y - L : y;
    // |u|^2 of the sector's members lies between 4/3 and 4 times u_y^2
    if (16 * uy * uy < lo2 || 16 * uy * uy >= 3 * hi2) continue;
    const long lo = lo2 - 4 * uy * uy;   // 4 ux^2 >= lo
    const long hi = hi2 - 4 * uy * uy;   // 4 ux^2 <  hi
    double s = 0.0;
    if (hi > 0) {
      long a = lo <= 0 ? 0 : (long)ceil(sqrt((double)lo / 4.0));
      while (a > 0 && 4 * (a - 1) * (a - 1) >= lo) --a;
      while (4 * a * a < lo) ++a;
      long bnd = (long)floor(sqrt((double)(hi - 1) / 4.0));
      while (4 * (bnd + 1) * (bnd + 1) < hi) ++bnd;
      while (bnd >= 0 && 4 * bnd * bnd >= hi) --bnd;
      for (long ux = a; ux <= bnd; ++ux) {
        for (int sg = 0; sg < 2; ++sg) {
          if (sg == 1 && ux == 0) continue;
          const long v = sg ? -ux : ux;
          if (v > L / 2 || v <= -L / 2) continue;
          if (v == 0 || uy == 0 || v * v > 3 * uy * uy || uy * uy > 3 * v * v) continue;
          s += (double)P[(long)y * L + (v >= 0 ? v : v + L)];
          ++c;
        }
      }
    }
    sum += s;
  }
  redc[t] = c;
  const double tot = block_sum256(sum, red);   // its barriers also order redc
  for (int h = 128; h > 0; h >>= 1) {
    if (t < h) redc[t] += redc[t + h];
    __syncthreads();
  }
  if (t == 0) {
    out[k] = redc[0] > 0 ? tot / (double)redc[0] : 0.0;
    if (counts) counts[k] = (int)redc[0];
  }
}

size_t al256(size_t x) { return (x + 255) & ~size_t(255); }

bool pow2(int L) { return L >= 16 && L <= 4096 && (L & (L - 1)) == 0; }

}  // namespace
}  // namespace mfbd

using namespace mfbd;

extern "C" {

int momfbd_power_spectrum_workspace(int L, int nbins, size_t* bytes) {
  if (!bytes || !pow2(L) || nbins < 1 || nbins > L) return MOMFBD_EINVAL;
  *bytes = al256(kMeanBlocks * sizeof(double)) + al256((size_t)L * L * sizeof(float2));
  return MOMFBD_OK;
}

int momfbd_power_spectrum(int L, const float* image, const float* window, float* power,
                          double* sector, int* counts, int nbins, void* ws, size_t ws_bytes,
                          void* stream) {
  size_t need = 0;
  int st = momfbd_power_spectrum_workspace(L, nbins, &need);
  if (st) return st;
  if (!image || !power) return MOMFBD_EINVAL;
  if (!ws || reinterpret_cast<uintptr_t>(ws) % 256 || ws_bytes < need) return MOMFBD_EWORKSPACE;
  if (hipGetLastError() != hipSuccess) return MOMFBD_EDEVICE;
  hipStream_t s = (hipStream_t)stream;
  char* w = static_cast<char*>(ws);
  double* mean_part = reinterpret_cast<double*>(w);
  float2* T = reinterpret_cast<float2*>(w + al256(kMeanBlocks * sizeof(double)));
  const int lg = __builtin_ctz(L), rows = fft_rows(L);
  const size_t lds = (rows * (size_t)fft_pitch(L) + fft_slot(L / 2)) * sizeof(float2);
  if (lds > 65536) {
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(&k_fft_rows<true>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess ||
        hipFuncSetAttribute(reinterpret_cast<const void*>(&k_fft_rows<false>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
      return MOMFBD_EDEVICE;
  }
  const dim3 grid(L / rows), block(rows * L / 8 < 64 ? 64 : rows * L / 8);
  hipLaunchKernelGGL(k_mean_part, dim3(kMeanBlocks), dim3(256), 0, s, (long)L * L, image,
                     mean_part);
  hipLaunchKernelGGL(k_fft_rows<true>, grid, block, lds, s, lg, image, window, mean_part, nullptr,
                     T, nullptr);
  hipLaunchKernelGGL(k_fft_rows<false>, grid, block, lds, s, lg, nullptr, nullptr, nullptr, T,
                     nullptr, power);
  if (sector)
    hipLaunchKernelGGL(k_sector_bins, dim3(nbins), dim3(256), 0, s, L, power, sector, counts);
  return hipGetLastError() == hipSuccess ? MOMFBD_OK : MOMFBD_EDEVICE;
}

}  // extern "C"
