// Unit kernels of the MOMFBD hot path for 64x64 patches (gfx950).
//
// One workgroup = one wavefront = one unit (patch p, channel c, frame j).
//   forward : phase -> pupil -> inverse 2-D DFT -> |.|^2 (unit-sum PSF)
//             -> forward 2-D DFT (OTF half spectrum)
//   fwdobj  : (a launch schedule) one workgroup of up to 12 waves per
//             (patch, object): the forward of its units, then the Wiener
//             object O_k = N_k / Q_k and the patch loss in FP64 with the
//             object kernel's own per-pair code (object.hip)
//   adjoint : G = conj(O)(D - O S) -> inverse DFT -> H = -4 w kappa g p
//             -> forward DFT on the pupil band -> dL/dphi = Im(conj(P) G_P)
//   prepare : patch cut, mean removal, apodization, mean restore, 2-D DFT
//   objimg  : object spectrum -> real image / N^2
//   burst   : phase -> OTF -> noisy frame of an object -> data spectrum
//   netin   : data spectrum -> the warm-start network's input
#include <hip/hip_runtime.h>

#include "bf16.h"
#include "internal.h"
#include "ops64.h"

#ifndef MFBD_HW_SINCOS
#define MFBD_HW_SINCOS 1
#endif

namespace mfbd {
using namespace n64;

namespace {

constexpr int kUnitF2 = N * HC;   // float2 elements per half spectrum (2112)

__device__ __forceinline__ void wave_sync() { __syncthreads(); }

// Ordering of a unit's LDS exchanges: SYNC 0, the workgroup barrier (a
// one-wave workgroup); SYNC 1, for a unit that is one wave of a larger
// workgroup, the wave's own order only: a wave's LDS accesses complete in
// issue order, so fences at wavefront scope that keep the compiler from
// moving accesses across them are enough.
template <int SYNC>
__device__ __forceinline__ void unit_sync() {
  if constexpr (SYNC == 0) {
    __syncthreads();
  } else {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
}

// Workgroups are dispatched round-robin over the 8 XCDs, each with its own L2.
// Remapping block b to unit (b mod 8) * per + b / 8 gives every XCD a
// contiguous run of units, so the frames of one patch-object (which share the
// object spectrum) meet in the same L2.  The grid has 8 * per blocks.
constexpr int kXcds = 8;
__device__ __forceinline__ int xcd_unit(int per) {
  const int b = blockIdx.x;
  return (b % kXcds) * per + b / kXcds;
}
__host__ __device__ inline int xcd_per(int units) { return (units + kXcds - 1) / kXcds; }

// exp(2 pi i t) for a phase t in turns.  The hardware sine/cosine take
// turns directly; the argument is first reduced to [0,1).
__device__ __forceinline__ float2 expi_turns(float t) {
#if MFBD_HW_SINCOS
  const float f = __builtin_amdgcn_fractf(t);
  return make_float2(__builtin_amdgcn_cosf(f), __builtin_amdgcn_sinf(f));
#else
  float s, c;
  sincospif(2.0f * t, &s, &c);
  return make_float2(c, s);
#endif
}

// Input of op1_cols for lane (q,b): y[n] = P(16+n, 16+q) W64^{+b(16+n)} with
// P = A exp(2 pi i t) on the band; the modulation is a phase ramp of
// b (16+n)/64 turns added before the exponential.
__device__ __forceinline__ void build_pupil(const float* __restrict__ A, const float* __restrict__ ph,
                                            int lane, float2 (&y)[32]) {
  const int q = lane >> 1, b = lane & 1;
#pragma unroll
  for (int n = 0; n < 32; ++n) {
    const float a = A[n * kBand + q];
    const float t = ph[n * kBand + q] + (b ? (16 + n) * (1.0f / 64.0f) : 0.0f);
    y[n] = cscale(expi_turns(t), a);
  }
}

// The two transposes go through a half-size buffer (real parts, then
// imaginary parts): 9.2 KB of LDS per wave lets a CU hold the 12 waves its
// registers allow, against 9 with the full-size buffer.
// Unit u of a field on the wave's LDS (Th, Taux); the OTF is stored to S
// (STORE) and left in X (lane's values at sl_index) and x32 (at sl_index32).
template <bool WANT_PSF, int SYNC, bool STORE = true>
__device__ __forceinline__ void forward64_core(float2* Th, float2* Taux, int u, const ChanTab& ct,
                                               int C, int J, const int* __restrict__ active,
                                               const float* __restrict__ Ab,
                                               const float* __restrict__ phi,
                                               float* __restrict__ psf,
                                               float2* __restrict__ S, float2 (&X)[32],
                                               float2& x32) {
  float* Tf = reinterpret_cast<float*>(Th);
  if (active && !active[u / (J * C)]) return;
  const int lane = threadIdx.x & 63;
  const int c = (u / J) % C;
  float2 pe[32], po[32];
  {
    float2 y[32];
    // a wave that is issuing its loads runs at raised priority, so that
    // they go out ahead of the transform work of the waves beside it
    __builtin_amdgcn_s_setprio(2);
    build_pupil(Ab + c * kBandPix, phi + (size_t)u * kBandPix, lane, y);
    __builtin_amdgcn_s_setprio(0);
    fft32<+1>(y);
    op1_cols_put<0>(y, Tf, lane);
    unit_sync<SYNC>();
    op1_rows_get0(Tf, lane, pe);
    unit_sync<SYNC>();
    op1_cols_put<1>(y, Tf, lane);
  }
  unit_sync<SYNC>();
  op1_rows_get1(Tf, lane, pe, po);
  // half the PSF row (op2_rows_values takes s / 2; the factor is exact)
  const float kap_half = 0.5f * ct.kappa[c];
  float se[32], so[32];
#pragma unroll
  for (int n = 0; n < 32; ++n) {
    se[n] = kap_half * cabs2(pe[n]);
    so[n] = kap_half * cabs2(po[n]);
  }
  if (WANT_PSF) {
    float* row = psf + (size_t)u * N * N + lane * N;
#pragma unroll
    for (int n = 0; n < 32; ++n) {
      row[2 * n] = 2.0f * se[n];
      row[2 * n + 1] = 2.0f * so[n];
    }
  }
  float2 v[32];
  op2_rows_values(se, so, v);
  unit_sync<SYNC>();
  op2_rows_put<0>(v, Tf, lane);
  unit_sync<SYNC>();
  op2_cols_get<0>(Tf, lane, X);
  unit_sync<SYNC>();
  op2_rows_put<1>(v, Tf, lane);
  unit_sync<SYNC>();
  op2_cols_get<1>(Tf, lane, X);
  op2_cols_finish(X, Taux, lane);
  unit_sync<SYNC>();
  x32 = op2_unpack(Taux, Th, lane);
  unit_sync<SYNC>();
  op2_collect(Th, lane, X);
  if constexpr (STORE) {
    float2* out = S + (size_t)u * kUnitF2;
#pragma unroll
    for (int m = 0; m < 32; ++m) out[sl_index(lane, m)] = X[m];
    out[sl_index32(lane)] = x32;
  }
}

// Unit u of a field (the kernel of one plan and the group kernel both
// resolve u, then run this).
template <bool WANT_PSF>
__device__ __forceinline__ void forward64_unit(int u, const ChanTab& ct, int C, int J,
                                               const int* __restrict__ active,
                                               const float* __restrict__ Ab,
                                               const float* __restrict__ phi,
                                               float* __restrict__ psf,
                                               float2* __restrict__ S) {
  __shared__ float2 Th[LDS_HALF / 2];
  __shared__ float2 Taux[LDS_AUX];
  float2 X[32], x32;
  forward64_core<WANT_PSF, 0>(Th, Taux, u, ct, C, J, active, Ab, phi, psf, S, X, x32);
}

template <bool WANT_PSF>
__global__ __launch_bounds__(64) void k_forward64(int units, int xcd, ChanTab ct, int C, int J,
                                                  const int* __restrict__ active,
                                                  const float* __restrict__ Ab,
                                                  const float* __restrict__ phi,
                                                  float* __restrict__ psf,
                                                  float2* __restrict__ S) {
  const int u = xcd ? xcd_unit(xcd_per(units)) : blockIdx.x;
  if (u >= units) return;
  forward64_unit<WANT_PSF>(u, ct, C, J, active, Ab, phi, psf, S);
}

// Every unit of every field of a group; the XCD order runs over the group's
// unit sequence (fields in order, each field's units in order).
__global__ __launch_bounds__(64) void k_forward64_group(GroupArgs ga, int xcd) {
  const int g = xcd ? xcd_unit(xcd_per(ga.total)) : blockIdx.x;
  if (g >= ga.total) return;
  const int2 it = ga.item[g];
  const FieldDesc& F = ga.fd[it.x];
  forward64_unit<false>(it.y, F.ct, F.d.C, F.d.J, F.active, F.Ab, F.w.phi, nullptr,
                        F.w.S);
}

// Forward and Wiener object of one (patch, object) plane per workgroup of
// kFusedWaves waves.  Wave w computes unit w of the plane (the object's
// channels in order, each channel's frames in order) and stores its OTF to
// S as k_forward64 does; after the barrier the workgroup's threads take the
// plane's frequency pairs as k_object<64, 1> does (blocks of 256 pairs, one
// pair per thread, the same per-pair code and the same tree sums of the loss
// terms), so that O and the loss partials equal those of the two separate
// launches bit for bit.  The OTFs it reads back were written by its own
// waves moments before and come from the caches, not HBM: per step S
// crosses HBM once less, and one launch is saved.  The workgroup holds
// 110.6 KB of LDS, so a CU runs one at a time: the 12 waves its registers
// allow the forward transforms in any case.  But every CU then alternates a
// transform phase and a memory phase in step with the others, and no second
// workgroup fills the gaps: measured no faster than the two launches, it is
// a launch schedule (object_fused), off by default.
constexpr int kWaveLds = LDS_HALF / 2 + LDS_AUX;   // float2 per wave (transforms)
constexpr int kObjParts = object_blocks(N, 1);     // 256-pair blocks of a plane
constexpr int kFusedThreads = 64 * kFusedWaves;
static_assert(kObjParts * 256 * sizeof(double) <= kFusedWaves * kWaveLds * sizeof(float2),
              "the loss terms of a plane fit the transforms' LDS");

__global__ __launch_bounds__(kFusedThreads) void k_fwdobj64(int K, ChanTab ct, int C, int J,
                                                            LossArgs la,
                                                            const int* __restrict__ active,
                                                            const float* __restrict__ Ab,
                                                            const float* __restrict__ phi,
                                                            float2* __restrict__ S,
                                                            float2* __restrict__ O,
                                                            double* __restrict__ loss_part) {
  __shared__ float2 lds[kFusedWaves * kWaveLds];
  const int plane = blockIdx.x, p = plane / K, k = plane % K;
  if (active && !active[p]) return;
  const int w = threadIdx.x >> 6;
  const int c0 = ct.obj_first[k];
  if (w < (ct.obj_first[k + 1] - c0) * J) {
    float2 X[32], x32;
    const int u = (p * C + ct.obj_chans[c0 + w / J]) * J + w % J;
    forward64_core<false, 1>(lds + w * kWaveLds, lds + w * kWaveLds + LDS_HALF / 2, u, ct, C,
                             J, nullptr, Ab, phi, nullptr, S, X, x32);
  }
  // every unit's S is written (visible to the workgroup after the barrier)
  // and the transforms are done with LDS
  __syncthreads();
  constexpr int kPairs = kUnitF2 / 2;
  double* red = reinterpret_cast<double*>(lds);
  for (int f2 = threadIdx.x; f2 < kObjParts * 256; f2 += kFusedThreads) {
    double acc = 0.0;
    if (f2 < kPairs) acc += object_pair<N>(f2, p, k, C, J, K, ct, la, S, O);
    red[f2] = acc;
  }
  __syncthreads();
  // the object kernel's sums over each block of 256 pairs, all blocks at once
  for (int s2 = 128; s2 > 0; s2 >>= 1) {
    for (int t = threadIdx.x; t < kObjParts * s2; t += kFusedThreads) {
      const int part = t / s2, i = t % s2;
      red[part * 256 + i] += red[part * 256 + i + s2];
    }
    __syncthreads();
  }
  if ((int)threadIdx.x < kObjParts)
    loss_part[(size_t)plane * kObjParts + threadIdx.x] = red[threadIdx.x * 256];
}

__device__ __forceinline__ void adjoint64_unit(int u, const ChanTab& ct, int C, int J, int K,
                                               const LossArgs& la,
                                               const int* __restrict__ active,
                                               const float* __restrict__ Ab,
                                               const float* __restrict__ phi,
                                               const float2* __restrict__ S,
                                               const float2* __restrict__ O,
                                               float* __restrict__ gphi) {
  __shared__ float2 T[LDS_MAIN];
  __shared__ float2 Taux[LDS_AUX];
  const int lane = threadIdx.x;
  const int j = u % J;
  const int c = (u / J) % C;
  const int p = u / (J * C);
  if (active && !active[p]) return;
  const int k = ct.chan_obj[c];
  const float w2 = -2.0f * (la.weights ? la.weights[c * J + j] : 1.0f);
  const float2* Su = S + (size_t)u * kUnitF2;
  const float2* Du = la.D + (size_t)u * kUnitF2;
  const float2* Ok = O + ((size_t)p * K + k) * kUnitF2;
  const float* Ac = Ab + c * kBandPix;
  const float* phu = phi + (size_t)u * kBandPix;
  // the pupil band field (recomputed below to form p) depends only on phi:
  // build it first so that its loads overlap those of G
  // raised priority while the loads of phi, D, S and O are issued
  __builtin_amdgcn_s_setprio(2);
  float2 y[32];
  build_pupil(Ac, phu, lane, y);

  // G = conj(O) (D - O S) in spectral layout (the frame factor -2 w is
  // applied with 2 kappa after the inverse transform); zero outside the
  // object's spectral support, where D, S and O are not read
  constexpr int kOut = kUnitF2 * 8;
  const __amdgpu_buffer_rsrc_t rD = raw_buffer(Du, kOut), rS = raw_buffer(Su, kOut),
                               rO = raw_buffer(Ok, kOut);
  const int fm = la.supp[k * HC + (lane >> 1)];
  float2 G[32];
#pragma unroll
  for (int m = 0; m < 32; ++m) {
    const int off = in_support(2 * m + (lane & 1), N, fm) ? sl_index(lane, m) * 8 : kOut;
    const float2 o = buffer_load_f2(rO, off);
    G[m] = cmul(cconj(o), csub(buffer_load_f2(rD, off), cmul(o, buffer_load_f2(rS, off))));
  }
  float2 g32;
  {
    const int off = in_support(lane, N, la.supp[k * HC + 32]) ? sl_index32(lane) * 8 : kOut;
    const float2 o = buffer_load_f2(rO, off);
    g32 = cmul(cconj(o), csub(buffer_load_f2(rD, off), cmul(o, buffer_load_f2(rS, off))));
  }
  __builtin_amdgcn_s_setprio(0);
  op3_gather(g32, Taux, lane);
  wave_sync();
  op3_cols(G, Taux, T, lane);
  wave_sync();
  float ge[32], go[32];
  op3_rows(T, lane, ge, go);
  wave_sync();

  // recompute the pupil band transform, then H = -4 w kappa g p and its
  // forward transform to the band, half a row spectrum at a time
  op1_cols(y, T, lane);
  wave_sync();
  float2 Gr[32];
  op14_rows(T, lane, ge, go, 2.0f * ct.kappa[c] * w2, Gr);   // w2: the frame's -2 w
  wave_sync();
  op14_write(Gr, T, lane);
  wave_sync();
  float2 GP[16];
  op4_cols(T, lane, GP);
  const int b = lane & 1, q = lane >> 1;
  float* gout = gphi + (size_t)u * kBandPix;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int n = 2 * i + b;
    const float2 pk = cscale(expi_turns(phu[n * kBand + q]), Ac[n * kBand + q]);
    const float2 gp = GP[i];
    gout[n * kBand + q] = pk.x * gp.y - pk.y * gp.x;   // Im(conj(P) G_P)
  }
}

__global__ __launch_bounds__(64) void k_adjoint64(int units, int xcd, ChanTab ct, int C, int J,
                                                  int K,
                                                  LossArgs la, const int* __restrict__ active,
                                                  const float* __restrict__ Ab,
                                                  const float* __restrict__ phi,
                                                  const float2* __restrict__ S,
                                                  const float2* __restrict__ O,
                                                  float* __restrict__ gphi) {
  const int u = xcd ? xcd_unit(xcd_per(units)) : blockIdx.x;
  if (u >= units) return;
  adjoint64_unit(u, ct, C, J, K, la, active, Ab, phi, S, O, gphi);
}

__global__ __launch_bounds__(64) void k_adjoint64_group(GroupArgs ga, int xcd) {
  const int g = xcd ? xcd_unit(xcd_per(ga.total)) : blockIdx.x;
  if (g >= ga.total) return;
  const int2 it = ga.item[g];
  const FieldDesc& F = ga.fd[it.x];
  adjoint64_unit(it.y, F.ct, F.d.C, F.d.J, F.d.K, F.la, F.active, F.Ab, F.w.phi,
                 F.w.S, F.w.O, F.w.gphi);
}

// Column layout v (lane x: all rows of column x) of a patch -> D = DFT(W (v -
// m) + m), m its mean, stored as a half spectrum.  Whole rows of the window
// are used in the column layout (in row layout every load instruction touched
// 64 lines).
template <int SYNC>
__device__ __forceinline__ void apodized_spectrum(float (&v)[64], const float* __restrict__ apod,
                                                  float2* Th, float2* Taux, int lane,
                                                  float2* __restrict__ out) {
  float* Tf = reinterpret_cast<float*>(Th);
  float s[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int r = 0; r < 64; ++r) s[r & 3] += v[r];
  float sum = (s[0] + s[1]) + (s[2] + s[3]);
  for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off);
  const float mean = sum * (1.0f / (N * N));
  // half the apodized image (op2_rows_values takes s / 2)
#pragma unroll
  for (int r = 0; r < 64; ++r) v[r] = 0.5f * (apod[r * N + lane] * (v[r] - mean) + mean);
  float se[32], so[32];
  image_cols_put<0>(v, Tf, lane);
  unit_sync<SYNC>();
  image_rows_get<0>(Tf, lane, se, so);
  unit_sync<SYNC>();
  image_cols_put<1>(v, Tf, lane);
  unit_sync<SYNC>();
  image_rows_get<1>(Tf, lane, se, so);
  float2 w[32], X[32];
  op2_rows_values(se, so, w);
  unit_sync<SYNC>();
  op2_rows_put<0>(w, Tf, lane);
  unit_sync<SYNC>();
  op2_cols_get<0>(Tf, lane, X);
  unit_sync<SYNC>();
  op2_rows_put<1>(w, Tf, lane);
  unit_sync<SYNC>();
  op2_cols_get<1>(Tf, lane, X);
  op2_cols_finish(X, Taux, lane);
  unit_sync<SYNC>();
  const float2 x32 = op2_unpack(Taux, Th, lane);
  unit_sync<SYNC>();
  op2_collect(Th, lane, X);
#pragma unroll
  for (int m = 0; m < 32; ++m) out[sl_index(lane, m)] = X[m];
  out[sl_index32(lane)] = x32;
}

// A workgroup of WAVES units, one per wave.  Four: the window is loaded into LDS
// once for all of them, beside the loads of the frames.  The 23 064 units of 24
// frames of 1024 x 1024 take 138 us (490 MB to move, 94 us at the rate of a
// large copy; 144 with one unit to a workgroup, which reads the window from
// memory, and 202 us with the window read row by row).  VALU busy 46%, LDS 14%,
// and a wave waits 55% of its cycles: the rest is the latency of one chain of
// loads, transposes and stores per wave.  One unit to a workgroup up to
// kPrepFewUnits units: a chip that they do not fill waits for the window's way
// through LDS (200 units 8.3 against 9.4 us, 512 8.6 against 10.0, 2880 17.7
// against 18.0; no difference up to 11 532).
constexpr int kPrepWaves = 4, kPrepFewUnits = 4096;
template <int WAVES>
__global__ __launch_bounds__(64 * WAVES) void k_prepare64(CutOrder order, int P, int frames_n,
                                                          int H, int W, int stride, int nx,
                                                          const float* __restrict__ frames,
                                                          const float* __restrict__ apod,
                                                          float2* __restrict__ D) {
  __shared__ float2 lds[WAVES][LDS_HALF / 2 + LDS_AUX];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int g = order.block(blockIdx.x) * WAVES + wave, p = g % P, f = g / P;
  const bool on = f < frames_n;
  float v[64];
  if (on) {
    const int y0 = (p / nx) * stride, x0 = (p % nx) * stride;
    const float* src = frames + ((size_t)f * H + y0) * W + x0;
#pragma unroll
    for (int r = 0; r < N; ++r) v[r] = src[(size_t)r * W + lane];
  }
  float2* out = D + ((size_t)p * frames_n + f) * kUnitF2;
  if constexpr (WAVES > 1) {
    __shared__ float win[N * N];
#pragma unroll
    for (int i = 0; i < N * N / (64 * WAVES); ++i)
      win[threadIdx.x + 64 * WAVES * i] = apod[threadIdx.x + 64 * WAVES * i];
    __syncthreads();
    if (!on) return;
    apodized_spectrum<1>(v, win, lds[wave], lds[wave] + LDS_HALF / 2, lane, out);
  } else {
    if (!on) return;
    apodized_spectrum<0>(v, apod, lds[0], lds[0] + LDS_HALF / 2, lane, out);
  }
}

// Spectrum in the lanes' layout (X, x32) -> its image IDFT / N^2 in column
// layout.
__device__ __forceinline__ void inverse_cols(float2 (&X)[32], float2 x32, float2* Th, float2* Taux,
                                             int lane, float (&v)[64]) {
  float* Tf = reinterpret_cast<float*>(Th);
  op3_gather(x32, Taux, lane);
  wave_sync();
  op3_cols_fft(X, Taux, lane);
  float ge[32], go[32];
  {
    float2 Xr[32];
    op3_cols_put<0>(X, Tf, lane);
    wave_sync();
    op3_rows_get<0>(Tf, lane, Xr);
    wave_sync();
    op3_cols_put<1>(X, Tf, lane);
    wave_sync();
    op3_rows_get<1>(Tf, lane, Xr);
    wave_sync();
    op3_rows_finish(Xr, ge, go);
  }
  image_rows_put<0>(ge, go, Tf, lane);
  wave_sync();
  image_cols_get<0>(Tf, lane, v);
  wave_sync();
  image_rows_put<1>(ge, go, Tf, lane);
  wave_sync();
  image_cols_get<1>(Tf, lane, v);
  wave_sync();
#pragma unroll
  for (int r = 0; r < 64; ++r) v[r] *= 1.0f / (N * N);
}

// Item it = (it / per, it % per) of spectra laid out with `stride` items
// between consecutive values of it / per (object images: per = items,
// stride 0; channel 0 of bursts [B][C][J]: per = J, stride = C J).
__global__ __launch_bounds__(64) void k_objimg64(int items, int per, int stride,
                                                 const float2* __restrict__ O,
                                                 float* __restrict__ obj) {
  __shared__ float2 Th[LDS_HALF / 2];
  __shared__ float2 Taux[LDS_AUX];
  const int it = blockIdx.x;
  if (it >= items) return;
  const int lane = threadIdx.x;
  const float2* A = O + ((size_t)(it / per) * stride + it % per) * kUnitF2;
  float2 X[32];
#pragma unroll
  for (int m = 0; m < 32; ++m) X[m] = A[sl_index(lane, m)];
  float v[64];
  inverse_cols(X, A[sl_index32(lane)], Th, Taux, lane, v);
  float* out = obj + (size_t)it * N * N + lane;
#pragma unroll
  for (int r = 0; r < 64; ++r) out[r * N] = v[r];
}

// Input of the warm-start network: frame f = IDFT(D) / N^2 of item `it` (as
// k_objimg64), then 10 (f / mean f - 1) in bfloat16, one plane per frame:
// x[it][N][N].  The image stays in LDS between the transform and the
// normalisation (in two launches it crossed HBM twice in FP32).  The mean is
// the sum of 256 strided partial sums of 16 pixels (pixel i to partial i % 256,
// in order) and a tree over them, the order k_norm_frames uses too.  3072
// frames take 21.7 us (52 MB read, 25 MB written); the transform and a
// normalisation pass over NHWC took 29 + 55 us.
__global__ __launch_bounds__(64) void k_netin64(int items, int per, int stride,
                                                const float2* __restrict__ D,
                                                uint16_t* __restrict__ x) {
  __shared__ float2 T[LDS_MAIN];
  __shared__ float2 Taux[LDS_AUX];
  constexpr int LD = N + 1;
  static_assert(N * LD <= 2 * LDS_MAIN, "the image fits the transform's buffer");
  const int it = blockIdx.x;
  if (it >= items) return;
  const int lane = threadIdx.x;
  const float2* A = D + ((size_t)(it / per) * stride + it % per) * kUnitF2;
  float* Tf = reinterpret_cast<float*>(T);
  {
    float2 X[32];
#pragma unroll
    for (int m = 0; m < 32; ++m) X[m] = A[sl_index(lane, m)];
    op3_gather(A[sl_index32(lane)], Taux, lane);
    wave_sync();
    op3_cols(X, Taux, T, lane);
    wave_sync();
    float ge[32], go[32];
    op3_rows(T, lane, ge, go);
    wave_sync();
    const float inv = 1.0f / (N * N);
#pragma unroll
    for (int n = 0; n < 32; ++n) {
      Tf[lane * LD + 2 * n] = ge[n] * inv;
      Tf[lane * LD + 2 * n + 1] = go[n] * inv;
    }
  }
  wave_sync();
  // partial 64 q + lane: rows q, q + 4, ... of column `lane`
  float s[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    s[q] = 0.f;
#pragma unroll
    for (int t = 0; t < 16; ++t) s[q] += Tf[(q + 4 * t) * LD + lane];
  }
  float r = (s[0] + s[2]) + (s[1] + s[3]);
  for (int h = 32; h > 0; h >>= 1) r += __shfl_down(r, h);
  const float inv = (float)(N * N) / __shfl(r, 0);
  uint2* out = reinterpret_cast<uint2*>(x + (size_t)it * N * N);
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int row = 4 * i + (lane >> 4), col = 4 * (lane & 15);
    const float* v = Tf + row * LD + col;
    uint16_t h[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) h[e] = f2bf(10.f * (v[e] * inv - 1.f));
    out[i * 64 + lane] = make_uint2(h[0] | ((uint32_t)h[1] << 16), h[2] | ((uint32_t)h[3] << 16));
  }
}

// Synthetic bursts: unit u = (p, c, j) from its phase to its data spectrum in
// one pass: the OTF S (as k_forward64), the frame i = IDFT(O_k S) / N^2 +
// sigma_p n, written to the field layout [C][J][P*N][N], and D = DFT(W (i - m)
// + m) (as k_prepare64).  S and the frame stay on chip (in three launches S
// crossed HBM twice and the frames came back once: 23 + 54 + 33 us for 3072
// units, now 47).  Three waves per SIMD hold those units in one round, at the
// cost of 16 bytes of scratch a lane (55 us with two).  Without SPECTRA the frames
// only, for a D that overlaps what other units still read.
template <bool SPECTRA>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(3))) void k_burst64(int units, int P, int C, int J, int K, ChanTab ct,
                                                const float* __restrict__ Ab,
                                                const float* __restrict__ phi,
                                                const float2* __restrict__ O,
                                                const float* __restrict__ noise,
                                                const float* __restrict__ sigma,
                                                const float* __restrict__ apod,
                                                float* __restrict__ field,
                                                float2* __restrict__ D) {
  __shared__ float2 Th[LDS_HALF / 2];
  __shared__ float2 Taux[LDS_AUX];
  const int u = blockIdx.x;
  if (u >= units) return;
  const int lane = threadIdx.x;
  const int j = u % J, c = (u / J) % C, p = u / (J * C);
  float2 X[32], x32;
  forward64_core<false, 0, false>(Th, Taux, u, ct, C, J, nullptr, Ab, phi, nullptr, nullptr, X,
                                  x32);
  wave_sync();
  const float2* Ok = O + ((size_t)p * K + ct.chan_obj[c]) * kUnitF2;
#pragma unroll
  for (int m = 0; m < 32; ++m) X[m] = cmul(Ok[sl_index(lane, m)], X[m]);
  float v[64];
  inverse_cols(X, cmul(Ok[sl_index32(lane)], x32), Th, Taux, lane, v);
  const float sg = sigma[p];
  const float* nz = noise + (size_t)u * N * N + lane;
  float* out = field + ((size_t)(c * J + j) * P + p) * N * N + lane;
#pragma unroll
  for (int r = 0; r < 64; ++r) {
    v[r] += sg * nz[r * N];
    out[r * N] = v[r];
  }
  if constexpr (SPECTRA) apodized_spectrum<0>(v, apod, Th, Taux, lane, D + (size_t)u * kUnitF2);
}

}  // namespace

hipError_t launch_burst64(const Dims& d, const ChanTab& ct, const float* Ab, const float* phi,
                          const float2* O, const float* noise, const float* sigma,
                          const float* apod, float* field, float2* D, hipStream_t s) {
  const int units = d.P * d.C * d.J;
  auto* kernel = D ? &k_burst64<true> : &k_burst64<false>;
  hipLaunchKernelGGL(kernel, dim3(units), dim3(64), 0, s, units, d.P, d.C, d.J, d.K, ct, Ab, phi, O,
                     noise, sigma, apod, field, D);
  return hipGetLastError();
}

hipError_t launch_forward64(const Dims& d, const ChanTab& ct, const int* active, const float* Ab,
                            const float* phi, float* psf, float2* S, hipStream_t s) {
  const int units = d.P * d.C * d.J;
  const dim3 grid(d.xcd_fwd ? kXcds * xcd_per(units) : units);
  if (psf)
    hipLaunchKernelGGL(k_forward64<true>, grid, dim3(64), 0, s, units, d.xcd_fwd, ct, d.C, d.J,
                       active, Ab, phi, psf, S);
  else
    hipLaunchKernelGGL(k_forward64<false>, grid, dim3(64), 0, s, units, d.xcd_fwd, ct, d.C, d.J,
                       active, Ab, phi, psf, S);
  return hipGetLastError();
}

hipError_t launch_fwdobj64(const Dims& d, const ChanTab& ct, const LossArgs& la,
                           const int* active, const float* Ab, const float* phi, float2* S,
                           float2* O, double* loss_pk, hipStream_t s) {
  hipLaunchKernelGGL(k_fwdobj64, dim3(d.P * d.K), dim3(kFusedThreads), 0, s, d.K, ct, d.C, d.J,
                     la, active, Ab, phi, S, O, loss_pk);
  return hipGetLastError();
}

hipError_t launch_adjoint64(const Dims& d, const ChanTab& ct, const LossArgs& la,
                            const int* active, const float* Ab, const float* phi, const float2* S,
                            const float2* O, float* gphi, hipStream_t s) {
  const int units = d.P * d.C * d.J;
  const dim3 grid(d.xcd_adj ? kXcds * xcd_per(units) : units);
  hipLaunchKernelGGL(k_adjoint64, grid, dim3(64), 0, s, units, d.xcd_adj, ct, d.C, d.J, d.K, la,
                     active, Ab, phi, S, O, gphi);
  return hipGetLastError();
}

hipError_t launch_forward64_group(const GroupArgs& ga, int xcd, hipStream_t s) {
  const dim3 grid(xcd ? kXcds * xcd_per(ga.total) : ga.total);
  hipLaunchKernelGGL(k_forward64_group, grid, dim3(64), 0, s, ga, xcd);
  return hipGetLastError();
}

hipError_t launch_adjoint64_group(const GroupArgs& ga, int xcd, hipStream_t s) {
  const dim3 grid(xcd ? kXcds * xcd_per(ga.total) : ga.total);
  hipLaunchKernelGGL(k_adjoint64_group, grid, dim3(64), 0, s, ga, xcd);
  return hipGetLastError();
}

hipError_t launch_prepare64(const Dims& d, const float* frames, int H, int W, int stride,
                            const float* apod, float2* D, hipStream_t s) {
  const int units = d.P * d.C * d.J;
  const int nx = (W - N) / stride + 1;
  const int waves = units <= kPrepFewUnits ? 1 : kPrepWaves;
  const CutOrder order = CutOrder::of(units, waves);
  auto* kernel = waves == 1 ? &k_prepare64<1> : &k_prepare64<kPrepWaves>;
  hipLaunchKernelGGL(kernel, dim3(order.grid()), dim3(64 * waves), 0, s, order, d.P, d.C * d.J, H, W,
                     stride, nx, frames, apod, D);
  return hipGetLastError();
}

hipError_t launch_objimg64(const Dims& d, const float2* O, float* obj, hipStream_t s) {
  const int items = d.P * d.K;
  hipLaunchKernelGGL(k_objimg64, dim3(items), dim3(64), 0, s, items, items, 0, O, obj);
  return hipGetLastError();
}

hipError_t launch_frames64(int items, int per, int stride, const float2* D, float* out,
                           hipStream_t s) {
  hipLaunchKernelGGL(k_objimg64, dim3(items), dim3(64), 0, s, items, per, stride, D, out);
  return hipGetLastError();
}

hipError_t launch_netin64(int items, int per, int stride, const float2* D, uint16_t* x,
                          hipStream_t s) {
  hipLaunchKernelGGL(k_netin64, dim3(items), dim3(64), 0, s, items, per, stride, D, x);
  return hipGetLastError();
}

}  // namespace mfbd
