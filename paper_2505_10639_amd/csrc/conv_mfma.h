// Kernels of the warm-start network's layers on the matrix cores (gfx950):
// 3x3 stride-2 convolutions as implicit GEMMs (no im2col in memory) and the
// dense layers, forward and backward, BF16 operands with FP32 accumulation.
//
// Operand layout of v_mfma_f32_16x16x16_bf16: lane l (i = l % 16, g = l / 16)
// supplies A[i][4g + 0..3] and B[4g + 0..3][i] and receives D[4g + e][i],
// e = 0..3.  The weights are the A operand and the pixels (or bursts) the B
// operand, so a lane ends with four consecutive output channels of one pixel:
// one 8-byte store.
//
// Order of the sums that are rounded to bfloat16 (activations and their
// gradients; the network is sensitive to those roundings): the k range of an
// output is cut into chunks of `kchunk` (a multiple of 32; split_chunk in
// cnn.hip); a chunk is one chain of matrix instructions in k order from zero,
// and the chunks are added in order.  Whatever the tiling, an output has the
// same bits; but kchunk depends on the rows of the launch, so a burst's bits may
// differ between batches of different sizes.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "bf16.h"

namespace mfbd {
namespace conv {

typedef short short4v __attribute__((ext_vector_type(4)));
typedef short short8v __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ u32x2 pack4(float a, float b, float c, float d) {
  return u32x2{(uint32_t)f2bf(a) | ((uint32_t)f2bf(b) << 16),
               (uint32_t)f2bf(c) | ((uint32_t)f2bf(d) << 16)};
}

__device__ __forceinline__ floatx4 mfma16(short4v a, short4v b, floatx4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0);
}

// A tile row of 32 k values in LDS is stored so that the 16-byte read of lane
// group g holds its k of both 16-wide steps: k = 16 s + 4 g + e sits at
// 8 g + 4 s + e.  Rows are 40 values apart (80 bytes: the 16 rows one read
// touches start on distinct banks).
constexpr int kLd = 40;

// the eight k values 8 t .. 8 t + 7 of a row's 32
__device__ __forceinline__ void put8(uint16_t* row, int t, u32x4 v) {
  const int s = t >> 1, g = 2 * (t & 1);
  *reinterpret_cast<u32x2*>(row + 8 * g + 4 * s) = u32x2{v[0], v[1]};
  *reinterpret_cast<u32x2*>(row + 8 * (g + 1) + 4 * s) = u32x2{v[2], v[3]};
}

struct Frag2 {
  short4v s0, s1;
};
__device__ __forceinline__ Frag2 get_frag(const uint16_t* row, int g) {
  const short8v v = *reinterpret_cast<const short8v*>(row + 8 * g);
  return Frag2{__builtin_shufflevector(v, v, 0, 1, 2, 3), __builtin_shufflevector(v, v, 4, 5, 6, 7)};
}

// Convolution of NHWC activations x [B][H][H][CI] with weights w [CO][9 CI]
// (tap by tap, channels fastest): y [B][H/2][H/2][CO] = bf16(ReLU(.. + bias)).
// A block of four waves computes BM output pixels x BN channels; wave
// (wm, wn) owns TM x TN tiles of 16.  Stages of BK k values (one tap each:
// BK divides CI) go global -> registers -> LDS, the next stage's loads in
// flight while the current one is multiplied; one barrier a stage.
// What bounds it: at 256 bursts of 12 frames of 64 x 64 the three layers are
// 6 GFLOP and move 45 MB, so a launch (10.3 to 11.7 us each) is mostly its
// start and the latency of its 9 to 18 stages (VALU busy 16 to 21% of it); BM
// and BN are the smallest tiles that lost nothing, to give every CU blocks at
// small batches too.  With im2col and partial products in memory the same layers
// took 55 to 100 us.
template <int CI, int CO, int BM, int BN, int WM, int BK>
__global__ __launch_bounds__(256) void k_conv(int M, int H, int kchunk,
                                              const uint16_t* __restrict__ x,
                                              const uint16_t* __restrict__ w,
                                              const float* __restrict__ bias,
                                              uint16_t* __restrict__ y) {
  constexpr int WN = 4 / WM, TM = BM / (16 * WM), TN = BN / (16 * WN);
  constexpr int K = 9 * CI, SUB = BK / 32, PER = BK / 8;     // 16-byte pieces of a stage row
  constexpr int NX = BM * PER / 256, NW = BN * PER / 256;    // pieces per thread
  static_assert(CI % BK == 0 && BM * PER % 256 == 0 && BN * PER % 256 == 0, "tile shape");
  __shared__ __align__(16) uint16_t xs[2][SUB][BM][kLd];
  __shared__ __align__(16) uint16_t ws[2][SUB][BN][kLd];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int i16 = lane & 15, g = lane >> 4;
  const int wm = wave % WM, wn = wave / WM;
  const int m0 = blockIdx.x * BM, n0 = blockIdx.y * BN;
  const int Ho = H / 2;
  // this thread's pieces: pixel rows and weight rows
  const uint16_t* xrow[NX];
  unsigned xmask[NX];        // valid taps, bit ky * 3 + kx
#pragma unroll
  for (int e = 0; e < NX; ++e) {
    const int m = m0 + (tid + 256 * e) / PER;
    const int mc = m < M ? m : 0;
    const int ox = mc % Ho, oy = (mc / Ho) % Ho, b = mc / (Ho * Ho);
    xrow[e] = x + (((long)b * H + 2 * oy - 1) * H + 2 * ox - 1) * CI + 8 * ((tid + 256 * e) % PER);
    // rows and columns 0..H-1 are hit by every tap but ky = 0 (kx = 0) at the
    // upper (left) edge; 2 oy + 1 and 2 ox + 1 never pass H - 1
    unsigned v = m < M ? 0x1ffu : 0u;
    if (oy == 0) v &= ~0x007u;
    if (ox == 0) v &= ~0x049u;
    xmask[e] = v;
  }
  const uint16_t* wrow[NW];
#pragma unroll
  for (int e = 0; e < NW; ++e)
    wrow[e] = w + (long)(n0 + (tid + 256 * e) / PER) * K + 8 * ((tid + 256 * e) % PER);
  u32x4 xv[NX], wv[NW];
  auto load = [&](int k0) {
    const int tap = k0 / CI, ky = tap / 3, kx = tap % 3;
    const long off = ((long)ky * H + kx) * CI + (k0 - tap * CI);
#pragma unroll
    for (int e = 0; e < NX; ++e)
      xv[e] = (xmask[e] >> tap) & 1 ? *reinterpret_cast<const u32x4*>(xrow[e] + off) : u32x4{0, 0, 0, 0};
#pragma unroll
    for (int e = 0; e < NW; ++e) wv[e] = *reinterpret_cast<const u32x4*>(wrow[e] + k0);
  };
  auto store = [&](int buf) {
#pragma unroll
    for (int e = 0; e < NX; ++e) {
      const int i = tid + 256 * e, t = i % PER;
      put8(xs[buf][t / 4][i / PER], t % 4, xv[e]);
    }
#pragma unroll
    for (int e = 0; e < NW; ++e) {
      const int i = tid + 256 * e, t = i % PER;
      put8(ws[buf][t / 4][i / PER], t % 4, wv[e]);
    }
  };
  floatx4 acc[TM][TN], tot[TM][TN];
#pragma unroll
  for (int a = 0; a < TM; ++a)
#pragma unroll
    for (int b = 0; b < TN; ++b) acc[a][b] = tot[a][b] = floatx4{0.f, 0.f, 0.f, 0.f};
  load(0);
  store(0);
  __syncthreads();
  int left = kchunk;         // k values left in the current chunk
  for (int k0 = 0, st = 0; k0 < K; k0 += BK, ++st) {
    const int buf = st & 1;
    if (k0 + BK < K) load(k0 + BK);
#pragma unroll
    for (int sub = 0; sub < SUB; ++sub) {
      Frag2 xf[TM], wf[TN];
#pragma unroll
      for (int a = 0; a < TM; ++a) xf[a] = get_frag(xs[buf][sub][(wm * TM + a) * 16 + i16], g);
#pragma unroll
      for (int b = 0; b < TN; ++b) wf[b] = get_frag(ws[buf][sub][(wn * TN + b) * 16 + i16], g);
#pragma unroll
      for (int a = 0; a < TM; ++a)
#pragma unroll
        for (int b = 0; b < TN; ++b) acc[a][b] = mfma16(wf[b].s0, xf[a].s0, acc[a][b]);
#pragma unroll
      for (int a = 0; a < TM; ++a)
#pragma unroll
        for (int b = 0; b < TN; ++b) acc[a][b] = mfma16(wf[b].s1, xf[a].s1, acc[a][b]);
      left -= 32;
      if (left == 0 || k0 + 32 * (sub + 1) >= K) {
        left = kchunk;
#pragma unroll
        for (int a = 0; a < TM; ++a)
#pragma unroll
          for (int b = 0; b < TN; ++b) {
            tot[a][b] += acc[a][b];
            acc[a][b] = floatx4{0.f, 0.f, 0.f, 0.f};
          }
      }
    }
    if (k0 + BK < K) store(buf ^ 1);
    __syncthreads();
  }
#pragma unroll
  for (int a = 0; a < TM; ++a) {
    const int m = m0 + (wm * TM + a) * 16 + i16;
    if (m >= M) continue;
#pragma unroll
    for (int b = 0; b < TN; ++b) {
      const int n = n0 + (wn * TN + b) * 16 + 4 * g;
      float v[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = fmaxf(tot[a][b][e] + bias[n + e], 0.f);
      *reinterpret_cast<u32x2*>(y + (long)m * CO + n) = pack4(v[0], v[1], v[2], v[3]);
    }
  }
}

// First convolution: the frames x [B][J][N][N] (bf16, one plane per frame, as
// the input kernels leave them) with weights w [32][9 J].  One block: one
// burst and RO = net_rows(N) rows of the output; its input rows are staged in
// LDS with the frames fastest ([row][column][J], a zero column on the left
// and, at the top, a zero row), the weights beside them, and every wave takes
// tiles of 16 pixels x 32 channels.  J % 4 == 0: the four k of a lane group
// are four frames of one tap, one 8-byte read; otherwise four 2-byte reads
// through a table of offsets.  A block reads 2 RO + 1 rows of 2 N bytes a frame,
// the first of which the block above it reads too.
__host__ __device__ inline int net_rows(int N) { return N == 64 ? 4 : 2; }
__host__ __device__ inline int conv1_ld(int J) { return (9 * J + 31) / 32 * 32 + 4; }
__host__ __device__ inline size_t conv1_tile(int N, int J) {
  return ((size_t)(2 * net_rows(N) + 1) * (N + 1) * J * 2 + 15) / 16 * 16;
}
__host__ __device__ inline size_t conv1_lds(int N, int J) {
  return conv1_tile(N, J) + (size_t)conv1_ld(J) * (J % 4 == 0 ? 4 : 68);
}

template <bool J4>
__global__ __launch_bounds__(256) void k_conv1(int N, int J, int kchunk,
                                               const uint16_t* __restrict__ x,
                                               const uint16_t* __restrict__ w,
                                               const float* __restrict__ bias,
                                               uint16_t* __restrict__ y) {
  extern __shared__ __align__(16) unsigned char lds1[];
  const int K = 9 * J, ld = conv1_ld(J), CW = N + 1, RO = net_rows(N), Wo = N / 2;
  uint16_t* xl = reinterpret_cast<uint16_t*>(lds1);         // [2 RO + 1][CW][J]
  int* koff = reinterpret_cast<int*>(lds1 + conv1_tile(N, J));   // [ld]
  uint16_t* wl = reinterpret_cast<uint16_t*>(koff + ld);    // [32][ld] (J % 4 != 0)
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int i16 = lane & 15, g = lane >> 4;
  const int per = Wo / RO, b = blockIdx.x / per, oy0 = (blockIdx.x % per) * RO;
  const int rows = 2 * RO + 1;
  for (int k = tid; k < ld; k += 256) {
    const int kk = k < K ? k : 0, tap = kk / J;             // weights past K are zero
    koff[k] = ((tap / 3) * CW + tap % 3) * J + kk % J;
  }
  if (!J4)
    for (int k = tid % 8; k < ld; k += 8)
      wl[(tid / 8) * ld + k] = k < K ? w[(tid / 8) * K + k] : (uint16_t)0;
  for (int i = tid; i < rows * J; i += 256) xl[(i / J) * CW * J + i % J] = 0;   // column 0
  // frames fastest over the threads: their 2-byte stores to LDS then fall on
  // neighbouring addresses (pieces fastest put 16 lanes on one bank)
  const int pieces = N / 8;                                 // 16-byte pieces of an input row
  for (int i = tid; i < J * rows * pieces; i += 256) {
    const int j = i % J, q = i / J, t = q % pieces, r = q / pieces;
    const int yy = 2 * oy0 - 1 + r;
    u32x4 v{0, 0, 0, 0};
    if (yy >= 0)
      v = *reinterpret_cast<const u32x4*>(x + (((long)b * J + j) * N + yy) * N + 8 * t);
    uint16_t* dst = xl + ((long)r * CW + 1 + 8 * t) * J + j;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      dst[(2 * e) * J] = (uint16_t)(v[e] & 0xffffu);
      dst[(2 * e + 1) * J] = (uint16_t)(v[e] >> 16);
    }
  }
  __syncthreads();
  // tiles t0 and t0 + 4 of a wave together: they share the weights
  const int tiles = RO * Wo / 16;
  for (int t0 = wave; t0 < tiles; t0 += 8) {
    const int n = t0 + 4 < tiles ? 2 : 1;
    const uint16_t* base[2];
    int oy[2], ox[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int pix = (t0 + (q < n ? 4 * q : 0)) * 16 + i16;
      oy[q] = pix / Wo;
      ox[q] = pix % Wo;
      base[q] = xl + ((2 * oy[q]) * CW + 2 * ox[q]) * J;
    }
    floatx4 acc[2][2], tot[2][2];
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
      for (int a = 0; a < 2; ++a) acc[q][a] = tot[q][a] = floatx4{0.f, 0.f, 0.f, 0.f};
    int left = kchunk;
    for (int k0 = 0; k0 < K; k0 += 32) {
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        const int k = k0 + 16 * s + 4 * g;
        short4v xf[2], wf[2];
#pragma unroll
        for (int a = 0; a < 2; ++a) {
          if (J4)
            wf[a] = k < K ? *reinterpret_cast<const short4v*>(w + (16 * a + i16) * K + k)
                          : short4v{0, 0, 0, 0};
          else
            wf[a] = *reinterpret_cast<const short4v*>(wl + (16 * a + i16) * ld + k);
        }
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          if (J4) {
            xf[q] = *reinterpret_cast<const short4v*>(base[q] + koff[k]);
          } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) xf[q][e] = (short)base[q][koff[k + e]];
          }
#pragma unroll
          for (int a = 0; a < 2; ++a) acc[q][a] = mfma16(wf[a], xf[q], acc[q][a]);
        }
      }
      left -= 32;
      if (left == 0 || k0 + 32 >= K) {
        left = kchunk;
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
          for (int a = 0; a < 2; ++a) {
            tot[q][a] += acc[q][a];
            acc[q][a] = floatx4{0.f, 0.f, 0.f, 0.f};
          }
      }
    }
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      if (q >= n) break;
      uint16_t* out = y + (((long)b * Wo + oy0 + oy[q]) * Wo + ox[q]) * 32 + 4 * g;
#pragma unroll
      for (int a = 0; a < 2; ++a) {
        float v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = fmaxf(tot[q][a][e] + bias[16 * a + 4 * g + e], 0.f);
        *reinterpret_cast<u32x2*>(out + 16 * a) = pack4(v[0], v[1], v[2], v[3]);
      }
    }
  }
}

// Dense layer: out[m][n] = sum_k x[m][k] w[n][k] + bias[n] (K a multiple of
// 32), ReLU and bf16 (out16), or FP32 times scale[n % smod] where given
// (out32).  One block per 16 x 16 outputs, so that a few rows (bursts) still
// keep the chip busy; the chunks of the k range are dealt to its four waves,
// the partial tiles left in LDS and added in chunk order.  The operands go
// through LDS in windows of 512 k: a wave reads a kilobyte of one row at a
// time (reading 16 rows at once, a power of two of bytes apart, put every
// request on one L2 channel: 19 against 8 us for 256 x 512 x 2048).
constexpr int kDenseK = 512, kDenseLd = kDenseK + 8, kDenseZ = kDenseK / 32;
__global__ __launch_bounds__(256) void k_dense(int M, int N, int K, int kchunk,
                                               const uint16_t* __restrict__ x,
                                               const uint16_t* __restrict__ w,
                                               const float* __restrict__ bias,
                                               uint16_t* __restrict__ out16,
                                               float* __restrict__ out32,
                                               const float* __restrict__ scale, int smod) {
  __shared__ __align__(16) uint16_t rows[32][kDenseLd];     // 16 of x, 16 of w
  __shared__ __align__(16) float part[kDenseZ][256];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int i16 = lane & 15, g = lane >> 4;
  const int n0 = blockIdx.x * 16, m0 = blockIdx.y * 16;
  // wave r reads rows r, r + 4, ...: lane l the eight k 8 l .. 8 l + 7
  u32x4 v[8];
  auto load = [&](int k0) {
    const int k = min(k0 + 8 * lane, K - 8);                // past the end: not used
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int r = wave + 4 * e;
      const uint16_t* src = r < 16 ? x + (long)min(m0 + r, M - 1) * K
                                   : w + (long)min(n0 + r - 16, N - 1) * K;
      v[e] = *reinterpret_cast<const u32x4*>(src + k);
    }
  };
  load(0);
  float sum = 0.f;
  floatx4 acc{0.f, 0.f, 0.f, 0.f};
  int z = 0, left = kchunk;      // the chunk at hand and what is left of it
  for (int k0 = 0; k0 < K; k0 += kDenseK) {
#pragma unroll
    for (int e = 0; e < 8; ++e)
      *reinterpret_cast<u32x4*>(&rows[wave + 4 * e][8 * lane]) = v[e];
    __syncthreads();
    if (k0 + kDenseK < K) load(k0 + kDenseK);
    const int kn = min(kDenseK, K - k0);
    int done = 0;                // chunks completed in this window
    for (int k = 0; k < kn; k += 32) {
      if ((z & 3) == wave) {
#pragma unroll
        for (int s = 0; s < 2; ++s)
          acc = mfma16(*reinterpret_cast<const short4v*>(&rows[16 + i16][k + 16 * s + 4 * g]),
                       *reinterpret_cast<const short4v*>(&rows[i16][k + 16 * s + 4 * g]), acc);
      }
      left -= 32;
      if (left == 0 || k0 + k + 32 >= K) {
        if ((z & 3) == wave) {
          *reinterpret_cast<floatx4*>(&part[done][i16 * 16 + 4 * g]) = acc;   // [m][n]
          acc = floatx4{0.f, 0.f, 0.f, 0.f};
        }
        ++done;
        ++z;
        left = kchunk;
      }
    }
    __syncthreads();
    for (int d = 0; d < done; ++d) sum += part[d][tid];
  }
  const int m = m0 + tid / 16, n = n0 + tid % 16;
  if (m >= M || n >= N) return;
  sum += bias[n];
  if (out16) out16[(long)m * N + n] = f2bf(fmaxf(sum, 0.f));
  if (out32) out32[(long)m * N + n] = scale ? sum * scale[n % smod] : sum;
}


// ------------------------------------------------------------------ backward

// Two rows k, k + 1 of eight consecutive columns, column by column: the pair
// of column e as one word (row k in the low half).
__device__ __forceinline__ void pair8(u32x4 r0, u32x4 r1, uint32_t (&out)[8]) {
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    out[2 * e] = __builtin_amdgcn_perm(r1[e], r0[e], 0x05040100);
    out[2 * e + 1] = __builtin_amdgcn_perm(r1[e], r0[e], 0x07060302);
  }
}

// position of k (of 32) in a row read by get_frag
__device__ __forceinline__ int frag_pos(int k) { return 8 * ((k & 15) >> 2) + 4 * (k >> 4) + (k & 3); }

// Gradient of a convolution's input: for one parity class (py, px) of the
// input pixels, dx[b][2 y + py][2 x + px][ci] = sum over the class's taps in
// (ky, kx) order of sum_co dz[b][oy][ox][co] w[co][tap][ci], kept where the
// input activation h is positive, as bf16.  A stride-2 convolution reads an
// even row (column) through tap 1 alone and an odd one through taps 0 and 2,
// so the four classes have 1, 2, 2 and 4 taps and nothing is multiplied for
// padding.  Per tap the sum over co is cut into chunks as in the forward
// layers, and the taps are added in order: the bits of the columns-and-gather
// form, without its FP32 columns (9 ci values a pixel) in memory: 23, 17 and
// 15 us for the three layers at 256 bursts of 64 x 64, against 75 to 110 us.
// A block: BM pixels x BN input channels; a wave 32 pixels of them.
template <int CI, int CO, int BM, int BN>
__global__ __launch_bounds__(256) void k_conv_dx(int M, int Ho, int kchunk,
                                                 const uint16_t* __restrict__ dz,
                                                 const uint16_t* __restrict__ w,
                                                 const uint16_t* __restrict__ h,
                                                 uint16_t* __restrict__ dx) {
  constexpr int WM = BM / 32, WN = 4 / WM, TM = 2, TN = BN / (16 * WN);
  constexpr int NX = BM * 4 / 256 > 0 ? BM * 4 / 256 : 1;   // 16-byte pieces of dz per thread
  constexpr int WT = BN / 8 * 16;                           // threads staging weights
  static_assert(BM * 4 % 256 == 0 && WT <= 256 && CO % 32 == 0, "tile shape");
  __shared__ __align__(16) uint16_t xs[2][BM][kLd];
  __shared__ __align__(16) uint16_t ws[2][BN][kLd];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int i16 = lane & 15, g = lane >> 4;
  const int wm = wave % WM, wn = wave / WM;
  const int m0 = blockIdx.x * BM, n0 = blockIdx.y * BN;
  const int py = blockIdx.z >> 1, px = blockIdx.z & 1;
  const int nx = px ? 2 : 1, taps = (py ? 2 : 1) * nx;
  // tap t: (ky, kx), reading dz at (y + oy, x + ox) of the class's pixel (y, x)
  auto tap_of = [&](int t, int& k, int& oy, int& ox) {
    const int a = t / nx, b = t % nx;
    const int ky = py ? 2 * a : 1, kx = px ? 2 * b : 1;
    oy = py && a == 0;
    ox = px && b == 0;
    k = ky * 3 + kx;
  };
  int yy[NX], xx[NX];
  long row[NX];
#pragma unroll
  for (int e = 0; e < NX; ++e) {
    const int m = m0 + (tid + 256 * e) / 4;
    const int mc = m < M ? m : 0;
    xx[e] = mc % Ho;
    yy[e] = m < M ? (mc / Ho) % Ho : Ho;       // Ho: never inside
    row[e] = (long)mc * CO + 8 * ((tid + 256 * e) % 4);
  }
  const int kp = tid % 16, piece = tid / 16;   // weights: rows co = 2 kp, + 1; columns 8 piece ..
  u32x4 xv[NX], w0, w1;
  auto load = [&](int st) {
    const int t = st / (CO / 32), c0 = (st % (CO / 32)) * 32;
    int k, oy, ox;
    tap_of(t, k, oy, ox);
#pragma unroll
    for (int e = 0; e < NX; ++e)
      xv[e] = yy[e] + oy < Ho && xx[e] + ox < Ho
                  ? *reinterpret_cast<const u32x4*>(dz + row[e] + (long)(oy * Ho + ox) * CO + c0)
                  : u32x4{0, 0, 0, 0};
    if (tid < WT) {
      const uint16_t* src = w + ((long)(c0 + 2 * kp) * 9 + k) * CI + n0 + 8 * piece;
      w0 = *reinterpret_cast<const u32x4*>(src);
      w1 = *reinterpret_cast<const u32x4*>(src + 9 * CI);
    }
  };
  auto store = [&](int buf) {
#pragma unroll
    for (int e = 0; e < NX; ++e) {
      const int i = tid + 256 * e;
      put8(xs[buf][i / 4], i % 4, xv[e]);
    }
    if (tid < WT) {
      uint32_t pr[8];
      pair8(w0, w1, pr);
#pragma unroll
      for (int e = 0; e < 8; ++e)
        *reinterpret_cast<uint32_t*>(&ws[buf][8 * piece + e][frag_pos(2 * kp)]) = pr[e];
    }
  };
  floatx4 acc[TM][TN], tot[TM][TN], sum[TM][TN];
#pragma unroll
  for (int a = 0; a < TM; ++a)
#pragma unroll
    for (int b = 0; b < TN; ++b) acc[a][b] = tot[a][b] = sum[a][b] = floatx4{0.f, 0.f, 0.f, 0.f};
  const int steps = taps * (CO / 32);
  load(0);
  store(0);
  __syncthreads();
  int left = kchunk;
  for (int st = 0; st < steps; ++st) {
    const int buf = st & 1;
    if (st + 1 < steps) load(st + 1);
    Frag2 xf[TM], wf[TN];
#pragma unroll
    for (int a = 0; a < TM; ++a) xf[a] = get_frag(xs[buf][(wm * TM + a) * 16 + i16], g);
#pragma unroll
    for (int b = 0; b < TN; ++b) wf[b] = get_frag(ws[buf][(wn * TN + b) * 16 + i16], g);
#pragma unroll
    for (int a = 0; a < TM; ++a)
#pragma unroll
      for (int b = 0; b < TN; ++b) {
        acc[a][b] = mfma16(wf[b].s0, xf[a].s0, acc[a][b]);
        acc[a][b] = mfma16(wf[b].s1, xf[a].s1, acc[a][b]);
      }
    left -= 32;
    const bool tap_end = st % (CO / 32) == CO / 32 - 1;
    if (left == 0 || tap_end) {
      left = kchunk;
#pragma unroll
      for (int a = 0; a < TM; ++a)
#pragma unroll
        for (int b = 0; b < TN; ++b) {
          tot[a][b] += acc[a][b];
          acc[a][b] = floatx4{0.f, 0.f, 0.f, 0.f};
          if (tap_end) {
            sum[a][b] += tot[a][b];
            tot[a][b] = floatx4{0.f, 0.f, 0.f, 0.f};
          }
        }
    }
    if (st + 1 < steps) store(buf ^ 1);
    __syncthreads();
  }
  const int H = 2 * Ho;
#pragma unroll
  for (int a = 0; a < TM; ++a) {
    const int m = m0 + (wm * TM + a) * 16 + i16;
    if (m >= M) continue;
    const int x = 2 * (m % Ho) + px, y = 2 * ((m / Ho) % Ho) + py, b = m / (Ho * Ho);
    const long o = (((long)b * H + y) * H + x) * CI;
#pragma unroll
    for (int t = 0; t < TN; ++t) {
      const int n = n0 + (wn * TN + t) * 16 + 4 * g;
      const u32x2 hv = *reinterpret_cast<const u32x2*>(h + o + n);
      float v[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const uint16_t he = (uint16_t)(hv[e / 2] >> (16 * (e & 1)));
        v[e] = bf2f(he) > 0.f ? sum[a][t][e] : 0.f;
      }
      *reinterpret_cast<u32x2*>(dx + o + n) = pack4(v[0], v[1], v[2], v[3]);
    }
  }
}

// Gradient of a dense layer's input: dh[m][n] = sum_k dz[m][k] w[k][n], kept
// where the input activation h is positive, as bf16.  w [K][N] (N a multiple
// of 32) is transposed on its way into LDS.  A block: 32 bursts x 32 inputs,
// in windows of 128 k (a few long stages rather than many short ones: their
// latency is what the launch costs); wave (a, b) one 16 x 16 tile.
__global__ __launch_bounds__(256) void k_dense_dx(int M, int N, int K, int kchunk,
                                                  const uint16_t* __restrict__ dz,
                                                  const uint16_t* __restrict__ w,
                                                  const uint16_t* __restrict__ h,
                                                  uint16_t* __restrict__ dx) {
  __shared__ __align__(16) uint16_t xs[4][32][kLd];
  __shared__ __align__(16) uint16_t ws[4][32][kLd];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int i16 = lane & 15, g = lane >> 4;
  const int n0 = blockIdx.x * 32, m0 = blockIdx.y * 32;
  const int ta = wave & 1, tb = wave >> 1;
  // dz: row tid / 8, k = 16 (tid % 8) .. + 15; w: rows 2 kp, 2 kp + 1 and
  // columns 8 piece .. + 7
  const int xr = tid / 8, xk = 16 * (tid % 8), kp = tid / 4, piece = tid % 4;
  const uint16_t* src = dz + (long)min(m0 + xr, M - 1) * K;
  u32x4 xv[2], w0, w1;
  auto load = [&](int k0) {
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int k = k0 + xk + 8 * q;
      xv[q] = u32x4{0, 0, 0, 0};
      if (K % 8 == 0) {
        if (k < K) xv[q] = *reinterpret_cast<const u32x4*>(src + k);
      } else {                                   // rows of any length
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (k + e < K) xv[q][e / 2] |= (uint32_t)src[k + e] << (16 * (e & 1));
      }
    }
    const int k = k0 + 2 * kp;
    const uint16_t* ww = w + (long)k * N + n0 + 8 * piece;
    w0 = k < K ? *reinterpret_cast<const u32x4*>(ww) : u32x4{0, 0, 0, 0};
    w1 = k + 1 < K ? *reinterpret_cast<const u32x4*>(ww + N) : u32x4{0, 0, 0, 0};
  };
  floatx4 acc{0.f, 0.f, 0.f, 0.f}, tot{0.f, 0.f, 0.f, 0.f};
  load(0);
  int left = kchunk;
  for (int k0 = 0; k0 < K; k0 += 128) {
#pragma unroll
    for (int q = 0; q < 2; ++q) put8(xs[xk / 32][xr], xk / 8 % 4 + q, xv[q]);
    uint32_t pr[8];
    pair8(w0, w1, pr);
#pragma unroll
    for (int e = 0; e < 8; ++e)
      *reinterpret_cast<uint32_t*>(&ws[kp / 16][8 * piece + e][frag_pos(2 * kp % 32)]) = pr[e];
    __syncthreads();
    if (k0 + 128 < K) load(k0 + 128);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (k0 + 32 * q >= K) break;
      const Frag2 xf = get_frag(xs[q][16 * ta + i16], g), wf = get_frag(ws[q][16 * tb + i16], g);
      acc = mfma16(wf.s0, xf.s0, acc);
      acc = mfma16(wf.s1, xf.s1, acc);
      left -= 32;
      if (left == 0 || k0 + 32 * q + 32 >= K) {
        left = kchunk;
        tot += acc;
        acc = floatx4{0.f, 0.f, 0.f, 0.f};
      }
    }
    __syncthreads();
  }
  const int m = m0 + 16 * ta + i16, n = n0 + 16 * tb + 4 * g;
  if (m >= M) return;
  const u32x2 hv = *reinterpret_cast<const u32x2*>(h + (long)m * N + n);
  float v[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const uint16_t he = (uint16_t)(hv[e / 2] >> (16 * (e & 1)));
    v[e] = bf2f(he) > 0.f ? tot[e] : 0.f;
  }
  *reinterpret_cast<u32x2*>(dx + (long)m * N + n) = pack4(v[0], v[1], v[2], v[3]);
}

// Parameter gradients: part[z][i][j] = sum over split z of the rows k of
// P[k][i] Q[k][j], i < M, j < N, with one more column j = N of ones for the
// bias (v_mfma_f32_16x16x32_bf16; these sums stay FP32, added over the splits
// by k_grad_sum).  P = dz [k][M].  Q: a dense layer's input [k][N], or (CI >
// 0) a convolution's: row k = output pixel, column j = tap CI + ci, gathered
// from the NHWC input.  Both have their columns, not their rows, contiguous:
// a thread takes two rows of eight columns and stores the eight pairs, so the
// matrix operands' eight consecutive k are one 16-byte read.  A block is a 64
// x 64 tile, wave (a, b) 32 x 32 of it, in stages of 32 rows, two of
// them in flight.  At 256 bursts of 64 x 64 the three convolutions take 20, 19
// and 14 us with four blocks a CU (24, 23 and 15 with two; then, blocks of one
// row range kept on one XCD: 21, 22, 14, and the dense layers, of few row ranges,
// 15 instead of 7).  Gathering and pairing the rows takes 26 to 34 VALU
// instructions to a matrix instruction, yet the VALU is busy only 26 to 32% of
// the time: the rest is the latency of the stages.
template <int CI>
__global__ __launch_bounds__(256) void k_wgrad(int M, int N, int K, int rows, int H,
                                               const uint16_t* __restrict__ P,
                                               const uint16_t* __restrict__ Q,
                                               float* __restrict__ part) {
  typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
  __shared__ __align__(16) uint16_t ts[2][128][kLd];   // 64 columns of P, 64 of Q
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int i16 = lane & 15, g = lane >> 4;
  const int j0 = blockIdx.x * 64, i0 = blockIdx.y * 64, z = blockIdx.z;
  const int wa = wave & 1, wb = wave >> 1;
  const int kb = z * rows, ke = min(K, kb + rows);
  const int kp = tid % 16, piece = (tid / 16) % 8;     // rows 2 kp, 2 kp + 1; columns 8 piece ..
  const bool isq = tid >= 128;
  const int Ho = H / 2;
  const int col = (isq ? j0 : i0) + 8 * piece;
  const int width = isq ? N : M;
  const int tap = CI > 0 ? col / (CI > 0 ? CI : 1) : 0, ky = tap / 3, kx = tap % 3;
  // output pixel of this thread's two rows, moved on by 32 rows a stage
  int ox[2], oy[2], b[2], dx = 0, dy = 0, db = 0;
  if (CI > 0) {
    dx = 32 % Ho;
    dy = 32 / Ho % Ho;
    db = 32 / (Ho * Ho);
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      const int k = kb + 2 * kp + r;
      ox[r] = k % Ho;
      oy[r] = k / Ho % Ho;
      b[r] = k / (Ho * Ho);
    }
  }
  auto load = [&](int k0, u32x4 (&v)[2]) {
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      const int k = k0 + 2 * kp + r;
      u32x4 t{0, 0, 0, 0};
      if (k < ke && col < width) {
        if (CI > 0 && isq) {
          const int y = 2 * oy[r] + ky - 1, x = 2 * ox[r] + kx - 1;
          if (y >= 0 && x >= 0)
            t = *reinterpret_cast<const u32x4*>(Q + (((long)b[r] * H + y) * H + x) * CI + col - tap * CI);
        } else {
          const uint16_t* src = (isq ? Q : P) + (long)k * width + col;
          if (width % 8 == 0) {
            t = *reinterpret_cast<const u32x4*>(src);
          } else {                           // rows of any length: two bytes at a time
#pragma unroll
            for (int e = 0; e < 8; ++e)
              if (col + e < width) t[e / 2] |= (uint32_t)src[e] << (16 * (e & 1));
          }
        }
      }
      if (k < ke && isq && col <= N && N < col + 8) {     // the column of ones
        const int e = N - col;
        const uint32_t one = 0x3f80u << (16 * (e & 1));
#pragma unroll
        for (int q = 0; q < 4; ++q)
          if (q == e / 2) t[q] |= one;
      }
      v[r] = t;
      if (CI > 0) {
        ox[r] += dx;
        oy[r] += dy;
        b[r] += db;
        if (ox[r] >= Ho) {
          ox[r] -= Ho;
          ++oy[r];
        }
        if (oy[r] >= Ho) {
          oy[r] -= Ho;
          ++b[r];
        }
      }
    }
  };
  auto store = [&](int buf, const u32x4 (&v)[2]) {
    uint32_t pr[8];
    pair8(v[0], v[1], pr);
#pragma unroll
    for (int e = 0; e < 8; ++e)
      *reinterpret_cast<uint32_t*>(&ts[buf][(isq ? 64 : 0) + 8 * piece + e][2 * kp]) = pr[e];
  };
  floatx4 acc[2][2];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) acc[a][b] = floatx4{0.f, 0.f, 0.f, 0.f};
  auto multiply = [&](int buf) {
    bf16x8 pf[2], qf[2];
#pragma unroll
    for (int a = 0; a < 2; ++a) {
      pf[a] = *reinterpret_cast<const bf16x8*>(&ts[buf][32 * wa + 16 * a + i16][8 * g]);
      qf[a] = *reinterpret_cast<const bf16x8*>(&ts[buf][64 + 32 * wb + 16 * a + i16][8 * g]);
    }
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int b = 0; b < 2; ++b)
        acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pf[a], qf[b], acc[a][b], 0, 0, 0);
  };
  // two stages of loads in flight (rows past ke come as zeros)
  u32x4 va[2], vb[2];
  load(kb, va);
  load(kb + 32, vb);
  store(0, va);
  __syncthreads();
  for (int k0 = kb; k0 < ke; k0 += 64) {
    load(k0 + 64, va);
    multiply(0);
    store(1, vb);
    __syncthreads();
    load(k0 + 96, vb);
    multiply(1);
    store(0, va);
    __syncthreads();
  }
  float* out = part + (long)z * M * (N + 1);
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int i = i0 + 32 * wa + 16 * a + 4 * g + e, j = j0 + 32 * wb + 16 * b + i16;
        if (i < M && j <= N) out[(long)i * (N + 1) + j] = acc[a][b][e];
      }
}

// The same for the first convolution, whose input x [B][J][N][N] keeps the
// frames as planes: column j = tap J + ci of eight consecutive output pixels
// of a row is every second value of an input row, so a thread reads 16 values
// of the row (and the one before them) and stores the eight even ones (kx =
// 1), the eight odd ones (kx = 2) and the odd ones one pixel earlier (kx =
// 0).  A block takes `rows` output pixels and all 32 x (9 J + 1) sums, its
// waves every fourth 16-column tile.  A stage is latency: 36 us in blocks of 32
// stages (one a CU at 256 bursts of 64 x 64), 21.5 us in blocks of 16.
__host__ __device__ inline int wgrad1_cols(int J) { return (9 * J + 1 + 15) / 16 * 16; }
__host__ __device__ inline size_t wgrad1_lds(int J) {
  return (size_t)(32 + wgrad1_cols(J)) * kLd * 2 * 2;
}
template <int TILES, int TASKS>
__global__ __launch_bounds__(256) void k_wgrad1(int N, int J, int K, int rows,
                                                const uint16_t* __restrict__ dz,
                                                const uint16_t* __restrict__ x,
                                                float* __restrict__ part) {
  typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
  extern __shared__ __align__(16) uint16_t tw[];            // [2][32 + wgrad1_cols][kLd]
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int i16 = lane & 15, g = lane >> 4;
  const int NC = 9 * J, cols = wgrad1_cols(J), Wo = N / 2;
  const int kb = blockIdx.x * rows, ke = min(K, kb + rows);
  const int size = (32 + cols) * kLd;                       // values of one buffer
  for (int i = tid; i < 2 * (cols - NC) * 32; i += 256) {   // ones, then zeros
    const int r = i / 32 % (cols - NC), buf = i / 32 / (cols - NC);
    tw[buf * size + (32 + NC + r) * kLd + i % 32] = r == 0 ? (uint16_t)0x3f80 : (uint16_t)0;
  }
  // this thread's pieces of a stage: TASKS (ky, ci, octet) of the input, and
  // for threads 0..63 a pair of pixels of dz (K is a multiple of 32)
  const int kp = tid % 16, piece = tid / 16;
  u32x4 r0[TASKS], r1[TASKS], d0, d1;
  uint32_t before[TASKS];
  auto load = [&](int k0) {
    if (tid < 64) {
      const uint16_t* src = dz + (long)(k0 + 2 * kp) * 32 + 8 * piece;
      d0 = *reinterpret_cast<const u32x4*>(src);
      d1 = *reinterpret_cast<const u32x4*>(src + 32);
    }
#pragma unroll
    for (int t = 0; t < TASKS; ++t) {
      const int i = tid + 256 * t;
      r0[t] = r1[t] = u32x4{0, 0, 0, 0};
      before[t] = 0u;
      if (i >= 12 * J) continue;
      const int o = i & 3, q = i >> 2, ky = q / J, ci = q - ky * J;
      const int k = k0 + 8 * o;                             // eight pixels of one row
      const int ox = k % Wo, oy = (k / Wo) % Wo, b = k / (Wo * Wo);
      const int y = 2 * oy + ky - 1;
      if (y >= 0) {
        const uint16_t* src = x + (((long)b * J + ci) * N + y) * N + 2 * ox;
        r0[t] = *reinterpret_cast<const u32x4*>(src);
        r1[t] = *reinterpret_cast<const u32x4*>(src + 8);
        if (ox > 0) before[t] = src[-1];
      }
    }
  };
  auto store = [&](uint16_t* buf) {
    if (tid < 64) {
      uint32_t pr[8];
      pair8(d0, d1, pr);
#pragma unroll
      for (int e = 0; e < 8; ++e)
        *reinterpret_cast<uint32_t*>(buf + (8 * piece + e) * kLd + 2 * kp) = pr[e];
    }
#pragma unroll
    for (int t = 0; t < TASKS; ++t) {
      const int i = tid + 256 * t;
      if (i >= 12 * J) continue;
      const int o = i & 3, q = i >> 2, ky = q / J, ci = q - ky * J;
      u32x4 ev, od, pv;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const uint32_t lo = e < 2 ? r0[t][2 * e] : r1[t][2 * e - 4];
        const uint32_t hi = e < 2 ? r0[t][2 * e + 1] : r1[t][2 * e - 3];
        ev[e] = __builtin_amdgcn_perm(hi, lo, 0x05040100);
        od[e] = __builtin_amdgcn_perm(hi, lo, 0x07060302);
      }
      pv[0] = (od[0] << 16) | before[t];
#pragma unroll
      for (int e = 1; e < 4; ++e) pv[e] = (od[e] << 16) | (od[e - 1] >> 16);
      uint16_t* dst = buf + (32 + ky * 3 * J + ci) * kLd + 8 * o;
      *reinterpret_cast<u32x4*>(dst) = pv;
      *reinterpret_cast<u32x4*>(dst + J * kLd) = ev;
      *reinterpret_cast<u32x4*>(dst + 2 * J * kLd) = od;
    }
  };
  floatx4 acc[TILES][2];
#pragma unroll
  for (int t = 0; t < TILES; ++t) acc[t][0] = acc[t][1] = floatx4{0.f, 0.f, 0.f, 0.f};
  load(kb);
  store(tw);
  __syncthreads();
  for (int k0 = kb, st = 0; k0 < ke; k0 += 32, ++st) {
    uint16_t* buf = tw + (st & 1) * size;
    if (k0 + 32 < ke) load(k0 + 32);
    bf16x8 pf[2];
#pragma unroll
    for (int a = 0; a < 2; ++a)
      pf[a] = *reinterpret_cast<const bf16x8*>(buf + (16 * a + i16) * kLd + 8 * g);
#pragma unroll
    for (int t = 0; t < TILES; ++t) {
      const int c0 = 16 * (wave + 4 * t);
      if (c0 >= cols) break;
      const bf16x8 qf = *reinterpret_cast<const bf16x8*>(buf + (32 + c0 + i16) * kLd + 8 * g);
      acc[t][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pf[0], qf, acc[t][0], 0, 0, 0);
      acc[t][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pf[1], qf, acc[t][1], 0, 0, 0);
    }
    if (k0 + 32 < ke) store(tw + ((st & 1) ^ 1) * size);
    __syncthreads();
  }
  float* out = part + (long)blockIdx.x * 32 * (NC + 1);
#pragma unroll
  for (int t = 0; t < TILES; ++t) {
    const int j = 16 * (wave + 4 * t) + i16;
    if (j > NC) continue;
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int e = 0; e < 4; ++e) out[(long)(16 * a + 4 * g + e) * (NC + 1) + j] = acc[t][a][e];
  }
}

// Parameter gradients of every layer from their split sums: a block takes 256
// parameters, or, of a layer with many splits, 64 parameters x 4 quarters of
// the splits (each quarter added in order, then the quarters in order).  The
// last block sums the bursts' losses.
constexpr int kManySplits = 16;
__host__ __device__ inline int grad_sum_params(int splits) { return splits >= kManySplits ? 64 : 256; }
struct GradSum {
  long part;          // floats into the partial buffer
  long out;           // weights, then biases, in the gradient vector
  int M, N, splits;   // [splits][M][N + 1]
  int block0;         // first block of this layer
};
struct GradSums {
  GradSum l[6];
  int blocks;         // of all layers
};
__global__ __launch_bounds__(256) void k_grad_sum(GradSums gs, const float* __restrict__ part,
                                                  float* __restrict__ grad, int B,
                                                  const double* __restrict__ loss_b,
                                                  double* __restrict__ loss) {
  __shared__ double red[256];
  const int tid = threadIdx.x;
  if ((int)blockIdx.x == gs.blocks) {
    double s = 0.0;
    for (int b = tid; b < B; b += 256) s += loss_b[b];
    red[tid] = s;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
      if (tid < h) red[tid] += red[tid + h];
      __syncthreads();
    }
    if (tid == 0) *loss = red[0];
    return;
  }
  int li = 0;
  while (li < 5 && (int)blockIdx.x >= gs.l[li + 1].block0) ++li;
  const GradSum L = gs.l[li];
  const int wide = grad_sum_params(L.splits), n1 = L.N + 1;
  const int e = tid % wide, quarter = tid / wide;
  const long total = (long)L.M * n1, i = (long)(blockIdx.x - L.block0) * wide + e;
  const int per = wide == 64 ? (L.splits + 3) / 4 : L.splits;
  float s = 0.f;
  if (i < total) {
    const float* src = part + L.part + i;
#pragma unroll 8
    for (int z = quarter * per; z < min(L.splits, (quarter + 1) * per); ++z) s += src[(long)z * total];
  }
  float* rf = reinterpret_cast<float*>(red);
  rf[tid] = s;
  __syncthreads();
  if (tid < wide && i < total) {
    const float v = wide == 64 ? ((rf[e] + rf[64 + e]) + rf[128 + e]) + rf[192 + e] : s;
    const int m = (int)(i / n1), n = (int)(i % n1);
    grad[L.out + (n < L.N ? (long)m * L.N + n : (long)L.M * L.N + m)] = v;
  }
}

}  // namespace conv
}  // namespace mfbd
