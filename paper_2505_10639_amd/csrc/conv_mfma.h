// Kernels of the warm-start network's layers on the matrix cores (gfx950):
// 3x3 stride-2 convolutions as implicit GEMMs (no im2col in memory) and the
// dense layers, BF16 operands with FP32 accumulation.
//
// Operand layout of v_mfma_f32_16x16x16_bf16: lane l (i = l % 16, g = l / 16)
// supplies A[i][4g + 0..3] and B[4g + 0..3][i] and receives D[4g + e][i],
// e = 0..3.  The weights are the A operand and the pixels (or bursts) the B
// operand, so a lane ends with four consecutive output channels of one pixel:
// one 8-byte store.
//
// Order of every sum: the k range of an output is cut into chunks of `kchunk`
// (a multiple of 32, fixed by the layer's sizes: split_chunk in cnn.hip); a
// chunk is one chain of matrix instructions in k order from zero, and the
// chunks are added in order.  Whatever the tiling, an output has the same bits.
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
// start and the latency of its 9 to 18 stages; BM and BN are the smallest
// tiles that lost nothing, to give every CU blocks at small batches too.  With
// im2col and partial products in memory the same layers took 55 to 100 us.
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
// through a table of offsets.  Read once from memory: 128 B a row and frame.
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


}  // namespace conv
}  // namespace mfbd
