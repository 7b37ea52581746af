// Warm-start network: a convolutional regressor from a burst of frames to
// per-frame modal coefficients, trained and run on the matrix cores
// (BF16 operands, FP32 accumulation: v_mfma_f32_16x16x16_bf16).
//
// Architecture (input: J frames of N x N, N = 64, 96 or 128, NHWC with the
// frames as channels):
//   conv 3x3 stride 2 pad 1, J -> 32, ReLU        N -> N/2
//   conv 3x3 stride 2 pad 1, 32 -> 64, ReLU       N/2 -> N/4
//   conv 3x3 stride 2 pad 1, 64 -> 128, ReLU      N/4 -> N/8
//   conv 3x3 stride 2 pad 1, 128 -> 128, ReLU     N/8 -> N/16
//   dense 128 (N/16)^2 -> 512, ReLU               (2048 at N = 64)
//   dense 512 -> J*M (linear), times the per-mode scale
// Convolutions are implicit GEMMs (conv_mfma.h): no columns and no products
// of a layer cross memory but its activations, their gradients and the split
// sums of its parameter gradients.  Weights and activations are stored in bfloat16, biases, master
// weights, gradients and Adam moments in FP32.  Every reduction runs in a
// fixed order, so results are bitwise reproducible.
//
// Loss (per frame): the burst mean of the tilt modes is removed from
// prediction and target, and the squared error is the smaller of those to
// the target and to the target with its even-radial-order modes negated,
// the two symmetries that leave the frames unchanged without diversity.
// Mode m's error is weighted by scale_m^2 / mean(scale^2): the loss is the
// wavefront error in units of the mean mode variance.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <new>
#include <vector>

#include "conv_mfma.h"
#include "internal.h"
#include "momfbd.h"

namespace mfbd {
namespace {

__global__ __launch_bounds__(256) void k_cast_bf16(long n, const float* __restrict__ x,
                                                   uint16_t* __restrict__ y) {
  const long i = (long)blockIdx.x * 256 + threadIdx.x;
  if (i < n) y[i] = f2bf(x[i]);
}

// frames [B*J][npix] FP32 -> the network's input, one bfloat16 plane per
// frame: 10 (f / mean - 1); one block per frame (k_netin64 does the same from
// the spectra at 64 x 64).  WIDE: those values as momfbd_cnn_input returns them,
// [B][npix][J] floats.
template <bool WIDE>
__global__ __launch_bounds__(256) void k_norm_frames(int npix, int J, const float* __restrict__ f,
                                                     uint16_t* __restrict__ x,
                                                     float* __restrict__ wide) {
  __shared__ float red[256];
  const int u = blockIdx.x, tid = threadIdx.x;
  const float* fu = f + (long)u * npix;
  float s = 0.f;
  for (int i = tid; i < npix; i += 256) s += fu[i];
  red[tid] = s;
  __syncthreads();
  for (int h = 128; h > 0; h >>= 1) {
    if (tid < h) red[tid] += red[tid + h];
    __syncthreads();
  }
  const float inv = (float)npix / red[0];
  for (int i = tid; i < npix; i += 256) {
    const uint16_t h = f2bf(10.f * (fu[i] * inv - 1.f));
    if (WIDE)
      wide[((long)(u / J) * npix + i) * J + u % J] = bf2f(h);
    else
      x[(long)u * npix + i] = h;
  }
}

// the network's input as momfbd_cnn_input returns it: [B][npix][J] floats
__global__ __launch_bounds__(256) void k_widen_input(long n, int J, int npix,
                                                     const uint16_t* __restrict__ x,
                                                     float* __restrict__ out) {
  const long i = (long)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const long r = i / J, b = r / npix;
  out[i] = bf2f(x[(b * J + i % J) * npix + r % npix]);
}

constexpr int kMaxJM = 2048;

// Per burst: loss and dL/dz (as the bfloat16 the backward pass reads).
// One block per burst; thread t handles (j, m) = (t / M, t % M) for
// t = tid, tid + 1024.
__global__ __launch_bounds__(1024) void k_burst_loss(int B, int J, int M,
                                                     const float* __restrict__ z,
                                                     const float* __restrict__ target,
                                                     const float* __restrict__ scale,
                                                     const float* __restrict__ weight,
                                                     const int* __restrict__ even,
                                                     double* __restrict__ loss_b,
                                                     uint16_t* __restrict__ dz) {
  __shared__ float p[kMaxJM], q[kMaxJM], d1[kMaxJM], d2[kMaxJM], g[kMaxJM];
  __shared__ float e1[64], e2[64];
  __shared__ float tm[4];
  const int b = blockIdx.x, tid = threadIdx.x, JM = J * M;
  // work in units of the per-mode scale (the network's own output units)
  for (int t = tid; t < JM; t += 1024) {
    p[t] = z[(long)b * JM + t];
    q[t] = target[(long)b * JM + t] / scale[t % M];
  }
  __syncthreads();
  if (tid < 4) {           // burst means of the two tilt modes
    const int mm = tid & 1;
    const float* src = tid < 2 ? p : q;
    float s = 0.f;
    for (int jj = 0; jj < J; ++jj) s += src[jj * M + mm];
    tm[tid] = s / J;
  }
  __syncthreads();
  // tilt-centred values replace p and q (each element is read and written by
  // its own thread only)
  for (int t = tid; t < JM; t += 1024) {
    const int m = t % M;
    const float pv = p[t] - (m < 2 ? tm[m] : 0.f);
    const float qv = q[t] - (m < 2 ? tm[2 + m] : 0.f);
    const float sg = even[m] ? -1.f : 1.f;
    d1[t] = weight[m] * (pv - qv) * (pv - qv);
    d2[t] = weight[m] * (pv - sg * qv) * (pv - sg * qv);
    p[t] = pv;
    q[t] = qv;
  }
  __syncthreads();
  if (tid < J) {
    float a = 0.f, c = 0.f;
    for (int mm = 0; mm < M; ++mm) {
      a += d1[tid * M + mm];
      c += d2[tid * M + mm];
    }
    e1[tid] = a;
    e2[tid] = c;
  }
  __syncthreads();
  const float inv = 1.f / ((float)B * J);
  for (int t = tid; t < JM; t += 1024) {
    const int j = t / M, m = t % M;
    const float sg = even[m] ? -1.f : 1.f;
    const bool flip = e2[j] < e1[j];
    g[t] = 2.f * weight[m] * (p[t] - (flip ? sg * q[t] : q[t])) * inv;
  }
  __syncthreads();
  for (int t = tid; t < JM; t += 1024) {
    const int m = t % M;
    float gv = g[t];
    if (m < 2) {
      float s = 0.f;
      for (int jj = 0; jj < J; ++jj) s += g[jj * M + m];
      gv -= s / J;
    }
    dz[(long)b * JM + t] = f2bf(gv);
  }
  if (tid == 0) {
    double s = 0.0;
    for (int jj = 0; jj < J; ++jj) s += (double)fminf(e1[jj], e2[jj]);
    loss_b[b] = s * (double)inv;
  }
}

__global__ __launch_bounds__(256) void k_adam(long n, float* __restrict__ w,
                                              const float* __restrict__ g, float* __restrict__ m1,
                                              float* __restrict__ m2, uint16_t* __restrict__ w16,
                                              float lr, float b1, float b2, float eps, float c1,
                                              float c2) {
  const long i = (long)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const float gi = g[i];
  const float a = b1 * m1[i] + (1.f - b1) * gi;
  const float v = b2 * m2[i] + (1.f - b2) * gi * gi;
  m1[i] = a;
  m2[i] = v;
  const float wi = w[i] - lr * (a / c1) / (sqrtf(v / c2) + eps);
  w[i] = wi;
  if (w16) w16[i] = f2bf(wi);
}

// scaled normals -> parameters: He initialisation of the weights, zero biases
__global__ __launch_bounds__(256) void k_init(long n, const float* __restrict__ normals,
                                              const float* __restrict__ std_of,
                                              float* __restrict__ w) {
  const long i = (long)blockIdx.x * 256 + threadIdx.x;
  if (i < n) w[i] = normals[i] * std_of[i];
}

unsigned blocks(long n) { return (unsigned)((n + 255) / 256); }

}  // namespace
}  // namespace mfbd

using namespace mfbd;

struct Layer {
  bool conv;
  int ci, co, h;         // conv: input channels, output channels, input side
  int n_in, n_out;       // dense
  long w_off, b_off;     // offsets into the flat parameter vector
  long rows;             // GEMM rows per burst (output pixels) and K
  int K;
};

struct momfbd_cnn_s {
  int N, J, M, batch_max;
  long n_params;
  std::vector<Layer> layers;
  float* scale = nullptr;     // [M] device
  float* weight = nullptr;    // [M] device: scale^2 / mean(scale^2)
  int* even = nullptr;        // [M] device
  float* init_std = nullptr;  // [n_params] device
  size_t ws_bytes = 0;
  // workspace offsets (bytes)
  size_t o_frames, o_x0, o_y[5], o_z, o_part, o_dz, o_dz2, o_w16, o_lossb;
  size_t part_floats;   // enters split_chunk
  int device = -1;
};

namespace {

size_t al256(size_t x) { return (x + 255) & ~size_t(255); }

// Chunk of the k range summed as one chain (a multiple of 32): as many splits
// of K as keep 64 x 64 tiles of the output near 2048 blocks and their partial
// products within part_floats (no such buffer exists: the rule is kept for the
// bits).  It fixes the order of every sum of a layer, whichever kernel forms it;
// M is the batch times the layer's rows and part_floats grows with batch_max, so
// the order, and with it an output's last bits, may change with either.
int split_chunk(const momfbd_cnn_s* n, int M, int N, int K) {
  const int tm = (M + 63) / 64, tn = (N + 63) / 64;
  const int kc32 = (K + 31) / 32;
  int splits = 1;
  while (splits * 2 <= kc32 && (long)tm * tn * splits * 2 <= 2048 && splits < 256) splits *= 2;
  while ((long)splits * M * N > (long)n->part_floats && splits > 1) splits /= 2;
  return ((kc32 + splits - 1) / splits) * 32;
}

// the network's input from the bursts' first channel: the apodized patches
// W(x - m) + m = IDFT(D) / N^2 of D [B][C][J][N][N/2+1], channel 0, each
// normalised, one bfloat16 plane per frame
hipError_t input_from_spectra(const momfbd_cnn_s* n, int B, int C, const void* D, char* ws,
                              hipStream_t s, float* wide = nullptr) {
  const float2* d = static_cast<const float2*>(D);
  uint16_t* x0 = reinterpret_cast<uint16_t*>(ws + n->o_x0);
  if (n->N == 64) return launch_netin64(B * n->J, n->J, C * n->J, d, x0, s);
  float* frames = reinterpret_cast<float*>(ws + n->o_frames);
  const hipError_t e = launch_frames(n->N, B * n->J, n->J, C * n->J, d, frames, s);
  if (e != hipSuccess) return e;
  auto* kernel = wide ? &k_norm_frames<true> : &k_norm_frames<false>;
  hipLaunchKernelGGL(kernel, dim3(B * n->J), dim3(256), 0, s, n->N * n->N, n->J, frames, x0, wide);
  return hipGetLastError();
}

// Frames up to which momfbd_cnn_input writes its floats from the normalisation
// itself at 96 x 96 and 128 x 128; with more, stores J floats apart cost more than
// the launch that gathers whole pixels (128 x 128, 64 bursts: 2 frames 40 us
// against 45, 5 frames 72 against 65, 24 frames 376 against 159).
constexpr int kDirectInputFrames = 4;

hipError_t run_conv1(const momfbd_cnn_s* n, int B, const uint16_t* x, const uint16_t* w,
                     const float* bias, uint16_t* y, hipStream_t s) {
  const Layer& L = n->layers[0];
  const int kchunk = split_chunk(n, (int)(B * L.rows), L.co, L.K);
  const size_t lds = conv::conv1_lds(n->N, n->J);
  const dim3 grid(B * (n->N / 2 / conv::net_rows(n->N)));
  auto* kernel = n->J % 4 == 0 ? &conv::k_conv1<true> : &conv::k_conv1<false>;
  if (lds > 65536) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(kernel, grid, dim3(256), lds, s, n->N, n->J, kchunk, x, w, bias, y);
  return hipGetLastError();
}

template <int CI, int CO, int BM, int BN, int WM, int BK>
hipError_t run_conv(const momfbd_cnn_s* n, const Layer& L, int B, const uint16_t* x,
                    const uint16_t* w, const float* bias, uint16_t* y, hipStream_t s) {
  const int M = (int)(B * L.rows);
  hipLaunchKernelGGL((conv::k_conv<CI, CO, BM, BN, WM, BK>), dim3((M + BM - 1) / BM, CO / BN),
                     dim3(256), 0, s, M, L.h, split_chunk(n, M, CO, L.K), x, w, bias, y);
  return hipGetLastError();
}

hipError_t run_dense(const momfbd_cnn_s* n, const Layer& L, int B, const uint16_t* x,
                     const uint16_t* w, const float* bias, uint16_t* out16, float* out32,
                     const float* scale, hipStream_t s) {
  hipLaunchKernelGGL(conv::k_dense, dim3((L.n_out + 15) / 16, (B + 15) / 16), dim3(256), 0, s, B,
                     L.n_out, L.n_in, split_chunk(n, B, L.n_out, L.n_in), x, w, bias, out16, out32,
                     scale, n->M);
  return hipGetLastError();
}

// Activations of every layer, and the last layer's output z into `out32`,
// times the mode scale where `scale` is given.
hipError_t run_forward(const momfbd_cnn_s* n, const float* params, const void* D, int B, int C,
                       char* ws, float* out32, const float* scale, hipStream_t s) {
  hipError_t e = input_from_spectra(n, B, C, D, ws, s);
  const uint16_t* w16 = reinterpret_cast<const uint16_t*>(ws + n->o_w16);
  const uint16_t* h = reinterpret_cast<const uint16_t*>(ws + n->o_x0);
  for (int l = 0; l < 6 && e == hipSuccess; ++l) {
    const Layer& L = n->layers[l];
    const uint16_t* w = w16 + L.w_off;
    const float* bias = params + L.b_off;
    uint16_t* y = l < 5 ? reinterpret_cast<uint16_t*>(ws + n->o_y[l]) : nullptr;
    switch (l) {
      case 0: e = run_conv1(n, B, h, w, bias, y, s); break;
      case 1: e = run_conv<32, 64, 64, 64, 4, 32>(n, L, B, h, w, bias, y, s); break;
      case 2: e = run_conv<64, 128, 32, 64, 2, 64>(n, L, B, h, w, bias, y, s); break;
      case 3: e = run_conv<128, 128, 32, 32, 2, 64>(n, L, B, h, w, bias, y, s); break;
      case 4: e = run_dense(n, L, B, h, w, bias, y, nullptr, nullptr, s); break;
      default: e = run_dense(n, L, B, h, w, bias, nullptr, out32, scale, s); break;
    }
    h = y;
  }
  return e;
}

// The rows (pixels or bursts) of one split of a layer's parameter gradients,
// a multiple of 32, and the splits: enough blocks of 64 x 64 sums for four on
// every CU, but at least four stages of 32 rows in each (256 bursts of 64 x 64:
// the convolutions' 62 us with two a CU, 53 with four, k_grad_sum 10.6 and
// 14.2; the pass 276 and 272).  The first layer's
// blocks hold all its sums, at least 16 stages each: 512 blocks at 256 bursts
// of 64 x 64, whose partial sums are 7 MB.
struct WgradSplit {
  int rows, splits;
};
// the most splits of a layer's K rows; never fewer for a larger K
int wgrad_max_splits(const Layer& L, int l, long K) {
  const long stages = (K + 31) / 32;
  const int Mo = L.conv ? L.co : L.n_out, tiles = (L.K + 64) / 64 * ((Mo + 63) / 64);
  const long splits =
      l == 0 ? (stages + 15) / 16 : std::min((stages + 3) / 4, std::max(1L, 1024L / tiles));
  return (int)std::max(1L, std::min(splits, 512L));
}
WgradSplit wgrad_split(const Layer& L, int l, int K) {
  const int stages = (K + 31) / 32, splits = wgrad_max_splits(L, l, K);
  const int rows = (stages + splits - 1) / splits * 32;
  return WgradSplit{rows, (K + rows - 1) / rows};
}

// floats that hold every layer's split sums at any batch up to `batch_max`
long wgrad_floats(const std::vector<Layer>& layers, int batch_max) {
  long n = 0;
  for (size_t l = 0; l < layers.size(); ++l) {
    const Layer& L = layers[l];
    n += (long)wgrad_max_splits(L, (int)l, batch_max * L.rows) * (L.conv ? L.co : L.n_out) *
         (L.K + 1);
  }
  return n;
}

hipError_t run_wgrad1(const momfbd_cnn_s* n, int K, const WgradSplit& sp, const uint16_t* dz,
                      const uint16_t* x, float* part, hipStream_t s) {
  const size_t lds = conv::wgrad1_lds(n->J);
  const int tiles = (conv::wgrad1_cols(n->J) / 16 + 3) / 4;
  // tiles a wave and pieces a thread holds in registers: up to 14, 28 and 64 frames
  auto* kernel = tiles <= 2 ? &conv::k_wgrad1<2, 1> : tiles <= 4 ? &conv::k_wgrad1<4, 2>
                                                                : &conv::k_wgrad1<10, 3>;
  if (lds > 65536) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(kernel, dim3(sp.splits), dim3(256), lds, s, n->N, n->J, K, sp.rows, dz, x, part);
  return hipGetLastError();
}

template <int CI, int CO, int BM, int BN>
hipError_t run_conv_dx(const momfbd_cnn_s* n, const Layer& L, int B, const uint16_t* dz,
                       const uint16_t* w, const uint16_t* h, uint16_t* dx, hipStream_t s) {
  const int M = (int)(B * L.rows);
  hipLaunchKernelGGL((conv::k_conv_dx<CI, CO, BM, BN>), dim3((M + BM - 1) / BM, CI / BN, 4),
                     dim3(256), 0, s, M, L.h / 2, split_chunk(n, M, L.K, CO), dz, w, h, dx);
  return hipGetLastError();
}

// A network and a workspace that is 256-byte aligned and at least
// momfbd_cnn_sizes' workspace_bytes long.
int check_ws(const momfbd_cnn_s* n, const void* ws, size_t ws_bytes) {
  if (!n) return MOMFBD_EINVAL;
  if (!ws || reinterpret_cast<uintptr_t>(ws) % 256 || ws_bytes < n->ws_bytes)
    return MOMFBD_EWORKSPACE;
  return MOMFBD_OK;
}

int check_net(const momfbd_cnn_s* n, const void* ws, size_t ws_bytes, int B) {
  const int st = check_ws(n, ws, ws_bytes);
  if (st) return st;
  if (B < 1 || B > n->batch_max) return MOMFBD_EINVAL;
  return MOMFBD_OK;
}

int status_of(hipError_t e) { return e == hipSuccess ? MOMFBD_OK : MOMFBD_EDEVICE; }

}  // namespace

extern "C" {

int momfbd_cnn_create(int N, int J, int M, int batch_max, const float* mode_scale,
                      momfbd_cnn* out) {
  if (!out || !mode_scale || J < 1 || M < 2 || batch_max < 1 || (long)J * M > kMaxJM ||
      J > 64)
    return MOMFBD_EINVAL;
  if (N != 64 && N != 96 && N != 128) return MOMFBD_EUNSUPPORTED;
  for (int m = 0; m < M; ++m)
    if (!(mode_scale[m] > 0.f) || !std::isfinite(mode_scale[m])) return MOMFBD_EINVAL;
  momfbd_cnn_s* n = new (std::nothrow) momfbd_cnn_s();
  if (!n) return MOMFBD_EDEVICE;
  n->N = N;
  n->J = J;
  n->M = M;
  n->batch_max = batch_max;
  const int chans[5] = {J, 32, 64, 128, 128};
  long off = 0;
  int side = N;
  for (int l = 0; l < 4; ++l) {
    Layer L{};
    L.conv = true;
    L.ci = chans[l];
    L.co = chans[l + 1];
    L.h = side;
    L.K = 9 * L.ci;
    L.rows = (long)(side / 2) * (side / 2);
    L.w_off = off;
    off += (long)L.co * L.K;
    L.b_off = off;
    off += L.co;
    n->layers.push_back(L);
    side /= 2;
  }
  const int dense_in[2] = {128 * side * side, 512}, dense_out[2] = {512, J * M};
  for (int l = 0; l < 2; ++l) {
    Layer L{};
    L.conv = false;
    L.n_in = dense_in[l];
    L.n_out = dense_out[l];
    L.K = L.n_in;
    L.rows = 1;
    L.w_off = off;
    off += (long)L.n_out * L.n_in;
    L.b_off = off;
    off += L.n_out;
    n->layers.push_back(L);
  }
  n->n_params = off;
  // workspace
  const long Bm = batch_max;
  size_t o = 0;
  n->o_frames = o;
  if (N != 64) o = al256(o + (size_t)Bm * J * N * N * sizeof(float));
  n->o_x0 = o;
  o = al256(o + (size_t)Bm * J * N * N * sizeof(uint16_t));
  size_t max_dz = (size_t)Bm * std::max(J * M, 512);   // gradients of a layer's activations
  for (int l = 0; l < 4; ++l) {
    const Layer& L = n->layers[l];
    n->o_y[l] = o;
    o = al256(o + (size_t)Bm * L.rows * L.co * sizeof(uint16_t));
    max_dz = std::max(max_dz, (size_t)Bm * L.rows * L.co);
  }
  n->o_y[4] = o;
  o = al256(o + (size_t)Bm * 512 * sizeof(uint16_t));
  n->o_z = o;
  o = al256(o + (size_t)Bm * J * M * sizeof(float));
  // the largest layer's products times a few splits
  size_t part = 0;
  for (const Layer& L : n->layers) {
    part = std::max(part, (size_t)Bm * L.rows * (L.conv ? L.co : L.n_out));
    part = std::max(part, (size_t)(L.conv ? L.co : L.n_out) * L.K * 64);
    part = std::max(part, (size_t)Bm * L.rows * L.K);
  }
  n->part_floats = part;
  // split sums of the parameter gradients
  n->o_part = o;
  o = al256(o + (size_t)wgrad_floats(n->layers, batch_max) * sizeof(float));
  n->o_dz = o;
  o = al256(o + max_dz * sizeof(uint16_t));
  n->o_dz2 = o;
  o = al256(o + max_dz * sizeof(uint16_t));
  n->o_w16 = o;
  o = al256(o + (size_t)n->n_params * sizeof(uint16_t));
  n->o_lossb = o;
  o = al256(o + (size_t)Bm * sizeof(double));
  n->ws_bytes = o;
  // tables
  std::vector<int> even(M);
  for (int m = 0; m < M; ++m) {
    const int j = m + 2;
    int r = 0;
    while ((r + 1) * (r + 2) / 2 < j) ++r;
    even[m] = (r % 2 == 0) ? 1 : 0;
  }
  std::vector<float> stdv(n->n_params, 0.f);
  for (const Layer& L : n->layers) {
    const float sd = std::sqrt(2.0f / (float)L.K);
    const long nw = L.conv ? (long)L.co * L.K : (long)L.n_out * L.n_in;
    for (long i = 0; i < nw; ++i) stdv[L.w_off + i] = sd;
  }
  // the last layer starts small: the first predictions are near zero
  const Layer& Ll = n->layers.back();
  for (long i = 0; i < (long)Ll.n_out * Ll.n_in; ++i) stdv[Ll.w_off + i] *= 0.1f;
  std::vector<float> wt(M);
  double mean2 = 0.0;
  for (int m = 0; m < M; ++m) mean2 += (double)mode_scale[m] * mode_scale[m] / M;
  for (int m = 0; m < M; ++m) wt[m] = (float)((double)mode_scale[m] * mode_scale[m] / mean2);
  bool ok = hipGetDevice(&n->device) == hipSuccess &&
            hipMalloc(&n->scale, M * sizeof(float)) == hipSuccess &&
            hipMalloc(&n->weight, M * sizeof(float)) == hipSuccess &&
            hipMemcpy(n->weight, wt.data(), M * sizeof(float), hipMemcpyHostToDevice) ==
                hipSuccess &&
            hipMalloc(&n->even, M * sizeof(int)) == hipSuccess &&
            hipMalloc(&n->init_std, n->n_params * sizeof(float)) == hipSuccess &&
            hipMemcpy(n->scale, mode_scale, M * sizeof(float), hipMemcpyHostToDevice) == hipSuccess &&
            hipMemcpy(n->even, even.data(), M * sizeof(int), hipMemcpyHostToDevice) == hipSuccess &&
            hipMemcpy(n->init_std, stdv.data(), n->n_params * sizeof(float),
                      hipMemcpyHostToDevice) == hipSuccess;
  if (!ok) {
    momfbd_cnn_destroy(n);
    return MOMFBD_EDEVICE;
  }
  *out = n;
  return MOMFBD_OK;
}

int momfbd_cnn_destroy(momfbd_cnn net) {
  if (!net) return MOMFBD_OK;
  if (net->scale) (void)hipFree(net->scale);
  if (net->weight) (void)hipFree(net->weight);
  if (net->even) (void)hipFree(net->even);
  if (net->init_std) (void)hipFree(net->init_std);
  delete net;
  return MOMFBD_OK;
}

int momfbd_cnn_sizes(momfbd_cnn net, size_t* n_params, size_t* workspace_bytes) {
  if (!net) return MOMFBD_EINVAL;
  if (n_params) *n_params = (size_t)net->n_params;
  if (workspace_bytes) *workspace_bytes = net->ws_bytes;
  return MOMFBD_OK;
}

int momfbd_cnn_init(momfbd_cnn net, const float* normals, float* params, void* ws,
                    size_t ws_bytes, void* stream) {
  const int st = check_ws(net, ws, ws_bytes);
  if (st) return st;
  if (!normals || !params) return MOMFBD_EINVAL;
  hipStream_t s = (hipStream_t)stream;
  hipLaunchKernelGGL(k_init, dim3(blocks(net->n_params)), dim3(256), 0, s, net->n_params, normals,
                     net->init_std, params);
  hipLaunchKernelGGL(k_cast_bf16, dim3(blocks(net->n_params)), dim3(256), 0, s, net->n_params,
                     params, reinterpret_cast<uint16_t*>(static_cast<char*>(ws) + net->o_w16));
  return status_of(hipGetLastError());
}

int momfbd_cnn_load(momfbd_cnn net, const float* params, void* ws, size_t ws_bytes,
                    void* stream) {
  const int st = check_ws(net, ws, ws_bytes);
  if (st) return st;
  if (!params) return MOMFBD_EINVAL;
  hipLaunchKernelGGL(k_cast_bf16, dim3(blocks(net->n_params)), dim3(256), 0, (hipStream_t)stream,
                     net->n_params, params,
                     reinterpret_cast<uint16_t*>(static_cast<char*>(ws) + net->o_w16));
  return status_of(hipGetLastError());
}

int momfbd_cnn_forward(momfbd_cnn net, const float* params, const void* D, int B, int C,
                       float* alpha, void* ws, size_t ws_bytes, void* stream) {
  int st = check_net(net, ws, ws_bytes, B);
  if (st) return st;
  if (!params || !D || !alpha || C < 1) return MOMFBD_EINVAL;
  hipStream_t s = (hipStream_t)stream;
  char* w = static_cast<char*>(ws);
  return status_of(run_forward(net, params, D, B, C, w, alpha, net->scale, s));
}

int momfbd_cnn_input(momfbd_cnn net, const void* D, int B, int C, float* x, void* ws,
                     size_t ws_bytes, void* stream) {
  int st = check_net(net, ws, ws_bytes, B);
  if (st) return st;
  if (!D || !x || C < 1) return MOMFBD_EINVAL;
  hipStream_t s = (hipStream_t)stream;
  char* w = static_cast<char*>(ws);
  const bool direct = net->N != 64 && net->J <= kDirectInputFrames;
  const hipError_t e = input_from_spectra(net, B, C, D, w, s, direct ? x : nullptr);
  if (e != hipSuccess) return MOMFBD_EDEVICE;
  if (direct) return MOMFBD_OK;
  const int npix = net->N * net->N;
  const long n = (long)B * npix * net->J;
  hipLaunchKernelGGL(k_widen_input, dim3(blocks(n)), dim3(256), 0, s, n, net->J, npix,
                     reinterpret_cast<const uint16_t*>(w + net->o_x0), x);
  return status_of(hipGetLastError());
}

int momfbd_cnn_loss_grad(momfbd_cnn net, const float* params, const void* D, int C,
                         const float* target, int B, double* loss, float* grad, void* ws,
                         size_t ws_bytes, void* stream) {
  int st = check_net(net, ws, ws_bytes, B);
  if (st) return st;
  if (!params || !D || !target || !loss || !grad || C < 1) return MOMFBD_EINVAL;
  hipStream_t s = (hipStream_t)stream;
  char* w = static_cast<char*>(ws);
  hipError_t e = run_forward(net, params, D, B, C, w, reinterpret_cast<float*>(w + net->o_z), nullptr, s);
  if (e != hipSuccess) return MOMFBD_EDEVICE;
  uint16_t* dz = reinterpret_cast<uint16_t*>(w + net->o_dz);
  uint16_t* dx = reinterpret_cast<uint16_t*>(w + net->o_dz2);
  const uint16_t* w16 = reinterpret_cast<const uint16_t*>(w + net->o_w16);
  float* part = reinterpret_cast<float*>(w + net->o_part);
  double* lb = reinterpret_cast<double*>(w + net->o_lossb);
  hipLaunchKernelGGL(k_burst_loss, dim3(B), dim3(1024), 0, s, B, net->J, net->M,
                     reinterpret_cast<const float*>(w + net->o_z), target, net->scale,
                     net->weight, net->even, lb, dz);
  conv::GradSums gs{};
  long used = 0;
  for (int l = 5; l >= 0 && e == hipSuccess; --l) {
    const Layer& L = net->layers[l];
    // input activation of this layer (bfloat16)
    const uint16_t* hin = reinterpret_cast<const uint16_t*>(w + (l == 0 ? net->o_x0 : net->o_y[l - 1]));
    const uint16_t* wl = w16 + L.w_off;
    const int Mo = L.conv ? L.co : L.n_out, K = (int)(B * L.rows);
    const WgradSplit ws_l = wgrad_split(L, l, K);
    gs.l[l] = conv::GradSum{used, L.w_off, Mo, L.K, ws_l.splits, 0};
    float* pl = part + used;
    used += (long)ws_l.splits * Mo * (L.K + 1);
    const dim3 grid((L.K + 64) / 64, (Mo + 63) / 64, ws_l.splits);
    switch (l) {
      case 0: e = run_wgrad1(net, K, ws_l, dz, hin, pl, s); break;
      case 1: hipLaunchKernelGGL(conv::k_wgrad<32>, grid, dim3(256), 0, s, Mo, L.K, K, ws_l.rows, L.h, dz, hin, pl); break;
      case 2: hipLaunchKernelGGL(conv::k_wgrad<64>, grid, dim3(256), 0, s, Mo, L.K, K, ws_l.rows, L.h, dz, hin, pl); break;
      case 3: hipLaunchKernelGGL(conv::k_wgrad<128>, grid, dim3(256), 0, s, Mo, L.K, K, ws_l.rows, L.h, dz, hin, pl); break;
      default: hipLaunchKernelGGL(conv::k_wgrad<0>, grid, dim3(256), 0, s, Mo, L.K, K, ws_l.rows, 0, dz, hin, pl); break;
    }
    switch (l) {
      case 0: break;
      case 1: e = run_conv_dx<32, 64, 64, 32>(net, L, B, dz, wl, hin, dx, s); break;
      case 2: e = run_conv_dx<64, 128, 64, 64>(net, L, B, dz, wl, hin, dx, s); break;
      case 3: e = run_conv_dx<128, 128, 64, 64>(net, L, B, dz, wl, hin, dx, s); break;
      default:
        hipLaunchKernelGGL(conv::k_dense_dx, dim3(L.n_in / 32, (B + 31) / 32), dim3(256), 0, s, B,
                           L.n_in, L.n_out, split_chunk(net, B, L.n_in, L.n_out), dz, wl, hin, dx);
        break;
    }
    std::swap(dz, dx);
  }
  if (e != hipSuccess) return MOMFBD_EDEVICE;
  for (int l = 0; l < 6; ++l) {
    gs.l[l].block0 = gs.blocks;
    const int per = conv::grad_sum_params(gs.l[l].splits);
    gs.blocks += (int)(((long)gs.l[l].M * (gs.l[l].N + 1) + per - 1) / per);
  }
  hipLaunchKernelGGL(conv::k_grad_sum, dim3(gs.blocks + 1), dim3(256), 0, s, gs, part, grad, B, lb,
                     loss);
  return status_of(hipGetLastError());
}

int momfbd_cnn_adam(momfbd_cnn net, float* params, const float* grad, float* m1, float* m2,
                    int step, float lr, float beta1, float beta2, float eps, void* ws,
                    size_t ws_bytes, void* stream) {
  const int st = check_ws(net, ws, ws_bytes);
  if (st) return st;
  if (!params || !grad || !m1 || !m2 || step < 1) return MOMFBD_EINVAL;
  const float c1 = 1.f - std::pow(beta1, (float)step), c2 = 1.f - std::pow(beta2, (float)step);
  hipLaunchKernelGGL(k_adam, dim3(blocks(net->n_params)), dim3(256), 0, (hipStream_t)stream,
                     net->n_params, params, grad, m1, m2,
                     reinterpret_cast<uint16_t*>(static_cast<char*>(ws) + net->o_w16), lr, beta1,
                     beta2, eps, c1, c2);
  return status_of(hipGetLastError());
}

}  // extern "C"
