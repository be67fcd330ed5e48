// Warm-start MLP training on the GPU with the library's own kernels.
//
// The network is the MLP of Eq. 3 with tanh hidden layers and an identity
// output, trained by minimising the mean squared error with Adam (the loss
// and optimiser the paper uses for its surrogate networks, Section 4.2).
// Every product is the same MFMA "NT" GEMM as the Hessian sweeps:
//   forward   A_l  = tanh(A_{l-1} W_l^T + b_l)        B operand W_l
//   dgrad     dA   = dZ_l W_l                         B operand W_l^T (copy)
//   wgrad     dW_l = dZ_l^T A_{l-1}                   both operands stored
//                                                     transposed (K = batch)
// with fused epilogues (bias + tanh + sigma', sigma' scaling, transposed
// copies for the next wgrad).  Master parameters and Adam moments are FP32;
// the GEMM copies of W and W^T are BF16 (or FP32).  All reductions are in a
// fixed order, so a step is deterministic.
//
// Networks whose products are all small (the warm-start network and anything
// with fewer than 128 tiles of 128 x 128 per product) take tr_mm_kernel and
// tr_wgrad_kernel below instead of the GEMM library: a step is then 2 L + 1
// launches.  Larger ones keep the LDS-tiled GEMMs, which read each operand
// from L2 a quarter as often, and separate bias-gradient and Adam launches.
#include <math.h>
#include <string.h>

#include <algorithm>
#include <random>
#include <string>
#include <vector>

#include "../../include/nnc.h"
#include "nnc_device.h"
#include "nnc_internal.h"

namespace nnc {

namespace {

inline int rup(int x, int a) { return (x + a - 1) / a * a; }

// One layer of the grouped weight-gradient launch.
struct TrLayer {
  const void *dZT, *AT;  // [dp_l][bp], [dp_{l-1}][bp]
  float *W, *m, *v, *dW;
  float *b, *mb, *vb, *db;
  void *Wc, *WTc;
  int rows, cols;  // dp_l, dp_{l-1}
  int tile0;       // first tile of the layer
};

// Most pinned host memory a trainer keeps.  Above it a copy's waits are a small
// part of its time.
constexpr size_t kStagingBytes = (size_t)32 << 20;

struct Trainer {
  bool small = false;         // tr_mm_kernel / tr_wgrad_kernel path
  TrLayer* dlayers = nullptr;  // device table of the grouped launch
  int wtiles = 0;
  int L = 0, batch = 0, bp = 0;
  DType ct = DT_BF16;
  size_t csz = 2;
  std::vector<int> d, dp;
  std::vector<float*> Wm, bm, mW, vW, mb, vb, dW, db;  // per layer (index l-1)
  std::vector<void*> Wc, WTc;
  std::vector<void*> A, AT;     // A[l] l = 0..L-1 (compute type), [bp][dp_l] and [dp_l][bp]
  std::vector<float*> D1;       // sigma' of hidden layers [bp][dp_l]
  std::vector<void*> dZ, dZT;   // per layer l = 1..L
  float* Yhat = nullptr;        // [bp][dp_L]
  double* partial = nullptr;    // loss partial sums
  double* lossd = nullptr;
  int npartial = 0;
  int step = 0;
  // pinned host copy of one set of parameters or gradients as laid out on the
  // device, for nnc_train_get_params / _get_grads (NULL: pageable copies, also
  // where it would be larger than kStagingBytes)
  float* staging = nullptr;
  std::vector<void*> allocs;
};

void* talloc(Trainer* t, size_t bytes) {
  void* p = nullptr;
  if (hipMalloc(&p, bytes ? bytes : 16) != hipSuccess) return nullptr;
  if (hipMemset(p, 0, bytes ? bytes : 16) != hipSuccess) {
    hipFree(p);
    return nullptr;
  }
  t->allocs.push_back(p);
  return p;
}

void free_trainer(Trainer* t) {
  if (!t) return;
  for (void* p : t->allocs) hipFree(p);
  if (t->staging) hipHostFree(t->staging);
  delete t;
}

// ---------------------------------------------------------------- kernels
// Input batch as GEMM operands, row-major and transposed, in 32 x 32 tiles
// through LDS so that both copies are written along their rows.
template <typename T>
__global__ void __launch_bounds__(256) tr_cast_input(const double* X, int rows, int d0, int bp, int dp0, T* A, T* AT) {
  __shared__ T tile[32][34];
  const int r0 = blockIdx.y * 32, c0 = blockIdx.x * 32;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
#pragma unroll
  for (int y = ty; y < 32; y += 8) {
    const int r = r0 + y, c = c0 + tx;
    const T v = from_d<T>(r < rows && c < d0 ? X[(long long)r * d0 + c] : 0.0);
    A[(long long)r * dp0 + c] = v;
    tile[y][tx] = v;
  }
  __syncthreads();
#pragma unroll
  for (int y = ty; y < 32; y += 8) AT[(long long)(c0 + y) * bp + r0 + tx] = tile[tx][y];
}

// dZ_L = 2 (Yhat - Y) / (batch * m) on the true region; per-block loss partials.
template <typename T>
__global__ void tr_mse_grad(const float* Yhat, const double* Y, int batch, int m, int bp, int dpL,
                            T* dZ, T* dZT, double* partial) {
  __shared__ double red[256];
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  double sq = 0.0;
  if (i < (long long)bp * dpL) {
    const int r = (int)(i / dpL);
    const int c = (int)(i % dpL);
    float g = 0.f;
    if (r < batch && c < m) {
      const double diff = (double)Yhat[i] - Y[(long long)r * m + c];
      sq = diff * diff;
      g = (float)(2.0 * diff / ((double)batch * m));
    }
    dZ[i] = from_f<T>(g);
    dZT[(long long)c * bp + r] = from_f<T>(g);
  }
  red[threadIdx.x] = sq;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) partial[blockIdx.x] = red[0];
}

// Sum of the loss partials by one workgroup: strided sums per thread, then a
// tree in LDS (one thread adding them in turn waited for each load: 51 us for
// the warm-start network's 832 partials).
__global__ void __launch_bounds__(256) tr_sum_partials(const double* partial, int n, double scale, double* out) {
  __shared__ double red[256];
  double s = 0.0;
  for (int i = threadIdx.x; i < n; i += 256) s += partial[i];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) *out = red[0] * scale;
}

// db[j] = sum_k dZT[j][k] in batch order, one thread per row, 16 bytes a load.
template <typename T>
__global__ void __launch_bounds__(64) tr_colsum(const T* dZT, int rows, int bp, float* db) {
  constexpr int V = 16 / (int)sizeof(T);
  const int j = blockIdx.x * 64 + threadIdx.x;
  if (j >= rows) return;
  float s = 0.f;
#pragma unroll 8
  for (int k = 0; k < bp; k += V) {
    float e[V];
    Vec16<T, float>::unpack(*(const uint4*)(dZT + (long long)j * bp + k), e);
#pragma unroll
    for (int q = 0; q < V; ++q) s += e[q];
  }
  db[j] = s;
}

struct AdamArgs {
  float lr, b1, b2, eps, c1, c2;
};

// The fused operations are written out: both kernels below round every step
// alike, whatever the compiler would contract in each.
__device__ __forceinline__ float adam_update(const AdamArgs& h, float g, float& m1, float& m2, float p) {
#pragma clang fp contract(off)
  m1 = fmaf(1.f - h.b1, g, h.b1 * m1);
  m2 = fmaf(g, (1.f - h.b2) * g, h.b2 * m2);
  return p - h.lr * (m1 / h.c1) / (sqrtf(m2 / h.c2) + h.eps);
}

// Adam on one parameter block; refreshes the GEMM copies (W and W^T) when
// `wc` is given.  rows x cols is the padded block shape.
template <typename T>
__global__ void tr_adam(float* p, float* m1, float* m2, const float* g, long long count, int cols, int rows,
                        AdamArgs h, T* wc, T* wtc) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= count) return;
  float a = m1[i], b = m2[i];
  const float np_ = adam_update(h, g[i], a, b, p[i]);
  m1[i] = a;
  m2[i] = b;
  p[i] = np_;
  if (wc) {
    const int r = (int)(i / cols);
    const int c = (int)(i % cols);
    wc[i] = from_f<T>(np_);
    wtc[(long long)c * rows + r] = from_f<T>(np_);
  }
}

// ---------------------------------------------------------------- small products
// C[r][c] = sum_k R[r][k] C[c][k] of a training step: 32 x 32 outputs per
// workgroup, one 16 x 16 block per wave, whose operand fragments go straight
// from L2 into registers (the next 8 K steps' on the way while these are
// multiplied); no LDS and no barrier stands between load and MFMA.  These
// products are a few dozen K steps of operands that fit L2, so what counts is
// how long the chain of loads is and how many CUs take part: the 64 x 64 LDS
// tiles put 256 x 512 x 832 on 32 CUs in 13 dependent rounds.  One wave runs
// the whole of K in order, as the LDS tiles do, so both give the same bits (a
// BF16 step that rounds one sum the other way moves the parameters after an
// epoch by 2e-4).  The lane's results are columns 4 (l / 16) .. + 3 of row
// l % 16.
// 256 x 512 x 832 in BF16: 10.1 -> 8.3 us; a step of the warm-start network
// 20 launches and 264 us of kernels -> 7 launches and 65 us.
template <typename T> struct TrMma;
template <> struct TrMma<bf16> {
  static constexpr int VEC = 8;
  __device__ __forceinline__ static void mma(floatx4& c, const uint4& a, const uint4& b) {
    c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0,
                                                0);
  }
};
template <> struct TrMma<float> {
  static constexpr int VEC = 4;
  __device__ __forceinline__ static void mma(floatx4& c, const uint4& a, const uint4& b) {
    float x[4], y[4];
    Vec16<float, float>::unpack(a, x);
    Vec16<float, float>::unpack(b, y);
#pragma unroll
    for (int e = 0; e < 4; ++e) c = __builtin_amdgcn_mfma_f32_16x16x4f32(x[e], y[e], c, 0, 0, 0);
  }
};

// C, R: this wave's 16 operand rows of the columns and of the rows, K a
// multiple of 64 (so of 2 BF16 and 4 FP32 steps).
template <typename T>
__device__ __forceinline__ floatx4 tr_block(const T* C, const T* R, int K) {
  using M = TrMma<T>;
  constexpr int KSTEP = 4 * M::VEC;
  constexpr int U = 8;
  const int lane = threadIdx.x & 63;
  const long long o = (long long)(lane & 15) * K + (lane >> 4) * M::VEC;
  const T* cp = C + o;
  const T* rp = R + o;
  const int steps = K / KSTEP;
  floatx4 acc = {0, 0, 0, 0};
  uint4 cf[U], rf[U], cn[U], rn[U];
  auto load = [&](int s, uint4 (&c)[U], uint4 (&r)[U]) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = min(s + u, steps - 1) * KSTEP;  // past the end: loaded again, not used
      c[u] = *(const uint4*)(cp + k);
      r[u] = *(const uint4*)(rp + k);
    }
  };
  auto mul = [&](int s, const uint4 (&c)[U], const uint4 (&r)[U]) {
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (s + u < steps) M::mma(acc, c[u], r[u]);
  };
  load(0, cf, rf);
  for (int s = 0; s < steps; s += 2 * U) {
    if (s + U < steps) load(s + U, cn, rn);
    mul(s, cf, rf);
    if (s + 2 * U < steps) load(s + 2 * U, cf, rf);
    if (s + U < steps) mul(s + U, cn, rn);
  }
  return acc;
}

// Four consecutive values into the row-major and the transposed copy.
template <typename T>
__device__ __forceinline__ void tr_put(T* o, T* ot, int row, int col, long long ldo, long long ldt, const float (&v)[4]) {
  union {
    T e[4];
    uint2 u2;
    uint4 u4;
  } w;
#pragma unroll
  for (int e = 0; e < 4; ++e) w.e[e] = from_f<T>(v[e]);
  if constexpr (sizeof(T) == 2)
    *(uint2*)(o + row * ldo + col) = w.u2;
  else
    *(uint4*)(o + row * ldo + col) = w.u4;
#pragma unroll
  for (int e = 0; e < 4; ++e) ot[(col + e) * ldt + row] = w.e[e];
}

enum { TRM_HIDDEN, TRM_OUT, TRM_BWD };

struct TrMm {
  const void *C, *R;  // [cols][K], [rows][K]
  int K, ld;          // ld of row-major outputs (= columns)
  int bp;             // ld of transposed outputs (= rows)
  const float* bias;
  void *out, *outT;
  float* d1;          // sigma': written by TRM_HIDDEN, read by TRM_BWD
  float* yhat;        // TRM_OUT
  const double* Y;    // TRM_OUT: targets, or NULL (prediction only)
  int batch, m;
  double* partial;    // TRM_OUT: one loss partial per wave
};

// Hidden layer forward (bias, tanh, sigma'), output layer forward (with the
// loss gradient dZ_L = 2 (Yhat - Y) / (batch m) when there are targets), or
// backward through a layer (times sigma').
template <typename T, int MODE>
__global__ void __launch_bounds__(256) tr_mm_kernel(TrMm g) {
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int c0 = blockIdx.x * 32 + (wave & 1) * 16, r0 = blockIdx.y * 32 + (wave >> 1) * 16;
  const floatx4 a = tr_block<T>((const T*)g.C + (long long)c0 * g.K, (const T*)g.R + (long long)r0 * g.K, g.K);
  const int row = r0 + (lane & 15);
  const int col = c0 + (lane >> 4) * 4;
  const long long o = (long long)row * g.ld + col;
  float v[4] = {a[0], a[1], a[2], a[3]};
  if constexpr (MODE == TRM_HIDDEN) {
    const float4 b = *(const float4*)(g.bias + col);
    v[0] = tanhf(v[0] + b.x);
    v[1] = tanhf(v[1] + b.y);
    v[2] = tanhf(v[2] + b.z);
    v[3] = tanhf(v[3] + b.w);
    tr_put<T>((T*)g.out, (T*)g.outT, row, col, g.ld, g.bp, v);
    *(float4*)(g.d1 + o) = make_float4(1.0f - v[0] * v[0], 1.0f - v[1] * v[1], 1.0f - v[2] * v[2], 1.0f - v[3] * v[3]);
  } else if constexpr (MODE == TRM_BWD) {
    const float4 d = *(const float4*)(g.d1 + o);
    v[0] *= d.x;
    v[1] *= d.y;
    v[2] *= d.z;
    v[3] *= d.w;
    tr_put<T>((T*)g.out, (T*)g.outT, row, col, g.ld, g.bp, v);
  } else {
    const float4 b = *(const float4*)(g.bias + col);
    v[0] += b.x;
    v[1] += b.y;
    v[2] += b.z;
    v[3] += b.w;
    *(float4*)(g.yhat + o) = make_float4(v[0], v[1], v[2], v[3]);
    if (!g.Y) return;
    double sq = 0.0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float dz = 0.f;
      if (row < g.batch && col + e < g.m) {
        const double diff = (double)v[e] - g.Y[(long long)row * g.m + col + e];
        sq += diff * diff;
        dz = (float)(2.0 * diff / ((double)g.batch * g.m));
      }
      v[e] = dz;
    }
    tr_put<T>((T*)g.out, (T*)g.outT, row, col, g.ld, g.bp, v);
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) sq += __shfl_xor(sq, off, 64);
    if (lane == 0) g.partial[((long long)blockIdx.y * gridDim.x + blockIdx.x) * 4 + wave] = sq;
  }
}

// Weight and bias gradients of every layer in one launch, with Adam on the
// tile while it is in registers: dW_l = dZ_l^T A_{l-1}, the new W in FP32 and
// as both GEMM copies.  The layer's first column of tiles also sums dZ over
// the batch for the bias, one thread per row in batch order.
template <typename T>
__global__ void __launch_bounds__(256) tr_wgrad_kernel(const TrLayer* __restrict__ layers, int L, int bp, AdamArgs h) {
  int l = 0;
  while (l + 1 < L && layers[l + 1].tile0 <= (int)blockIdx.x) ++l;
  const TrLayer y = layers[l];
  const int t = blockIdx.x - y.tile0;
  const int tc = y.cols / 32;
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int c0 = t % tc * 32 + (wave & 1) * 16, r0 = t / tc * 32 + (wave >> 1) * 16;
  const floatx4 a = tr_block<T>((const T*)y.AT + (long long)c0 * bp, (const T*)y.dZT + (long long)r0 * bp, bp);
  const int row = r0 + (lane & 15);
  const int col = c0 + (lane >> 4) * 4;
  const long long o = (long long)row * y.cols + col;
  *(float4*)(y.dW + o) = make_float4(a[0], a[1], a[2], a[3]);
  const float4 p4 = *(const float4*)(y.W + o), m4 = *(const float4*)(y.m + o), v4 = *(const float4*)(y.v + o);
  const float g[4] = {a[0], a[1], a[2], a[3]};
  float p[4] = {p4.x, p4.y, p4.z, p4.w}, m[4] = {m4.x, m4.y, m4.z, m4.w}, v[4] = {v4.x, v4.y, v4.z, v4.w};
#pragma unroll
  for (int e = 0; e < 4; ++e) p[e] = adam_update(h, g[e], m[e], v[e], p[e]);
  *(float4*)(y.W + o) = make_float4(p[0], p[1], p[2], p[3]);
  *(float4*)(y.m + o) = make_float4(m[0], m[1], m[2], m[3]);
  *(float4*)(y.v + o) = make_float4(v[0], v[1], v[2], v[3]);
  tr_put<T>((T*)y.Wc, (T*)y.WTc, row, col, y.cols, y.rows, p);
  if (t % tc == 0 && threadIdx.x < 32) {
    constexpr int V = 16 / (int)sizeof(T);
    const int i = t / tc * 32 + threadIdx.x;
    const T* z = (const T*)y.dZT + (long long)i * bp;
    float gb = 0.f;
#pragma unroll 8
    for (int k = 0; k < bp; k += V) {
      float e[V];
      Vec16<T, float>::unpack(*(const uint4*)(z + k), e);
#pragma unroll
      for (int q = 0; q < V; ++q) gb += e[q];
    }
    y.db[i] = gb;
    float mb = y.mb[i], vb = y.vb[i];
    y.b[i] = adam_update(h, gb, mb, vb, y.b[i]);
    y.mb[i] = mb;
    y.vb[i] = vb;
  }
}

template <typename T>
__global__ void tr_sync(const float* p, long long count, int cols, int rows, T* wc, T* wtc) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= count) return;
  const int r = (int)(i / cols);
  const int c = (int)(i % cols);
  wc[i] = from_f<T>(p[i]);
  wtc[(long long)c * rows + r] = from_f<T>(p[i]);
}

__global__ void tr_out_f64(const float* Yhat, int rows, int m, int dpL, double* out) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (long long)rows * m) return;
  const int r = (int)(i / m);
  const int c = (int)(i % m);
  out[i] = (double)Yhat[(long long)r * dpL + c];
}

inline unsigned nblk(long long n) { return (unsigned)((n + 255) / 256); }

#define TR_HIP(c, call)                                                             \
  do {                                                                              \
    hipError_t e_ = (call);                                                         \
    if (e_ != hipSuccess) {                                                         \
      (c)->err = std::string(#call) + " failed: " + hipGetErrorString(e_);           \
      return NNC_E_HIP;                                                             \
    }                                                                               \
  } while (0)

// Launch of a small-product kernel, profiled as a GEMM.
#define TR_MM(c, kernel, ...)                       \
  do {                                              \
    ProfRec pr_;                                    \
    prof_begin((c), NNC_KC_GEMM, &pr_);             \
    hipLaunchKernelGGL(kernel, __VA_ARGS__);        \
    prof_end((c), &pr_);                            \
  } while (0)

int get_trainer(Ctx* c, int id, Trainer** out) {
  if (!c) return NNC_E_ARG;
  if (id < 0 || id >= (int)c->trainers.size() || !c->trainers[id]) {
    c->err = "invalid trainer handle";
    return NNC_E_ARG;
  }
  *out = (Trainer*)c->trainers[id];
  return NNC_OK;
}

int tr_gemm(Ctx* c, Trainer* t, GemmArgs g) {
  const long long tiles = (long long)((g.M + 127) / 128) * ((g.N + 127) / 128);
  const int cfg = tiles >= 128 ? 0 : 3;
  g.kper = g.K;
  ProfRec pr;
  prof_begin(c, NNC_KC_GEMM, &pr);
  TR_HIP(c, launch_gemm(t->ct, cfg, false, g, 1, c->stream));
  prof_end(c, &pr);
  return NNC_OK;
}

GemmArgs gargs(const void* A, long long lda, const void* B, long long ldb, int M, int N, int K) {
  GemmArgs g;
  memset(&g, 0, sizeof(g));
  g.A = A;
  g.B = B;
  g.lda = lda;
  g.ldb = ldb;
  g.M = M;
  g.N = N;
  g.K = K;
  g.rdiv = 1;
  return g;
}

// Grid of the 32 x 32 tiles of a rows x cols product (both multiples of 64).
inline dim3 tr_grid(int rows, int cols) { return dim3(cols / 32, rows / 32); }

// Forward pass of `rows` samples; with targets Y (the small path) the output
// layer's launch also writes dZ_L and the loss partials.
template <typename T>
int tr_forward(Ctx* c, Trainer* t, const double* X, int rows, const double* Y) {
  hipStream_t s = c->stream;
  hipLaunchKernelGGL(tr_cast_input<T>, tr_grid(t->bp, t->dp[0]), dim3(256), 0, s, X, rows, t->d[0], t->bp, t->dp[0],
                     (T*)t->A[0], (T*)t->AT[0]);
  TR_HIP(c, hipGetLastError());
  for (int l = 1; l <= t->L; ++l) {
    if (t->small) {
      TrMm g{};
      g.C = t->Wc[l - 1];
      g.R = t->A[l - 1];
      g.K = t->dp[l - 1];
      g.ld = t->dp[l];
      g.bp = t->bp;
      g.bias = t->bm[l - 1];
      if (l < t->L) {
        g.out = t->A[l];
        g.outT = t->AT[l];
        g.d1 = t->D1[l];
        TR_MM(c, (tr_mm_kernel<T, TRM_HIDDEN>), tr_grid(t->bp, t->dp[l]), dim3(256), 0, s, g);
      } else {
        g.out = t->dZ[l];
        g.outT = t->dZT[l];
        g.yhat = t->Yhat;
        g.Y = Y;
        g.batch = t->batch;
        g.m = t->d[l];
        g.partial = t->partial;
        TR_MM(c, (tr_mm_kernel<T, TRM_OUT>), tr_grid(t->bp, t->dp[l]), dim3(256), 0, s, g);
      }
      TR_HIP(c, hipGetLastError());
      continue;
    }
    GemmArgs g = gargs(t->A[l - 1], t->dp[l - 1], t->Wc[l - 1], t->dp[l - 1], t->bp, t->dp[l],
                       t->dp[l - 1]);
    g.epi = EPI_TRAIN_FWD;
    g.bias = t->bm[l - 1];
    g.ldo = t->dp[l];
    g.ldt = t->bp;
    if (l < t->L) {
      g.act = ACT_TANH;
      g.out0 = t->A[l];
      g.out1 = t->AT[l];
      g.out2 = t->D1[l];
    } else {
      g.act = ACT_IDENTITY;
      g.out2 = t->Yhat;
    }
    int rc = tr_gemm(c, t, g);
    if (rc) return rc;
  }
  return NNC_OK;
}

// Backward pass and update by the small kernels: dZ down the layers, then
// every layer's gradients and Adam in one launch (the weights are read by the
// backward passes before).
template <typename T>
int tr_backward_small(Ctx* c, Trainer* t, const AdamArgs& h) {
  hipStream_t s = c->stream;
  for (int l = t->L; l >= 2; --l) {
    TrMm g{};
    g.C = t->WTc[l - 1];
    g.R = t->dZ[l];
    g.K = t->dp[l];
    g.ld = t->dp[l - 1];
    g.bp = t->bp;
    g.d1 = t->D1[l - 1];
    g.out = t->dZ[l - 1];
    g.outT = t->dZT[l - 1];
    TR_MM(c, (tr_mm_kernel<T, TRM_BWD>), tr_grid(t->bp, t->dp[l - 1]), dim3(256), 0, s, g);
    TR_HIP(c, hipGetLastError());
  }
  TR_MM(c, tr_wgrad_kernel<T>, dim3(t->wtiles), dim3(256), 0, s, (const TrLayer*)t->dlayers, t->L, t->bp, h);
  TR_HIP(c, hipGetLastError());
  return NNC_OK;
}

// The same by the LDS-tiled GEMMs, from Yhat on.
template <typename T>
int tr_backward_large(Ctx* c, Trainer* t, const double* Y, const AdamArgs& h) {
  hipStream_t s = c->stream;
  const int L = t->L;
  int rc;
  const long long nout = (long long)t->bp * t->dp[L];
  hipLaunchKernelGGL(tr_mse_grad<T>, dim3(nblk(nout)), dim3(256), 0, s, t->Yhat, Y, t->batch,
                     t->d[L], t->bp, t->dp[L], (T*)t->dZ[L], (T*)t->dZT[L], t->partial);
  TR_HIP(c, hipGetLastError());
  for (int l = L; l >= 1; --l) {
    // wgrad: dW_l[dp_l][dp_{l-1}] = dZT_l [dp_l][bp] x AT_{l-1} [dp_{l-1}][bp]^T
    GemmArgs g = gargs(t->dZT[l], t->bp, t->AT[l - 1], t->bp, t->dp[l], t->dp[l - 1], t->bp);
    g.epi = EPI_F32;
    g.out0 = t->dW[l - 1];
    g.ldo = t->dp[l - 1];
    if ((rc = tr_gemm(c, t, g))) return rc;
    hipLaunchKernelGGL(tr_colsum<T>, dim3((t->dp[l] + 63) / 64), dim3(64), 0, s, (const T*)t->dZT[l],
                       t->dp[l], t->bp, t->db[l - 1]);
    TR_HIP(c, hipGetLastError());
    if (l >= 2) {
      // dgrad: dZ_{l-1} = (dZ_l W_l) * sigma'_{l-1};  W_l = (W_l^T)^T
      GemmArgs b = gargs(t->dZ[l], t->dp[l], t->WTc[l - 1], t->dp[l], t->bp, t->dp[l - 1], t->dp[l]);
      b.epi = EPI_TRAIN_BWD;
      b.v0 = t->D1[l - 1];
      b.ldv = t->dp[l - 1];
      b.out0 = t->dZ[l - 1];
      b.out1 = t->dZT[l - 1];
      b.ldo = t->dp[l - 1];
      b.ldt = t->bp;
      if ((rc = tr_gemm(c, t, b))) return rc;
    }
  }
  for (int l = 1; l <= L; ++l) {
    const long long cw = (long long)t->dp[l] * t->dp[l - 1];
    hipLaunchKernelGGL(tr_adam<T>, dim3(nblk(cw)), dim3(256), 0, s, t->Wm[l - 1], t->mW[l - 1],
                       t->vW[l - 1], t->dW[l - 1], cw, t->dp[l - 1], t->dp[l], h, (T*)t->Wc[l - 1],
                       (T*)t->WTc[l - 1]);
    TR_HIP(c, hipGetLastError());
    hipLaunchKernelGGL(tr_adam<T>, dim3(nblk(t->dp[l])), dim3(256), 0, s, t->bm[l - 1], t->mb[l - 1],
                       t->vb[l - 1], t->db[l - 1], (long long)t->dp[l], t->dp[l], 1, h, (T*)nullptr, (T*)nullptr);
    TR_HIP(c, hipGetLastError());
  }
  return NNC_OK;
}

template <typename T>
int tr_step(Ctx* c, Trainer* t, const double* X, const double* Y, float lr, float* loss) {
  hipStream_t s = c->stream;
  int rc = tr_forward<T>(c, t, X, t->batch, Y);
  if (rc) return rc;
  const float b1 = 0.9f, b2 = 0.999f;
  const int step = t->step + 1;
  const AdamArgs h{lr, b1, b2, 1e-8f, 1.f - powf(b1, (float)step), 1.f - powf(b2, (float)step)};
  rc = t->small ? tr_backward_small<T>(c, t, h) : tr_backward_large<T>(c, t, Y, h);
  if (rc) return rc;
  t->step = step;
  if (loss) {
    hipLaunchKernelGGL(tr_sum_partials, dim3(1), dim3(256), 0, s, t->partial, t->npartial,
                       1.0 / ((double)t->batch * t->d[t->L]), t->lossd);
    TR_HIP(c, hipGetLastError());
    double v = 0.0;
    TR_HIP(c, hipMemcpyAsync(&v, t->lossd, sizeof(double), hipMemcpyDeviceToHost, s));
    TR_HIP(c, hipStreamSynchronize(s));
    *loss = (float)v;
  }
  return NNC_OK;
}

template <typename T>
int tr_sync_copies(Ctx* c, Trainer* t) {
  for (int l = 1; l <= t->L; ++l) {
    const long long cw = (long long)t->dp[l] * t->dp[l - 1];
    hipLaunchKernelGGL(tr_sync<T>, dim3(nblk(cw)), dim3(256), 0, c->stream, t->Wm[l - 1], cw,
                       t->dp[l - 1], t->dp[l], (T*)t->Wc[l - 1], (T*)t->WTc[l - 1]);
    TR_HIP(c, hipGetLastError());
  }
  return NNC_OK;
}

int sync_copies(Ctx* c, Trainer* t) {
  return t->ct == DT_BF16 ? tr_sync_copies<bf16>(c, t) : tr_sync_copies<float>(c, t);
}

long long num_params(const Trainer* t) {
  long long n = 0;
  for (int l = 1; l <= t->L; ++l) n += (long long)t->d[l] * t->d[l - 1] + t->d[l];
  return n;
}

}  // namespace

void free_trainers(Ctx* c) {
  for (void* p : c->trainers) free_trainer((Trainer*)p);
  c->trainers.clear();
}

}  // namespace nnc

using namespace nnc;

extern "C" {

int nnc_train_create(nnc_ctx ctx, int L, const int* dims, int batch, int prec,
                     unsigned long long seed, int* mlp) {
  Ctx* c = (Ctx*)ctx;
  if (!c || !dims || !mlp) return NNC_E_ARG;
  if (L < 1 || batch < 1) {
    c->err = "L and batch must be >= 1";
    return NNC_E_SHAPE;
  }
  for (int l = 0; l <= L; ++l)
    if (dims[l] < 1) {
      c->err = "layer widths must be >= 1";
      return NNC_E_SHAPE;
    }
  if (prec != NNC_BF16 && prec != NNC_FP32) {
    c->err = "trainer precision must be NNC_BF16 or NNC_FP32";
    return NNC_E_UNSUPPORTED;
  }
  if (hipSetDevice(c->device) != hipSuccess) return NNC_E_HIP;
  Trainer* t = new Trainer();
  t->L = L;
  t->batch = batch;
  t->bp = rup(batch, 64);
  t->ct = prec == NNC_BF16 ? DT_BF16 : DT_F32;
  t->csz = prec == NNC_BF16 ? 2 : 4;
  for (int l = 0; l <= L; ++l) {
    t->d.push_back(dims[l]);
    t->dp.push_back(rup(dims[l], 64));
  }
  bool ok = true;
  auto A = [&](size_t b) {
    void* p = talloc(t, b);
    if (!p) ok = false;
    return p;
  };
  for (int l = 1; l <= L; ++l) {
    const size_t cw = (size_t)t->dp[l] * t->dp[l - 1];
    t->Wm.push_back((float*)A(cw * 4));
    t->mW.push_back((float*)A(cw * 4));
    t->vW.push_back((float*)A(cw * 4));
    t->dW.push_back((float*)A(cw * 4));
    t->bm.push_back((float*)A(t->dp[l] * 4));
    t->mb.push_back((float*)A(t->dp[l] * 4));
    t->vb.push_back((float*)A(t->dp[l] * 4));
    t->db.push_back((float*)A(t->dp[l] * 4));
    t->Wc.push_back(A(cw * t->csz));
    t->WTc.push_back(A(cw * t->csz));
  }
  t->A.assign(L, nullptr);
  t->AT.assign(L, nullptr);
  t->D1.assign(L, nullptr);
  for (int l = 0; l < L; ++l) {
    t->A[l] = A((size_t)t->bp * t->dp[l] * t->csz);
    t->AT[l] = A((size_t)t->bp * t->dp[l] * t->csz);
    if (l > 0) t->D1[l] = (float*)A((size_t)t->bp * t->dp[l] * 4);
  }
  t->dZ.assign(L + 1, nullptr);
  t->dZT.assign(L + 1, nullptr);
  for (int l = 1; l <= L; ++l) {
    t->dZ[l] = A((size_t)t->bp * t->dp[l] * t->csz);
    t->dZT[l] = A((size_t)t->bp * t->dp[l] * t->csz);
  }
  t->Yhat = (float*)A((size_t)t->bp * t->dp[L] * 4);
  // small: every product of a step below 128 tiles of 128 x 128 (tr_gemm's own
  // line between its small and its large tiles)
  t->small = true;
  for (int l = 1; l <= L; ++l) {
    auto tiles = [](int a, int b) { return (long long)((a + 127) / 128) * ((b + 127) / 128); };
    if (tiles(t->bp, t->dp[l]) >= 128 || tiles(t->dp[l], t->dp[l - 1]) >= 128 || tiles(t->bp, t->dp[l - 1]) >= 128)
      t->small = false;
  }
  // loss partials: one per wave of 256 outputs (small), or per block of 256
  t->npartial = (int)nblk((long long)t->bp * t->dp[L]);
  t->partial = (double*)A((size_t)t->npartial * 8);
  t->dlayers = (TrLayer*)A(sizeof(TrLayer) * L);
  size_t words = 0;
  for (int l = 1; l <= L; ++l) words += ((size_t)t->dp[l - 1] + 1) * t->dp[l];
  if (words * 4 <= kStagingBytes &&
      hipHostMalloc((void**)&t->staging, words * 4, hipHostMallocDefault) != hipSuccess) {
    (void)hipGetLastError();
    t->staging = nullptr;
  }
  t->lossd = (double*)A(8);
  if (!ok) {
    free_trainer(t);
    c->err = "device allocation failed";
    return NNC_E_NOMEM;
  }
  std::vector<TrLayer> table(L);
  for (int l = 1; l <= L; ++l) {
    table[l - 1] = TrLayer{t->dZT[l],   t->AT[l - 1], t->Wm[l - 1], t->mW[l - 1], t->vW[l - 1], t->dW[l - 1],
                           t->bm[l - 1], t->mb[l - 1], t->vb[l - 1], t->db[l - 1], t->Wc[l - 1], t->WTc[l - 1],
                           t->dp[l],     t->dp[l - 1], t->wtiles};
    if (t->small) t->wtiles += t->dp[l] / 32 * (t->dp[l - 1] / 32);
  }
  if (hipMemcpy(t->dlayers, table.data(), sizeof(TrLayer) * L, hipMemcpyHostToDevice) != hipSuccess) {
    free_trainer(t);
    c->err = "layer table upload failed";
    return NNC_E_HIP;
  }
  // N(0, 1/fan_in) initial weights from `seed` (host generator), zero biases.
  std::mt19937_64 gen(seed);
  std::normal_distribution<double> nd(0.0, 1.0);
  for (int l = 1; l <= L; ++l) {
    std::vector<float> w((size_t)t->dp[l] * t->dp[l - 1], 0.f);
    const double sc = 1.0 / sqrt((double)dims[l - 1]);
    for (int r = 0; r < dims[l]; ++r)
      for (int q = 0; q < dims[l - 1]; ++q) w[(size_t)r * t->dp[l - 1] + q] = (float)(nd(gen) * sc);
    if (hipMemcpy(t->Wm[l - 1], w.data(), w.size() * 4, hipMemcpyHostToDevice) != hipSuccess) {
      free_trainer(t);
      c->err = "parameter upload failed";
      return NNC_E_HIP;
    }
  }
  int rc = sync_copies(c, t);
  if (rc == NNC_OK && hipStreamSynchronize(c->stream) != hipSuccess) rc = NNC_E_HIP;
  if (rc) {
    free_trainer(t);
    return rc;
  }
  c->trainers.push_back(t);
  *mlp = (int)c->trainers.size() - 1;
  return NNC_OK;
}

int nnc_train_destroy(nnc_ctx ctx, int id) {
  Ctx* c = (Ctx*)ctx;
  Trainer* t;
  int rc = get_trainer(c, id, &t);
  if (rc) return rc;
  hipStreamSynchronize(c->stream);
  free_trainer(t);
  c->trainers[id] = nullptr;
  return NNC_OK;
}

int nnc_train_step(nnc_ctx ctx, int id, const double* X, const double* Y, float lr, float* loss) {
  Ctx* c = (Ctx*)ctx;
  Trainer* t;
  int rc = get_trainer(c, id, &t);
  if (rc) return rc;
  if (!X || !Y) {
    c->err = "null X or Y";
    return NNC_E_ARG;
  }
  if (hipSetDevice(c->device) != hipSuccess) return NNC_E_HIP;
  return t->ct == DT_BF16 ? tr_step<bf16>(c, t, X, Y, lr, loss) : tr_step<float>(c, t, X, Y, lr, loss);
}

int nnc_train_predict(nnc_ctx ctx, int id, int B, const double* X, double* Yhat) {
  Ctx* c = (Ctx*)ctx;
  Trainer* t;
  int rc = get_trainer(c, id, &t);
  if (rc) return rc;
  if (B < 0 || B > t->batch) {
    c->err = "B outside [0, batch]";
    return NNC_E_SHAPE;
  }
  if (B == 0) return NNC_OK;
  if (!X || !Yhat) {
    c->err = "null X or Yhat";
    return NNC_E_ARG;
  }
  if (hipSetDevice(c->device) != hipSuccess) return NNC_E_HIP;
  rc = t->ct == DT_BF16 ? tr_forward<bf16>(c, t, X, B, nullptr) : tr_forward<float>(c, t, X, B, nullptr);
  if (rc) return rc;
  const int m = t->d[t->L];
  hipLaunchKernelGGL(tr_out_f64, dim3(nblk((long long)B * m)), dim3(256), 0, c->stream, t->Yhat, B, m,
                     t->dp[t->L], Yhat);
  TR_HIP(c, hipGetLastError());
  return NNC_OK;
}

int nnc_train_num_params(nnc_ctx ctx, int id, long long* count) {
  Ctx* c = (Ctx*)ctx;
  Trainer* t;
  int rc = get_trainer(c, id, &t);
  if (rc) return rc;
  if (!count) return NNC_E_ARG;
  *count = num_params(t);
  return NNC_OK;
}

// Parameters or gradients, unpadded and in FP64, layer by layer.  With staging
// all copies are queued behind the stream's work into pinned memory and waited
// for once (a pageable copy per array, each waiting on its own into fresh host
// memory: 15 steps of the warm-start network and its 1.1M parameters back
// 1,600 -> 1,380 us); without, one array at a time.
static int copy_out(Ctx* c, Trainer* t, double* host, bool grads) {
  auto unpad = [&](const float* from, int rows, int cols, int ld) {
    for (int r = 0; r < rows; ++r, host += cols)
      for (int q = 0; q < cols; ++q) host[q] = from[(size_t)r * ld + q];
  };
  std::vector<float> pageable;
  size_t o = 0;
  for (int l = 1; l <= t->L; ++l) {
    const size_t cw = (size_t)t->dp[l] * t->dp[l - 1], cb = t->dp[l];
    const float* w = grads ? t->dW[l - 1] : t->Wm[l - 1];
    const float* b = grads ? t->db[l - 1] : t->bm[l - 1];
    if (t->staging) {
      TR_HIP(c, hipMemcpyAsync(t->staging + o, w, cw * 4, hipMemcpyDeviceToHost, c->stream));
      TR_HIP(c, hipMemcpyAsync(t->staging + o + cw, b, cb * 4, hipMemcpyDeviceToHost, c->stream));
      o += cw + cb;
      continue;
    }
    pageable.resize(std::max(pageable.size(), std::max(cw, cb)));
    if (l == 1) TR_HIP(c, hipStreamSynchronize(c->stream));
    TR_HIP(c, hipMemcpy(pageable.data(), w, cw * 4, hipMemcpyDeviceToHost));
    unpad(pageable.data(), t->d[l], t->d[l - 1], t->dp[l - 1]);
    TR_HIP(c, hipMemcpy(pageable.data(), b, cb * 4, hipMemcpyDeviceToHost));
    unpad(pageable.data(), 1, t->d[l], t->dp[l]);
  }
  if (!t->staging) return NNC_OK;
  TR_HIP(c, hipStreamSynchronize(c->stream));
  const float* from = t->staging;
  for (int l = 1; l <= t->L; ++l) {
    unpad(from, t->d[l], t->d[l - 1], t->dp[l - 1]);
    from += (size_t)t->dp[l] * t->dp[l - 1];
    unpad(from, 1, t->d[l], t->dp[l]);
    from += t->dp[l];
  }
  return NNC_OK;
}

int nnc_train_get_params(nnc_ctx ctx, int id, double* host) {
  Ctx* c = (Ctx*)ctx;
  Trainer* t;
  int rc = get_trainer(c, id, &t);
  if (rc) return rc;
  if (!host) return NNC_E_ARG;
  return copy_out(c, t, host, false);
}

int nnc_train_get_grads(nnc_ctx ctx, int id, double* host) {
  Ctx* c = (Ctx*)ctx;
  Trainer* t;
  int rc = get_trainer(c, id, &t);
  if (rc) return rc;
  if (!host) return NNC_E_ARG;
  return copy_out(c, t, host, true);
}

int nnc_train_set_params(nnc_ctx ctx, int id, const double* host) {
  Ctx* c = (Ctx*)ctx;
  Trainer* t;
  int rc = get_trainer(c, id, &t);
  if (rc) return rc;
  if (!host) return NNC_E_ARG;
  TR_HIP(c, hipStreamSynchronize(c->stream));
  size_t off = 0;
  for (int l = 1; l <= t->L; ++l) {
    const size_t cw = (size_t)t->dp[l] * t->dp[l - 1];
    std::vector<float> w(cw, 0.f);
    std::vector<float> b(t->dp[l], 0.f);
    for (int r = 0; r < t->d[l]; ++r)
      for (int q = 0; q < t->d[l - 1]; ++q) w[(size_t)r * t->dp[l - 1] + q] = (float)host[off++];
    for (int r = 0; r < t->d[l]; ++r) b[r] = (float)host[off++];
    TR_HIP(c, hipMemcpy(t->Wm[l - 1], w.data(), cw * 4, hipMemcpyHostToDevice));
    TR_HIP(c, hipMemcpy(t->bm[l - 1], b.data(), b.size() * 4, hipMemcpyHostToDevice));
    // a new parameter set restarts Adam
    TR_HIP(c, hipMemset(t->mW[l - 1], 0, cw * 4));
    TR_HIP(c, hipMemset(t->vW[l - 1], 0, cw * 4));
    TR_HIP(c, hipMemset(t->mb[l - 1], 0, t->dp[l] * 4));
    TR_HIP(c, hipMemset(t->vb[l - 1], 0, t->dp[l] * 4));
  }
  t->step = 0;
  rc = sync_copies(c, t);
  if (rc) return rc;
  TR_HIP(c, hipStreamSynchronize(c->stream));
  return NNC_OK;
}

}  // extern "C"
