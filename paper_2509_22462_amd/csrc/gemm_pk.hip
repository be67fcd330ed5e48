// Sweep products on packed operands (gfx950 / CDNA4): FP32 by three BF16
// parts per element, BF16, and FP64.
//
// C[M][N] = P[M][K] W[N][K]^T, P the tangents (one row per tangent column), W
// the weights.  Both operands are stored in the order the matrix units read
// them: for each block of 16 rows, each 32 elements of K and each part, the
// 1 KiB that one wave reads as a v_mfma_f32_16x16x32_bf16 operand (lane l
// holds row l % 16, elements 8 (l / 16) .. + 7; FP64: blocks of 8 elements for
// v_mfma_f64_16x16x4_f64).  A wave's LDS-DMA load
// therefore reads one contiguous KiB of memory, lands it in LDS as it is, and
// a fragment read is 64 consecutive 16-byte lanes: no bank conflicts, no
// swizzle, no address arithmetic per row.
//
// FP32 (NP = 3): x = hi + mid + lo, each what is left rounded to 8 significant
// bits, so the three parts hold all 24 (cut_parts in pk_device.h), and
//   x y = hi hi + (hi mid + mid hi) + (hi lo + mid mid + lo hi) + what is left out,
// six BF16 products accumulated in FP32: at 16x the rate of the FP32
// instruction they cost 6/16 of its time.  What is left out, mid lo + lo mid +
// lo lo, is at most 2^-23 of a product, 2e-8 of it in the root mean square and of
// either sign: less than the rounding of one FP32 addition.  (Parts cut off
// instead of rounded left out 4e-8 on average, always with the product's sign: H
// of hidden widths up to 64 was off by 1.02 to 1.3 times the FP32 instruction's
// error.)  The five smaller products have accumulators of their own, so the
// large ones are rounded by one product in six.  Errors of H against FP64, this
// and the FP32 instruction: hidden widths of 16 1.1-1.3e-7 and 1.3-1.6e-7, of 64
// 1.3-1.6e-7 and 1.6-2.2e-7, of 512 1.4-1.7e-7 and 3.1-4.8e-7.
//
// What bounds it: the matrix cores and the LDS reads that feed them (each
// three-part fragment pair feeds six MFMAs, a BF16 pair one).  Measured with
// the sweep's epilogue, against the tuned tilings of the row-major kernels:
// FP32 25,088 x 8192 x 8192 24.2 -> 14.1 ms (139 -> 239 TF/s), 784 x 8192 x 8192
// 0.83 -> 0.55 ms; BF16 the same shapes 3.67 -> 3.15 ms and 0.118 -> 0.106 ms;
// FP64 784 x 8192 x 8192 1.93 -> 1.75 ms.
#include <algorithm>
#include <type_traits>

#include "lds_dma.h"
#include "nnc_device.h"
#include "nnc_internal.h"
#include "pk_device.h"

namespace nnc {

namespace {

// MFMA accumulators: FP32 for BF16 parts, FP64 for FP64.
template <typename T> struct PkAcc {
  using A = float;
  using V = floatx4;
};
template <> struct PkAcc<double> {
  using A = double;
  using V = doublex4;
};

// The sum of an FP32 product's large and small parts' accumulators.  Products
// that overflow take the large one to infinity; the small parts have either sign
// and may overflow to the other one.
__device__ __forceinline__ float with_low(float acc, float low) { return fabsf(acc) == INFINITY ? acc : acc + low; }

// Four consecutive elements of a row-major FP32, BF16 or FP64 array (aligned
// to the four).
template <typename T, typename A>
__device__ __forceinline__ void put4(T* o, const A (&x)[4]) {
  if constexpr (sizeof(T) == 8) {
    *(double2*)o = make_double2(x[0], x[1]);
    *(double2*)(o + 2) = make_double2(x[2], x[3]);
  } else if constexpr (sizeof(T) == 4) {
    *(float4*)o = make_float4(x[0], x[1], x[2], x[3]);
  } else {
    uint2 t[1];
    cut_parts<1>(x, t);
    *(uint2*)o = t[0];
  }
}

// The square roots of four |s|.  FP32: each in two parts, the second one Newton
// step, so that v sqrt|s| is rounded once (an FP32 root would be off alike in
// every row).
template <typename A>
struct Roots {
  A q[4];
  float c[4];
};
__device__ __forceinline__ void load_roots(const double* s, Roots<double>& r) {
  const double2 s0 = *(const double2*)s, s1 = *(const double2*)(s + 2);
  r.q[0] = sqrt(fabs(s0.x));
  r.q[1] = sqrt(fabs(s0.y));
  r.q[2] = sqrt(fabs(s1.x));
  r.q[3] = sqrt(fabs(s1.y));
}
__device__ __forceinline__ void load_roots(const double* s, Roots<float>& r) {
  const double2 s0 = *(const double2*)s, s1 = *(const double2*)(s + 2);
  const double a[4] = {fabs(s0.x), fabs(s0.y), fabs(s1.x), fabs(s1.y)};
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const float h = (float)a[e];
    r.q[e] = __builtin_amdgcn_sqrtf(h);
    r.c[e] = (fmaf(-r.q[e], r.q[e], h) + (float)(a[e] - (double)h)) * (0.5f * __builtin_amdgcn_rcpf(r.q[e]));
    if (!(h > 0x1p-80f && h < 0x1p80f)) {  // zero, the ends of the range, NaN
      const double d = sqrt(a[e]);
      r.q[e] = (float)d;
      r.c[e] = d < 0x1p100 ? (float)(d - (double)r.q[e]) : 0.f;
    }
  }
}
__device__ __forceinline__ double times_root(double v, const Roots<double>& r, int e) { return v * r.q[e]; }
__device__ __forceinline__ float times_root(float v, const Roots<float>& r, int e) {
  return fmaf(v, r.q[e], fabsf(v) < INFINITY ? v * r.c[e] : 0.f);
}

// Four consecutive elements of T (row i of point b) as U = sqrt|s| T (r: the
// roots) and, from the point's first row, the signs of s.
template <typename T, typename A>
__device__ __forceinline__ void put_u(const PackedU& u, int b, int i, int col, const double* s, const Roots<A>& r,
                                      const A (&v)[4]) {
  A x[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) x[e] = times_root(v[e], r, e);
  put_packed<T>(u.U, b * u.np16 + i, col, u.kt, x);
  if (i != 0) return;
  char* o = (char*)u.sgn + (long long)b * u.kt * 64;
  uint32_t h[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) h[e] = (uint32_t)__double2hiint(s[e]) & 0x80000000u;
  if constexpr (sizeof(T) == 8) {
    *(uint4*)(o + (long long)col * 8) = make_uint4(0u, h[0], 0u, h[1]);
    *(uint4*)(o + (long long)col * 8 + 16) = make_uint4(0u, h[2], 0u, h[3]);
  } else {
    *(uint2*)(o + (long long)col * 2) = make_uint2((h[0] >> 16) | h[1], (h[2] >> 16) | h[3]);
  }
}

// Four consecutive results of one row through the epilogue of g.epi; r: the roots
// of point rb's columns, if that is this row's point.
template <typename T>
__device__ __forceinline__ void pk_epilogue(const GemmArgs& g, int row, int col, int b,
                                            const typename PkAcc<T>::A (&v)[4], int split,
                                            Roots<typename PkAcc<T>::A>& r, int& rb) {
  using A = typename PkAcc<T>::A;
  if (g.epi == EPI_PART) {
    put4<A, A>((A*)g.out0 + (long long)split * g.split_stride + (long long)row * g.ldo + col, v);
    return;
  }
  const long long vi = (long long)b * g.ldv + col;
  if (g.out0) put4<T, A>((T*)g.out0 + (long long)row * g.ldo + col, v);
  if (g.out2) {
    const double* sv = (const double*)g.v1 + vi;
    if constexpr (sizeof(T) == 2) {  // BF16: S_l, row-major
      const A x[4] = {v[0] * (A)sv[0], v[1] * (A)sv[1], v[2] * (A)sv[2], v[3] * (A)sv[3]};
      put4<T, A>((T*)g.out2 + (long long)row * g.ldo + col, x);
    } else {
      if (b != rb) load_roots(sv, r);
      rb = b;
      put_u<T>(g.u, b, row - b * g.u.n, g.ucol + col, sv, r, v);
    }
  }
  if (g.out1) {
    const A* d = (const A*)g.v0 + vi;
    const A x[4] = {v[0] * d[0], v[1] * d[1], v[2] * d[2], v[3] * d[3]};
    put_packed<T>(g.out1, row, col, (int)(g.ldo1 / PkElem<T>::KB), x);
  }
}

// One output tile: WN x WM waves, each FN x FM blocks of 16 neurons x 16
// tangent rows; NS LDS stages of KS K blocks.  The weights are the MFMA's
// first operand, so lane l holds neurons 4 (l / 16) .. + 3 of tangent row
// l % 16: four consecutive columns of the row-major outputs.  (The FP64
// instruction gives lane l its rows l / 16 + 4 e; pack_operand_kernel orders
// the 16 rows of a weight block to match.)
template <typename T, int WN, int WM, int FN, int FM, int KS, int NS>
struct PkTile {
  static constexpr int NP = PkElem<T>::NP;
  static constexpr int NW = WN * WM;
  static constexpr int BNB = WN * FN, BMB = WM * FM;  // 16-row blocks of W and P per tile
  static constexpr int CW = BNB * KS * NP, CP = BMB * KS * NP;  // KiB per stage
  static constexpr int LW = (CW + NW - 1) / NW, LP = (CP + NW - 1) / NW;
  static constexpr int CPT = LW + LP;  // DMA loads per wave and stage
  static constexpr int PBASE = LW * NW * 1024;  // P's blocks follow W's in a stage
  static constexpr int STAGE = CPT * NW * 1024;
};

// (GROUPED only names the caller: one instantiation per kernel.)
template <typename T, int WN, int WM, int FN, int FM, int KS, int NS, bool GROUPED>
__device__ __forceinline__ void pk_tile(const GemmArgs& g, int t, int split, char* st0, char* st1, char* st2,
                                        char* st3) {
  using S = PkTile<T, WN, WM, FN, FM, KS, NS>;
  // distinct LDS arrays, chosen at compile time in each step: the compiler then
  // waits, before a fragment read, only for loads into that stage
  auto st = [&](int i) -> char* { return i == 0 ? st0 : i == 1 ? st1 : i == 2 ? st2 : st3; };
  const int tm = t % g.tiles_m, tn = t / g.tiles_m;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wn = wave % WN, wm = wave / WN;
  constexpr int NP = S::NP, KB = PkElem<T>::KB;
  const int kt = g.K / KB;
  const int k0 = split * (g.kper / KB);
  const int nk = (min(kt, k0 + g.kper / KB) - k0) / KS;  // stages (K and kper are multiples of KB KS)
  const int nb0 = tn * S::BNB, mb0 = tm * S::BMB;
  const int nbw = (g.N + 15) >> 4, mbw = (g.M + 15) >> 4;
  // One buffer resource per operand, from the tile's first block on.
  const unsigned rowb = (unsigned)kt * NP * 1024u;  // bytes of one 16-row block
  const int nbv = min(S::BNB, nbw - nb0), mbv = min(S::BMB, mbw - mb0);  // the tile's blocks inside the operands
  const __amdgpu_buffer_rsrc_t rsW = __builtin_amdgcn_make_buffer_rsrc(
      (void*)((const char*)g.B + (long long)nb0 * rowb), (short)0, (int)(nbv * rowb), 0x00020000);
  const __amdgpu_buffer_rsrc_t rsP = __builtin_amdgcn_make_buffer_rsrc(
      (void*)((const char*)g.A + (long long)mb0 * rowb), (short)0, (int)(mbv * rowb), 0x00020000);
  const int vofs = lane * 16;
  // Chunk c of a stage's operand: block c / (KS NP), K block and part c % (KS NP),
  // which follow one another in memory as in LDS.  What lies past the tile's
  // last block, and the loads that only fill a wave's count, read the last
  // block again (their results are not stored), so every wave issues the same
  // number of loads per stage and none of them is conditional.
  int so0[S::CPT];
#pragma unroll
  for (int p = 0; p < S::CPT; ++p) {
    const bool isw = p < S::LW;
    const int c = (isw ? p : p - S::LW) * S::NW + wave;
    so0[p] = (int)(min(c / (KS * NP), (isw ? nbv : mbv) - 1) * rowb + (unsigned)(c % (KS * NP)) * 1024u);
  }
  auto dma = [&](int s, char* dst) {  // stages past the last one read it again
    const int ko = (k0 + min(s, nk - 1) * KS) * NP * 1024;
#pragma unroll
    for (int p = 0; p < S::CPT; ++p) {
      const lds_ptr d = (lds_ptr)(dst + (p * S::NW + wave) * 1024);
      if (p < S::LW)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rsW, d, 16, vofs, so0[p] + ko, 0, 0);
      else
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rsP, d, 16, vofs, so0[p] + ko, 0, 0);
    }
  };
  using V = typename PkAcc<T>::V;
  V acc[FN][FM], low[FN][FM];  // low: the products of the smaller parts (NP = 3)
#pragma unroll
  for (int i = 0; i < FN; ++i)
#pragma unroll
    for (int j = 0; j < FM; ++j) acc[i][j] = low[i][j] = V{0, 0, 0, 0};
  const int wbase = wn * FN * KS * NP * 1024 + lane * 16;
  const int pbase = S::PBASE + wm * FM * KS * NP * 1024 + lane * 16;
  using Frag = typename std::conditional<sizeof(T) == 8, double2, bf16x8>::type;
  struct Frags {
    Frag w[NP][FN], x[NP][FM];
  };
  // one K block's fragments, in the order the products below want them: the
  // first product waits for two of the six groups (all planes of one operand
  // first: 6 % slower.  Two halves of the workgroup taking turns at reading and
  // multiplying, a barrier between: 12 % slower)
  auto load = [&](const char* sb, int ks, Frags& f) {
    auto lw = [&](int p) {
#pragma unroll
      for (int i = 0; i < FN; ++i) f.w[p][i] = *(const Frag*)(sb + wbase + ((i * KS + ks) * NP + p) * 1024);
    };
    auto lx = [&](int p) {
#pragma unroll
      for (int j = 0; j < FM; ++j) f.x[p][j] = *(const Frag*)(sb + pbase + ((j * KS + ks) * NP + p) * 1024);
    };
    if constexpr (NP == 3) {
      lx(0);
      lw(2);
      lw(1);
      lx(1);
      lw(0);
      lx(2);
    } else {
      lw(0);
      lx(0);
    }
  };
  auto mul = [&](const Frags& f) {
    if constexpr (sizeof(T) == 8) {
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int i = 0; i < FN; ++i)
#pragma unroll
          for (int j = 0; j < FM; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(h ? f.w[0][i].y : f.w[0][i].x,
                                                             h ? f.x[0][j].y : f.x[0][j].x, acc[i][j], 0, 0, 0);
    } else {
      auto prod = [&](int a, int b, V(&to)[FN][FM]) {
#pragma unroll
        for (int i = 0; i < FN; ++i)
#pragma unroll
          for (int j = 0; j < FM; ++j)
            to[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f.w[a][i], f.x[b][j], to[i][j], 0, 0, 0);
      };
      if constexpr (NP == 3) {
        prod(2, 0, low);
        prod(1, 0, low);
        prod(1, 1, low);
        prod(0, 1, low);
        prod(0, 0, acc);
        prod(0, 2, low);
      } else {
        prod(0, 0, acc);
      }
    }
  };
  auto compute = [&](const char* sb) {
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      Frags f;
      load(sb, ks, f);
      mul(f);
      if constexpr (NP == 1 && sizeof(T) == 2) __builtin_amdgcn_sched_barrier(0);  // one K block in registers
    }
  };
#pragma unroll
  for (int s = 0; s < NS - 1; ++s) dma(s, st(s));
  for (int s0 = 0;; s0 += NS) {
#pragma unroll
    for (int u = 0; u < NS; ++u) {
      wait_stage<(NS - 2) * S::CPT>();
      dma(s0 + u + NS - 1, st((u + NS - 1) % NS));
      compute(st(u));
      if (s0 + u + 1 >= nk) goto done;
    }
  }
done:
  wait_loads<0>();
  int pt[FM];  // the rows' points
#pragma unroll
  for (int j = 0; j < FM; ++j) pt[j] = ((mb0 + wm * FM + j) * 16 + (lane & 15)) / g.rdiv;
  Roots<typename PkAcc<T>::A> r;
  int rb = -1;
  auto out = [&](int i, int j) {
    const int col = (nb0 + wn * FN + i) * 16 + (lane >> 4) * 4;
    const int row = (mb0 + wm * FM + j) * 16 + (lane & 15);
    if (row >= g.M || col >= g.N) return;
    typename PkAcc<T>::A v[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if constexpr (NP == 3)
        v[e] = with_low(acc[i][j][e], low[i][j][e]);
      else
        v[e] = acc[i][j][e];
    }
    pk_epilogue<T>(g, row, col, pt[j], v, split, r, rb);
  };
  if constexpr (sizeof(T) == 2) {  // row-major outputs: along the row
#pragma unroll
    for (int j = 0; j < FM; ++j)
#pragma unroll
      for (int i = 0; i < FN; ++i) out(i, j);
  } else {  // a column's roots serve its rows
#pragma unroll
    for (int i = 0; i < FN; ++i) {
      rb = -1;
#pragma unroll
      for (int j = 0; j < FM; ++j) out(i, j);
    }
  }
}

// Each XCD takes a contiguous run of tiles (which share weight blocks in its L2).
__device__ __forceinline__ int pk_xcd(int t, int tiles) {
  const int full = tiles - tiles % 8;
  return t < full ? (t % 8) * (full / 8) + t / 8 : t;
}

#define PK_STAGES                                                                                 \
  using S = PkTile<T, WN, WM, FN, FM, KS, NS>;                                                   \
  static_assert(NS >= 2 && NS <= 4 && S::STAGE * NS <= 160 * 1024, "LDS");                        \
  __shared__ __attribute__((aligned(16))) char st0[S::STAGE];                                     \
  __shared__ __attribute__((aligned(16))) char st1[S::STAGE];                                     \
  __shared__ __attribute__((aligned(16))) char st2[NS > 2 ? S::STAGE : 16];                       \
  __shared__ __attribute__((aligned(16))) char st3[NS > 3 ? S::STAGE : 16]

template <typename T, int WN, int WM, int FN, int FM, int KS, int NS>
__global__ void __launch_bounds__(WN * WM * 64) gemm_pk_kernel(GemmArgs g) {
  PK_STAGES;
  pk_tile<T, WN, WM, FN, FM, KS, NS, false>(g, pk_xcd(blockIdx.x, g.tiles_m * g.tiles_n), blockIdx.y, st0, st1, st2, st3);
}


// Persistent grouped launch: workgroup w takes work items w, w + gridDim.x, ...
// (as gemm_grouped_kernel).
template <typename T, int WN, int WM, int FN, int FM, int KS, int NS>
__global__ void __launch_bounds__(WN * WM * 64)
gemm_pk_grouped_kernel(const GemmArgs* __restrict__ groups, const int* __restrict__ offsets, int ngroups) {
  PK_STAGES;
  const int total = offsets[ngroups];
  for (int w = blockIdx.x; w < total; w += gridDim.x) {
    int gi = 0;
    while (gi + 1 < ngroups && offsets[gi + 1] <= w) ++gi;
    const GemmArgs g = groups[gi];
    pk_tile<T, WN, WM, FN, FM, KS, NS, true>(g, pk_xcd(w - offsets[gi], g.tiles_m * g.tiles_n), 0, st0, st1, st2, st3);
    __syncthreads();  // every wave done with the stages before the next item refills them
  }
}
#undef PK_STAGES

// Sum of the K slices in slice order through the product's epilogue, four
// columns per lane.  FP32 and FP64: a wave takes 16 rows x 16 columns as in the
// tiles, so that the packed results leave in half KiB blocks (lanes along a row
// wrote an eighth of each: 784 x 4096 in FP32, two slices: 19.7 -> 12.0 us).
// BF16, whose row-major results are as many bytes as the packed ones: along a
// row (15 us, against 24).
template <typename T>
__global__ void __launch_bounds__(256) pk_reduce_kernel(GemmArgs g, const void* __restrict__ part, int splits) {
  using A = typename PkAcc<T>::A;
  using V = typename PkAcc<T>::V;
  const int lane = threadIdx.x & 63;
  int row, col;
  if constexpr (sizeof(T) == 2) {
    const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
    row = (int)(i / (g.N / 4));
    col = (int)(i % (g.N / 4)) * 4;
  } else {
    const int wc = g.N / 16;
    const long long w = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
    row = (int)(w / wc) * 16 + (lane & 15);
    col = (int)(w % wc) * 16 + (lane >> 4) * 4;
  }
  if (row >= g.M) return;
  const long long MN = (long long)g.M * g.N;
  const A* p = (const A*)part + (long long)row * g.N + col;
  V t = *(const V*)p;
#pragma unroll 4
  for (int s = 1; s < splits; ++s) t += *(const V*)(p + s * MN);
  const A v[4] = {t[0], t[1], t[2], t[3]};
  Roots<A> r;
  int rb = -1;
  pk_epilogue<T>(g, row, col, row / g.rdiv, v, 0, r, rb);
}

template <typename T>
__global__ void __launch_bounds__(256) pack_operand_kernel(const T* __restrict__ W, long long ldw, long long total, int K,
                                                           void* __restrict__ out) {
  using A = typename PkAcc<T>::A;
  const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
  if (i >= total) return;
  const int q = K / 4;
  const int row = (int)(i / q);
  const int col = (int)(i - (long long)row * q) * 4;
  const T* w = W + row * ldw + col;
  const A v[4] = {(A)w[0], (A)w[1], (A)w[2], (A)w[3]};
  const int r16 = row & 15;
  const int prow = sizeof(T) == 8 ? (row - r16) + (r16 >> 2) + 4 * (r16 & 3) : row;
  put_packed<T>(out, prow, col, K / PkElem<T>::KB, v);
}

// ---------------------------------------------------------------- symmetric product
// H_b = sum_k sign(s_k) U_ik U_jk over all layers' columns: the lower block
// triangle of square tiles, both operands from the one packed U; a stage holds
// the tile's row blocks, its column blocks and the K blocks' signs, which are
// XORed into the column fragments.  FP32 sums are added into FP64 every 64
// elements of K, as the row-major kernel does.  One operand is written by the
// sweep and read here where T and S = diag(s) T were.  137M network, FP32: 229
// -> 150 us at one point, 5.8 -> 4.0 ms at 32; the surrogate batch's 5.2 -> 3.8.
template <typename T, int WN, int WM, int FN, int FM, int KS, int NS>
struct SymTile {
  static constexpr int NP = PkElem<T>::NP;
  static constexpr int NW = WN * WM;
  static constexpr int EB = WN * FN;  // 16-row blocks of the tile's edge
  static_assert(EB == WM * FM, "square tiles");
  static constexpr int CW = EB * KS * NP;             // KiB per stage and operand
  static constexpr int LW = (CW + NW - 1) / NW;       // loads per wave and operand
  static constexpr int CPT = 2 * LW + 1;              // and one of signs
  static constexpr int PBASE = LW * NW * 1024;
  static constexpr int SBASE = 2 * PBASE;
  static constexpr int STAGE = SBASE + NW * 1024;
};

// One entry of the product element by element, where the parts' products came to
// NaN: past the FP32 range the small ones may overflow against the large ones,
// which have one accumulator here (a second one, as in pk_tile, spills: 137M
// network 2 % slower).  The entry of a NaN element is known at that element.
__device__ double sym_entry(const GemmArgs& g, int b, int row, int col, int k0, int k1) {
  auto elem = [&](int r, int k) {
    const char* p = (const char*)g.u.U + packed_offset<float>(b * g.u.np16 + r, k, g.u.kt);
    auto part = [&](int i) { return __uint_as_float((uint32_t) * (const uint16_t*)(p + i * 1024) << 16); };
    const float lo = part(2);
    return fabsf(lo) == INFINITY ? lo : part(0) + part(1) + lo;
  };
  const uint16_t* sgn = (const uint16_t*)((const char*)g.u.sgn + (long long)b * g.u.kt * 64);
  double sum = 0.0;
  float acc = 0.f;
  for (int k = k0; k < k1; ++k) {
    const float x = elem(row, k), y = elem(col, k);
    if (x != x || y != y) return NAN;
    acc = fmaf(sgn[k] ? -x : x, y, acc);
    if ((k & 63) == 63) {
      sum += (double)acc;
      acc = 0.f;
    }
  }
  return sum + (double)acc;
}

// (GROUPED only names the caller.)
template <typename T, int WN, int WM, int FN, int FM, int KS, int NS, bool GROUPED>
__device__ __forceinline__ void sym_tile(const GemmArgs& g, int t, int split, char* st0, char* st1, char* st2) {
  using S = SymTile<T, WN, WM, FN, FM, KS, NS>;
  constexpr int NP = S::NP, KB = PkElem<T>::KB;
  constexpr int FOLD = 2;  // K blocks per fold into FP64 (FP32)
  static_assert(KS <= S::NW && FOLD % KS == 0, "one K block of signs per wave; whole stages per fold");
  auto st = [&](int i) -> char* { return i == 0 ? st0 : i == 1 ? st1 : st2; };
  const int per = g.tiles_m * (g.tiles_m + 1) / 2;
  const int b = t / per;
  t -= b * per;
  int ti = (int)((sqrtf(8.0f * (float)t + 1.0f) - 1.0f) * 0.5f);
  while (ti > 0 && ti * (ti + 1) / 2 > t) --ti;
  while ((ti + 1) * (ti + 2) / 2 <= t) ++ti;
  const int tj = t - ti * (ti + 1) / 2;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wn = wave % WN, wm = wave / WN;
  const int kt = g.u.kt;
  const int k0 = split * (g.kper / KB);
  const int nk = (min(kt, k0 + g.kper / KB) - k0) / KS;
  const int nb = g.u.np16 >> 4;
  const unsigned rowb = (unsigned)kt * NP * 1024u;
  const char* U = (const char*)g.u.U + (long long)b * nb * rowb;
  const int nvi = min(S::EB, nb - ti * S::EB), nvj = min(S::EB, nb - tj * S::EB);
  const __amdgpu_buffer_rsrc_t rsI = __builtin_amdgcn_make_buffer_rsrc(
      (void*)(U + (long long)ti * S::EB * rowb), (short)0, (int)(nvi * rowb), 0x00020000);
  const __amdgpu_buffer_rsrc_t rsJ = __builtin_amdgcn_make_buffer_rsrc(
      (void*)(U + (long long)tj * S::EB * rowb), (short)0, (int)(nvj * rowb), 0x00020000);
  const __amdgpu_buffer_rsrc_t rsS = __builtin_amdgcn_make_buffer_rsrc(
      (void*)((const char*)g.u.sgn + (long long)b * kt * 64), (short)0, kt * 64, 0x00020000);
  const int vofs = lane * 16;
  const int sofs = (lane >> 4) * 16;
  int so0[2 * S::LW];  // as in pk_tile: what lies past the last block reads it again
#pragma unroll
  for (int p = 0; p < 2 * S::LW; ++p) {
    const bool isi = p < S::LW;
    const int c = (isi ? p : p - S::LW) * S::NW + wave;
    so0[p] = (int)(min(c / (KS * NP), (isi ? nvi : nvj) - 1) * rowb + (unsigned)(c % (KS * NP)) * 1024u);
  }
  auto dma = [&](int s, char* dst) {
    const int kb = k0 + min(s, nk - 1) * KS;
#pragma unroll
    for (int p = 0; p < 2 * S::LW; ++p) {
      const lds_ptr d = (lds_ptr)(dst + (p * S::NW + wave) * 1024);
      if (p < S::LW)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rsI, d, 16, vofs, so0[p] + kb * NP * 1024, 0, 0);
      else
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rsJ, d, 16, vofs, so0[p] + kb * NP * 1024, 0, 0);
    }
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsS, (lds_ptr)(dst + S::SBASE + wave * 1024), 16, sofs,
                                             (kb + wave % KS) * 64, 0, 0);
  };
  using V = typename PkAcc<T>::V;
  V acc[FN][FM];
  double sum[sizeof(T) == 8 ? 1 : FN][sizeof(T) == 8 ? 1 : FM][4];
#pragma unroll
  for (int i = 0; i < FN; ++i)
#pragma unroll
    for (int j = 0; j < FM; ++j) {
      acc[i][j] = V{0, 0, 0, 0};
      if constexpr (sizeof(T) < 8) {
#pragma unroll
        for (int e = 0; e < 4; ++e) sum[i][j][e] = 0.0;
      }
    }
  auto fold = [&]() {
    if constexpr (sizeof(T) < 8) {
#pragma unroll
      for (int i = 0; i < FN; ++i)
#pragma unroll
        for (int j = 0; j < FM; ++j) {
#pragma unroll
          for (int e = 0; e < 4; ++e) sum[i][j][e] += (double)acc[i][j][e];
          acc[i][j] = V{0, 0, 0, 0};
        }
    }
  };
  const int ibase = wn * FN * KS * NP * 1024 + lane * 16;
  const int jbase = S::PBASE + wm * FM * KS * NP * 1024 + lane * 16;
  auto compute = [&](const char* sb) {
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      uint4 w[NP][FN], x[NP][FM];
      const uint4 sg = *(const uint4*)(sb + S::SBASE + ks * 1024 + lane * 16);
      auto lw = [&](int p) {
#pragma unroll
        for (int i = 0; i < FN; ++i) w[p][i] = *(const uint4*)(sb + ibase + ((i * KS + ks) * NP + p) * 1024);
      };
      auto lx = [&](int p) {
#pragma unroll
        for (int j = 0; j < FM; ++j) {
          const uint4 v = *(const uint4*)(sb + jbase + ((j * KS + ks) * NP + p) * 1024);
          x[p][j] = make_uint4(v.x ^ sg.x, v.y ^ sg.y, v.z ^ sg.z, v.w ^ sg.w);
        }
      };
      if constexpr (NP == 3) {  // in the order the products want them
        lx(0);
        lw(2);
        lw(1);
        lx(1);
        lw(0);
        lx(2);
      } else {
        lw(0);
        lx(0);
      }
      if constexpr (sizeof(T) == 8) {
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int i = 0; i < FN; ++i)
#pragma unroll
            for (int j = 0; j < FM; ++j) {
              const double2 wd = __builtin_bit_cast(double2, w[0][i]), xd = __builtin_bit_cast(double2, x[0][j]);
              acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(h ? wd.y : wd.x, h ? xd.y : xd.x, acc[i][j], 0, 0, 0);
            }
      } else {
        auto prod = [&](int pa, int pb) {
#pragma unroll
          for (int i = 0; i < FN; ++i)
#pragma unroll
            for (int j = 0; j < FM; ++j)
              acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w[pa][i]),
                                                                  __builtin_bit_cast(bf16x8, x[pb][j]), acc[i][j], 0, 0, 0);
        };
        if constexpr (NP == 3) {
          prod(2, 0);
          prod(1, 0);
          prod(1, 1);
          prod(0, 1);
          prod(0, 0);
          prod(0, 2);
        } else {
          prod(0, 0);
        }
      }
    }
  };
#pragma unroll
  for (int s = 0; s < NS - 1; ++s) dma(s, st(s));
  for (int s0 = 0;; s0 += NS) {
#pragma unroll
    for (int u = 0; u < NS; ++u) {
      wait_stage<(NS - 2) * S::CPT>();
      dma(s0 + u + NS - 1, st((u + NS - 1) % NS));
      compute(st(u));
      if ((s0 + u + 1) % (FOLD / KS) == 0) fold();
      if (s0 + u + 1 >= nk) goto done;
    }
  }
done:
  wait_loads<0>();
  fold();
  double* H = (double*)g.out0 + (long long)split * g.split_stride + b * g.bsO;
#pragma unroll
  for (int i = 0; i < FN; ++i)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int row = (ti * S::EB + wn * FN + i) * 16 + (sizeof(T) == 8 ? (lane >> 4) + 4 * e : (lane >> 4) * 4 + e);
      if (row >= g.M) continue;
#pragma unroll
      for (int j = 0; j < FM; ++j) {
        const int col = (tj * S::EB + wm * FM + j) * 16 + (lane & 15);
        if (col < g.N) {
          if constexpr (sizeof(T) == 8)
            H[(long long)row * g.ldo + col] = acc[i][j][e];
          else
            H[(long long)row * g.ldo + col] =
                sum[i][j][e] == sum[i][j][e] ? sum[i][j][e] : sym_entry(g, b, row, col, k0 * KB, min(kt * KB, k0 * KB + g.kper));
        }
      }
    }
}

#define SYM_STAGES                                                                \
  using S = SymTile<T, WN, WM, FN, FM, KS, NS>;                                   \
  static_assert(NS >= 2 && NS <= 3 && S::STAGE * NS <= 160 * 1024, "LDS");        \
  __shared__ __attribute__((aligned(16))) char st0[S::STAGE];                     \
  __shared__ __attribute__((aligned(16))) char st1[S::STAGE];                     \
  __shared__ __attribute__((aligned(16))) char st2[NS > 2 ? S::STAGE : 16]

template <typename T, int WN, int WM, int FN, int FM, int KS, int NS>
__global__ void __launch_bounds__(WN * WM * 64) gemm_pk_sym_kernel(GemmArgs g) {
  SYM_STAGES;
  sym_tile<T, WN, WM, FN, FM, KS, NS, false>(g, pk_xcd(blockIdx.x, gemm_tiles_per_split(g)), blockIdx.y, st0, st1, st2);
}

template <typename T, int WN, int WM, int FN, int FM, int KS, int NS>
__global__ void __launch_bounds__(WN * WM * 64)
gemm_pk_sym_grouped_kernel(const GemmArgs* __restrict__ groups, const int* __restrict__ offsets, int ngroups) {
  SYM_STAGES;
  const int total = offsets[ngroups];
  for (int w = blockIdx.x; w < total; w += gridDim.x) {
    int gi = 0;
    while (gi + 1 < ngroups && offsets[gi + 1] <= w) ++gi;
    const GemmArgs g = groups[gi];
    const int local = w - offsets[gi];
    const int tiles = gemm_tiles_per_split(g);
    sym_tile<T, WN, WM, FN, FM, KS, NS, true>(g, pk_xcd(local % tiles, tiles), local / tiles, st0, st1, st2);
    __syncthreads();
  }
}
#undef SYM_STAGES

// U from row-major T: a wave takes 16 rows of a point and 32 columns of a
// layer, lane l row l % 16 and columns 4 (l / 16) .. + 3 of each half.  With P
// also the first product's operand, of the elements it holds already: a launch
// and a read of W_1 less than seeding it apart.
template <typename T>
__global__ void __launch_bounds__(256) pack_u_kernel(PackUArgs a) {
  using A = typename PkAcc<T>::A;
  const int lane = threadIdx.x & 63;
  const int nb = a.u.np16 >> 4;
  const int b = blockIdx.x / nb;
  const int i = (blockIdx.x - b * nb) * 16 + (lane & 15);
  int cx = blockIdx.y, l = 0;  // blocks of 128 columns, layer by layer
  for (; l < a.layers; ++l) {
    const int nch = (a.dp[l] + 127) / 128;
    if (cx < nch) break;
    cx -= nch;
  }
  if (l >= a.layers || i >= a.u.n) return;
  const int dp = a.dp[l];
  const T* t = l == 0 && a.T1 ? (const T*)a.T1 + (long long)i * a.ld1
                              : (const T*)a.Tc + (long long)(b * a.u.n + i) * a.ld + a.koff[l];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int c = cx * 128 + (threadIdx.x >> 6) * 32 + h * 16 + (lane >> 4) * 4;
    if (c >= dp) return;
    const A v[4] = {(A)t[c], (A)t[c + 1], (A)t[c + 2], (A)t[c + 3]};
    const double* s = a.s[l] + (long long)b * dp + c;
    Roots<A> r;
    load_roots(s, r);
    put_u<T>(a.u, b, i, a.koff[l] + c, s, r, v);
    if (a.P && l == 0) {
      const A* d = (const A*)a.d1 + (long long)b * dp + c;
      const A x[4] = {v[0] * d[0], v[1] * d[1], v[2] * d[2], v[3] * d[3]};
      put_packed<T>(a.P, b * a.u.n + i, c, dp / PkElem<T>::KB, x);
    }
  }
}

// The tilings.  us1 / us2: time 32 elements of K take a CU for one tile,
// with one workgroup on it and (us2) with several in turn or at once, measured
// at 25088 x 8192 x 8192 and 784 x 8192 x 8192 (us2, us1 of the large tiles),
// 117 x 4032 x 4032 (us1 of the small ones) and 5488 x 512 x 1024 (the last of
// FP32: 172 tiles in 38 us, where 64 x 128 and 64 x 64 take 47 and 49).
struct PkCfg {
  int bm, bn, ks, occ;
  double us1, us2;
};
constexpr int kPkCfgs = 4;   // BF16, FP64
constexpr int kPkCfgs32 = 5;  // FP32
constexpr PkCfg kPkF32[kPkCfgs32] = {
    {128, 256, 32, 1, 2.00, 2.20},  // 8 waves of 64 x 64
    {112, 256, 32, 1, 1.87, 2.04},  // 8 waves of 32 x 112: whole tiles of 784 rows
    {64, 128, 32, 2, 1.00, 0.70},   // 4 waves of 64 x 32
    {64, 64, 32, 2, 0.75, 0.45},    // 4 waves of 32 x 32
    {128, 128, 32, 1, 1.20, 1.30},  // 8 waves of 32 x 64: about one round of tiles
};
constexpr PkCfg kPkBf16[kPkCfgs] = {
    {256, 256, 32, 1, 0.80, 0.97},  // 8 waves of 64 x 128
    {112, 256, 64, 1, 0.41, 0.49},  // 8 waves of 32 x 112
    {128, 64, 64, 2, 0.23, 0.29},   // 8 waves of 16 x 64
    {64, 64, 64, 3, 0.17, 0.15},    // 4 waves of 32 x 32
};
constexpr PkCfg kPkF64[kPkCfgs] = {
    {128, 256, 16, 1, 7.20, 7.20},  // 8 waves of 64 x 64
    {112, 256, 16, 1, 6.30, 6.30},  // 8 waves of 32 x 112
    {64, 128, 16, 2, 2.60, 1.90},   // 4 waves of 64 x 32
    {64, 64, 16, 3, 1.30, 0.95},    // 4 waves of 32 x 32
};

inline int pk_cfgs(DType t) { return t == DT_F32 ? kPkCfgs32 : kPkCfgs; }
inline const PkCfg& pk_cfg(DType t, int cfg) {
  return t == DT_F32 ? kPkF32[cfg] : t == DT_BF16 ? kPkBf16[cfg] : kPkF64[cfg];
}

// CALL(type, WN, WM, FN, FM, KS, NS) of tiling cfg.
#define PK_DISPATCH(T, CALL)                        \
  do {                                              \
    if constexpr (sizeof(T) == 4) {                 \
      switch (cfg) {                                \
        case 0: CALL(float, 4, 2, 4, 4, 1, 2);      \
        case 1: CALL(float, 8, 1, 2, 7, 1, 2);      \
        case 2: CALL(float, 2, 2, 4, 2, 1, 2);      \
        case 3: CALL(float, 2, 2, 2, 2, 1, 3);      \
        case 4: CALL(float, 4, 2, 2, 4, 1, 3);      \
        default: return hipErrorInvalidValue;       \
      }                                             \
    } else if constexpr (sizeof(T) == 2) {          \
      switch (cfg) {                                \
        case 0: CALL(bf16, 4, 2, 4, 8, 1, 4);       \
        case 1: CALL(bf16, 8, 1, 2, 7, 2, 3);       \
        case 2: CALL(bf16, 4, 2, 1, 4, 2, 3);       \
        case 3: CALL(bf16, 2, 2, 2, 2, 2, 3);       \
        default: return hipErrorInvalidValue;       \
      }                                             \
    } else {                                        \
      switch (cfg) {                                \
        case 0: CALL(double, 4, 2, 4, 4, 2, 3);     \
        case 1: CALL(double, 8, 1, 2, 7, 2, 3);     \
        case 2: CALL(double, 2, 2, 4, 2, 2, 3);     \
        case 3: CALL(double, 2, 2, 2, 2, 2, 3);     \
        default: return hipErrorInvalidValue;       \
      }                                             \
    }                                               \
  } while (0)

template <typename T>
hipError_t pk_launch(int cfg, const GemmArgs& g, int splits, hipStream_t s) {
  const dim3 grid(g.tiles_m * g.tiles_n, splits);
#define PK_CALL(T_, WN, WM, FN, FM, KS, NS)                                                            \
  hipLaunchKernelGGL((gemm_pk_kernel<T_, WN, WM, FN, FM, KS, NS>), grid, dim3(WN * WM * 64), 0, s, g); \
  return hipGetLastError()
  PK_DISPATCH(T, PK_CALL);
#undef PK_CALL
}

template <typename T>
hipError_t pk_launch_grouped(int cfg, const GemmArgs* groups, const int* offsets, int ngroups, int grid, hipStream_t s) {
#define PK_CALL(T_, WN, WM, FN, FM, KS, NS)                                                                    \
  hipLaunchKernelGGL((gemm_pk_grouped_kernel<T_, WN, WM, FN, FM, KS, NS>), dim3(grid), dim3(WN * WM * 64), 0, \
                     s, groups, offsets, ngroups);                                                                \
  return hipGetLastError()
  PK_DISPATCH(T, PK_CALL);
#undef PK_CALL
}

inline int pk_kper(const PkCfg& c, int K, int ks) {
  return ((K + ks - 1) / ks + c.ks - 1) / c.ks * c.ks;
}

}  // namespace

// The tiling and K split of the least estimated time: the rounds of tiles a CU
// takes, each K / ksplit long, and with a split the partials written and read
// at 4.5 TB/s by one more launch (7 us: at 4 a 302 x 256 x 256 product was split
// for no gain and a call of 28 such launches took 236 instead of 219 us).
PkChoice pk_choose(DType t, int M, int N, int K, size_t part_bytes) {
  PkChoice best{0, 1};
  double best_us = 1e30;
  const double psz = t == DT_F64 ? 8.0 : 4.0;  // bytes of a partial
  for (int i = 0; i < pk_cfgs(t); ++i) {
    const PkCfg& c = pk_cfg(t, i);
    const long long tiles = (long long)((M + c.bm - 1) / c.bm) * ((N + c.bn - 1) / c.bn);
    for (int ks = 1; ks <= 8; ++ks) {
      const int kper = pk_kper(c, K, ks);
      if ((K + kper - 1) / kper != ks) continue;
      if (ks > 1 && ks * psz * M * N > (double)part_bytes) break;
      const long long rounds = (tiles * ks + 255) / 256;
      double us = kper / 32.0 * (rounds == 1 ? c.us1 : rounds * c.us2) + 4.0;
      if (ks > 1) us += 7.0 + 2.0 * psz * ks * M * N / 4.5e6;
      if (us < best_us) {
        best_us = us;
        best = PkChoice{i, ks};
      }
    }
  }
  return best;
}

int pk_num_cfgs(DType t) { return pk_cfgs(t); }

int pk_slices(DType t, int cfg, int K, int ks) {
  const int kper = pk_kper(pk_cfg(t, cfg), K, ks);
  return (K + kper - 1) / kper;
}

size_t pk_operand_bytes(DType t, long long rows, int K) {
  return (size_t)((rows + 15) / 16 * 16) * K * (t == DT_F32 ? 6 : t == DT_BF16 ? 2 : 8);
}

hipError_t launch_pack_operand(DType t, const void* W, long long ldw, int rows, int K, void* out, hipStream_t s) {
  if (rows <= 0 || rows % 16 != 0 || K <= 0 || K % 64 != 0) return hipErrorInvalidValue;
  const long long total = (long long)rows * (K / 4);
  const long long blocks = (total + 255) / 256;
  if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
#define PK_PACK(T)                                                                                            \
  hipLaunchKernelGGL(pack_operand_kernel<T>, dim3((unsigned)blocks), dim3(256), 0, s, (const T*)W, ldw, total, K, \
                     out)
  switch (t) {
    case DT_F32: PK_PACK(float); break;
    case DT_BF16: PK_PACK(bf16); break;
    case DT_F64: PK_PACK(double); break;
  }
#undef PK_PACK
  return hipGetLastError();
}

void pk_set_tiles(DType t, int cfg, GemmArgs& g) {
  const PkCfg& c = pk_cfg(t, cfg);
  g.tiles_m = (g.M + c.bm - 1) / c.bm;
  g.tiles_n = (g.N + c.bn - 1) / c.bn;
}

int pk_grouped_occupancy(DType t, int cfg) { return pk_cfg(t, cfg).occ; }

hipError_t launch_gemm_pk(DType t, PkChoice ch, GemmArgs g, void* part, hipStream_t s) {
  if (g.M <= 0 || g.N <= 0) return hipSuccess;
  if (t != DT_BF16 && g.out2 && (!g.u.U || !g.u.sgn || g.u.n <= 0)) return hipErrorInvalidValue;
  if (ch.cfg < 0 || ch.cfg >= pk_cfgs(t) || g.K <= 0 || g.K % 64 != 0 || g.N % 16 != 0 ||
      (ch.ksplit > 1 && !part))
    return hipErrorInvalidValue;
  pk_set_tiles(t, ch.cfg, g);
  GemmArgs p = g;
  p.kper = pk_kper(pk_cfg(t, ch.cfg), g.K, ch.ksplit);
  const int splits = (g.K + p.kper - 1) / p.kper;
  if (splits > 1) {
    p.epi = EPI_PART;
    p.out0 = part;
    p.ldo = g.N;
    p.split_stride = (long long)g.M * g.N;
  }
  hipError_t e = t == DT_F32    ? pk_launch<float>(ch.cfg, p, splits, s)
                 : t == DT_BF16 ? pk_launch<bf16>(ch.cfg, p, splits, s)
                                : pk_launch<double>(ch.cfg, p, splits, s);
  if (e != hipSuccess || splits == 1) return e;
  const long long blocks = ((long long)((g.M + 15) / 16) * (g.N / 16) + 3) / 4;
  if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
  const dim3 grid((unsigned)blocks);
  switch (t) {
    case DT_F32: hipLaunchKernelGGL(pk_reduce_kernel<float>, grid, dim3(256), 0, s, g, (const void*)part, splits); break;
    case DT_BF16: hipLaunchKernelGGL(pk_reduce_kernel<bf16>, grid, dim3(256), 0, s, g, (const void*)part, splits); break;
    case DT_F64: hipLaunchKernelGGL(pk_reduce_kernel<double>, grid, dim3(256), 0, s, g, (const void*)part, splits); break;
  }
  return hipGetLastError();
}

// Tile edge: 128 where its tiles, at two thirds of the 64-wide ones' time per
// area, take less than those.
int pk_sym_edge(int n) {
  const double t64 = (n + 63) / 64, t128 = (n + 127) / 128;
  return t128 * (t128 + 1) * 128 * 128 * 0.67 < t64 * (t64 + 1) * 64 * 64 ? 128 : 64;
}

int pk_sym_occupancy(int edge) { return edge == 128 ? 1 : 2; }

size_t pk_u_bytes(DType t, int n, int B, int K) {
  return pk_operand_bytes(t, (long long)B * ((n + 15) / 16 * 16), K);
}

#define SYM_DISPATCH(CALL)                                                     \
  do {                                                                         \
    if (edge == 128) {                                                         \
      switch (t) {                                                             \
        case DT_F32: CALL(float, 2, 4, 4, 2, 1, 2);                            \
        case DT_F64: CALL(double, 2, 4, 4, 2, 2, 3);                           \
        default: break;                                                        \
      }                                                                        \
    } else if (edge == 64) {                                                   \
      switch (t) {                                                             \
        case DT_F32: CALL(float, 2, 2, 2, 2, 1, 2);                            \
        case DT_F64: CALL(double, 2, 2, 2, 2, 2, 3);                           \
        default: break;                                                        \
      }                                                                        \
    }                                                                          \
    return hipErrorInvalidValue;                                               \
  } while (0)

hipError_t launch_gemm_pk_sym(DType t, GemmArgs g, int splits, hipStream_t s) {
  if (g.M <= 0 || g.nbat <= 0) return hipSuccess;
  if (g.M != g.N || g.kper <= 0 || g.kper % 64 != 0 || g.u.kt <= 0) return hipErrorInvalidValue;
  const int edge = g.sym;
  g.tiles_m = g.tiles_n = edge > 0 ? (g.M + edge - 1) / edge : 0;
  const dim3 grid(gemm_tiles_per_split(g), splits);
#define SYM_CALL(T, WN, WM, FN, FM, KS, NS)                                                                     \
  hipLaunchKernelGGL((gemm_pk_sym_kernel<T, WN, WM, FN, FM, KS, NS>), grid, dim3(WN * WM * 64), 0, s, g); \
  return hipGetLastError()
  SYM_DISPATCH(SYM_CALL);
#undef SYM_CALL
}

hipError_t launch_gemm_pk_sym_grouped(DType t, int edge, const GemmArgs* groups, const int* offsets, int ngroups,
                                      int grid, hipStream_t s) {
  if (grid <= 0) return hipErrorInvalidValue;
#define SYM_CALL(T, WN, WM, FN, FM, KS, NS)                                                                      \
  hipLaunchKernelGGL((gemm_pk_sym_grouped_kernel<T, WN, WM, FN, FM, KS, NS>), dim3(grid), dim3(WN * WM * 64), 0, \
                     s, groups, offsets, ngroups);                                                              \
  return hipGetLastError()
  SYM_DISPATCH(SYM_CALL);
#undef SYM_CALL
}

// Time of a round of tiles (32 elements of K: 1.1 / 3.6 us at edge 128 in
// FP32 / FP64, 0.37 of it per tile at edge 64) against the partials
// written and read back.  A slice keeps 128 elements or more.  (The rounds take
// no less than the tiles' time over all CUs: where that and the partials of sp
// slices exceed the best, so do those of more.  A network is sized by asking for
// every number of points up to max_points.)
int pk_sym_splits(DType t, int n, int B, int K) {
  const int edge = pk_sym_edge(n);
  const double tt = (n + edge - 1) / edge;
  const double tiles = B * tt * (tt + 1) / 2;
  const double us = (t == DT_F32 ? 1.1 : 3.6) * (edge == 128 ? 1.0 : 0.37);
  int best = 1;
  double best_us = 1e30;
  const double least = tiles * (K / 32.0) * us / 256.0 * (1.0 - 1e-9);
  for (int sp = 1; sp <= 256 && (sp == 1 || K / sp >= 128); ++sp) {
    const double rounds = (double)(((long long)(tiles * sp) + 255) / 256);
    const double parts = sp * (0.1 + (double)B * n * n * 16.0 / 4.5e6);
    if (least + parts >= best_us) break;
    const double c = rounds * (K / 32.0 / sp) * us + parts + (sp > 16 ? 5.0 : 0.0);
    if (c < best_us) {
      best_us = c;
      best = sp;
    }
  }
  return best;
}

hipError_t launch_pack_u(DType t, const PackUArgs& a, hipStream_t s) {
  if (a.B <= 0 || a.layers <= 0) return hipSuccess;
  if (a.layers > kMaxScaleLayers || a.ld % 4 != 0 || a.ld1 % 4 != 0) return hipErrorInvalidValue;
  long long chunks = 0;
  for (int l = 0; l < a.layers; ++l) {
    if (a.dp[l] % 64 != 0 || a.koff[l] % 64 != 0) return hipErrorInvalidValue;
    chunks += (a.dp[l] + 127) / 128;
  }
  if (chunks > 65535) return hipErrorInvalidValue;
  const dim3 grid((unsigned)(a.B * (a.u.np16 / 16)), (unsigned)chunks);
  switch (t) {
    case DT_F32: hipLaunchKernelGGL(pack_u_kernel<float>, grid, dim3(256), 0, s, a); break;
    case DT_BF16: return hipErrorInvalidValue;
    case DT_F64: hipLaunchKernelGGL(pack_u_kernel<double>, grid, dim3(256), 0, s, a); break;
  }
  return hipGetLastError();
}

hipError_t launch_gemm_pk_grouped(DType t, int cfg, const GemmArgs* groups, const int* offsets, int ngroups, int grid,
                                  hipStream_t s) {
  if (grid <= 0) return hipErrorInvalidValue;
  switch (t) {
    case DT_F32: return pk_launch_grouped<float>(cfg, groups, offsets, ngroups, grid, s);
    case DT_BF16: return pk_launch_grouped<bf16>(cfg, groups, offsets, ngroups, grid, s);
    case DT_F64: return pk_launch_grouped<double>(cfg, groups, offsets, ngroups, grid, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace nnc
