#pragma once
// gfx950 kernels of the state-vector library.
//
// State layout in HBM: two planes (re, im) of 2^n elements (double for
// complex128, float for complex64).  Gate action follows the paper's gather /
// multiply / scatter over the amplitudes that differ only on the targets
// (Section 5.3), but indices are computed by bit insertion instead of an index
// table, and many gates are applied per HBM round trip (see sv_internal.h).
#include <hip/hip_runtime.h>

#include <type_traits>
#include <stdint.h>

#include "sv_internal.h"

namespace svk {

template <typename T> struct C2T;
template <> struct C2T<double> { using type = double2; };
template <> struct C2T<float> { using type = float2; };

template <typename T> struct V4T;   // 16-byte global vector of T
template <> struct V4T<double> { using type = double2; static constexpr int N = 2; };
template <> struct V4T<float> { using type = float4; static constexpr int N = 4; };

// Read-only views in the constant address space: the data (plan descriptors,
// coefficients) is written before the kernel and never during it, so loads
// through these pointers are invariant and go to the scalar cache (SGPRs)
// when the address is wave-uniform.
#define SVI_CONST __attribute__((address_space(4)))
template <typename T>
__device__ __forceinline__ const SVI_CONST T *cptr(const T *p) {
  return (const SVI_CONST T *)p;
}

// Workgroup barrier that orders LDS only: the fences are scoped to the local
// address space, so outstanding global loads (the next tile's prefetch) are
// not waited for, unlike __syncthreads().
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

template <typename T>
__device__ __forceinline__ int swz(int i) {
  return svi_swz(i, sizeof(T) == 8 ? 3 : 4);
}

// Insert a zero bit at each position of pos[0..np) (ascending).
__device__ __forceinline__ uint64_t insert_zeros64(uint64_t x, const int32_t *pos, int np) {
  for (int k = 0; k < np; k++) {
    const int p = pos[k];
    const uint64_t lo = x & ((1ull << p) - 1ull);
    x = ((x >> p) << (p + 1)) | lo;
  }
  return x;
}

// Micro-op o, read through the constant address space (uniform index:
// scalar loads, not vector loads whose waits would also wait for other
// memory traffic in flight).
__device__ __forceinline__ MicroOp op_at(const MicroOp *ops, int o) {
  const SVI_CONST MicroOp &s = cptr(ops)[o];
  MicroOp m;
  m.type = s.type;
  m.t0 = s.t0;
  m.t1 = s.t1;
  m.mask = s.mask;
  m.cm = s.cm;
  m.cv = s.cv;
  m.coef = s.coef;
  m.gz = s.gz;
  m.galpha = s.galpha;
  m.gbeta = s.gbeta;
  return m;
}

// Tile-local base index of a thread in a stage: thread-index bit k placed on
// tile bit tpos[k] (the group bits stay zero), as the lane's part (k < 6) and
// the wave's, which is uniform: scalar work.  tpos is read as aligned 32-bit
// words (scalar loads; byte loads of the descriptor would become vector loads,
// whose waits also wait for the tile prefetch in flight).
__device__ __forceinline__ int lane_base(int lane, const SVI_CONST StageDesc &sd) {
  const SVI_CONST int32_t *w = (const SVI_CONST int32_t *)sd.tpos;
  int b = 0;
#pragma unroll
  for (int k = 0; k < 6; k++) b |= ((lane >> k) & 1) << ((w[k >> 2] >> (8 * (k & 3))) & 0xff);
  return b;
}

template <int M, int R>
__device__ __forceinline__ int wave_base(int wave, const SVI_CONST StageDesc &sd) {
  const SVI_CONST int32_t *w = (const SVI_CONST int32_t *)sd.tpos;
  int b = 0;
#pragma unroll
  for (int k = 6; k < M - R; k++)
    b |= ((wave >> (k - 6)) & 1) << ((w[k >> 2] >> (8 * (k & 3))) & 0xff);
  return b;
}

// Brings a sweep's descriptors, micro-ops and coefficients into the XCD's L2
// (one load per 64-byte line, spread over the workgroup's NT threads), so that
// the stages' scalar loads, which come one after the other, miss no further
// than that.  Returns a value to be used once the loads may be waited for.
// For the serving kernel, whose stages on one tile are a latency chain (burst
// of 48 requests 1241 -> 1029 us); the sweep kernels gain 3% at 12 qubits and
// nothing at 20 and 21, and lost 1% at 30, so they do without.
template <int NT, typename Args>
__device__ __forceinline__ int warm_sweep(const Args &a) {
  int x = 0;
  auto lines = [&](const void *p, int64_t b, int64_t e) {
    const char *q = (const char *)p;
    for (int64_t o = b + (int64_t)threadIdx.x * 64; o < e; o += NT * 64) x ^= *(const int *)(q + o);
  };
  lines(a.stages, (int64_t)a.stage_begin * sizeof(StageDesc), (int64_t)a.stage_end * sizeof(StageDesc));
  lines(a.coef, (int64_t)a.coef_begin * 8, (int64_t)a.coef_end * 8);
  lines(a.ops, (int64_t)a.op_begin * sizeof(MicroOp), (int64_t)a.op_end * sizeof(MicroOp));
  return x;
}

// Global offset of tile row r: bit k of r goes to qubit hb[k].
__device__ __forceinline__ uint64_t spread_row(int r, const int32_t *hb, int nh) {
  uint64_t o = 0;
  for (int k = 0; k < nh; k++) o |= (uint64_t)((r >> k) & 1) << hb[k];
  return o;
}

// Offset of tile element i from its tile's base: the low c bits stay, bit
// c + k goes to qubit hb[k].
__device__ __forceinline__ uint64_t tile_off(int i, int c, const int32_t *hb, int nh) {
  return spread_row(i >> c, hb, nh) + (uint64_t)(i & ((1 << c) - 1));
}

// Base index of tile `tile`: zeros inserted at the tile's qubits (0..c-1 and hb).
__device__ __forceinline__ uint64_t tile_base(int64_t tile, int c, const int32_t *hb, int nh) {
  uint64_t x = (uint64_t)tile << c;
  return insert_zeros64(x, hb, nh);
}

// Tile-local index whose bits land on output index i under the output bit
// permutation pm (output bit k <- bit pm[k]).
__device__ __forceinline__ int perm_bits(int i, const int32_t *pm, int m) {
  int j = 0;
  for (int b = 0; b < m; b++) j |= ((i >> b) & 1) << pm[b];
  return j;
}

// ------------------------------------------------------------ micro-ops
// All group arrays are indexed with compile-time indices only.

template <typename T, int R, int TB>
__device__ __forceinline__ void mo_u(T *re, T *im, const double *cf, uint32_t cm, uint32_t cv) {
  const T a0r = (T)cf[0], a0i = (T)cf[1], a1r = (T)cf[2], a1i = (T)cf[3];
  const T b0r = (T)cf[4], b0i = (T)cf[5], b1r = (T)cf[6], b1i = (T)cf[7];
  if (cm == 0) {
#pragma unroll
    for (int j = 0; j < (1 << R); j++) {
      if (j & (1 << TB)) continue;
      const int k = j | (1 << TB);
      const T xr = re[j], xi = im[j], yr = re[k], yi = im[k];
      re[j] = a0r * xr - a0i * xi + a1r * yr - a1i * yi;
      im[j] = a0r * xi + a0i * xr + a1r * yi + a1i * yr;
      re[k] = b0r * xr - b0i * xi + b1r * yr - b1i * yi;
      im[k] = b0r * xi + b0i * xr + b1r * yi + b1i * yr;
    }
  } else {
#pragma unroll
    for (int j = 0; j < (1 << R); j++) {
      if (j & (1 << TB)) continue;
      if ((j & cm) != cv) continue;
      const int k = j | (1 << TB);
      const T xr = re[j], xi = im[j], yr = re[k], yi = im[k];
      re[j] = a0r * xr - a0i * xi + a1r * yr - a1i * yi;
      im[j] = a0r * xi + a0i * xr + a1r * yi + a1i * yr;
      re[k] = b0r * xr - b0i * xi + b1r * yr - b1i * yi;
      im[k] = b0r * xi + b0i * xr + b1r * yi + b1i * yr;
    }
  }
}

template <typename T, int R, int TB>
__device__ __forceinline__ void mo_r(T *re, T *im, const double *cf, uint32_t cm, uint32_t cv) {
  const T r00 = (T)cf[0], r01 = (T)cf[1], r10 = (T)cf[2], r11 = (T)cf[3];
  if (cm == 0) {
#pragma unroll
    for (int j = 0; j < (1 << R); j++) {
      if (j & (1 << TB)) continue;
      const int k = j | (1 << TB);
      const T xr = re[j], xi = im[j], yr = re[k], yi = im[k];
      re[j] = r00 * xr + r01 * yr;
      im[j] = r00 * xi + r01 * yi;
      re[k] = r10 * xr + r11 * yr;
      im[k] = r10 * xi + r11 * yi;
    }
  } else {
#pragma unroll
    for (int j = 0; j < (1 << R); j++) {
      if (j & (1 << TB)) continue;
      if ((j & cm) != cv) continue;
      const int k = j | (1 << TB);
      const T xr = re[j], xi = im[j], yr = re[k], yi = im[k];
      re[j] = r00 * xr + r01 * yr;
      im[j] = r00 * xi + r01 * yi;
      re[k] = r10 * xr + r11 * yr;
      im[k] = r10 * xi + r11 * yi;
    }
  }
}

template <typename T, int R>
__device__ __forceinline__ void mo_p(T *re, T *im, const double *cf, uint32_t mask, uint32_t cm,
                                     uint32_t cv) {
  const T d0r = (T)cf[0], d0i = (T)cf[1], d1r = (T)cf[2], d1i = (T)cf[3];
#pragma unroll
  for (int j = 0; j < (1 << R); j++) {
    if ((j & cm) != cv) continue;
    const bool odd = __builtin_popcount((uint32_t)j & mask) & 1;
    const T dr = odd ? d1r : d0r;
    const T di = odd ? d1i : d0i;
    const T xr = re[j], xi = im[j];
    re[j] = xr * dr - xi * di;
    im[j] = xr * di + xi * dr;
  }
}

template <typename T, int R, int TB>
__device__ __forceinline__ void mo_x(T *re, T *im, uint32_t cm, uint32_t cv) {
#pragma unroll
  for (int j = 0; j < (1 << R); j++) {
    if (j & (1 << TB)) continue;
    if ((j & cm) != cv) continue;
    const int k = j | (1 << TB);
    T t = re[j]; re[j] = re[k]; re[k] = t;
    t = im[j]; im[j] = im[k]; im[k] = t;
  }
}

template <typename T, int R, int A, int B>
__device__ __forceinline__ void mo_swap(T *re, T *im, uint32_t cm, uint32_t cv) {
#pragma unroll
  for (int j = 0; j < (1 << R); j++) {
    if (!((j >> A) & 1) || ((j >> B) & 1)) continue;
    if ((j & cm) != cv) continue;
    const int k = j ^ (1 << A) ^ (1 << B);
    T t = re[j]; re[j] = re[k]; re[k] = t;
    t = im[j]; im[j] = im[k]; im[k] = t;
  }
}

template <typename T, int R>
__device__ __forceinline__ void mo_neg(T *re, T *im, uint32_t cm, uint32_t cv) {
#pragma unroll
  for (int j = 0; j < (1 << R); j++) {
    if ((j & cm) != cv) continue;
    re[j] = -re[j];
    im[j] = -im[j];
  }
}

// 4x4 on (bit A = low local bit, bit B = high local bit).
template <typename T, int R, int A, int B>
__device__ __forceinline__ void mo_q(T *re, T *im, const double *cf, uint32_t cm, uint32_t cv) {
  T u[32];
#pragma unroll
  for (int q = 0; q < 32; q++) u[q] = (T)cf[q];
#pragma unroll
  for (int j = 0; j < (1 << R); j++) {
    if ((j >> A) & 1) continue;
    if ((j >> B) & 1) continue;
    if ((j & cm) != cv) continue;
    constexpr int a1 = 1 << A, b1 = 1 << B;
    const T x0r = re[j], x0i = im[j], x1r = re[j | a1], x1i = im[j | a1];
    const T x2r = re[j | b1], x2i = im[j | b1], x3r = re[j | a1 | b1], x3i = im[j | a1 | b1];
#define SVI_ROW(r, dst)                                                                   \
    {                                                                                     \
      const T ar = u[8 * r + 0] * x0r - u[8 * r + 1] * x0i + u[8 * r + 2] * x1r -         \
                   u[8 * r + 3] * x1i + u[8 * r + 4] * x2r - u[8 * r + 5] * x2i +         \
                   u[8 * r + 6] * x3r - u[8 * r + 7] * x3i;                               \
      const T ai = u[8 * r + 0] * x0i + u[8 * r + 1] * x0r + u[8 * r + 2] * x1i +         \
                   u[8 * r + 3] * x1r + u[8 * r + 4] * x2i + u[8 * r + 5] * x2r +         \
                   u[8 * r + 6] * x3i + u[8 * r + 7] * x3r;                               \
      re[dst] = ar;                                                                       \
      im[dst] = ai;                                                                       \
    }
    SVI_ROW(0, j) SVI_ROW(1, j | a1) SVI_ROW(2, j | b1) SVI_ROW(3, j | a1 | b1)
#undef SVI_ROW
  }
}

// Real rotation between the two local patterns of a two-level subspace:
// for every j with (j & tm) == pa, partner k = j ^ XM:
//   (x_j, x_k) <- (r00 x_j + r01 x_k, r10 x_j + r11 x_k).
template <typename T, int R, int XM>
__device__ __forceinline__ void mo_2l(T *re, T *im, const double *cf, uint32_t tm, uint32_t pa,
                                      uint32_t cm, uint32_t cv) {
  const T r00 = (T)cf[0], r01 = (T)cf[1], r10 = (T)cf[2], r11 = (T)cf[3];
#pragma unroll
  for (int j = 0; j < (1 << R); j++) {
    if (((uint32_t)j & tm) != pa) continue;
    if ((j & cm) != cv) continue;
    const int k = j ^ XM;
    const T xr = re[j], xi = im[j], yr = re[k], yi = im[k];
    re[j] = r00 * xr + r01 * yr;
    im[j] = r00 * xi + r01 * yi;
    re[k] = r10 * xr + r11 * yr;
    im[k] = r10 * xi + r11 * yi;
  }
}

// 2^K x 2^K on group bits 0..K-1.
template <typename T, int R, int K>
__device__ __forceinline__ void mo_dense(T *re, T *im, const double *cf, uint32_t cm,
                                         uint32_t cv) {
  constexpr int D = 1 << K;
#pragma clang loop unroll(full)
  for (int o = 0; o < (1 << (R - K)); o++) {
    const int base = o << K;
    if ((base & cm) != cv) continue;
    T xr[D], xi[D];
#pragma unroll
    for (int q = 0; q < D; q++) { xr[q] = re[base + q]; xi[q] = im[base + q]; }
#pragma unroll
    for (int r = 0; r < D; r++) {
      T ar = 0, ai = 0;
#pragma unroll
      for (int q = 0; q < D; q++) {
        const T ur = (T)cf[(r * D + q) * 2], ui = (T)cf[(r * D + q) * 2 + 1];
        ar += ur * xr[q] - ui * xi[q];
        ai += ur * xi[q] + ui * xr[q];
      }
      re[base + r] = ar;
      im[base + r] = ai;
    }
  }
}

template <typename T, int R, typename CP = const double *>
__device__ __forceinline__ void mo_diagt(T *re, T *im, CP cf) {
#pragma unroll
  for (int j = 0; j < (1 << R); j++) {
    const T dr = (T)cf[2 * j], di = (T)cf[2 * j + 1];
    const T xr = re[j], xi = im[j];
    re[j] = xr * dr - xi * di;
    im[j] = xr * di + xi * dr;
  }
}

// The same on FP32 amplitudes with the table and the products in FP64: one
// rounding for each part, none of the table, whose rounded entries shift phases
// and weights the same way all over the state.  400 expectation values of
// complex64 circuits (19 to 28 qubits, 8 to 22 layers) are 2.5e-7 off on the
// mean with it, 6.9e-7 with the table in FP32; 28 qubits, 20 layers take 21.4 ms
// against 19.2.
template <int R, typename CP>
__device__ __forceinline__ void mo_diagt_wide(float *re, float *im, CP cf) {
#pragma unroll
  for (int j = 0; j < (1 << R); j++) {
    const double dr = cf[2 * j], di = cf[2 * j + 1], xr = (double)re[j], xi = (double)im[j];
    re[j] = (float)(xr * dr - xi * di);
    im[j] = (float)(xr * di + xi * dr);
  }
}

// Im <lam| G |psi> over one group from the generator's per-slot table (see
// GRAD_ODD / GRAD_BETA in sv_internal.h); XM is the generator's x-mask.
template <typename T, int R, int XM, bool ODD, typename CP>
__device__ __forceinline__ double mo_grad(const T *pr, const T *pi, const T *lr, const T *li,
                                          CP tab) {
  constexpr int G = 1 << R;
  double acc = 0.0;
#pragma unroll
  for (int j = 0; j < G; j++) {
    const int k = j ^ XM;
    const double ljr = (double)lr[j], lji = (double)li[j];
    const double f = ODD ? ljr * (double)pr[k] + lji * (double)pi[k]
                         : ljr * (double)pi[k] - lji * (double)pr[k];
    acc += (double)tab[j] * f;
  }
  return acc;
}

// Fast-Givens rotation on group bit TB (record {form, k, scale, 0}, form 0 or
// 1; the scale is applied separately).  Gentleman's scaled rotation: each
// output is one FMA with a +-1 coefficient on one input.  F0: the form is 0
// (FP64 always, CF_FORM0; FP32 nearly always): straight-line FMAs, with no
// branch whose two arms the compiler would merge with copies.
template <typename T, int R, int TB, bool F0, typename CP>
__device__ __forceinline__ void mo_fastr(T *re, T *im, CP cf) {
  const T k = (T)cf[1];
#define SVI_FR(XR, XI, YR, YI)                                   \
  _Pragma("unroll") for (int j = 0; j < (1 << R); j++) {         \
    if (j & (1 << TB)) continue;                                 \
    const int l = j | (1 << TB);                                 \
    const T xr = re[j], xi = im[j], yr = re[l], yi = im[l];      \
    re[j] = XR; im[j] = XI; re[l] = YR; im[l] = YI;              \
  }
  if constexpr (F0) {
    SVI_FR(xr - k * yr, xi - k * yi, k * xr + yr, k * xi + yi)
  } else {
    const int form = (int)cf[0];
    if (form == 0) {
      SVI_FR(xr - k * yr, xi - k * yi, k * xr + yr, k * xi + yi)
    } else {
      SVI_FR(k * xr - yr, k * xi - yi, xr + k * yr, xi + k * yi)
    }
  }
#undef SVI_FR
}

// Static Kronecker stage: s * D_after * (R~_{R-1} (x) ... (x) R~_0) * D_before,
// in three parts so that gradient terms can be taken between them.
template <typename T, int R, typename CP>
__device__ __forceinline__ void kron_pre(T *re, T *im, CP cf, int dflags) {
  if (dflags & 1) mo_diagt<T, R>(re, im, cf + 4 * R);
}

template <typename T, int R, bool F0 = sizeof(T) == 8, typename CP>
__device__ __forceinline__ void kron_rot(T *re, T *im, CP cf, uint32_t rmask) {
  if (rmask & 1u) mo_fastr<T, R, 0, F0>(re, im, cf + 0);
  if (rmask & 2u) mo_fastr<T, R, 1, F0>(re, im, cf + 4);
  if constexpr (R > 2) { if (rmask & 4u) mo_fastr<T, R, 2, F0>(re, im, cf + 8); }
  if constexpr (R > 3) { if (rmask & 8u) mo_fastr<T, R, 3, F0>(re, im, cf + 12); }
  if constexpr (R > 4) { if (rmask & 16u) mo_fastr<T, R, 4, F0>(re, im, cf + 16); }
}

// Every group bit rotated (rmask full), no conditionals.
template <typename T, int R, bool F0 = sizeof(T) == 8, typename CP>
__device__ __forceinline__ void kron_rot_all(T *re, T *im, CP cf) {
  mo_fastr<T, R, 0, F0>(re, im, cf + 0);
  mo_fastr<T, R, 1, F0>(re, im, cf + 4);
  if constexpr (R > 2) mo_fastr<T, R, 2, F0>(re, im, cf + 8);
  if constexpr (R > 3) mo_fastr<T, R, 3, F0>(re, im, cf + 12);
  if constexpr (R > 4) mo_fastr<T, R, 4, F0>(re, im, cf + 16);
}

// Whether a stage's rotations all have form 0 (uniform, on the forms' bits).
template <typename T, int R, typename CP>
__device__ __forceinline__ bool kron_form0(CP cf, uint32_t rmask) {
  if constexpr (sizeof(T) == 8) return true;
  uint32_t f = 0;
#pragma unroll
  for (int t = 0; t < R; t++) f |= (rmask >> t) & 1u ? __float_as_uint((float)cf[4 * t]) : 0u;
  return f == 0;
}

template <typename T, int R, typename CP>
__device__ __forceinline__ void kron_post(T *re, T *im, CP cf, int dflags) {
  constexpr int G = 1 << R;
  CP ta = cf + 4 * R + 2 * G;
  if (dflags & 2) mo_diagt<T, R>(re, im, ta);
  if (dflags & 4) {
    const T sc = (T)ta[2 * G];
#pragma unroll
    for (int j = 0; j < G; j++) { re[j] *= sc; im[j] *= sc; }
  }
}

template <typename T, int R, bool F0 = sizeof(T) == 8, typename CP>
__device__ __forceinline__ void kron_stage(T *re, T *im, CP cf, uint32_t rmask, int dflags) {
  kron_pre<T, R>(re, im, cf, dflags);
  kron_rot<T, R, F0>(re, im, cf, rmask);
  kron_post<T, R>(re, im, cf, dflags);
}

#define SVI_T5(F, t, ...)                                   \
  switch (t) {                                              \
    case 0: F<T, R, 0>(__VA_ARGS__); break;                 \
    case 1: F<T, R, 1>(__VA_ARGS__); break;                 \
    case 2: if constexpr (R > 2) F<T, R, 2>(__VA_ARGS__); break; \
    case 3: if constexpr (R > 3) F<T, R, 3>(__VA_ARGS__); break; \
    case 4: if constexpr (R > 4) F<T, R, 4>(__VA_ARGS__); break; \
    default: break;                                         \
  }

template <typename T, int R>
__device__ __forceinline__ void dispatch_swap(int a, int b, T *re, T *im, uint32_t cm, uint32_t cv) {
#define SVI_SW(A, B) if (a == A && b == B) { if constexpr (A < R && B < R) mo_swap<T, R, A, B>(re, im, cm, cv); return; }
  SVI_SW(0, 1) SVI_SW(0, 2) SVI_SW(0, 3) SVI_SW(0, 4) SVI_SW(1, 0) SVI_SW(1, 2) SVI_SW(1, 3)
  SVI_SW(1, 4) SVI_SW(2, 0) SVI_SW(2, 1) SVI_SW(2, 3) SVI_SW(2, 4) SVI_SW(3, 0) SVI_SW(3, 1)
  SVI_SW(3, 2) SVI_SW(3, 4) SVI_SW(4, 0) SVI_SW(4, 1) SVI_SW(4, 2) SVI_SW(4, 3)
#undef SVI_SW
}

template <typename T, int R>
__device__ __forceinline__ void dispatch_q(int a, int b, T *re, T *im, const double *cf,
                                           uint32_t cm, uint32_t cv) {
#define SVI_Q(A, B) if (a == A && b == B) { if constexpr (A < R && B < R) mo_q<T, R, A, B>(re, im, cf, cm, cv); return; }
  SVI_Q(0, 1) SVI_Q(0, 2) SVI_Q(0, 3) SVI_Q(0, 4) SVI_Q(1, 0) SVI_Q(1, 2) SVI_Q(1, 3)
  SVI_Q(1, 4) SVI_Q(2, 0) SVI_Q(2, 1) SVI_Q(2, 3) SVI_Q(2, 4) SVI_Q(3, 0) SVI_Q(3, 1)
  SVI_Q(3, 2) SVI_Q(3, 4) SVI_Q(4, 0) SVI_Q(4, 1) SVI_Q(4, 2) SVI_Q(4, 3)
#undef SVI_Q
}

template <typename T, int R>
__device__ __forceinline__ void apply_op(const MicroOp &op, T *re, T *im, const double *coef) {
  const double *cf = coef + op.coef;
  switch (op.type) {
    case MO_U: SVI_T5(mo_u, op.t0, re, im, cf, op.cm, op.cv) break;
    case MO_R: SVI_T5(mo_r, op.t0, re, im, cf, op.cm, op.cv) break;
    case MO_P: mo_p<T, R>(re, im, cf, op.mask, op.cm, op.cv); break;
    case MO_X:
      switch (op.t0) {
        case 0: mo_x<T, R, 0>(re, im, op.cm, op.cv); break;
        case 1: mo_x<T, R, 1>(re, im, op.cm, op.cv); break;
        case 2: if constexpr (R > 2) mo_x<T, R, 2>(re, im, op.cm, op.cv); break;
        case 3: if constexpr (R > 3) mo_x<T, R, 3>(re, im, op.cm, op.cv); break;
        case 4: if constexpr (R > 4) mo_x<T, R, 4>(re, im, op.cm, op.cv); break;
        default: break;
      }
      break;
    case MO_SWAP: dispatch_swap<T, R>(op.t0, op.t1, re, im, op.cm, op.cv); break;
    case MO_NEG: mo_neg<T, R>(re, im, op.cm, op.cv); break;
    case MO_Q: dispatch_q<T, R>(op.t0, op.t1, re, im, cf, op.cm, op.cv); break;
    case MO_DENSE:
      switch (op.mask) {
        case 1: mo_dense<T, R, 1>(re, im, cf, op.cm, op.cv); break;
        case 2: mo_dense<T, R, 2>(re, im, cf, op.cm, op.cv); break;
        case 3: if constexpr (R >= 3) mo_dense<T, R, 3>(re, im, cf, op.cm, op.cv); break;
        default: break;
      }
      break;
    case MO_DIAGT: mo_diagt<T, R>(re, im, cf); break;
    case MO_2L:
      switch (op.t1) {
#define SVI_L(XV) case XV: if constexpr (XV < (1 << R)) mo_2l<T, R, XV>(re, im, cf, op.mask, op.gz, op.cm, op.cv); break;
        SVI_L(1) SVI_L(2) SVI_L(3) SVI_L(4) SVI_L(5) SVI_L(6) SVI_L(7) SVI_L(8) SVI_L(9) SVI_L(10)
        SVI_L(11) SVI_L(12) SVI_L(13) SVI_L(14) SVI_L(15) SVI_L(16) SVI_L(17) SVI_L(18) SVI_L(19)
        SVI_L(20) SVI_L(21) SVI_L(22) SVI_L(23) SVI_L(24) SVI_L(25) SVI_L(26) SVI_L(27) SVI_L(28)
        SVI_L(29) SVI_L(30) SVI_L(31)
#undef SVI_L
        default: break;
      }
      break;
    default: break;
  }
}

// Im <lam| G |psi> over one group for the generator of a two-level rotation
// between the slot patterns a ((j & tm) == pa) and b = a ^ XM: G a = i b,
// G b = -i a, so the term is Re(conj(lam_b) psi_a) - Re(conj(lam_a) psi_b).
template <typename T, int R, int XM>
__device__ __forceinline__ double mo_grad2l(const T *pr, const T *pi, const T *lr, const T *li,
                                            uint32_t tm, uint32_t pa, uint32_t cm, uint32_t cv) {
  double acc = 0.0;
#pragma unroll
  for (int j = 0; j < (1 << R); j++) {
    if (((uint32_t)j & tm) != pa) continue;
    if ((j & cm) != cv) continue;
    const int k = j ^ XM;
    acc += ((double)lr[k] * (double)pr[j] + (double)li[k] * (double)pi[j]) -
           ((double)lr[j] * (double)pr[k] + (double)li[j] * (double)pi[k]);
  }
  return acc;
}

// MO_GRAD: generator alpha * (Pauli string) + beta * I on the control subspace,
// through its per-slot table in the coefficient buffer.
template <typename T, int R>
__device__ __forceinline__ double grad_op(const MicroOp &op, const T *pr, const T *pi, const T *lr,
                                          const T *li, const double *coef) {
  const SVI_CONST double *tab = cptr(coef) + op.t0;
  const uint32_t x = op.mask;   // x-mask over group bits
  // diagonal generators (Z strings, phases): one table, the even form on j itself
  if (x == 0) return mo_grad<T, R, 0, false>(pr, pi, lr, li, tab);
  const bool odd = (op.t1 & GRAD_ODD) != 0;
  switch (x) {
#define SVI_G(XV) case XV: if constexpr (XV < (1 << R)) { \
      if (odd) return mo_grad<T, R, XV, true>(pr, pi, lr, li, tab); \
      return mo_grad<T, R, XV, false>(pr, pi, lr, li, tab); } break;
    SVI_G(1) SVI_G(2) SVI_G(3) SVI_G(4) SVI_G(5) SVI_G(6) SVI_G(7) SVI_G(8) SVI_G(9)
    SVI_G(10) SVI_G(11) SVI_G(12) SVI_G(13) SVI_G(14) SVI_G(15) SVI_G(16) SVI_G(17) SVI_G(18)
    SVI_G(19) SVI_G(20) SVI_G(21) SVI_G(22) SVI_G(23) SVI_G(24) SVI_G(25) SVI_G(26) SVI_G(27)
    SVI_G(28) SVI_G(29) SVI_G(30) SVI_G(31)
#undef SVI_G
    default: break;
  }
  return 0.0;
}

// Gradient of an uncontrolled RY on group bit TB (generator Y):
// Im <lam| Y |psi> over one group.
template <typename T, int R, int TB>
__device__ __forceinline__ double ry_grad(const T *pr, const T *pi, const T *lr, const T *li) {
  double up = 0.0, down = 0.0;
#pragma unroll
  for (int j = 0; j < (1 << R); j++) {
    if (j & (1 << TB)) continue;
    const int k = j | (1 << TB);
    up += (double)lr[k] * (double)pr[j] + (double)li[k] * (double)pi[j];
    down += (double)lr[j] * (double)pr[k] + (double)li[j] * (double)pi[k];
  }
  return up - down;
}

template <typename T, int R>
__device__ __forceinline__ double ry_grad_at(int t, const T *pr, const T *pi, const T *lr,
                                             const T *li) {
  switch (t) {
    case 0: return ry_grad<T, R, 0>(pr, pi, lr, li);
    case 1: return ry_grad<T, R, 1>(pr, pi, lr, li);
    case 2: if constexpr (R > 2) return ry_grad<T, R, 2>(pr, pi, lr, li); break;
    case 3: if constexpr (R > 3) return ry_grad<T, R, 3>(pr, pi, lr, li); break;
    case 4: if constexpr (R > 4) return ry_grad<T, R, 4>(pr, pi, lr, li); break;
    default: break;
  }
  return 0.0;
}

// Gradient slot of a Kronecker stage's RY on group bit t (StageDesc::ry; -1: none).
__device__ __forceinline__ int ry_slot(const SVI_CONST StageDesc &sd, int t) {
  const uint32_t v = (sd.ry[t >> 1] >> (16 * (t & 1))) & 0xffffu;
  return v == 0xffffu ? -1 : (int)v;
}

// MO_GRAD or MO_GRAD2L (the micro-op interpreter; Kronecker stages hold MO_GRAD only).
template <typename T, int R>
__device__ __forceinline__ double grad_any(const MicroOp &op, const T *pr, const T *pi,
                                           const T *lr, const T *li, const double *coef) {
  if (op.type == MO_GRAD2L) {
    switch (op.t1) {
#define SVI_G2(XV) case XV: if constexpr (XV < (1 << R)) return mo_grad2l<T, R, XV>(pr, pi, lr, li, op.mask, op.gz, op.cm, op.cv); break;
      SVI_G2(3) SVI_G2(5) SVI_G2(6) SVI_G2(9) SVI_G2(10) SVI_G2(12) SVI_G2(15) SVI_G2(17)
      SVI_G2(18) SVI_G2(20) SVI_G2(23) SVI_G2(24) SVI_G2(27) SVI_G2(29) SVI_G2(30)
#undef SVI_G2
      default: break;
    }
    return 0.0;
  }
  return grad_op<T, R>(op, pr, pi, lr, li, coef);
}

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// ------------------------------------------------------------ tile sweep
// One persistent workgroup loops over tiles.  NS = 1 (forward) or 2 (adjoint:
// state 0 = psi, state 1 = lambda, micro-ops applied to both, MO_GRAD
// accumulates gradient partials).

#define SVI_GSLOTS 256
#define SVI_GSLOTS_WIDE 128  // gradient slots per sweep of the two-state Kronecker kernel

// Sum of v over the 64 lanes of a wave, valid in lane 63, by DPP lane moves
// (VALU only): partial sums within rows of 16 lanes (shifts by 1, 2, 4, 8),
// then row 0 into row 1 and row 2 into row 3 (broadcast of lane 15), then
// rows 0-1 into rows 2-3 (broadcast of lane 31).  Lanes outside a shift's row
// read 0.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ double dpp_d(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(b & 0xffffffffll), CTRL, ROW_MASK, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, ROW_MASK, 0xf, true);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

__device__ __forceinline__ double wave_total63(double v) {
  v += dpp_d<0x111, 0xf>(v);   // row_shr:1
  v += dpp_d<0x112, 0xf>(v);   // row_shr:2
  v += dpp_d<0x114, 0xf>(v);   // row_shr:4
  v += dpp_d<0x118, 0xf>(v);   // row_shr:8
  v += dpp_d<0x142, 0xa>(v);   // row_bcast:15 into rows 1 and 3
  v += dpp_d<0x143, 0xc>(v);   // row_bcast:31 into rows 2 and 3
  return v;
}

// Swaps the upper 32 lanes of x with the lower 32 lanes of y (64-bit values,
// v_permlane32_swap on each half).
__device__ __forceinline__ void swap32_d(double &x, double &y) {
  const long long xb = __double_as_longlong(x), yb = __double_as_longlong(y);
  const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)xb, (unsigned)yb, false, false);
  const auto hi =
      __builtin_amdgcn_permlane32_swap((unsigned)(xb >> 32), (unsigned)(yb >> 32), false, false);
  x = __longlong_as_double(((long long)hi[0] << 32) | (unsigned)lo[0]);
  y = __longlong_as_double(((long long)hi[1] << 32) | (unsigned)lo[1]);
}

// Sums over the 64 lanes of a wave of two per-lane values in one chain: the
// halves exchange and add, so that lanes 0-31 hold half-sums of v0 and lanes
// 32-63 of v1; row shifts by 1, 2, 4, 8 sum each row of 16 lanes, and the
// broadcast of lane 15 into rows 1 and 3 adds row 0 to row 1 and row 2 to
// row 3.  The total of v0 is valid in lane 31, that of v1 in lane 63: 18 VALU
// instructions for both, against 18 for each through wave_total63.  Needs
// every lane of the wave active.
__device__ __forceinline__ double wave_total2(double v0, double v1) {
  swap32_d(v0, v1);
  double t = v0 + v1;
  t += dpp_d<0x111, 0xf>(t);   // row_shr:1
  t += dpp_d<0x112, 0xf>(t);   // row_shr:2
  t += dpp_d<0x114, 0xf>(t);   // row_shr:4
  t += dpp_d<0x118, 0xf>(t);   // row_shr:8
  t += dpp_d<0x142, 0xa>(t);   // row_bcast:15 into rows 1 and 3
  return t;
}

// Adds the two wave totals of wave_total2 to slots s0 and s1 of the wave's LDS
// row (a slot < 0: none) with adds that return nothing, lanes 31 and 63.
__device__ __forceinline__ void wave_deposit2(double *row, int s0, int s1, double t, int lane) {
  const int slot = lane == 31 ? s0 : s1;
  if ((lane == 31 || lane == 63) && slot >= 0) atomicAdd(&row[slot], t);
}

template <typename T, int M, int R, int NS>
__global__ void __launch_bounds__(1 << (M - R)) k_sweep(SweepArgs a) {
  constexpr int NT = 1 << (M - R);
  constexpr int G = 1 << R;
  constexpr int VN = V4T<T>::N;
  constexpr int LV = VN == 2 ? 1 : 2;
  constexpr int NIT = (1 << M) / (VN * NT);   // vector loads per thread per plane (full tile)
  constexpr int NWAVE = (NT + 63) / 64;
  using C2 = typename C2T<T>::type;
  using V4 = typename V4T<T>::type;
  __shared__ C2 lds[NS][1 << M];
  __shared__ double wsum[NS == 2 ? NWAVE : 1][NS == 2 ? SVI_GSLOTS : 1];
  __shared__ double gacc[NS == 2 ? SVI_GSLOTS : 1];
  __shared__ int32_t hb_s[SVI_MMAX];

  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int m = a.m, c = a.c, nh = a.nh;
  const int mm = m > R ? m : R;              // tile bits including phantom padding
  const int ntile_el = 1 << m;               // real amplitudes per tile
  const int ngroups = 1 << (mm - R);
  const bool vec = c >= LV;                  // rows hold whole 16-byte vectors

  if (tid < SVI_MMAX) hb_s[tid] = a.hb[tid < nh ? tid : 0];
  if constexpr (NS == 2) {
    for (int s = tid; s < SVI_GSLOTS; s += NT) gacc[s] = 0.0;
  }
  __syncthreads();

  // Row offsets of this thread's elements, the same for every tile.
  uint64_t roff[NIT];
#pragma unroll
  for (int k = 0; k < NIT; k++) {
    const int i = (tid + k * NT) * (vec ? VN : 1);
    roff[k] = spread_row(i >> c, hb_s, nh) + (uint64_t)(i & ((1 << c) - 1));
  }

  const int tsw = swz<T>(tid * VN);          // swizzled slot of this thread's first element
  T *const pre0 = (T *)a.re, *const pim0 = (T *)a.im;
  T *const pre1 = (T *)a.re2, *const pim1 = (T *)a.im2;

  for (int64_t tile = blockIdx.x; tile < a.ntiles; tile += gridDim.x) {
    const uint64_t base = tile_base(tile, c, hb_s, nh);
    // ---- load tile (rows of 2^c contiguous amplitudes) into LDS
    if (mm > m) {
      for (int i = tid; i < (1 << mm); i += NT) {
        lds[0][swz<T>(i)] = C2{0, 0};
        if constexpr (NS == 2) lds[1][swz<T>(i)] = C2{0, 0};
      }
      __syncthreads();
    }
#pragma unroll
    for (int s = 0; s < NS; s++) {
      const T *pr = s == 0 ? pre0 : pre1;
      const T *pi = s == 0 ? pim0 : pim1;
      if (s == 0 && (a.flags & SW_INIT_ZERO)) {
        for (int i = tid; i < ntile_el; i += NT) {
          const T v = (base == 0 && i == 0) ? (T)1 : (T)0;
          lds[0][swz<T>(i)] = C2{v, 0};
        }
      } else if (vec) {
#pragma unroll
        for (int k = 0; k < NIT; k++) {
          const int i = (tid + k * NT) * VN;
          if (i < ntile_el) {
            const uint64_t g = base + roff[k];
            const V4 vr = *(const V4 *)(pr + g);
            const V4 vi = *(const V4 *)(pi + g);
            const int si = tsw ^ swz<T>(k * NT * VN);
            if constexpr (VN == 2) {
              lds[s][si] = C2{vr.x, vi.x};
              lds[s][si ^ 1] = C2{vr.y, vi.y};
            } else {
              lds[s][si] = C2{vr.x, vi.x};
              lds[s][si ^ 1] = C2{vr.y, vi.y};
              lds[s][si ^ 2] = C2{vr.z, vi.z};
              lds[s][si ^ 3] = C2{vr.w, vi.w};
            }
          }
        }
      } else {
        for (int i = tid; i < ntile_el; i += NT) {
          const uint64_t g = base + spread_row(i >> c, hb_s, nh) + (uint64_t)(i & ((1 << c) - 1));
          lds[s][swz<T>(i)] = C2{pr[g], pi[g]};
        }
      }
    }
    __syncthreads();

    // ---- stages
    for (int st = a.stage_begin; st < a.stage_end; st++) {
      const SVI_CONST StageDesc &sd = cptr(a.stages)[st];
      // Every thread runs the stage (keeps wave shuffles uniform).  Threads
      // beyond the tile's groups work on LDS slots above 2^mm, which are
      // never written back.
      const bool active = tid < ngroups;
      const int gbs =
          (swz<T>(lane_base(tid & 63, sd)) ^ swz<T>(wave_base<M, R>(wave, sd))) * (int)sizeof(C2);
      T re[NS][G], im[NS][G];
#pragma unroll
      for (int s = 0; s < NS; s++) {
        const char *lb = (const char *)lds[s];
#pragma unroll
        for (int j = 0; j < G; j++) {
          const C2 v = *(const C2 *)(lb + (gbs ^ sd.off[j]));
          re[s][j] = v.x;
          im[s][j] = v.y;
        }
      }
      if (sd.kind == ST_KRON) {
        const SVI_CONST double *kc = cptr(a.coef) + sd.kcoef;
        if constexpr (NS == 2) {
          // gradient terms Im <lam| G |psi> at the stage point where each
          // record's generator commutes with the rest of the stage; terms taken
          // after the fast-Givens rotations see both states divided by the
          // stage scale s, so they are multiplied by s^2
          auto grads = [&](int b, int e, double mult) {
            for (int o = b; o < e; o++) {
              const MicroOp op = op_at(a.ops, o);
              double v = active ? mult * mo_grad<T, R, 0, false>(re[0], im[0], re[1], im[1],
                                                                 cptr(a.coef) + op.t0) : 0.0;
              v = wave_sum(v);
              if ((tid & 63) == 0) wsum[tid >> 6][op.coef] = v;
            }
          };
          grads(sd.op_begin, sd.g1, 1.0);
          kron_pre<T, R>(re[0], im[0], kc, sd.dflags);
          kron_pre<T, R>(re[1], im[1], kc, sd.dflags);
          for (int t = 0; t < R; t++) {
            const int slot = ry_slot(sd, t);
            if (slot < 0) continue;
            const double v = wave_sum(active ? ry_grad_at<T, R>(t, re[0], im[0], re[1], im[1]) : 0.0);
            if ((tid & 63) == 0) wsum[tid >> 6][slot] = v;
          }
          kron_rot<T, R>(re[0], im[0], kc, sd.rmask);
          kron_rot<T, R>(re[1], im[1], kc, sd.rmask);
          if (sd.g1 < sd.op_end) {
            const double sc = kc[4 * R + 4 * G];
            grads(sd.g1, sd.op_end, sc * sc);
          }
          kron_post<T, R>(re[0], im[0], kc, sd.dflags);
          kron_post<T, R>(re[1], im[1], kc, sd.dflags);
        } else {
          kron_stage<T, R>(re[0], im[0], kc, sd.rmask, sd.dflags);
        }
      } else
      for (int o = sd.op_begin; o < sd.op_end; o++) {
        const MicroOp op = op_at(a.ops, o);
        if constexpr (NS == 2) {
          if (op.type == MO_GRAD || op.type == MO_GRAD2L) {
            double v = active ? grad_any<T, R>(op, re[0], im[0], re[1], im[1], a.coef) : 0.0;
            v = wave_sum(v);
            if ((tid & 63) == 0) wsum[tid >> 6][op.coef] = v;
            continue;
          }
        }
        apply_op<T, R>(op, re[0], im[0], a.coef);
        if constexpr (NS == 2) apply_op<T, R>(op, re[1], im[1], a.coef);
      }
      if (sd.dflags & SD_XCHG) lds_barrier();
#pragma unroll
      for (int s = 0; s < NS; s++) {
        char *lb = (char *)lds[s];
#pragma unroll
        for (int j = 0; j < G; j++) *(C2 *)(lb + (gbs ^ sd.off[G + j])) = C2{re[s][j], im[s][j]};
      }
      __syncthreads();
    }

    if constexpr (NS == 2) {
      // fold this tile's per-wave sums into the workgroup accumulators
      for (int s = tid; s < a.n_gslots; s += NT) {
        double v = 0.0;
        for (int w = 0; w < NWAVE; w++) v += wsum[w][s];
        gacc[s] += v;
      }
    }

    // ---- store tile (through the output bit permutation of a remapping sweep)
    const bool operm = (a.flags & SW_OPERM) != 0;
#pragma unroll
    for (int s = 0; s < NS; s++) {
      T *pr = s == 0 ? pre0 : pre1;
      T *pi = s == 0 ? pim0 : pim1;
      if (vec) {
        const int so1 = operm ? swz<T>(perm_bits(1, a.operm, m)) : 1;
        const int so2 = operm ? swz<T>(perm_bits(2, a.operm, m)) : 2;
#pragma unroll
        for (int k = 0; k < NIT; k++) {
          const int i = (tid + k * NT) * VN;
          if (i < ntile_el) {
            const uint64_t g = base + roff[k];
            const int si = operm ? swz<T>(perm_bits(i, a.operm, m)) : tsw ^ swz<T>(k * NT * VN);
            V4 vr, vi;
            if constexpr (VN == 2) {
              const C2 p0 = lds[s][si], p1 = lds[s][si ^ so1];
              vr = V4{p0.x, p1.x};
              vi = V4{p0.y, p1.y};
            } else {
              const C2 p0 = lds[s][si], p1 = lds[s][si ^ so1];
              const C2 p2 = lds[s][si ^ so2], p3 = lds[s][si ^ so1 ^ so2];
              vr = V4{p0.x, p1.x, p2.x, p3.x};
              vi = V4{p0.y, p1.y, p2.y, p3.y};
            }
            *(V4 *)(pr + g) = vr;
            *(V4 *)(pi + g) = vi;
          }
        }
      } else {
        for (int i = tid; i < ntile_el; i += NT) {
          const uint64_t g = base + spread_row(i >> c, hb_s, nh) + (uint64_t)(i & ((1 << c) - 1));
          const C2 p = lds[s][swz<T>(operm ? perm_bits(i, a.operm, m) : i)];
          pr[g] = p.x;
          pi[g] = p.y;
        }
      }
    }
    __syncthreads();
  }

  if constexpr (NS == 2) {
    for (int s = tid; s < a.n_gslots; s += NT)
      a.gpart[(int64_t)(a.gslot_begin + s) * gridDim.x + blockIdx.x] = gacc[s];
  }
}


// ------------------------------------------------- Kronecker-only sweep
// Lean variant for sweeps whose every stage is a Kronecker stage or (DN) a dense
// one.  Stage descriptors and coefficients are uniform and read with scalar loads; LDS
// holds only the tile, and the code holds only the static stage body, so the
// register groups stay in VGPRs with no interpreter paths competing for them.

// Tile order: XCD-aware.  Workgroup b runs on XCD b % 8; in every round the
// workgroups of one XCD take a contiguous run of tiles, so tiles that share
// HBM lines and DRAM pages are fetched through the same L2 at the same time.
__device__ __forceinline__ int64_t tile_of(int64_t round_base, int b, int grid) {
  const int per = grid >> 3;
  return grid >= 8 && (grid & 7) == 0 ? round_base + (int64_t)(b & 7) * per + (b >> 3)
                                      : round_base + b;
}

// A dense stage (ST_DENSE) on a group held in registers: output row r, formed
// from row r of the matrix, goes to out(r).  Entries that are exactly zero
// (nz) are passed over: gates on fewer qubits than the group, controlled ones
// and permutations leave most of the matrix empty, and an amplitude that is
// not finite stays where the gates leave it.  The entries are uniform: a row
// is held in SGPRs.  Measured over 200 gates of all kinds on 27 qubits: every
// entry formed 40.8 ms (bound by the FP64 FMAs), a branch per entry 28.4 ms
// (31 sweeps, 0.92 ms each: near the 0.88 ms that the state's traffic takes),
// with a copy for full rows besides 29.6, real and imaginary parts branched
// separately 32.2.
template <int R, typename Out>
__device__ __forceinline__ void dense_rows(const double *re, const double *im,
                                           const SVI_CONST double *u, Out out) {
  constexpr int G = 1 << R;
  const uint64_t nz = *(const SVI_CONST uint64_t *)(u + 2 * G * G);
#pragma unroll
  for (int r = 0; r < G; r++) {
    double c[2 * G];
#pragma unroll
    for (int q = 0; q < 2 * G; q++) c[q] = u[2 * G * r + q];
#pragma unroll
    for (int q = 0; q < 2 * G; q++) asm volatile("" : "+s"(c[q]));
    const uint32_t row = (uint32_t)(nz >> (G * r)) & ((1u << G) - 1);
    double ar = 0, ai = 0;
    auto entry = [&](int q) {
      ar = fma(c[2 * q], re[q], ar);
      ai = fma(c[2 * q], im[q], ai);
      ar = fma(-c[2 * q + 1], im[q], ar);
      ai = fma(c[2 * q + 1], re[q], ai);
    };
#pragma unroll
    for (int q = 0; q < G; q++) {
      if (!((row >> q) & 1u)) continue;
      asm volatile("" ::);   // a branch: the compiler would form every entry and select
      entry(q);
    }
    out(r, ar, ai);
  }
}

// DN: the sweep has dense stages too (FP64).
template <typename T, int M, int R, bool DN = false>
__global__ void __launch_bounds__(1 << (M - R)) k_sweep_kron(SweepArgs a) {
  constexpr int NT = 1 << (M - R);
  constexpr int G = 1 << R;
  using C2 = typename C2T<T>::type;
  // Per-stage thread bases (tile-local slot offset of the thread's register
  // group) depend on the thread and the stage, not on the tile: a workgroup
  // that runs several tiles takes those of the first GTAB stages from a table
  // built once per launch in the LDS the tile leaves free (sized so the
  // workgroups per CU stay as they are).  One that runs a single tile forms
  // them as it goes: building the table cost it 3 us a launch (21 qubits in
  // 13-bit tiles, 11 sweeps: 619 -> 588 us a pass), while forming them in every tile costs the
  // large states 2% (30 qubits: 202 -> 207 ms).
  constexpr int TILE_BYTES = (1 << M) * (int)sizeof(C2);
  constexpr int GTAB_BYTES = TILE_BYTES >= 131072 ? 30720 : TILE_BYTES >= 65536 ? 14336 : 6144;
  constexpr int GTAB = GTAB_BYTES / (2 * NT) > 0 ? GTAB_BYTES / (2 * NT) : 1;
  __shared__ C2 lds[1 << M];
  __shared__ int32_t hb_s[SVI_MMAX];
  __shared__ uint16_t gtab[GTAB * NT];   // swizzled element index (tiles hold <= 2^14)

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int m = a.m, c = a.c, nh = a.nh;
  const int ntile_el = 1 << m;
  const bool init0 = (a.flags & SW_INIT_ZERO) != 0;
  const SVI_CONST StageDesc *stages = cptr(a.stages + a.stage_begin);
  const int nst = a.stage_end - a.stage_begin;
  // FP32: the rotations' coefficients are rounded once, where they are formed
  // (28 qubits, 20 layers, 5-qubit groups: 33.9 ms with every wave converting
  // all of a stage's at every use and a branch on each rotation's form, 30.3
  // with neither); the tables stay in FP64 (mo_diagt_wide).
  const SVI_CONST T *coef;
  if constexpr (sizeof(T) == 8) coef = cptr(a.coef);
  else coef = cptr(a.coef32);

  if (tid < SVI_MMAX) hb_s[tid] = a.hb[tid < nh ? tid : 0];
  auto base_of = [&](int st) {
    return swz<T>(lane_base(lane, stages[st])) ^ swz<T>(wave_base<M, R>(wave, stages[st]));
  };
  const int ntab = a.ntiles <= gridDim.x ? 0 : nst < GTAB ? nst : GTAB;
  for (int st = 0; st < ntab; st++)   // each thread reads back only its own entries
    gtab[st * NT + tid] = (uint16_t)base_of(st);
  // waves whose threads hold no part of a small state (m < M) have no group
  const bool on = wave * 64 < (m > R ? 1 << (m - R) : 1);
  __syncthreads();

  // Lane tid moves tile elements i = tid + k * NT (k < G) between HBM and
  // LDS, one amplitude per access: consecutive lanes take consecutive
  // addresses along the tile's contiguous qubits, and every loaded value is
  // already the register that the (re, im) LDS write takes.  (Loading pairs
  // of amplitudes of one plane would need a register shuffle into (re, im)
  // pairs, which the compiler places, with a wait for the load, right after
  // the load.)
  //
  // Element i sits at tile_base + tile_off(i); tile_off is a bit deposit, so
  // it splits over the disjoint bit fields of tid and k * NT into a per-lane
  // part and wave-uniform parts.  Past the end of a small tile (i >= 2^m) the
  // deposit drops the missing tile bits, so the address stays inside the tile:
  // loads there are issued (and discarded) rather than branched around, and
  // stores are skipped.
  const uint64_t loff = tile_off(tid, c, hb_s, nh);
  uint64_t kb[R];
#pragma unroll
  for (int r = 0; r < R; r++) kb[r] = tile_off(NT << r, c, a.hb, nh);
  uint64_t loff_p;
  auto goff = [&](int k) {
    uint64_t o = loff_p;
#pragma unroll
    for (int r = 0; r < R; r++)
      if ((k >> r) & 1) o += kb[r];
    return o;
  };
  // LDS slots: element i is written to swz(i) and, for the store, read from
  // swz(P(i)) with P the identity or the output bit permutation of a
  // remapping sweep; swz and P are linear over XOR, so each is a per-lane
  // slot XOR wave-uniform parts.
  const bool operm = (a.flags & SW_OPERM) != 0;
  const int tsl = swz<T>(tid);
  const int ssl = swz<T>(operm ? perm_bits(tid, a.operm, m) : tid);
  int wsb[R], ssb[R];
#pragma unroll
  for (int r = 0; r < R; r++) {
    wsb[r] = swz<T>(NT << r);
    ssb[r] = swz<T>(operm ? perm_bits(NT << r, a.operm, m) : NT << r);
  }
  auto slot = [&](int base, const int *sb, int k) {
    int o = base;
#pragma unroll
    for (int r = 0; r < R; r++)
      if ((k >> r) & 1) o ^= sb[r];
    return o;
  };
  T *const pre = (T *)a.re, *const pim = (T *)a.im;
  char *const lb = (char *)lds;
  // tile t's base: t's bits deposited on the qubits outside the tile (for a
  // sparse sweep, on those of them inside the support only)
  const bool sparse = (a.flags & SW_SPARSE) != 0;
  auto tbase = [&](int64_t t) {
    return sparse ? tile_base(t, c, a.bz, a.nbz) : tile_base(t, c, hb_s, nh);
  };
  // The per-lane bases are re-declared opaque before each phase, so the
  // compiler recomputes the (cheap) per-element addresses next to their use
  // instead of hoisting all of them out of the tile loop and spilling them:
  // a scratch reload would wait on every outstanding HBM access.
  loff_p = loff;
  int tsl_p = tsl, ssl_p = ssl;
  auto opaque = [](auto &v) { asm volatile("" : "+v"(v)); };

  // Software pipeline: the next tile's HBM loads are issued into registers
  // before the current tile's stages run, so their latency hides behind the
  // LDS / VALU work, and the current tile's stores drain behind the next
  // tile's stages.  Inside the loop the next tile enters LDS after this
  // tile's stores, on one straight path: every HBM access sits in fixed-count
  // unrolled code, so the wait for the loads leaves the stores (issued after
  // them) in flight.  The loop is instantiated separately for a sweep that
  // synthesises |0..0> (no loads), so neither copy merges a path with loads
  // in flight into one without.  A full tile (m == M, every n >= M) takes a
  // copy with no per-element guards, so no HBM access or LDS write sits
  // under a lane branch whose skipped path would make the waits conservative.
  auto run = [&](auto synth, auto full) {
    constexpr bool I0 = decltype(synth)::value;
    constexpr bool FULL = decltype(full)::value;
    T nr[G], ni[G];
    auto fetch = [&](int64_t t) {
      const uint64_t b0 = tbase(t);
#pragma unroll
      for (int k = 0; k < G; k++) {
        const uint64_t g = b0 + goff(k);
        nr[k] = pre[g];
        ni[k] = pim[g];
      }
    };
    auto tile_in = [&](int64_t t) {
      opaque(tsl_p);
#pragma unroll
      for (int k = 0; k < G; k++) {
        if (FULL || tid + k * NT < ntile_el) {
          if constexpr (I0) {
            const T v = (t == 0 && tid + k * NT == 0) ? (T)1 : (T)0;
            lds[slot(tsl_p, wsb, k)] = C2{v, 0};
          } else {
            lds[slot(tsl_p, wsb, k)] = C2{nr[k], ni[k]};
          }
        }
      }
    };
    // Prefetch distance one tile: the loads of tile t+1 are issued right after
    // tile t enters LDS (in the same straight-line block that consumed the
    // previous prefetch registers, so no wait precedes them) and run behind
    // tile t's stages; tile t's stores drain behind tile t+1's stages.
    int64_t r0 = 0;
    int64_t tile = tile_of(0, blockIdx.x, gridDim.x);
    if (tile >= a.ntiles) return;
    int64_t next = tile_of(r0 + gridDim.x, blockIdx.x, gridDim.x);
    if constexpr (!I0) fetch(tile);
    tile_in(tile);
    lds_barrier();
    if constexpr (!I0) {
      if (next < a.ntiles) {
        opaque(loff_p);
        fetch(next);
      }
    }

    while (true) {
      const uint64_t base = tbase(tile);
      // From |0..0> only tile 0 holds a nonzero amplitude, and a sweep's
      // gates act within tiles, so every other tile stays zero: it skips the
      // stages and is written as zeros (uniform over the workgroup).
      const bool live = !I0 || tile == 0;
      // ---- stages
      for (int st = 0; live && st < nst; st++) {
        const SVI_CONST StageDesc &sd = stages[st];
        const int gbs = (st < ntab ? (int)gtab[st * NT + tid] : base_of(st)) * (int)sizeof(C2);
        // The common stage (every group bit rotated, then D_after) runs as its
        // own straight-line body from loads to stores; the general body
        // branches on the stage's parts, and in FP32 a third one on the forms
        // too.  Separate bodies leave nothing to merge, so none pays register
        // copies for another's branches.
        auto body = [&](auto full_stage, auto form0) {
          constexpr bool F0 = decltype(form0)::value;
          T re[G], im[G];
#pragma unroll
          for (int j = 0; j < G; j++) {
            const C2 v = *(const C2 *)(lb + (gbs ^ sd.off[j]));
            re[j] = v.x;
            im[j] = v.y;
          }
          const SVI_CONST double *tab = cptr(a.coef) + sd.kcoef + 4 * R;
          if constexpr (decltype(full_stage)::value) {
            kron_rot_all<T, R, F0>(re, im, coef + sd.kcoef);
            if constexpr (sizeof(T) == 4) mo_diagt_wide<R>(re, im, tab + 2 * G);
            else mo_diagt<T, R>(re, im, tab + 2 * G);
          } else if constexpr (sizeof(T) == 4) {
            if (sd.dflags & 1) mo_diagt_wide<R>(re, im, tab);
            kron_rot<T, R, F0>(re, im, coef + sd.kcoef, sd.rmask);
            if (sd.dflags & 2) mo_diagt_wide<R>(re, im, tab + 2 * G);
            if (sd.dflags & 4) kron_post<T, R>(re, im, coef + sd.kcoef, 4);
          } else {
            kron_stage<T, R, F0>(re, im, coef + sd.kcoef, sd.rmask, sd.dflags);
          }
          if (sd.dflags & SD_XCHG) lds_barrier();
#pragma unroll
          for (int j = 0; j < G; j++) *(C2 *)(lb + (gbs ^ sd.off[G + j])) = C2{re[j], im[j]};
        };
        bool dense = false;
        if constexpr (DN) dense = sd.kind == ST_DENSE;
        if (!FULL && !on) {
          if (sd.dflags & SD_XCHG) lds_barrier();
        } else if (dense) {
          if constexpr (DN) {
            if (((uint32_t)tid & sd.pm) == sd.pv) {
              T re[G], im[G];
#pragma unroll
              for (int j = 0; j < G; j++) {
                const C2 v = *(const C2 *)(lb + (gbs ^ sd.off[j]));
                re[j] = v.x;
                im[j] = v.y;
              }
              dense_rows<R>(re, im, coef + sd.kcoef, [&](int r, T x, T y) {
                *(C2 *)(lb + (gbs ^ sd.off[r])) = C2{x, y};
              });
            }
          }
        } else if (!kron_form0<T, R>(coef + sd.kcoef, sd.rmask)) {
          if constexpr (sizeof(T) == 4) body(std::false_type{}, std::false_type{});
        } else if (sd.rmask == (1u << R) - 1 && (sd.dflags & 7) == 2) {
          body(std::true_type{}, std::true_type{});
        } else {
          body(std::false_type{}, std::true_type{});
        }
        if (sd.dflags & SD_WLOCAL) {
          // the next stage reads only slots this wave wrote: keep the wave's
          // LDS accesses in order, no workgroup barrier
          __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
          __builtin_amdgcn_wave_barrier();
          __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
        } else {
          lds_barrier();
        }
      }
      // ---- LDS to HBM
      opaque(ssl_p);
      opaque(loff_p);
      if (live) {
#pragma unroll
        for (int k = 0; k < G; k++) {
          if (FULL || tid + k * NT < ntile_el) {
            const C2 p = lds[slot(ssl_p, ssb, k)];
            const uint64_t g = base + goff(k);
            pre[g] = p.x;
            pim[g] = p.y;
          }
        }
      } else {
#pragma unroll
        for (int k = 0; k < G; k++) {
          if (FULL || tid + k * NT < ntile_el) {
            const uint64_t g = base + goff(k);
            pre[g] = (T)0;
            pim[g] = (T)0;
          }
        }
      }
      lds_barrier();
      if (next >= a.ntiles) break;
      // ---- next tile into LDS (a synthesised sweep's later tiles are zero:
      // nothing to stage), then the prefetch of the one after
      if (!I0) tile_in(next);
      lds_barrier();
      r0 += gridDim.x;
      tile = next;
      next = tile_of(r0 + gridDim.x, blockIdx.x, gridDim.x);
      if constexpr (!I0) {
        if (next < a.ntiles) {
          opaque(loff_p);
          fetch(next);
        }
      }
    }
  };
  if (m == M) {
    if (init0)
      run(std::true_type{}, std::true_type{});
    else
      run(std::false_type{}, std::true_type{});
  } else {
    if (init0)
      run(std::true_type{}, std::false_type{});
    else
      run(std::false_type{}, std::false_type{});
  }
}

// ------------------------------------------------ tile sweep, one workgroup
// State accesses of kernels whose workgroups hand a state on to each other
// within one launch: relaxed agent-scope accesses, which go past the L1
// and the XCD's L2 to memory that every XCD sees.  A workgroup publishes its
// stores by waiting for them (stores_done) and then counting up; a reader
// needs no more than to see the count.  (Ordinary accesses with agent-scope
// fences write back and invalidate the whole L2 at every hand-over: the
// 96-circuit batch took 13.1 ms that way.)
template <typename T>
__device__ __forceinline__ T state_load(const T *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <typename T>
__device__ __forceinline__ void state_store(T *p, T v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Every store of this wave has reached memory.
__device__ __forceinline__ void stores_done() {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

// The stages of one sweep on the tile in LDS (a workgroup of 2^(M-R) threads);
// ends with a barrier after the last stage.
template <typename T, int M, int R, bool KO>
__device__ __forceinline__ void tile_stages(const SVI_CONST SweepArgs &a,
                                            typename C2T<T>::type *lt) {
  constexpr int G = 1 << R;
  using C2 = typename C2T<T>::type;
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int mm = a.m > R ? a.m : R;
  const int st_begin = a.stage_begin, st_end = a.stage_end;
  const SVI_CONST StageDesc *stages = cptr(a.stages);
  const MicroOp *ops = a.ops;
  const double *coef = a.coef;
  char *const lb = (char *)lt;
  // waves whose threads hold no part of a small state (m < M) have no group
  const bool on = wave * 64 < (1 << (mm - R));
  for (int st = st_begin; st < st_end; st++) {
    const SVI_CONST StageDesc &sd = stages[st];
    const int gbs =
        (swz<T>(lane_base(tid & 63, sd)) ^ swz<T>(wave_base<M, R>(wave, sd))) * (int)sizeof(C2);
    // a full Kronecker stage (every group bit rotated, then D_after) runs as
    // its own straight-line body, loads to stores; the general body branches
    auto body = [&](auto full_stage) {
      T re[G], im[G];
#pragma unroll
      for (int j = 0; j < G; j++) {
        const C2 v = *(const C2 *)(lb + (gbs ^ sd.off[j]));
        re[j] = v.x;
        im[j] = v.y;
      }
      if constexpr (decltype(full_stage)::value) {
        kron_rot_all<T, R>(re, im, cptr(coef) + sd.kcoef);
        mo_diagt<T, R>(re, im, cptr(coef) + sd.kcoef + 4 * R + 2 * G);
      } else if (KO || sd.kind == ST_KRON) {
        kron_stage<T, R>(re, im, cptr(coef) + sd.kcoef, sd.rmask, sd.dflags);
      } else {
        for (int o = sd.op_begin; o < sd.op_end; o++) {
          const MicroOp op = op_at(ops, o);
          apply_op<T, R>(op, re, im, coef);
        }
      }
      if (sd.dflags & SD_XCHG) lds_barrier();
#pragma unroll
      for (int j = 0; j < G; j++) *(C2 *)(lb + (gbs ^ sd.off[G + j])) = C2{re[j], im[j]};
    };
    if (!on) {
      if (sd.dflags & SD_XCHG) lds_barrier();
    } else if (sd.kind == ST_KRON && sd.rmask == (1u << R) - 1 && (sd.dflags & 7) == 2) {
      body(std::true_type{});
    } else {
      body(std::false_type{});
    }
    if (sd.dflags & SD_WLOCAL) {
      // the next stage reads only slots this wave wrote
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
    } else {
      lds_barrier();
    }
  }
}

// Tiles [t0, t1) of one sweep of one state, run by one workgroup of 2^(M-R)
// threads through the LDS tile `lt` (2^M amplitudes).  No qubit remapping
// on the way out (SW_OPERM is not taken).  KO: every stage is a Kronecker
// stage (no micro-op interpreter in the caller's kernel).
template <typename T, int M, int R, bool KO>
__device__ void sweep_tiles(const SVI_CONST SweepArgs &a, int64_t t0, int64_t t1,
                            typename C2T<T>::type *lt) {
  constexpr int NT = 1 << (M - R);
  constexpr int G = 1 << R;
  using C2 = typename C2T<T>::type;
  const int tid = threadIdx.x;
  const int m = a.m, c = a.c, nh = a.nh;
  const int mm = m > R ? m : R;
  const int ntile_el = 1 << m;
  const bool init0 = (a.flags & SW_INIT_ZERO) != 0;
  T *const pre = (T *)a.re, *const pim = (T *)a.im;
  // Amplitudes of a thread in flight at a time.  The values and addresses of all G
  // at once spilled beside the stages' registers (96 bytes a lane in FP64 with
  // 3-qubit groups, 856 in the general kernel's 5-qubit ones; now 0 and 88): 96
  // ragged circuits of 8 to 20 qubits 6.29 -> 4.93 ms, 16 of 16 qubits with gates of
  // all kinds 586 -> 464 us (559 with cached 16-byte accesses; 8 at a time 6.28 and
  // 462).  FP32 in 5-qubit groups, which never spilled here, is 1% slower with 4.
  constexpr int LC = sizeof(T) == 8 || R == 3 ? 4 : 8;

  // Thread tid moves tile elements i = tid + k * NT, one amplitude per access
  // (consecutive lanes on consecutive addresses).  Offsets: a deposit of the
  // element index by the descriptor's positions, read as scalars, so it splits
  // into the thread's part and a uniform part of k.
  auto off_of = [&](int i) {
    uint64_t o = (uint64_t)(i & ((1 << c) - 1));
    for (int k = 0; k < nh; k++) o |= (uint64_t)((i >> (c + k)) & 1) << a.hb[k];
    return o;
  };
  uint64_t toff = off_of(tid);
  uint64_t kb[R];
#pragma unroll
  for (int r = 0; r < R; r++) kb[r] = off_of(NT << r);
  // (re-declared opaque in every tile: the addresses are formed next to their
  // use, not hoisted into registers that the stages need)
  auto koff = [&](int k) {
    uint64_t o = 0;
#pragma unroll
    for (int r = 0; r < R; r++)
      if ((k >> r) & 1) o += kb[r];
    return o;
  };
  const int tsl = swz<T>(tid);

  // tile bases: a sparse sweep deposits the tile index on the support's
  // qubits outside the tile only (bz, read from the descriptor)
  const bool sparse = (a.flags & SW_SPARSE) != 0;
  const int nz = sparse ? a.nbz : nh;
  for (int64_t tile = t0; tile < t1; tile++) {
    uint64_t base = (uint64_t)tile << c;
    for (int k = 0; k < nz; k++) {
      const int p = sparse ? a.bz[k] : a.hb[k];
      base = ((base >> p) << (p + 1)) | (base & ((1ull << p) - 1ull));
    }
    T *const tr = pre + base, *const ti = pim + base;
    asm volatile("" : "+v"(toff));
    if (init0 && base != 0) {
      // From |0..0> every tile but the one holding index 0 stays zero (a
      // sweep's gates act within tiles): it is written as zeros, with no
      // stages and no LDS (uniform over the workgroup)
#pragma unroll
      for (int k = 0; k < G; k++)
        if (tid + k * NT < ntile_el) {
          state_store(tr + koff(k) + toff, (T)0);
          state_store(ti + koff(k) + toff, (T)0);
        }
      continue;
    }
    if (mm > m) {
      // tiles smaller than one register group: padding slots hold zeros
      for (int i = tid; i < (1 << mm); i += NT) lt[swz<T>(i)] = C2{0, 0};
      __syncthreads();
    }
    if (init0) {
      for (int i = tid; i < ntile_el; i += NT) {
        const T v = i == 0 ? (T)1 : (T)0;
        lt[swz<T>(i)] = C2{v, 0};
      }
    } else {
#pragma unroll
      for (int k0 = 0; k0 < G; k0 += LC) {
        T vr[LC], vi[LC];
#pragma unroll
        for (int k = 0; k < LC; k++)
          if (tid + (k0 + k) * NT < ntile_el) {
            vr[k] = state_load(tr + koff(k0 + k) + toff);
            vi[k] = state_load(ti + koff(k0 + k) + toff);
          }
#pragma unroll
        for (int k = 0; k < LC; k++)
          if (tid + (k0 + k) * NT < ntile_el) lt[tsl ^ swz<T>((k0 + k) * NT)] = C2{vr[k], vi[k]};
        asm volatile("" : "+v"(toff)::"memory");
      }
    }
    __syncthreads();

    tile_stages<T, M, R, KO>(a, lt);

    asm volatile("" : "+v"(toff));
#pragma unroll
    for (int k0 = 0; k0 < G; k0 += LC) {
#pragma unroll
      for (int k = k0; k < k0 + LC; k++)
        if (tid + k * NT < ntile_el) {
          const C2 p = lt[tsl ^ swz<T>(k * NT)];
          state_store(tr + koff(k) + toff, p.x);
          state_store(ti + koff(k) + toff, p.y);
        }
      asm volatile("" : "+v"(toff)::"memory");
    }
    __syncthreads();
  }
}

// ------------------------------------------- two-state Kronecker stage
// One Kronecker stage applied to the psi and lambda tiles held side by side in
// LDS (lb0, lb1), with the gradient terms Im <lam| G |psi> taken at the three
// stage points: diagonal generators (the stage's micro-ops) on the stage input
// and after the rotations, the RYs (StageDesc::ry) after D_before.  The RYs
// come from the descriptor, one straight-line sum for each group bit: as
// micro-ops with a table each, their loads came one after the other and the
// choice among the generators' forms cost 45 more registers (26 qubits, 10 HEA
// layers: 40.1 -> 36.0 ms a gradient; complex64, 24 qubits: 6.40 -> 4.71, the
// kernel no longer spills).  Terms go through in pairs: sink(s0, s1, t)
// receives the pair's wave_total2 result t and the pair's slots (s1 = -1: a
// single term), uniform across the wave.  Ends with the barrier (or the wave
// fence of a wave-local stage) that makes the stores visible to the next stage.
template <typename T, int R, typename Sink>
__device__ __forceinline__ void kron2_stage(char *lb0, char *lb1, int gbs,
                                            const SVI_CONST StageDesc &sd,
                                            const SVI_CONST T *coef, const MicroOp *ops,
                                            const double *gcoef, bool active, Sink &&sink) {
  constexpr int G = 1 << R;
  using C2 = typename C2T<T>::type;
  char *const lb[2] = {lb0, lb1};
  T re[2][G], im[2][G];
#pragma unroll
  for (int s = 0; s < 2; s++) {
#pragma unroll
    for (int j = 0; j < G; j++) {
      const C2 v = *(const C2 *)(lb[s] + (gbs ^ sd.off[j]));
      re[s][j] = v.x;
      im[s][j] = v.y;
    }
  }
  const SVI_CONST T *kc = coef + sd.kcoef;
  // terms go through in pairs, summed over the wave in one chain of lane moves
  // (groups of four, in any arrangement, measured slower): the first of a pair
  // waits here
  double wait_v = 0.0;
  int wait_s = -1;
  auto put = [&](int slot, double v) {
    if (!active) v = 0.0;
    if (wait_s < 0) {
      wait_v = v;
      wait_s = slot;
    } else {
      sink(wait_s, slot, wave_total2(wait_v, v));
      wait_s = -1;
    }
  };
  // diagonal generators: one array of the products Im(conj(lam_j) psi_j), then
  // a dot product with each term's table
  auto grads = [&](int b, int e, double mult) {
    if (b >= e) return;
    double fz[G];
#pragma unroll
    for (int j = 0; j < G; j++)
      fz[j] = (double)re[1][j] * (double)im[0][j] - (double)im[1][j] * (double)re[0][j];
#pragma clang loop unroll(disable)
    for (int o = b; o < e; o++) {
      const MicroOp op = op_at(ops, o);
      const SVI_CONST double *tab = cptr(gcoef) + op.t0;
      double acc = 0.0;
#pragma unroll
      for (int j = 0; j < G; j++) acc += (double)tab[j] * fz[j];
      put(op.coef, mult * acc);
    }
  };
  grads(sd.op_begin, sd.g1, 1.0);
  kron_pre<T, R>(re[0], im[0], kc, sd.dflags);
  kron_pre<T, R>(re[1], im[1], kc, sd.dflags);
  {
    auto ry = [&](auto bit) {
      constexpr int TB = decltype(bit)::value;
      const int slot = ry_slot(sd, TB);
      if (slot >= 0) put(slot, ry_grad<T, R, TB>(re[0], im[0], re[1], im[1]));
    };
    ry(std::integral_constant<int, 0>{});
    ry(std::integral_constant<int, 1>{});
    if constexpr (R > 2) ry(std::integral_constant<int, 2>{});
    if constexpr (R > 3) ry(std::integral_constant<int, 3>{});
    if constexpr (R > 4) ry(std::integral_constant<int, 4>{});
  }
  if (__builtin_expect(kron_form0<T, R>(kc, sd.rmask), 1)) {
    kron_rot<T, R, true>(re[0], im[0], kc, sd.rmask);
    kron_rot<T, R, true>(re[1], im[1], kc, sd.rmask);
  } else if constexpr (sizeof(T) == 4) {
    kron_rot<T, R>(re[0], im[0], kc, sd.rmask);
    kron_rot<T, R>(re[1], im[1], kc, sd.rmask);
  }
  if (sd.g1 < sd.op_end) {
    const double sc = cptr(gcoef)[sd.kcoef + 4 * R + 4 * G];
    grads(sd.g1, sd.op_end, sc * sc);
  }
  if (wait_s >= 0) sink(wait_s, -1, wave_total2(wait_v, 0.0));
  kron_post<T, R>(re[0], im[0], kc, sd.dflags);
  kron_post<T, R>(re[1], im[1], kc, sd.dflags);
  if (sd.dflags & SD_XCHG) lds_barrier();
#pragma unroll
  for (int s = 0; s < 2; s++) {
#pragma unroll
    for (int j = 0; j < G; j++) *(C2 *)(lb[s] + (gbs ^ sd.off[G + j])) = C2{re[s][j], im[s][j]};
  }
  if (sd.dflags & SD_WLOCAL) {
    // the next stage reads only slots this wave wrote
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
  } else {
    lds_barrier();
  }
}

// One micro-op stage (the interpreter) applied to the psi and lambda tiles
// in LDS: each gate micro-op acts on both states, each gradient micro-op sends
// its term Im <lam| G |psi> to sink(slot, -1, wave total) at its place in the
// stage.
// Ends with the barrier that makes the stores visible to the next stage.
template <typename T, int R, typename Sink>
__device__ __forceinline__ void ops2_stage(char *lb0, char *lb1, int gbs,
                                           const SVI_CONST StageDesc &sd, const MicroOp *ops,
                                           const double *coef, bool active, Sink &&sink) {
  constexpr int G = 1 << R;
  using C2 = typename C2T<T>::type;
  char *const lb[2] = {lb0, lb1};
  T re[2][G], im[2][G];
#pragma unroll
  for (int s = 0; s < 2; s++) {
#pragma unroll
    for (int j = 0; j < G; j++) {
      const C2 v = *(const C2 *)(lb[s] + (gbs ^ sd.off[j]));
      re[s][j] = v.x;
      im[s][j] = v.y;
    }
  }
  for (int o = sd.op_begin; o < sd.op_end; o++) {
    const MicroOp op = op_at(ops, o);
    if (op.type == MO_GRAD || op.type == MO_GRAD2L) {
      const double v = active ? grad_any<T, R>(op, re[0], im[0], re[1], im[1], coef) : 0.0;
      sink(op.coef, -1, wave_total2(v, 0.0));
      continue;
    }
    apply_op<T, R>(op, re[0], im[0], coef);
    apply_op<T, R>(op, re[1], im[1], coef);
  }
  if (sd.dflags & SD_XCHG) lds_barrier();
#pragma unroll
  for (int s = 0; s < 2; s++) {
#pragma unroll
    for (int j = 0; j < G; j++) *(C2 *)(lb[s] + (gbs ^ sd.off[G + j])) = C2{re[s][j], im[s][j]};
  }
  lds_barrier();
}

// ------------------------------------------- two-state Kronecker sweep
// Adjoint backward sweeps whose every stage is a Kronecker stage: psi and
// lambda tiles side by side in LDS, the stage applied to both, and the
// gradient terms Im <lam| G |psi> taken at the three stage points (stage
// input, after D_before, after the rotations) and reduced per workgroup.
template <typename T, int M, int R>
__global__ void __launch_bounds__(1 << (M - R)) k_sweep_kron2(SweepArgs a) {
  constexpr int NT = 1 << (M - R);
  constexpr int G = 1 << R;
  constexpr int VN = V4T<T>::N;
  constexpr int NIT = (1 << M) / (VN * NT);
  constexpr int NWAVE = NT / 64;
  using C2 = typename C2T<T>::type;
  using V4 = typename V4T<T>::type;
  // the lane parts of the stages' thread bases from a table built once per
  // launch (as in k_sweep_kron), in the LDS left by the tiles and the per-wave
  // sums within the workgroup's share of the CU (one workgroup per CU for
  // 128 KiB of tiles, two for 64 KiB)
  constexpr int TILE_BYTES = 2 * (1 << M) * (int)sizeof(C2);
  constexpr int WG_LDS = TILE_BYTES >= 131072 ? 163840 : TILE_BYTES >= 65536 ? 81920 : 40960;
  constexpr int LTAB_BYTES = WG_LDS - TILE_BYTES - NWAVE * SVI_GSLOTS_WIDE * 8 - 4 * SVI_MMAX - 256;
  constexpr int LTAB = LTAB_BYTES / 128 > 0 ? LTAB_BYTES / 128 : 1;
  __shared__ C2 lds[2][1 << M];
  __shared__ double wacc[NWAVE][SVI_GSLOTS_WIDE];   // per-wave sums of the gradient slots
  __shared__ int32_t hb_s[SVI_MMAX];
  __shared__ uint16_t ltab[LTAB * 64];   // swizzled element index

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int m = a.m, c = a.c, nh = a.nh;
  const int ntile_el = 1 << m;
  const bool vec = c >= (VN == 2 ? 1 : 2);
  const SVI_CONST StageDesc *stages = cptr(a.stages + a.stage_begin);
  const int nst = a.stage_end - a.stage_begin;
  const SVI_CONST T *coef;   // FP32: rounded once, where they are formed
  if constexpr (sizeof(T) == 8) coef = cptr(a.coef);
  else coef = cptr(a.coef32);

  if (tid < SVI_MMAX) hb_s[tid] = a.hb[tid < nh ? tid : 0];
  const int ntab = nst < LTAB ? nst : LTAB;
  for (int st = wave; st < ntab; st += NWAVE)
    ltab[st * 64 + lane] = (uint16_t)swz<T>(lane_base(lane, stages[st]));
  for (int k = tid; k < NWAVE * SVI_GSLOTS_WIDE; k += NT) (&wacc[0][0])[k] = 0.0;
  __syncthreads();

  uint64_t roff[NIT];
#pragma unroll
  for (int k = 0; k < NIT; k++) {
    const int i = (tid + k * NT) * (vec ? VN : 1);
    roff[k] = spread_row(i >> c, hb_s, nh) + (uint64_t)(i & ((1 << c) - 1));
  }
  const int tsw = swz<T>(tid * VN);
  T *const pr[2] = {(T *)a.re, (T *)a.re2};
  T *const pi[2] = {(T *)a.im, (T *)a.im2};
  const T *const qr[2] = {(const T *)a.src_re, (const T *)a.re2};
  const T *const qi[2] = {(const T *)a.src_im, (const T *)a.im2};
  const bool active = tid < (1 << (m > R ? m - R : 0));
  auto stages_run = [&]() {
    for (int st = 0; st < nst; st++) {
      const SVI_CONST StageDesc &sd = stages[st];
      const int gbs = ((st < ntab ? (int)ltab[st * 64 + lane] : swz<T>(lane_base(lane, sd))) ^
                       swz<T>(wave_base<M, R>(wave, sd))) * (int)sizeof(C2);
      kron2_stage<T, R>((char *)lds[0], (char *)lds[1], gbs, sd, coef, a.ops, a.coef, active,
                        [&](int s0, int s1, double t) {
        // this tile's wave totals into the wave's LDS rows of their slots
        // (LDS adds without return: the wave does not wait)
        wave_deposit2(wacc[tid >> 6], s0, s1, t, tid & 63);
      });
    }
  };
  auto tile_in = [&](int s, int k, const V4 &vr, const V4 &vi) {
    const int si = tsw ^ swz<T>(k * NT * VN);
    lds[s][si] = C2{vr.x, vi.x};
    lds[s][si ^ 1] = C2{vr.y, vi.y};
    if constexpr (VN == 4) {
      lds[s][si ^ 2] = C2{vr.z, vi.z};
      lds[s][si ^ 3] = C2{vr.w, vi.w};
    }
  };
  auto tile_out = [&](int s, int k, uint64_t g) {
    const int si = tsw ^ swz<T>(k * NT * VN);
    V4 vr, vi;
    if constexpr (VN == 2) {
      const C2 p0 = lds[s][si], p1 = lds[s][si ^ 1];
      vr = V4{p0.x, p1.x};
      vi = V4{p0.y, p1.y};
    } else {
      const C2 p0 = lds[s][si], p1 = lds[s][si ^ 1], p2 = lds[s][si ^ 2], p3 = lds[s][si ^ 3];
      vr = V4{p0.x, p1.x, p2.x, p3.x};
      vi = V4{p0.y, p1.y, p2.y, p3.y};
    }
    *(V4 *)(pr[s] + g) = vr;
    *(V4 *)(pi[s] + g) = vi;
  };

  int64_t r0 = 0;
  // Full tiles, FP64: the next tile's loads are in flight behind this tile's
  // stages (as in k_sweep_kron), in registers that the stages leave free at
  // two waves per SIMD; FP32 stages leave none.
  if (sizeof(T) == 8 && m == M && vec) {
    V4 nr[2][NIT], ni[2][NIT];
    auto fetch = [&](int64_t t) {
      const uint64_t b0 = tile_base(t, c, hb_s, nh);
#pragma unroll
      for (int s = 0; s < 2; s++)
#pragma unroll
        for (int k = 0; k < NIT; k++) {
          nr[s][k] = *(const V4 *)(qr[s] + b0 + roff[k]);
          ni[s][k] = *(const V4 *)(qi[s] + b0 + roff[k]);
        }
    };
    auto all_in = [&]() {
#pragma unroll
      for (int s = 0; s < 2; s++)
#pragma unroll
        for (int k = 0; k < NIT; k++) tile_in(s, k, nr[s][k], ni[s][k]);
    };
    int64_t tile = tile_of(0, blockIdx.x, gridDim.x);
    if (tile < a.ntiles) {
      int64_t next = tile_of(gridDim.x, blockIdx.x, gridDim.x);
      fetch(tile);
      all_in();
      lds_barrier();
      if (next < a.ntiles) fetch(next);
      while (true) {
        const uint64_t base = tile_base(tile, c, hb_s, nh);
        stages_run();
#pragma unroll
        for (int s = 0; s < 2; s++)
#pragma unroll
          for (int k = 0; k < NIT; k++) tile_out(s, k, base + roff[k]);
        lds_barrier();
        if (next >= a.ntiles) break;
        all_in();
        lds_barrier();
        r0 += gridDim.x;
        tile = next;
        next = tile_of(r0 + gridDim.x, blockIdx.x, gridDim.x);
        if (next < a.ntiles) fetch(next);
      }
    }
  } else
  for (int64_t tile = tile_of(0, blockIdx.x, gridDim.x); tile < a.ntiles;) {
    const uint64_t base = tile_base(tile, c, hb_s, nh);
    // ---- both tiles into LDS
#pragma unroll
    for (int s = 0; s < 2; s++) {
      if (vec) {
#pragma unroll
        for (int k = 0; k < NIT; k++) {
          const int i = (tid + k * NT) * VN;
          if (i < ntile_el) {
            const uint64_t g = base + roff[k];
            tile_in(s, k, *(const V4 *)(qr[s] + g), *(const V4 *)(qi[s] + g));
          }
        }
      } else {
        for (int i = tid; i < ntile_el; i += NT) {
          const uint64_t g = base + spread_row(i >> c, hb_s, nh) + (uint64_t)(i & ((1 << c) - 1));
          lds[s][swz<T>(i)] = C2{qr[s][g], qi[s][g]};
        }
      }
    }
    lds_barrier();
    stages_run();
    // ---- LDS to HBM
#pragma unroll
    for (int s = 0; s < 2; s++) {
      if (vec) {
#pragma unroll
        for (int k = 0; k < NIT; k++) {
          const int i = (tid + k * NT) * VN;
          if (i < ntile_el) {
            tile_out(s, k, base + roff[k]);
          }
        }
      } else {
        for (int i = tid; i < ntile_el; i += NT) {
          const uint64_t g = base + spread_row(i >> c, hb_s, nh) + (uint64_t)(i & ((1 << c) - 1));
          const C2 p = lds[s][swz<T>(i)];
          pr[s][g] = p.x;
          pi[s][g] = p.y;
        }
      }
    }
    __syncthreads();
    r0 += gridDim.x;
    tile = tile_of(r0, blockIdx.x, gridDim.x);
  }
  __syncthreads();
  for (int sl = tid; sl < a.n_gslots; sl += NT) {
    double v = 0.0;
    for (int w = 0; w < NWAVE; w++) v += wacc[w][sl];
    a.gpart[(int64_t)(a.gslot_begin + sl) * gridDim.x + blockIdx.x] = v;
  }
}

}  // namespace svk
