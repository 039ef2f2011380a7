// Device-side building blocks for gfx950: storage precisions, complex
// arithmetic, and the chiral-basis spin projectors (1 -+ gamma_mu).
#pragma once
#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include <stdint.h>
#include <type_traits>

namespace dwf {

// ----------------------------------------------------------------- complex
template <typename R>
struct cx {
  R re, im;
};

template <typename R>
__device__ __forceinline__ cx<R> cmake(R a, R b) { return {a, b}; }
template <typename R>
__device__ __forceinline__ cx<R> operator+(cx<R> a, cx<R> b) { return {a.re + b.re, a.im + b.im}; }
template <typename R>
__device__ __forceinline__ cx<R> operator-(cx<R> a, cx<R> b) { return {a.re - b.re, a.im - b.im}; }
template <typename R>
__device__ __forceinline__ cx<R> operator*(R s, cx<R> a) { return {s * a.re, s * a.im}; }
template <typename R>
__device__ __forceinline__ cx<R> cmul(cx<R> a, cx<R> b) {
  return {a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re};
}
// conj(a) * b
template <typename R>
__device__ __forceinline__ cx<R> cmulc(cx<R> a, cx<R> b) {
  return {a.re * b.re + a.im * b.im, a.re * b.im - a.im * b.re};
}
// i * a
template <typename R>
__device__ __forceinline__ cx<R> ci(cx<R> a) { return {-a.im, a.re}; }
template <typename R>
__device__ __forceinline__ cx<R> cfma(cx<R> a, cx<R> b, cx<R> acc) {  // acc + a*b
  acc.re = fma(a.re, b.re, acc.re);
  acc.re = fma(-a.im, b.im, acc.re);
  acc.im = fma(a.re, b.im, acc.im);
  acc.im = fma(a.im, b.re, acc.im);
  return acc;
}

// ----------------------------------------------------------------- bf16 (round to nearest even)
__device__ __forceinline__ uint16_t f32_to_bf16(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7f800000u) == 0x7f800000u) return uint16_t((u >> 16) | ((u & 0xffffu) ? 0x40u : 0u));
  u += 0x7fffu + ((u >> 16) & 1u);
  return uint16_t(u >> 16);
}
__device__ __forceinline__ float bf16_to_f32(uint16_t h) { return __uint_as_float(uint32_t(h) << 16); }

// ----------------------------------------------------------------- storage precisions
// Each precision stores one complex number as a pair (re, im) of its storage
// type; arithmetic is FP64 for FP64 and FP32 for everything else.  FP16 spinors
// carry a per-(site, s) FP32 norm (max |component| of the 5D site).
struct P64 {
  using S = double2;
  using R = double;
  static constexpr bool NORM = false;
  static constexpr int ID = 0;
  __device__ __forceinline__ static cx<R> ld(const S& v) { return {v.x, v.y}; }
  __device__ __forceinline__ static S st(cx<R> a) { return make_double2(a.re, a.im); }
};
struct P32 {
  using S = float2;
  using R = float;
  static constexpr bool NORM = false;
  static constexpr int ID = 1;
  __device__ __forceinline__ static cx<R> ld(const S& v) { return {v.x, v.y}; }
  __device__ __forceinline__ static S st(cx<R> a) { return make_float2(a.re, a.im); }
};
struct P16 {
  using S = __half2;
  using R = float;
  static constexpr bool NORM = true;
  static constexpr int ID = 2;
  __device__ __forceinline__ static cx<R> ld(const S& v) {
    float2 f = __half22float2(v);
    return {f.x, f.y};
  }
  __device__ __forceinline__ static S st(cx<R> a) { return __floats2half2_rn(a.re, a.im); }
};
struct PB16 {
  using S = uint32_t;
  using R = float;
  static constexpr bool NORM = false;
  static constexpr int ID = 3;
  __device__ __forceinline__ static cx<R> ld(const S& v) {
    return {bf16_to_f32(uint16_t(v & 0xffffu)), bf16_to_f32(uint16_t(v >> 16))};
  }
  __device__ __forceinline__ static S st(cx<R> a) {
    return uint32_t(f32_to_bf16(a.re)) | (uint32_t(f32_to_bf16(a.im)) << 16);
  }
};

// A half field of one parity: data[(x_cb*12 + k)*Ls + s], norm[x_cb*Ls + s] (FP16 only)
template <typename P>
struct Half {
  typename P::S* data;
  float* norm;
};
template <typename P>
struct CHalf {
  const typename P::S* data;
  const float* norm;
};

// bytes of one half field (nsites 4D checkerboard sites, Ls slices)
template <typename P>
__host__ __device__ inline size_t half_bytes(long nsites, int Ls) {
  size_t b = size_t(nsites) * 12 * Ls * sizeof(typename P::S);
  if (P::NORM) b += size_t(nsites) * Ls * sizeof(float);
  b = (b + 255) & ~size_t(255);
  return b;
}

template <typename P>
__host__ __device__ inline Half<P> half_view(void* base, long nsites, int Ls) {
  Half<P> h;
  h.data = reinterpret_cast<typename P::S*>(base);
  h.norm = P::NORM ? reinterpret_cast<float*>(reinterpret_cast<char*>(base) +
                                              size_t(nsites) * 12 * Ls * sizeof(typename P::S))
                   : nullptr;
  return h;
}
template <typename P>
__host__ __device__ inline CHalf<P> chalf_view(const void* base, long nsites, int Ls) {
  Half<P> h = half_view<P>(const_cast<void*>(base), nsites, Ls);
  return {h.data, h.norm};
}

// one element read or written, optionally with the non-temporal hint
template <typename T>
struct nt_type { typedef T type; };
template <>
struct nt_type<double2> { typedef double type __attribute__((ext_vector_type(2))); };
template <>
struct nt_type<float2> { typedef float type __attribute__((ext_vector_type(2))); };
template <>
struct nt_type<__half2> { typedef uint32_t type; };
template <bool NT, typename T>
__device__ __forceinline__ T get(const T* p) {
  if constexpr (!NT) return *p;
  typedef typename nt_type<T>::type V;
  return __builtin_bit_cast(T, __builtin_nontemporal_load(reinterpret_cast<const V*>(p)));
}
template <bool NT, typename T>
__device__ __forceinline__ void put(T* p, const T& v) {
  typedef typename nt_type<T>::type V;
  if constexpr (NT) __builtin_nontemporal_store(__builtin_bit_cast(V, v), reinterpret_cast<V*>(p));
  else *p = v;
}

// Load the 12 complex components of 5D site (x, s) (NT: see store_spinor)
template <typename P, bool NT = false>
__device__ __forceinline__ void load_spinor(CHalf<P> f, long x, int s, int Ls, cx<typename P::R> v[12]) {
  using R = typename P::R;
  const typename P::S* p = f.data + size_t(x) * 12 * Ls + s;
#pragma unroll
  for (int k = 0; k < 12; ++k) v[k] = P::ld(get<NT>(p + k * Ls));
  if constexpr (P::NORM) {
    const R n = get<NT>(f.norm + size_t(x) * Ls + s);
#pragma unroll
    for (int k = 0; k < 12; ++k) v[k] = n * v[k];
  }
}

// Load spin components [k0, k0+6) of 5D site (x, s)
template <typename P>
__device__ __forceinline__ void load_half_spinor(CHalf<P> f, long x, int s, int Ls, int k0, cx<typename P::R> v[6]) {
  using R = typename P::R;
  const typename P::S* p = f.data + (size_t(x) * 12 + k0) * Ls + s;
#pragma unroll
  for (int k = 0; k < 6; ++k) v[k] = P::ld(p[k * Ls]);
  if constexpr (P::NORM) {
    const R n = f.norm[size_t(x) * Ls + s];
#pragma unroll
    for (int k = 0; k < 6; ++k) v[k] = n * v[k];
  }
}

// NT: non-temporal, for fields a kernel streams beside gathers (see hop_body)
template <typename P, bool NT = false>
__device__ __forceinline__ void store_spinor(Half<P> f, long x, int s, int Ls, const cx<typename P::R> v[12]) {
  using R = typename P::R;
  typename P::S* p = f.data + size_t(x) * 12 * Ls + s;
  if constexpr (P::NORM) {
    R m = R(0);
#pragma unroll
    for (int k = 0; k < 12; ++k) m = fmaxf(m, fmaxf(fabsf(v[k].re), fabsf(v[k].im)));
    const R n = m > R(0) ? m : R(1);
    const R inv = R(1) / n;
    put<NT>(f.norm + size_t(x) * Ls + s, n);
#pragma unroll
    for (int k = 0; k < 12; ++k) put<NT>(p + k * Ls, P::st(inv * v[k]));
  } else {
#pragma unroll
    for (int k = 0; k < 12; ++k) put<NT>(p + k * Ls, P::st(v[k]));
  }
}

// ----------------------------------------------------------------- spin projection
// Chiral basis: g_k = [[0, -i s_k], [i s_k, 0]], g_4 = [[0, 1], [1, 0]].
// For the projector (1 + sg g_mu), sg = +-1, the two independent rows are
//   h0 = psi0 + a0 psi_j0,  h1 = psi1 + a1 psi_j1
// and rows 2, 3 are multiples of h0/h1.  (Derived from the matrices above.)
//   mu=x: h0 = psi0 - sg i psi3, h1 = psi1 - sg i psi2; r2 = sg i h1, r3 = sg i h0
//   mu=y: h0 = psi0 - sg psi3,   h1 = psi1 + sg psi2;   r2 = sg h1,   r3 = -sg h0
//   mu=z: h0 = psi0 - sg i psi2, h1 = psi1 + sg i psi3; r2 = sg i h0, r3 = -sg i h1
//   mu=t: h0 = psi0 + sg psi2,   h1 = psi1 + sg psi3;   r2 = sg h0,   r3 = sg h1
// the two rows for one colour, from the four spin components p0..p3 of that colour
template <int MU, int SG, typename R>
__device__ __forceinline__ void project_colour(cx<R> p0, cx<R> p1, cx<R> p2, cx<R> p3, cx<R>& h0, cx<R>& h1) {
  const R sg = R(SG);
  if constexpr (MU == 0) {
    h0 = p0 - sg * ci(p3);
    h1 = p1 - sg * ci(p2);
  } else if constexpr (MU == 1) {
    h0 = p0 - sg * p3;
    h1 = p1 + sg * p2;
  } else if constexpr (MU == 2) {
    h0 = p0 - sg * ci(p2);
    h1 = p1 + sg * ci(p3);
  } else {
    h0 = p0 + sg * p2;
    h1 = p1 + sg * p3;
  }
}
template <int MU, int SG, typename R>
__device__ __forceinline__ void project(const cx<R> psi[12], cx<R> h[6]) {
#pragma unroll
  for (int c = 0; c < 3; ++c) project_colour<MU, SG, R>(psi[c], psi[3 + c], psi[6 + c], psi[9 + c], h[c], h[3 + c]);
}

// acc += (1 + sg g_mu)-reconstruction of the projected, link-multiplied half spinor u
template <int MU, int SG, typename R>
__device__ __forceinline__ void reconstruct_acc(const cx<R> u[6], cx<R> acc[12]) {
  const R sg = R(SG);
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const cx<R> u0 = u[c], u1 = u[3 + c];
    acc[0 * 3 + c] = acc[0 * 3 + c] + u0;
    acc[1 * 3 + c] = acc[1 * 3 + c] + u1;
    if constexpr (MU == 0) {
      acc[2 * 3 + c] = acc[2 * 3 + c] + sg * ci(u1);
      acc[3 * 3 + c] = acc[3 * 3 + c] + sg * ci(u0);
    } else if constexpr (MU == 1) {
      acc[2 * 3 + c] = acc[2 * 3 + c] + sg * u1;
      acc[3 * 3 + c] = acc[3 * 3 + c] - sg * u0;
    } else if constexpr (MU == 2) {
      acc[2 * 3 + c] = acc[2 * 3 + c] + sg * ci(u0);
      acc[3 * 3 + c] = acc[3 * 3 + c] - sg * ci(u1);
    } else {
      acc[2 * 3 + c] = acc[2 * 3 + c] + sg * u0;
      acc[3 * 3 + c] = acc[3 * 3 + c] + sg * u1;
    }
  }
}

// u = M h for both half-spinor rows (M: 3x3 complex, row-major)
template <typename R>
__device__ __forceinline__ void su3_mul_half(const cx<R> M[9], const cx<R> h[6], cx<R> u[6]) {
#pragma unroll
  for (int r = 0; r < 2; ++r)
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      cx<R> s = cmul(M[a * 3 + 0], h[r * 3 + 0]);
      s = cfma(M[a * 3 + 1], h[r * 3 + 1], s);
      s = cfma(M[a * 3 + 2], h[r * 3 + 2], s);
      u[r * 3 + a] = s;
    }
}

// ----------------------------------------------------------------- fifth-dimension operators along s
// Each site-local operator of the even-odd DWF/Moebius system is, per chirality, a
// bidiagonal factor (a1 + b1 S_d1) followed optionally by the inverse of another
// bidiagonal (alpha + beta S_d2), where S_{-1} x_s = x_{s-1} (x_{-1} = -m x_{Ls-1}) and
// S_{+1} x_s = x_{s+1} (x_{Ls} = -m x_0).  Chirality 0 = spins 0,1 (P+), 1 = spins 2,3 (P-).
template <typename R>
struct FifthChir {
  R a1, b1;           // bidiagonal factor; b1 == 0: scalar
  R inv_alpha, a;     // inverse of (alpha + beta S_d2): 1/alpha and a = -beta/alpha
  R corr;             // m / (1 + m a^Ls)
  R inv_den;          // 1 / (1 + m a^Ls)
  int d1, d2;         // shift directions (-1 or +1)
  int has_inv;
};
template <typename R>
struct FifthScan {
  FifthChir<R> ch[2];
  R m;
};

// Site-local operators along s on the 12 components held by this lane (slice s) when the LSEG
// lanes of a site are the consecutive lanes [seg LSEG, (seg + 1) LSEG) of one wave.
//
// The inverse of (alpha + beta S_d) is the recurrence y_s = u_s + a y_{s-+1}, u = w / alpha: a scan over
// the segment with zero start, log2 LSEG steps v_s += a^off v_{s -+ off}, then the cyclic boundary
// y_{-1} = -m y_{LSEG-1} (resp. y_LSEG = -m y_0) in closed form:
//   y_s = P_s - m a^{s+1} P_{LSEG-1} / (1 + m a^LSEG)  or  y_s = Q_s - m a^{LSEG-s} Q_0 / (1 + m a^LSEG).
// In FP32 a segment of 16 lanes is one DPP row: a step is one v_fmac_f32 whose shifted operand is 0
// beyond the row, and the boundary one with the row's last (first) value.  A segment of 32 lanes is two
// rows: the scan inside each row, then the two rows' carries, which only need the rows' last (first)
// values, in closed form.  Two segments of 8 lanes share a row.  FP64 moves both words of a value with DPP
// (32 lanes: with ds_bpermute) and multiplies and adds them.
// Moving every value with ds_bpermute and selecting took 144 of them and about 340 VALU instructions per
// lane in FP32: the FP16 hops with this epilogue at 24^3 x 64, Ls = 32 went from 676 to 599 us, those with
// two of them from 920 to 752 us; M_prec in FP64, Ls = 16 at 16^3 x 32 344 -> 301 us (DPP and the rest of that
// hop's changes), A^-1 in FP32, Ls = 8 at 12^3 x 24 7.7 -> 5.7 us.
// Rotations with the boundary's factor -m in the wrapped lanes need no closing step, but round every
// lane in every step and the common factor 1 / (1 + m a^LSEG) once more: FP32 A^-1 at Ls = 8 was 1.38 times as
// far from the exact result, at Ls = 16 1.04 times.
// (The fmac steps are inline asm because the compiler emits a DPP move and a separate fma.  Each
// block starts with the five wait states that DPP needs after an EXEC or operand write; inside a
// block a value is read again only twelve instructions after it was written.)
template <int LSEG, typename R>
__device__ __forceinline__ R seg_shfl(R v, int src) {
  return __shfl(v, src, LSEG);
}

#define DWF_DPP12_BANKS(CTRL, COEF, BANKS)                                                          \
  "v_fmac_f32_dpp %0, %0, " COEF " " CTRL " row_mask:0xf bank_mask:" BANKS " bound_ctrl:1\n"        \
  "v_fmac_f32_dpp %1, %1, " COEF " " CTRL " row_mask:0xf bank_mask:" BANKS " bound_ctrl:1\n"        \
  "v_fmac_f32_dpp %2, %2, " COEF " " CTRL " row_mask:0xf bank_mask:" BANKS " bound_ctrl:1\n"        \
  "v_fmac_f32_dpp %3, %3, " COEF " " CTRL " row_mask:0xf bank_mask:" BANKS " bound_ctrl:1\n"        \
  "v_fmac_f32_dpp %4, %4, " COEF " " CTRL " row_mask:0xf bank_mask:" BANKS " bound_ctrl:1\n"        \
  "v_fmac_f32_dpp %5, %5, " COEF " " CTRL " row_mask:0xf bank_mask:" BANKS " bound_ctrl:1\n"        \
  "v_fmac_f32_dpp %6, %6, " COEF " " CTRL " row_mask:0xf bank_mask:" BANKS " bound_ctrl:1\n"        \
  "v_fmac_f32_dpp %7, %7, " COEF " " CTRL " row_mask:0xf bank_mask:" BANKS " bound_ctrl:1\n"        \
  "v_fmac_f32_dpp %8, %8, " COEF " " CTRL " row_mask:0xf bank_mask:" BANKS " bound_ctrl:1\n"        \
  "v_fmac_f32_dpp %9, %9, " COEF " " CTRL " row_mask:0xf bank_mask:" BANKS " bound_ctrl:1\n"        \
  "v_fmac_f32_dpp %10, %10, " COEF " " CTRL " row_mask:0xf bank_mask:" BANKS " bound_ctrl:1\n"      \
  "v_fmac_f32_dpp %11, %11, " COEF " " CTRL " row_mask:0xf bank_mask:" BANKS " bound_ctrl:1\n"
#define DWF_DPP12(CTRL, COEF) DWF_DPP12_BANKS(CTRL, COEF, "0xf")
#define DWF_DPP_STEPS(STEPS, ...)                                                                  \
  asm("s_nop 4\n" STEPS                                                                            \
      : "+v"(v[0].re), "+v"(v[0].im), "+v"(v[1].re), "+v"(v[1].im), "+v"(v[2].re), "+v"(v[2].im), "+v"(v[3].re), \
        "+v"(v[3].im), "+v"(v[4].re), "+v"(v[4].im), "+v"(v[5].re), "+v"(v[5].im)                  \
      : __VA_ARGS__)
#define DWF_DPP_SCAN(SH)                                                                           \
  DWF_DPP12(SH ":1", "%12") DWF_DPP12(SH ":2", "%13") DWF_DPP12(SH ":4", "%14") DWF_DPP12(SH ":8", "%15")

// the four steps of the scan on six components in a 16-lane row (from s - off, BACK from s + off; 0
// beyond the row)
template <bool BACK>
__device__ __forceinline__ void row_scan(cx<float>* v, float c1, float c2, float c4, float c8) {
  if constexpr (BACK) DWF_DPP_STEPS(DWF_DPP_SCAN("row_shl"), "v"(c1), "v"(c2), "v"(c4), "v"(c8));
  else DWF_DPP_STEPS(DWF_DPP_SCAN("row_shr"), "v"(c1), "v"(c2), "v"(c4), "v"(c8));
}
// ... and w times the row's last (BACK first) value added
template <bool BACK>
__device__ __forceinline__ void row_scan_close(cx<float>* v, float c1, float c2, float c4, float c8, float w) {
  if constexpr (BACK)
    DWF_DPP_STEPS(DWF_DPP_SCAN("row_shl") DWF_DPP12("row_newbcast:0", "%16"), "v"(c1), "v"(c2), "v"(c4), "v"(c8), "v"(w));
  else
    DWF_DPP_STEPS(DWF_DPP_SCAN("row_shr") DWF_DPP12("row_newbcast:15", "%16"), "v"(c1), "v"(c2), "v"(c4), "v"(c8), "v"(w));
}
// The same in segments of 8 lanes, two to a row: in the steps of 1 and 2 the lanes whose source lies in
// the other segment (vcc) take 0 (never a product with its value, which may be infinite); the step of 4
// and the boundary's values fall into whole banks of four lanes.
#define DWF_MASKED(K, CTRL, COEF)                                                                  \
  "v_cndmask_b32_dpp %12, %" #K ", %13, vcc " CTRL " row_mask:0xf bank_mask:0xf bound_ctrl:1\n"    \
  "v_fmac_f32 %" #K ", " COEF ", %12\n"
#define DWF_MASKED12(CTRL, COEF)                                                                   \
  DWF_MASKED(0, CTRL, COEF) DWF_MASKED(1, CTRL, COEF) DWF_MASKED(2, CTRL, COEF) DWF_MASKED(3, CTRL, COEF)    \
  DWF_MASKED(4, CTRL, COEF) DWF_MASKED(5, CTRL, COEF) DWF_MASKED(6, CTRL, COEF) DWF_MASKED(7, CTRL, COEF)    \
  DWF_MASKED(8, CTRL, COEF) DWF_MASKED(9, CTRL, COEF) DWF_MASKED(10, CTRL, COEF) DWF_MASKED(11, CTRL, COEF)
#define DWF_HALF_ROW(SH, BANKS4, LOW, HIGH)                                                        \
  asm("s_mov_b64 vcc, %18\ns_nop 4\n" DWF_MASKED12(SH ":1", "%14") "s_mov_b64 vcc, %19\n"         \
      DWF_MASKED12(SH ":2", "%15") DWF_DPP12_BANKS(SH ":4", "%16", BANKS4)                         \
      DWF_DPP12_BANKS("row_newbcast:" LOW, "%17", "0x3") DWF_DPP12_BANKS("row_newbcast:" HIGH, "%17", "0xc") \
      : "+v"(v[0].re), "+v"(v[0].im), "+v"(v[1].re), "+v"(v[1].im), "+v"(v[2].re), "+v"(v[2].im), "+v"(v[3].re), \
        "+v"(v[3].im), "+v"(v[4].re), "+v"(v[4].im), "+v"(v[5].re), "+v"(v[5].im), "=&v"(t)        \
      : "v"(0.0f), "v"(c1), "v"(c2), "v"(c4), "v"(w), "s"(out1), "s"(out2)                         \
      : "vcc")
template <bool BACK>
__device__ __forceinline__ void half_row_scan_close(cx<float>* v, float c1, float c2, float c4, float w) {
  float t;
  const uint64_t out1 = BACK ? 0x8080808080808080ULL : 0x0101010101010101ULL;
  const uint64_t out2 = BACK ? 0xc0c0c0c0c0c0c0c0ULL : 0x0303030303030303ULL;
  if constexpr (BACK) DWF_HALF_ROW("row_shl", "0x5", "0", "8");
  else DWF_HALF_ROW("row_shr", "0xa", "7", "15");
}
// the value of lane LANE of this lane's group of 32
template <int LANE>
__device__ __forceinline__ float bcast32(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_ds_swizzle(__builtin_bit_cast(int, v), LANE << 5));
}

// one DPP move within a 16-lane row; lanes whose source lies beyond the row get 0, lanes of the banks (groups
// of four) outside BANKS keep old
template <int CTRL, int BANKS = 0xf>
__device__ __forceinline__ float row_move(float v, float old = 0.0f) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, old), __builtin_bit_cast(int, v),
                                                               CTRL, 0xf, BANKS, true));
}
template <int CTRL, int BANKS = 0xf>
__device__ __forceinline__ double row_move(double v, double old = 0.0) {
  const uint2 x = __builtin_bit_cast(uint2, v), o = __builtin_bit_cast(uint2, old);
  return __builtin_bit_cast(double, uint2{(unsigned)__builtin_amdgcn_update_dpp((int)o.x, (int)x.x, CTRL, 0xf, BANKS, true),
                                          (unsigned)__builtin_amdgcn_update_dpp((int)o.y, (int)x.y, CTRL, 0xf, BANKS, true)});
}
constexpr int ROW_SHL = 0x100, ROW_SHR = 0x110, ROW_NEWBCAST = 0x150;
// the value OFF slices before this lane's (BACK: after it), 0 beyond the segment
template <int LSEG, bool BACK, int OFF, typename R>
__device__ __forceinline__ R seg_shift(R v, int s) {
  const int src = BACK ? s + OFF : s - OFF;
  const bool inside = src >= 0 && src < LSEG;
  if constexpr (LSEG <= 16) {
    const R t = row_move<(BACK ? ROW_SHL : ROW_SHR) + OFF>(v);
    return LSEG == 16 || inside ? t : R(0);
  } else {
    const R t = seg_shfl<LSEG>(v, src & (LSEG - 1));
    return inside ? t : R(0);
  }
}
// the value of the segment's last (BACK: first) slice
template <int LSEG, bool BACK, typename R>
__device__ __forceinline__ R seg_end(R v) {
  if constexpr (LSEG == 16) return row_move<ROW_NEWBCAST + (BACK ? 0 : 15)>(v);
  else if constexpr (LSEG == 8)
    return row_move<ROW_NEWBCAST + (BACK ? 8 : 15), 0xc>(v, row_move<ROW_NEWBCAST + (BACK ? 0 : 7), 0x3>(v));
  else return seg_shfl<LSEG>(v, BACK ? 0 : LSEG - 1);
}

// a^n, 1 <= n <= LSEG
template <int LSEG, typename R>
__device__ __forceinline__ R power(R a, int n) {
  R p = (n & 1) ? a : R(1);
#pragma unroll
  for (int bit = 2; bit <= LSEG; bit <<= 1) {
    a *= a;
    p = (n & bit) ? p * a : p;
  }
  return p;
}

// the scan's steps from OFF on, ap = a^OFF
template <int LSEG, bool BACK, int OFF, typename R>
__device__ __forceinline__ void seg_scan(cx<R>* v, int s, R ap) {
#pragma unroll
  for (int k = 0; k < 6; ++k) {
    const R tr = seg_shift<LSEG, BACK, OFF>(v[k].re, s), ti = seg_shift<LSEG, BACK, OFF>(v[k].im, s);
    v[k] = {fma(ap, tr, v[k].re), fma(ap, ti, v[k].im)};
  }
  if constexpr (2 * OFF < LSEG) seg_scan<LSEG, BACK, 2 * OFF>(v, s, ap * ap);
}

// (1 - a S_d)^-1 on six components
template <int LSEG, bool BACK, typename R>
__device__ __forceinline__ void seg_inverse(cx<R>* v, int s, const FifthChir<R>& c) {
  if constexpr (std::is_same<R, float>::value && LSEG == 16) {
    const R a2 = c.a * c.a, a4 = a2 * a2, a8 = a4 * a4;
    row_scan_close<BACK>(v, c.a, a2, a4, a8, -c.corr * power<LSEG>(c.a, BACK ? LSEG - s : s + 1));
  } else if constexpr (std::is_same<R, float>::value && LSEG == 8) {
    const R a2 = c.a * c.a, a4 = a2 * a2;
    half_row_scan_close<BACK>(v, c.a, a2, a4, -c.corr * power<LSEG>(c.a, BACK ? LSEG - s : s + 1));
  } else if constexpr (std::is_same<R, float>::value && LSEG == 32) {
    const R a2 = c.a * c.a, a4 = a2 * a2, a8 = a4 * a4, a16 = a8 * a8;
    row_scan<BACK>(v, c.a, a2, a4, a8);
    // carries: c0 enters the row that holds the wrap, c1 the other; with n, f the near and far
    // rows' end values (the row entered first is the far one's successor across the wrap)
    //   c0 = -m (f + a^16 n) / den,  c1 = (n - m a^16 f) / den,  den = 1 + m a^32
    const int i = BACK ? 15 - (s & 15) : s & 15;
    R w = c.a;  // a^{i+1}
    w *= (i & 1) ? c.a : R(1);
    w *= (i & 2) ? a2 : R(1);
    w *= (i & 4) ? a4 : R(1);
    w *= (i & 8) ? a8 : R(1);
    const bool first = BACK ? s >= 16 : s < 16;
    const R wm = -w * c.corr;  // corr = m / den
    const R kn = first ? wm * a16 : w * c.inv_den, kf = first ? wm : wm * a16;
#pragma unroll
    for (int k = 0; k < 6; ++k) {
      const R nr = bcast32<BACK ? 16 : 15>(v[k].re), ni = bcast32<BACK ? 16 : 15>(v[k].im);
      const R fr = bcast32<BACK ? 0 : 31>(v[k].re), fi = bcast32<BACK ? 0 : 31>(v[k].im);
      v[k] = {fma(kf, fr, fma(kn, nr, v[k].re)), fma(kf, fi, fma(kn, ni, v[k].im))};
    }
  } else {
    seg_scan<LSEG, BACK, 1>(v, s, c.a);
    const R w = -c.corr * power<LSEG>(c.a, BACK ? LSEG - s : s + 1);
#pragma unroll
    for (int k = 0; k < 6; ++k) {
      const R er = seg_end<LSEG, BACK>(v[k].re), ei = seg_end<LSEG, BACK>(v[k].im);
      v[k] = {fma(w, er, v[k].re), fma(w, ei, v[k].im)};
    }
  }
}

// the bidiagonal factors of an operator (operators without an inverse: all of it)
// (one path with a run-time source lane: a DPP path per direction raised the fused CG hop from
// 110 to 128 registers and spilled)
template <int LSEG, typename R>
__device__ __forceinline__ void fifth_bidiagonal_apply(cx<R> v[12], int s, const FifthScan<R>& e) {
#pragma unroll
  for (int ch = 0; ch < 2; ++ch) {
    const FifthChir<R> c = e.ch[ch];
    if (c.b1 != R(0)) {
      const int src = (s + c.d1) & (LSEG - 1);
      const bool wrap = (c.d1 < 0) ? (s == 0) : (s == LSEG - 1);
      const R f = wrap ? -e.m * c.b1 : c.b1;
#pragma unroll
      for (int k = ch * 6; k < ch * 6 + 6; ++k) {
        const R nr = seg_shfl<LSEG>(v[k].re, src), ni = seg_shfl<LSEG>(v[k].im, src);
        v[k] = {c.a1 * v[k].re + f * nr, c.a1 * v[k].im + f * ni};
      }
    } else if (c.a1 != R(1)) {
#pragma unroll
      for (int k = ch * 6; k < ch * 6 + 6; ++k) v[k] = c.a1 * v[k];
    }
  }
}

template <int LSEG, typename R>
__device__ __forceinline__ void fifth_scan_apply(cx<R> v[12], int s, const FifthScan<R>& e) {
  fifth_bidiagonal_apply<LSEG>(v, s, e);
#pragma unroll
  for (int ch = 0; ch < 2; ++ch) {
    const FifthChir<R> c = e.ch[ch];
    if (!__builtin_amdgcn_readfirstlane(c.has_inv)) continue;
    cx<R>* vc = v + ch * 6;
#pragma unroll
    for (int k = 0; k < 6; ++k) vc[k] = c.inv_alpha * vc[k];
    if (__builtin_amdgcn_readfirstlane(c.d2) < 0) seg_inverse<LSEG, false, R>(vc, s, c);
    else seg_inverse<LSEG, true, R>(vc, s, c);
  }
}

// XCD-aware block order: the hardware deals workgroups round-robin over the 8
// XCDs; remap so that each XCD walks one contiguous range of the lattice and
// neighbouring sites share its L2.
__device__ __forceinline__ long xcd_block(long bid, long nblocks) {
  const long q = nblocks >> 3, r = nblocks & 7;
  const long xcd = bid & 7, idx = bid >> 3;
  return xcd < r ? xcd * (q + 1) + idx : r * (q + 1) + (xcd - r) * q + idx;
}

}  // namespace dwf
