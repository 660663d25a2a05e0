// gfx950 kernels of one cPINN / XPINN training step.
//
// Each workgroup (4 waves) evaluates one network on a tile of 64 points,
// 16 points per wave.  The network value and its input derivatives are carried
// forward as four "streams" per (neuron, point): value, d/dz0, d/dz1 and the
// second-order sum over the set S the operator needs (S = {x, y} for the
// Laplacian, S = {x} for Burgers' u_xx).  For a hidden layer
//     a = W h + b,  a_i = W h_i,  a_S = W h_S          (Sec. 3 recurrence)
// and through tanh, with t = tanh a, s1 = sech^2 a, s2 = -2 t s1:
//     h = t,  h_i = s1 a_i,  h_S = s1 a_S + s2 sum_{i in S} a_i^2.
// The four streams of 16 points are the columns of one contraction per layer
// on the matrix cores (float32 values split into three bf16 parts, weights from
// LDS); the output layout of one layer is the B operand of the next with the K
// index permuted, so the tanh rule stays lane-local.  What the reverse pass
// needs of a layer is stashed per workgroup in global memory.
//
// The reverse (adjoint) pass differentiates the subdomain loss of
// Eq. cPINNLoss / Eq. XPINNLoss with respect to the subdomain's own
// parameters: seeds at the output from the PDE residual, data and interface
// terms, the adjoint of the tanh rule (s3 = -2 s1 (1 - 3 t^2))
//     abar_S = s1 g_S
//     abar_i = s1 g_i + 2 s2 a_i g_S            (i in S; s1 g_i otherwise)
//     abar   = s1 g + s2 sum_i a_i g_i + (s2 a_S + s3 sum_{i in S} a_i^2) g_S
// then dW = sum over points and streams of abar h_prev^T (MFMA over LDS-staged
// tiles) and g_prev = W^T abar (MFMA).  Every work item writes its own
// gradient partial row; a second kernel sums the rows of each subdomain in a
// fixed order (deterministic, no float atomics) and applies Adam.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>

#include "act_math.h"
#include "ddp_internal.h"
#include "kernels.h"

namespace ddp {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef __bf16 b2 __attribute__((ext_vector_type(2)));
typedef __bf16 b4 __attribute__((ext_vector_type(4)));
typedef __bf16 b8 __attribute__((ext_vector_type(8)));
typedef short s4 __attribute__((ext_vector_type(4)));

constexpr int TP = kTilePts;      // points per tile
// Items with nonzero output seeds below this run in float32 (Plain): the split
// loses nothing yet there, and 1e-9 of a gradient at 2^-90.
constexpr float kTinySeed = 0x1p-80f;
constexpr int NT = 64 * kWaves;   // threads per workgroup

// One 16-byte-per-lane store into the activation stash, followed by wait
// states before anything may overwrite its data registers.  The compiler
// treats a buffer store with an SGPR offset as free of the store-data
// overwrite hazard and will reuse the data VGPRs in the next instruction; with
// two waves per SIMD such stores were seen to write the later value now and
// then (values read back from the stash came back wrong for a few points),
// and the padding below removes that.
__device__ __forceinline__ void stash_put(f4 v, __amdgpu_buffer_rsrc_t rs, int voff, int soff) {
  __builtin_amdgcn_raw_buffer_store_b128(v, rs, voff, soff, 0);
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_nop 4");
  __builtin_amdgcn_sched_barrier(0);
}

// Per-item copy of the thread index the compiler cannot treat as loop
// invariant: keeps per-lane address arithmetic of every width class from being
// hoisted out of the persistent item loop (where it would pin registers).
__device__ __forceinline__ int item_tid() {
  int t = (int)threadIdx.x;
  asm volatile("" : "+v"(t));
  return t;
}

// Asynchronous copy of n4 float4 (16-byte aligned at both ends) from global
// memory straight into LDS (gfx950 LDS DMA, no registers): wave `wave`
// copies the 1 KB blocks wave, wave + kWaves, ...; lane l of a block moves
// its 16 bytes to block base + 16 l.  A wave's copies are counted by its
// vector-memory counter; the compiler waits on it only before that wave's own
// LDS reads, so the barrier that hands the buffer to the other waves must be
// preceded by dma_landed() in every wave.
__device__ __forceinline__ void dma_to_lds(float* dst, const float* src, int n4, int wave, int lane) {
  for (int b = wave; b * 64 < n4; b += kWaves) {
    const int c = b * 64 + lane;
    if (c < n4)
      __builtin_amdgcn_global_load_lds(src + 4 * c, (__attribute__((address_space(3))) void*)(dst + 256 * b), 16, 0,
                                       0);
  }
}

// The wave's own LDS accesses (in order in hardware) stay in order for the
// compiler.
__device__ __forceinline__ void wave_fence() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_wave_barrier();
}

// Wait until every vector-memory operation of this wave has completed
// (s_waitcnt vmcnt(0), the other counters left alone), so its LDS DMA copies
// have landed; gfx950 does not wait for them at a barrier by itself.
__device__ __forceinline__ void dma_landed() { __builtin_amdgcn_s_waitcnt(0x0F70); }

// Sum over the 16 lanes of each row (the 16 points of one lane group) with
// DPP moves: pairs, quads, half rows, rows.  Every lane of the row receives
// the same (bitwise) sum.
__device__ __forceinline__ float dpp_add(float v, int ctrl) {
  switch (ctrl) {   // the control must be a constant
    case 0xB1: return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0xB1, 0xf, 0xf, false));
    case 0x4E: return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x4E, 0xf, 0xf, false));
    case 0x141: return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x141, 0xf, 0xf, false));
    default: return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x140, 0xf, 0xf, false));
  }
}
__device__ __forceinline__ float row_sum16(float v) {
  v = dpp_add(v, 0xB1);    // quad_perm [1, 0, 3, 2]
  v = dpp_add(v, 0x4E);    // quad_perm [2, 3, 0, 1]
  v = dpp_add(v, 0x141);   // row_half_mirror
  return dpp_add(v, 0x140);   // row_mirror
}

// Sum over the four lane groups of a wave (lanes 16 apart), the same bits in
// every lane: the swaps exchange odd 16-lane rows, then halves, of two copies.
__device__ __forceinline__ float group_sum(float v) {
  const unsigned u = __float_as_uint(v);
  const auto a = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  const unsigned s = __float_as_uint(__uint_as_float(a[0]) + __uint_as_float(a[1]));
  const auto b = __builtin_amdgcn_permlane32_swap(s, s, false, false);
  return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// FP32 contractions on the bf16 matrix cores.  A float32 x is the sum of three
// bf16 values, hi = bf16(x), mid = bf16(x - hi), lo = bf16(x - hi - mid) (both
// differences are exact), and a product of two such sums keeps the six terms
// of relative size 2^-17 and up:
//     hi hi + (hi mid + mid hi) + (mid mid + hi lo + lo hi),
// accumulated in float32; what is left out, mostly mid lo + lo mid, is at most
// about 2^-24 of the product, as much as one float32 rounding.  Six 16x16x32
// bf16 MFMAs (16.8 cycles each, measured) replace eight 16x16x4 float32 ones (32
// cycles each) per 32 terms, and with eight times fewer float32 additions the
// measured error against float64 is smaller too (2-norm of 16x16 blocks: K = 32
// 3.6e-8 against 1.05e-7, K = 96 1.2e-7 / 1.8e-7, K = 256 2.7e-7 / 3.0e-7).
// What is no such sum (infinities, and the last bits of values below 2^-109) is
// left to the float32 run of Plain.
__device__ __forceinline__ f4 mma(b8 a, b8 b, f4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0); }
// (the same output layout: lane group g holds element g of the four terms)
__device__ __forceinline__ f4 mma_f32(float a, float b, f4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

// The split of two values: the remainders x - hi come from the bf16 dot
// product x + (hi0, hi1) . (-1, 0), exact like the subtraction (checked on
// random values over the range of the exponents; an infinite value makes both
// remainders NaN) and without unpacking the parts first: 7 instructions a pair
// instead of 11.  (The constants are made opaque: folded into the instruction as
// an inline literal they land in the wrong half.)
__device__ __forceinline__ void split2(float x0, float x1, b2& h, b2& m, b2& l) {
  unsigned c0 = 0x0000bf80u, c1 = 0xbf800000u;   // (-1, 0) and (0, -1)
  asm("" : "+s"(c0));
  asm("" : "+s"(c1));
  const b2 n0 = __builtin_bit_cast(b2, c0), n1 = __builtin_bit_cast(b2, c1);
  h = b2{(__bf16)x0, (__bf16)x1};
  const float r0 = __builtin_amdgcn_fdot2_f32_bf16(h, n0, x0, false);
  const float r1 = __builtin_amdgcn_fdot2_f32_bf16(h, n1, x1, false);
  m = b2{(__bf16)r0, (__bf16)r1};
  l = b2{(__bf16)__builtin_amdgcn_fdot2_f32_bf16(m, n0, r0, false),
         (__bf16)__builtin_amdgcn_fdot2_f32_bf16(m, n1, r1, false)};
}
__device__ __forceinline__ void split4(f4 x, b4& h, b4& m, b4& l) {
  b2 h0, h1, m0, m1, l0, l1;
  split2(x[0], x[1], h0, m0, l0);
  split2(x[2], x[3], h1, m1, l1);
  h = b4{h0[0], h0[1], h1[0], h1[1]};
  m = b4{m0[0], m0[1], m1[0], m1[1]};
  l = b4{l0[0], l0[1], l1[0], l1[1]};
}
__device__ __forceinline__ b8 join(b4 x, b4 y) { return b8{x[0], x[1], x[2], x[3], y[0], y[1], y[2], y[3]}; }

// tanh(a) and sech^2(a) from e = exp(-2|a|):  t = sign(a)(1-e)/(1+e),
// s1 = 4e/(1+e)^2 (no cancellation for large |a|); below 0.7, where 1 - e
// cancels, t = |a| + |a|^3 P(a^2) (as in tanh_value) and s1 = 1 - t^2.  Without
// that branch a step is 4 to 10 % faster, but the error of one gradient against 64
// bits is 1.3e-7 instead of 7e-8 (8 strips of 50) and, repeating at every step,
// it adds up: after 20 Adam steps of the 16-subdomain mix 1.57 against 0.89 times
// the float32-MFMA step's (geometric means of 7 seeds).
__device__ __forceinline__ void tanh_s1(float a, float& t, float& s1) {
  const float b = fabsf(a), u = b * b;
  const float e = __expf(-2.f * b);
  const float r = __builtin_amdgcn_rcpf(1.f + e);
  float p = -0.0051385928f;
  p = fmaf(p, u, 0.020091895f);
  p = fmaf(p, u, -0.053558834f);
  p = fmaf(p, u, 0.13329111f);
  p = fmaf(p, u, -0.33333191f);
  const float s = fmaf(b * u, p, b);
  const bool small = b < 0.7f;
  t = copysignf(small ? s : (1.f - e) * r, a);
  s1 = small ? fmaf(-s, s, 1.f) : 4.f * e * r * r;
}

template <bool S2>
__device__ __forceinline__ void tanh_rule(float a, float ax, float ay, float al, float& h, float& hx,
                                          float& hy, float& hl) {
  float t, s1;
  tanh_s1(a, t, s1);
  const float s2 = -2.f * t * s1;
  h = t;
  hx = s1 * ax;
  hy = s1 * ay;
  const float q = S2 ? fmaf(ax, ax, ay * ay) : ax * ax;
  hl = fmaf(s1, al, s2 * q);
}

template <bool S2>
__device__ __forceinline__ void tanh_adj(float a, float ax, float ay, float al, float g, float gx,
                                         float gy, float gl, float& ab, float& abx, float& aby,
                                         float& abl) {
  float t, s1;
  tanh_s1(a, t, s1);
  const float s2 = -2.f * t * s1;
  const float s3 = -2.f * s1 * (1.f - 3.f * t * t);
  const float q = S2 ? fmaf(ax, ax, ay * ay) : ax * ax;
  abl = s1 * gl;
  abx = fmaf(s1, gx, 2.f * s2 * ax * gl);
  aby = S2 ? fmaf(s1, gy, 2.f * s2 * ay * gl) : s1 * gy;
  ab = fmaf(s1, g, fmaf(s2, fmaf(ax, gx, ay * gy), fmaf(s2, al, s3 * q) * gl));
}

// The same adjoint from the post-activation streams: with hx = s1 ax, hy = s1 ay,
// hl = s1 al + s2 sum_{i in S} a_i^2 every term that held a_i is a polynomial in
// t and the h-streams (s2 a_i = -2 t h_i; s2 a_S + s3 sum a_i^2 = -2 t h_S -
// 2 sum h_i^2), so (a, hx, hy, hl) of a layer is all its reverse pass needs,
// both for this rule and as h^{k-1} of the next layer's dW.  t and s1 come
// from a, so nothing cancels when the neuron saturates.
template <bool S2>
__device__ __forceinline__ void tanh_adj_h(float a, float hx, float hy, float hl, float g, float gx, float gy,
                                           float gl, float& ab, float& abx, float& aby, float& abl) {
  float t, s1;
  tanh_s1(a, t, s1);
  const float m = -2.f * t;
  abl = s1 * gl;
  abx = fmaf(s1, gx, 2.f * m * hx * gl);
  aby = S2 ? fmaf(s1, gy, 2.f * m * hy * gl) : s1 * gy;
  const float q = S2 ? fmaf(hx, hx, hy * hy) : hx * hx;
  ab = fmaf(s1, g, fmaf(m, fmaf(hx, gx, hy * gy), fmaf(m, hl, -2.f * q) * gl));
}

// sin_cos (act_math.h): Cody-Waite reduction and the Cephes single-precision
// polynomials, register-light where pre-activations are small.

// General activation (Sec. 3): h = Phi(c a) with the effective slope c = n a^k
// of the layer and Phi in {tanh, sin, cos}.  The Taylor streams of y = c a are
// c times those of a, so the rule is the unit-slope one on the scaled streams:
// h = Phi(y), d_i h = Phi'(y) d_i y, Delta_S h = Phi'(y) Delta_S y +
// Phi''(y) sum_{i in S} (d_i y)^2.
__device__ __forceinline__ void act_derivs(int act, float y, float& f0, float& f1, float& f2, float& f3) {
  if (act == ACT_TANH) {
    float t, s1;
    tanh_s1(y, t, s1);
    f0 = t;
    f1 = s1;
    f2 = -2.f * t * s1;
    f3 = -2.f * s1 * (1.f - 3.f * t * t);
  } else {
    float sn, cs;
    sin_cos(y, sn, cs);
    f0 = act == ACT_SIN ? sn : cs;
    f1 = act == ACT_SIN ? cs : -sn;
    f2 = -f0;
    f3 = -f1;
  }
}

template <bool S2>
__device__ __forceinline__ void act_rule(int act, float c, float a, float ax, float ay, float al, float& h,
                                         float& hx, float& hy, float& hl) {
  const float y = c * a, yx = c * ax, yy = c * ay, yl = c * al;
  float f0, f1, f2, f3;
  act_derivs(act, y, f0, f1, f2, f3);
  h = f0;
  hx = f1 * yx;
  hy = f1 * yy;
  const float q = S2 ? fmaf(yx, yx, yy * yy) : yx * yx;
  hl = fmaf(f1, yl, f2 * q);
}

// Adjoint of act_rule: from the adjoints g of (h, d_i h, Delta_S h) the
// adjoints of the unscaled streams a (c times those of the scaled streams y),
// and dc += the derivative of the layer's share of J with respect to c, i.e.
// the adjoints of y dotted with the streams of a.
template <bool S2>
__device__ __forceinline__ void act_adj(int act, float c, float a, float ax, float ay, float al, float g, float gx,
                                        float gy, float gl, float& ab, float& abx, float& aby, float& abl,
                                        float& dc) {
  const float y = c * a, yx = c * ax, yy = c * ay, yl = c * al;
  float f0, f1, f2, f3;
  act_derivs(act, y, f0, f1, f2, f3);
  const float q = S2 ? fmaf(yx, yx, yy * yy) : yx * yx;
  const float bl = f1 * gl;
  const float bx = fmaf(f1, gx, 2.f * f2 * yx * gl);
  const float by = S2 ? fmaf(f1, gy, 2.f * f2 * yy * gl) : f1 * gy;
  const float b = fmaf(f1, g, fmaf(f2, fmaf(yx, gx, yy * gy), fmaf(f2, yl, f3 * q) * gl));
  dc = fmaf(b, a, fmaf(bx, ax, fmaf(by, ay, fmaf(bl, al, dc))));
  ab = c * b;
  abx = c * bx;
  aby = c * by;
  abl = c * bl;
}

// ---------------------------------------------------------------------------
// Operators.  u[c][s]: output c, stream s = (value, d/dz0, d/dz1, second order).

template <int PDE> struct Op;

// -Lap u = f   (F = -u_S - f; flux f = -grad u)
template <> struct Op<PDE_POISSON> {
  static constexpr int DO = 1, NEQ = 1;
  static constexpr bool S2 = true;
  __device__ static void residual(const float (&u)[DO][4], const float* f, float coef, float (&F)[NEQ]) {
    F[0] = -u[0][3] - f[0];
  }
  __device__ static void residual_adj(const float (&u)[DO][4], const float (&c)[NEQ], float coef,
                                      float (&ub)[DO][4]) {
    ub[0][3] -= c[0];
  }
  __device__ static void flux(const float (&u)[DO][4], float nx, float ny, float coef, float (&fl)[NEQ]) {
    fl[0] = -(nx * u[0][1] + ny * u[0][2]);
  }
  __device__ static void flux_adj(const float (&u)[DO][4], float nx, float ny, float coef, const float (&c)[NEQ],
                                  float (&ub)[DO][4]) {
    ub[0][1] -= c[0] * nx;
    ub[0][2] -= c[0] * ny;
  }
};

// u_t + u u_x - nu u_xx = f, inputs (x, t); space-time flux (u^2/2 - nu u_x, u)
template <> struct Op<PDE_BURGERS> {
  static constexpr int DO = 1, NEQ = 1;
  static constexpr bool S2 = false;
  __device__ static void residual(const float (&u)[DO][4], const float* f, float nu, float (&F)[NEQ]) {
    F[0] = u[0][2] + u[0][0] * u[0][1] - nu * u[0][3] - f[0];
  }
  __device__ static void residual_adj(const float (&u)[DO][4], const float (&c)[NEQ], float nu,
                                      float (&ub)[DO][4]) {
    ub[0][2] += c[0];
    ub[0][0] += c[0] * u[0][1];
    ub[0][1] += c[0] * u[0][0];
    ub[0][3] -= nu * c[0];
  }
  __device__ static void flux(const float (&u)[DO][4], float nx, float ny, float nu, float (&fl)[NEQ]) {
    fl[0] = nx * (0.5f * u[0][0] * u[0][0] - nu * u[0][1]) + ny * u[0][0];
  }
  __device__ static void flux_adj(const float (&u)[DO][4], float nx, float ny, float nu, const float (&c)[NEQ],
                                  float (&ub)[DO][4]) {
    ub[0][0] += c[0] * (nx * u[0][0] + ny);
    ub[0][1] -= c[0] * nx * nu;
  }
};

// steady incompressible Navier-Stokes, outputs (u, v, p), coef = Re; the
// conservative fluxes of Table 1 (x-momentum, y-momentum, mass) dotted with n:
//   (u^2 + p - u_x/Re, uv - u_y/Re), (uv - v_x/Re, v^2 + p - v_y/Re), (u, v)
template <> struct Op<PDE_NS> {
  static constexpr int DO = 3, NEQ = 3;
  static constexpr bool S2 = true;
  __device__ static void residual(const float (&u)[DO][4], const float* f, float re, float (&F)[NEQ]) {
    const float ir = 1.f / re;
    F[0] = u[0][0] * u[0][1] + u[1][0] * u[0][2] + u[2][1] - ir * u[0][3] - f[0];
    F[1] = u[0][0] * u[1][1] + u[1][0] * u[1][2] + u[2][2] - ir * u[1][3] - f[1];
    F[2] = u[0][1] + u[1][2] - f[2];
  }
  __device__ static void residual_adj(const float (&u)[DO][4], const float (&c)[NEQ], float re,
                                      float (&ub)[DO][4]) {
    const float ir = 1.f / re;
    ub[0][0] += c[0] * u[0][1] + c[1] * u[1][1];
    ub[0][1] += c[0] * u[0][0] + c[2];
    ub[0][2] += c[0] * u[1][0];
    ub[0][3] -= c[0] * ir;
    ub[1][0] += c[0] * u[0][2] + c[1] * u[1][2];
    ub[1][1] += c[1] * u[0][0];
    ub[1][2] += c[1] * u[1][0] + c[2];
    ub[1][3] -= c[1] * ir;
    ub[2][1] += c[0];
    ub[2][2] += c[1];
  }
  __device__ static void flux(const float (&u)[DO][4], float nx, float ny, float re, float (&fl)[NEQ]) {
    const float ir = 1.f / re;
    const float U = u[0][0], V = u[1][0], P = u[2][0];
    // the viscous parts are -(n . grad u)/Re and -(n . grad v)/Re
    const float un = fmaf(nx, u[0][1], ny * u[0][2]), vn = fmaf(nx, u[1][1], ny * u[1][2]);
    fl[0] = fmaf(nx, fmaf(U, U, P), fmaf(ny, U * V, -ir * un));
    fl[1] = fmaf(nx, U * V, fmaf(ny, fmaf(V, V, P), -ir * vn));
    fl[2] = fmaf(nx, U, ny * V);
  }
  __device__ static void flux_adj(const float (&u)[DO][4], float nx, float ny, float re, const float (&c)[NEQ],
                                  float (&ub)[DO][4]) {
    const float ir = 1.f / re;
    const float U = u[0][0], V = u[1][0];
    ub[0][0] += c[0] * (2.f * nx * U + ny * V) + c[1] * nx * V + c[2] * nx;
    ub[1][0] += c[0] * ny * U + c[1] * (nx * U + 2.f * ny * V) + c[2] * ny;
    ub[2][0] += c[0] * nx + c[1] * ny;
    ub[0][1] -= c[0] * ir * nx;
    ub[0][2] -= c[0] * ir * ny;
    ub[1][1] -= c[1] * ir * nx;
    ub[1][2] -= c[1] * ir * ny;
  }
};

// inverse diffusion div(K grad u) = f: both networks carry the (x, y)
// Laplacian stream set; the operator couples the u-network's streams with
// the K-network's and is evaluated in the paired epilogue of Tile, not here
template <> struct Op<PDE_INV> : Op<PDE_POISSON> {};

// epilogue modes of a train tile
enum {
  EPI_OWN = 0,    // the item's own loss terms and output seeds
  EPI_INV_U = 1,  // u-network of a paired inverse item: loss, u seeds, and the K seeds into LDS
  EPI_SEED = 2    // K-network of a paired inverse item: output seeds read from LDS, no loss
};
// parts of a train tile
enum {
  PH_ALL = 0,  // forward, loss / seeds, reverse pass
  PH_FWD = 1,  // forward only (stashed), output streams (value, d/dz0, d/dz1) to LDS
  PH_BWD = 2   // reverse pass only, from the stash of an earlier PH_FWD of the same tile
};
// values_tile modes
enum {
  VAL_OWN = 0,     // interface values of the item's method (u, then flux.n or L(u))
  VAL_STREAMS = 1, // output streams (value, d/dz0, d/dz1) of a one-output network
  VAL_INV_NB = 2   // inverse problem, neighbour u-network: (u, K, L(u, K)) with K from LDS
};

// ---------------------------------------------------------------------------
// Tile processor for one padded width class WP.
//
// LDS of a class (bytes): one split weight matrix is WP^2 x 3 parts x 2.
constexpr int split_matrix_bytes(int wp) { return 6 * wp * wp; }
// Whether each wave accumulates dW over its own 16 points (all blocks in its
// registers, one sum over the waves at the end of the layer) instead of a
// share of the blocks over all 64 points: classes up to 48, where the blocks
// take at most 36 registers.  No barriers between the streams, and each
// fragment read from LDS serves a row or column of blocks.  (16 networks of 20:
// 169 us a step with shared blocks, 159 with private ones.)
constexpr bool private_dw(int wp) { return wp <= 48; }
constexpr int stage_bytes(int wp) { return 2 * 3 * 2 * TP * (wp + 4); }
// Whether the staging area takes the place of W^T, which is then loaded after
// dW: where the two together exceed half a compute unit's LDS (class 80,
// two workgroups per unit) or all of it (class 112).
constexpr bool stage_over_weights(int wp) { return wp == 80 || wp == 112; }
// The sums over the waves of the output layer's and layer 1's gradients: in the
// second forward buffer, or behind the staging area where that is written
// without a barrier after the output layer (private_dw).
constexpr int sums_offset(int wp) {
  return private_dw(wp) ? split_matrix_bytes(wp) + stage_bytes(wp) : split_matrix_bytes(wp) + 4 * wp;
}
// weights and staging of a tile: two forward buffers; W^T and the staging
// area; the sums
constexpr int tile_bytes(int wp, int d_out) {
  const int buf = split_matrix_bytes(wp) + 4 * wp;
  const int rev = stage_bytes(wp) + (stage_over_weights(wp) ? 0 : split_matrix_bytes(wp));
  const int n = 2 * buf > rev ? 2 * buf : rev;
  const int sums = sums_offset(wp) + 4 * kWaves * (d_out > 3 ? d_out : 3) * (wp + 1);
  return ((n > sums ? n : sums) + 15) / 16 * 16;
}
//
// Lane layout (one wave = 16 points): lane = 16 g + pc holds point pc and,
// for output block mb and register i, neuron 16 mb + 4 g + i.  This is the
// C/D layout of the 16x16x32 MFMA, and with the K index of the next
// contraction permuted the same way (element e of lane group g is neuron
// 4 g + (e & 3) of block 2 kb + (e >> 2)) it is also its B-operand layout.

// one stream of the general activation rule (slope c, activation act)
template <bool S2>
__device__ __forceinline__ float act_stream_ga(int s, int act, float c, float a, float ax, float ay, float al) {
  const float y = c * a, yx = c * ax, yy = c * ay, yl = c * al;
  float f0, f1, f2, f3;
  act_derivs(act, y, f0, f1, f2, f3);
  if (s == 0) return f0;
  if (s == 1) return f1 * yx;
  if (s == 2) return f1 * yy;
  const float q = S2 ? fmaf(yx, yx, yy * yy) : yx * yx;
  return fmaf(f1, yl, f2 * q);
}

template <int WP, int PDE>
struct Tile {
  static constexpr int MB = WP / 16;
  static constexpr int DO = Op<PDE>::DO;
  static constexpr int NEQ = Op<PDE>::NEQ;
  static constexpr bool S2 = Op<PDE>::S2;
  static constexpr int KB = MB / 2;                         // 32-neuron steps of a contraction; an odd last block is
  static constexpr bool TAIL = (MB & 1) != 0;               // a 16-neuron step of its own
  // blocks of dW per wave: rows of blocks 4 r + wave, then the blocks of the
  // rows left over, dealt out one by one
  static constexpr int ROWS = MB / kWaves;
  static constexpr int REM = (MB % kWaves) * MB;
  static constexpr int NREM = (REM + kWaves - 1) / kWaves;
  static constexpr int WBYTES = split_matrix_bytes(WP);     // one split weight matrix
  static constexpr int BUF = WBYTES + 4 * WP;               // with its bias
  static constexpr bool PRIV = private_dw(WP);
  static constexpr int SROWS = PRIV ? 16 : TP;              // rows (points) of a staging area
  static constexpr int KL = (DO * WP + NT - 1) / NT;        // output-layer slots per thread
  static constexpr int STASH_LAYER = kWaves * 4 * MB * 1024;  // bytes of one layer's stash

  typedef f4 Streams[4][MB];

  // layer 1: a = W^1 z + b^1, a_0 = W^1[:,0], a_1 = W^1[:,1], a_S = 0
  __device__ static void layer1(const float* K, float x, float y, int g, Streams& A) {
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const f4 c = *reinterpret_cast<const f4*>(K + (16 * mb + 4 * g + i) * 4);
        A[0][mb][i] = fmaf(c[0], x, fmaf(c[1], y, c[2]));
        A[1][mb][i] = c[0];
        A[2][mb][i] = c[1];
        A[3][mb][i] = 0.f;
      }
    }
  }

  // GA: a network with another activation than tanh or with trainable
  // slopes (activation act, effective slope c of the layer); else plain tanh
  template <bool GA>
  __device__ static void activate(const Streams& A, Streams& H, int act, float c) {
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        float h, hx, hy, hl;
        if constexpr (GA) act_rule<S2>(act, c, A[0][mb][i], A[1][mb][i], A[2][mb][i], A[3][mb][i], h, hx, hy, hl);
        else tanh_rule<S2>(A[0][mb][i], A[1][mb][i], A[2][mb][i], A[3][mb][i], h, hx, hy, hl);
        H[0][mb][i] = h;
        H[1][mb][i] = hx;
        H[2][mb][i] = hy;
        H[3][mb][i] = hl;
      }
    }
  }

  // Forward weights alternate between two LDS buffers (weights, then bias), so
  // that layer k + 1's stream in while layer k computes; the last hidden layer
  // D always uses the first one.
  __device__ static char* wbuf(char* sW, int D, int k) { return ((D - k) & 1) ? sW + BUF : sW; }
  __device__ static void fetch_wb(char* dst, const float* K, const Layout& L, int k, int wave, int lane) {
    dma_to_lds(reinterpret_cast<float*>(dst), K + L.k_w(k), BUF / 16, wave, lane);
  }
  __device__ static void fetch_wt(char* sW, const float* K, const Layout& L, int k, int wave, int lane) {
    dma_to_lds(reinterpret_cast<float*>(sW), K + L.k_wt(k), WBYTES / 16, wave, lane);
  }
  // Y_s += W X_s for streams S0 .. S0 + NS - 1 (w: a split matrix in LDS, in
  // fragment order, so every read is 16 bytes a lane without bank conflicts).
  // Each weight fragment read feeds 6 NS MFMAs; a stream's values are split
  // once per 32-neuron step.  The odd last block packs two of the six
  // products into the two halves of each MFMA's K, so it costs three.
  template <int S0, int NS>
  __device__ __forceinline__ static void contract(const char* w, int lane, const Streams& X, Streams& Y) {
    // fragments are read one 16-row block ahead of their MFMAs
    auto load = [&](int mb, int kb, b8 (&f)[3]) {
      const b8* p = reinterpret_cast<const b8*>(w + mb * 96 * WP + kb * 3072) + lane;
      f[0] = p[0];
      f[1] = p[64];
      f[2] = p[128];
    };
    auto load_tail = [&](int mb, b8 (&f)[3]) {   // {mid, hi}, {hi, lo}
      const b4* p = reinterpret_cast<const b4*>(w + mb * 96 * WP + KB * 3072) + lane;
      const b4 wm = p[0], wh = p[64], wl = p[128];
      f[0] = join(wm, wh);
      f[1] = join(wh, wl);
    };
    b8 f[3], fn[3];
    if constexpr (KB > 0) load(0, 0, f);
    else load_tail(0, f);
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
      b8 xh[NS], xm[NS], xl[NS];
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        b4 h0, h1, m0, m1, l0, l1;
        split4(X[S0 + s][2 * kb], h0, m0, l0);
        split4(X[S0 + s][2 * kb + 1], h1, m1, l1);
        xh[s] = join(h0, h1);
        xm[s] = join(m0, m1);
        xl[s] = join(l0, l1);
      }
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) {
        if (mb + 1 < MB) load(mb + 1, kb, fn);
        else if (kb + 1 < KB) load(0, kb + 1, fn);
        else if constexpr (TAIL) load_tail(0, fn);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s = 0; s < NS; ++s) Y[S0 + s][mb] = mma(f[2], xh[s], Y[S0 + s][mb]);
#pragma unroll
        for (int s = 0; s < NS; ++s) Y[S0 + s][mb] = mma(f[1], xl[s], Y[S0 + s][mb]);
#pragma unroll
        for (int s = 0; s < NS; ++s) Y[S0 + s][mb] = mma(f[0], xm[s], Y[S0 + s][mb]);
#pragma unroll
        for (int s = 0; s < NS; ++s) Y[S0 + s][mb] = mma(f[0], xh[s], Y[S0 + s][mb]);
#pragma unroll
        for (int s = 0; s < NS; ++s) Y[S0 + s][mb] = mma(f[1], xm[s], Y[S0 + s][mb]);
#pragma unroll
        for (int s = 0; s < NS; ++s) Y[S0 + s][mb] = mma(f[1], xh[s], Y[S0 + s][mb]);
        f[0] = fn[0];
        f[1] = fn[1];
        f[2] = fn[2];
      }
    }
    if constexpr (TAIL) {
      b8 hh[NS], mm[NS], lh[NS];
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        b4 h, m, l;
        split4(X[S0 + s][MB - 1], h, m, l);
        hh[s] = join(h, h);
        mm[s] = join(m, m);
        lh[s] = join(l, h);
      }
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) {
        if (mb + 1 < MB) load_tail(mb + 1, fn);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s = 0; s < NS; ++s) Y[S0 + s][mb] = mma(f[1], lh[s], Y[S0 + s][mb]);
#pragma unroll
        for (int s = 0; s < NS; ++s) Y[S0 + s][mb] = mma(f[0], mm[s], Y[S0 + s][mb]);
#pragma unroll
        for (int s = 0; s < NS; ++s) Y[S0 + s][mb] = mma(f[0], hh[s], Y[S0 + s][mb]);
        f[0] = fn[0];
        f[1] = fn[1];
      }
    }
  }
  // The same Y_s += W X_s in float32, on the 16x16x4 float32 MFMA, for values
  // that are no sum of three bf16 (infinities, and NaN beside them): the parts
  // of a weight are added up again, element e of a fragment being the A operand
  // of the step that takes element e of the streams.  2.7 times the matrix
  // cycles; taken only where contract's result turned out not finite.
  template <int S0, int NS>
  __device__ __forceinline__ static void contract_f32(const char* w, int lane, const Streams& X, Streams& Y) {
    auto weight = [](__bf16 m, __bf16 h, __bf16 l) { return (float)h + ((float)m + (float)l); };
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
#pragma unroll
      for (int kb = 0; kb < KB; ++kb) {
        const b8* p = reinterpret_cast<const b8*>(w + mb * 96 * WP + kb * 3072) + lane;
        const b8 fm = p[0], fh = p[64], fl = p[128];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float v = weight(fm[e], fh[e], fl[e]);
#pragma unroll
          for (int s = S0; s < S0 + NS; ++s) Y[s][mb] = mma_f32(v, X[s][2 * kb + (e >> 2)][e & 3], Y[s][mb]);
        }
      }
      if constexpr (TAIL) {
        const b4* p = reinterpret_cast<const b4*>(w + mb * 96 * WP + KB * 3072) + lane;
        const b4 fm = p[0], fh = p[64], fl = p[128];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float v = weight(fm[e], fh[e], fl[e]);
#pragma unroll
          for (int s = S0; s < S0 + NS; ++s) Y[s][mb] = mma_f32(v, X[s][MB - 1][e], Y[s][mb]);
        }
      }
    }
  }
  // the values are computed by here, and nothing is known about them afterwards
  __device__ __forceinline__ static void pin(Streams& X) {
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) asm volatile("" : "+v"(X[s][mb]));
  }
  // any values
  __device__ __forceinline__ static void forget(Streams& X) {
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) asm volatile("" : "=v"(X[s][mb]));
  }
  // all four streams: at once where the registers allow it (half the weight
  // reads), else in two pairs
  template <bool PAIRS>
  __device__ __forceinline__ static void contract4(const char* w, int lane, const Streams& X, Streams& Y) {
    if constexpr (PAIRS) {
      contract<0, 2>(w, lane, X, Y);
      contract<2, 2>(w, lane, X, Y);
    } else {
      contract<0, 4>(w, lane, X, Y);
    }
  }

  // What the reverse pass keeps of a layer: the value pre-activation a and
  // the post-activation streams h_x, h_y, h_S (tanh: half of what a and h are
  // together), or for other activations and trainable slopes the four
  // pre-activation streams, from which h is rebuilt (class 80, without the
  // registers for that, keeps h as well, kMaxDepth layers further on).
  template <bool GA>
  __device__ static bool h_form(const NetDesc& nd) {
    return !GA || (nd.act == ACT_TANH && !nd.adaptive);
  }
  template <bool GA>
  __device__ static void stash_put_layer(const NetDesc& nd, __amdgpu_buffer_rsrc_t rs, int layer, int wave, int lane,
                                         const Streams& A, const Streams& H, bool values_only = false) {
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) stash_put(A[0][mb], rs, lane * 16, stash_off(layer, wave, 0, mb));
    if (values_only) return;
    const bool hf = h_form<GA>(nd);
#pragma unroll
    for (int s = 1; s < 4; ++s)
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) {
        if (hf) stash_put(H[s][mb], rs, lane * 16, stash_off(layer, wave, s, mb));
        else stash_put(A[s][mb], rs, lane * 16, stash_off(layer, wave, s, mb));
      }
    if (!KEEP && !hf) {
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
          stash_put(H[s][mb], rs, lane * 16, stash_off(layer + kMaxDepth, wave, s, mb));
    }
  }
  // one stream of h from what is kept
  template <bool GA>
  __device__ __forceinline__ static void h_stream(const NetDesc& nd, int s, float c, const Streams& S, f4 (&h)[MB]) {
    const bool hf = h_form<GA>(nd);
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (hf) {
          float t = S[s][mb][i], s1;
          if (s == 0) tanh_s1(S[0][mb][i], t, s1);
          h[mb][i] = t;
        } else {
          h[mb][i] = act_stream_ga<S2>(s, nd.act, c, S[0][mb][i], S[1][mb][i], S[2][mb][i], S[3][mb][i]);
        }
      }
  }
  // One hidden layer in place: a^k = W^k h^{k-1} (+ b^k on the value stream)
  // for all four streams, the activation rule, and what the reverse pass keeps
  // (values_only: of the pre-activations' value stream alone).
  template <bool STASH, bool GA>
  __device__ static void hidden_layer(const char* w, int g, Streams& H, __amdgpu_buffer_rsrc_t rs, int layer, int wave,
                                      int lane, const NetDesc& nd, float c, bool values_only = false) {
    const float* bias = reinterpret_cast<const float*>(w + WBYTES);
    Streams A;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      A[0][mb] = *reinterpret_cast<const f4*>(bias + 16 * mb + 4 * g);
      A[1][mb] = f4{0.f, 0.f, 0.f, 0.f};
      A[2][mb] = f4{0.f, 0.f, 0.f, 0.f};
      A[3][mb] = f4{0.f, 0.f, 0.f, 0.f};
    }
    contract4<MB == 5>(w, lane, H, A);
    activate<GA>(A, H, nd.act, c);
    if constexpr (STASH) {
      stash_put_layer<GA>(nd, rs, layer, wave, lane, A, H, values_only);
    }
  }

  // Staging area of dW (one per wave where PRIV): [operand abar, h][part][row]
  // [WP + 4] bf16, a row per point of one stream and the neurons along it, so that a lane writes its four
  // neurons of a block in 8 bytes; the operand fragments, which run along the
  // points, come out of the transposing LDS read (ds_read_b64_tr_b16).  LDS
  // takes 16 lanes and 32 banks at a time: rows an odd multiple of 8 bytes apart
  // put the writes of the 16 points of a lane group on all 32 banks (6 cycles a
  // wave and 8-byte write, measured; 16 with rows of WP neurons).  The reads, 4
  // rows of 32 bytes at a time, still collide two ways (four at class 64): bank
  // conflicts are a quarter of the LDS instructions' cycles on the 16-subdomain
  // mix.
  static constexpr int ROW = 2 * (WP + 4);      // bytes
  static constexpr int PART = SROWS * ROW;      // bytes of one part of one operand
  __device__ __forceinline__ static void stage_put(char* base, int row, int g, const f4 (&X)[MB]) {
    char* p = base + row * ROW + 8 * g;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      b4 h, m, l;
      split4(X[mb], h, m, l);
      *reinterpret_cast<b4*>(p + 32 * mb) = m;
      *reinterpret_cast<b4*>(p + 32 * mb + PART) = h;
      *reinterpret_cast<b4*>(p + 32 * mb + 2 * PART) = l;
    }
  }
  // fragment (neurons of block mb) x (32 rows from row 32 c): lane group g
  // holds rows 4 g .. 4 g + 3 and 16 more
  __device__ __forceinline__ static b8 stage_frag(const char* base, int c, int mb, int lane) {
    const char* p = base + (4 * (lane >> 4) + ((lane & 15) >> 2)) * ROW + 8 * (lane & 3) + 32 * mb + c * (32 * ROW);
    typedef __attribute__((address_space(3))) s4* lp;
    const s4 x = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lp)(p));
    const s4 y = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lp)(p + 16 * ROW));
    return join(__builtin_bit_cast(b4, x), __builtin_bit_cast(b4, y));
  }
  // the operands of a 16-row step: the parts of 16 rows in pairs, so that
  // three MFMAs hold the six products (as in contract's last block)
  struct Frag16 {
    b4 m, h, l;
  };
  __device__ __forceinline__ static Frag16 stage_parts16(const char* base, int mb, int lane) {
    const char* p = base + (4 * (lane >> 4) + ((lane & 15) >> 2)) * ROW + 8 * (lane & 3) + 32 * mb;
    typedef __attribute__((address_space(3))) s4* lp;
    return Frag16{__builtin_bit_cast(b4, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lp)(p))),
                  __builtin_bit_cast(b4, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lp)(p + PART))),
                  __builtin_bit_cast(b4, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lp)(p + 2 * PART)))};
  }
  struct Frag {
    b8 m, h, l;
  };
  __device__ __forceinline__ static Frag stage_parts(const char* base, int c, int mb, int lane) {
    return Frag{stage_frag(base, c, mb, lane), stage_frag(base + PART, c, mb, lane),
                stage_frag(base + 2 * PART, c, mb, lane)};
  }
  __device__ __forceinline__ static f4 mma6(const Frag& a, const Frag& b, f4 c) {
    c = mma(a.l, b.h, c);
    c = mma(a.h, b.l, c);
    c = mma(a.m, b.m, c);
    c = mma(a.m, b.h, c);
    c = mma(a.h, b.m, c);
    return mma(a.h, b.h, c);
  }
  // the sum over 32 rows: the fragment times ones
  __device__ __forceinline__ static f4 row_sums(const Frag& a, f4 c) {
    const __bf16 o = (__bf16)1.f;
    const b8 one = {o, o, o, o, o, o, o, o};
    return mma(a.h, one, mma(a.m, one, mma(a.l, one, c)));
  }

  // Whether the registers hold two layers' shares of the stash beside the
  // adjoint streams (not at two waves per SIMD and 80 neurons).
  static constexpr bool KEEP = MB != 5;

  // Activation stash of the workgroup's slot, [layer 1..D][wave][stream][mblock][lane]
  // float4, addressed through a buffer resource.
  __device__ static int stash_off(int layer, int wave, int s, int mb) {
    return (layer - 1) * STASH_LAYER + ((wave * 4 + s) * MB + mb) * 1024;
  }
  // Stash loads read at device scope (SC1): a slot is rewritten by the same
  // wave on every tile, and the per-CU vector L1 must not serve a copy from
  // before the rewrite.
  static constexpr int kStashLoadPolicy = 16;
  __device__ __forceinline__ static void stash_load_block(__amdgpu_buffer_rsrc_t rs, int layer, int wave, int lane,
                                                          int s, int mb, f4& v) {
    v = __builtin_amdgcn_raw_buffer_load_b128(rs, lane * 16, stash_off(layer, wave, s, mb), kStashLoadPolicy);
  }
  __device__ static void stash_load_stream(__amdgpu_buffer_rsrc_t rs, int layer, int wave, int lane, int s,
                                           f4 (&As)[MB]) {
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) stash_load_block(rs, layer, wave, lane, s, mb, As[mb]);
  }
  __device__ static void stash_load(__amdgpu_buffer_rsrc_t rs, int layer, int wave, int lane, Streams& A) {
#pragma unroll
    for (int s = 0; s < 4; ++s) stash_load_stream(rs, layer, wave, lane, s, A[s]);
  }

  // output layer u = W^L h + b^L for DO outputs; every lane group ends with
  // the full sums for its point (bitwise identical across groups)
  __device__ static void out_fwd(const float* WL, const float* bL, int g, const Streams& H, float (&u)[DO][4]) {
#pragma unroll
    for (int c = 0; c < DO; ++c) {
      float acc[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) {
        const f4 wv = *reinterpret_cast<const f4*>(WL + c * WP + 16 * mb + 4 * g);
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int s = 0; s < 4; ++s) acc[s] = fmaf(wv[i], H[s][mb][i], acc[s]);
      }
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const float v = group_sum(acc[s]);
        u[c][s] = s == 0 ? v + bL[c] : v;
      }
    }
  }

  __device__ __forceinline__ static bool finite4(const float (&v)[4]) {
    return fmaf(v[0], 0.f, fmaf(v[1], 0.f, fmaf(v[2], 0.f, v[3] * 0.f))) == 0.f;
  }
  __device__ __forceinline__ static bool finite_streams(const float (&u)[DO][4]) {
    bool f = finite4(u[0]);
#pragma unroll
    for (int c = 1; c < DO; ++c) f = f && finite4(u[c]);
    return f;
  }
  __device__ __forceinline__ static bool tiny_seeds(const float (&ub)[DO][4]) {
    float top = 0.f;
#pragma unroll
    for (int c = 0; c < DO; ++c)
#pragma unroll
      for (int s = 0; s < 4; ++s) top = fmaxf(top, fabsf(ub[c][s]));
    return top > 0.f && top < kTinySeed;
  }

  // values this network contributes on an interface: u (DO) then the normal
  // flux (cPINN) or the operator value L_x(u) without forcing (XPINN)
  __device__ static void own_values(int method, const float (&u)[DO][4], float nx, float ny, float coef,
                                    float (&ov)[DO + NEQ]) {
#pragma unroll
    for (int c = 0; c < DO; ++c) ov[c] = u[c][0];
    if (method == METHOD_XPINN) {
      const float zero[NEQ] = {};
      float F[NEQ];
      Op<PDE>::residual(u, zero, coef, F);
#pragma unroll
      for (int e = 0; e < NEQ; ++e) ov[DO + e] = F[e];
    } else {
      float fl[NEQ];
      Op<PDE>::flux(u, nx, ny, coef, fl);
#pragma unroll
      for (int e = 0; e < NEQ; ++e) ov[DO + e] = fl[e];
    }
  }

  // the point's forcing (residual points) or target values, loaded at the top
  // of the tile
  static constexpr int NTGT = DO > NEQ ? DO : NEQ;
  // loss contributions and output seeds of one point (the derivative of the
  // item's share of J_q with respect to the output streams)
  //
  // EPI_INV_U: inv holds the K-network's streams (K, K_x, K_y) per tile point
  // and nb the neighbour's (u, K, L) on interfaces; F = L - f with
  // L = K Lap u + K_x u_x + K_y u_y (Eq. heq expanded), and kb receives the
  // seeds of (K, K_x, K_y).  EPI_SEED: the seeds come from inv + 3 TP.
  template <int MODE>
  __device__ __forceinline__ static void epilogue(const KArgs& ka, const Item& it, const NetDesc& nd, int tp, bool valid,
                                  const float (&tgt)[NTGT], const float* nb, const float* inv, const float (&u)[DO][4], float (&ub)[DO][4],
                                  float (&loss)[kLossTerms], float (&kb)[3]) {
#pragma unroll
    for (int c = 0; c < DO; ++c)
#pragma unroll
      for (int s = 0; s < 4; ++s) ub[c][s] = 0.f;
#pragma unroll
    for (int t = 0; t < kLossTerms; ++t) loss[t] = 0.f;
    kb[0] = kb[1] = kb[2] = 0.f;
    if (!valid) return;
    const float inv_n = it.inv_n;
    if constexpr (MODE == EPI_SEED) {
#pragma unroll
      for (int s = 0; s < 3; ++s) ub[0][s] = inv[3 * TP + 3 * tp + s];
      return;
    } else if constexpr (MODE == EPI_INV_U) {
      const float K = inv[3 * tp], Kx = inv[3 * tp + 1], Ky = inv[3 * tp + 2];
      const float L = fmaf(K, u[0][3], fmaf(Kx, u[0][1], Ky * u[0][2]));
      float c;
      if (it.kind == KIND_RES) {
        const float F = L - tgt[0];
        loss[1] += F * F;
        c = 2.f * nd.loss_w[1] * F * inv_n;
      } else {
        const float dT = u[0][0] - nb[0], dK = K - nb[1], dL = L - nb[2];
        loss[2] += 0.25f * (dT * dT + dK * dK);
        ub[0][0] += 0.5f * nd.loss_w[2] * dT * inv_n;
        kb[0] += 0.5f * nd.loss_w[2] * dK * inv_n;
        loss[3] += dL * dL;
        c = 2.f * nd.loss_w[3] * dL * inv_n;
      }
      ub[0][1] += c * Kx;
      ub[0][2] += c * Ky;
      ub[0][3] += c * K;
      kb[0] += c * u[0][3];
      kb[1] += c * u[0][1];
      kb[2] += c * u[0][2];
      return;
    }
    if (it.kind == KIND_RES) {
      float F[NEQ];
      Op<PDE>::residual(u, tgt, ka.coef0, F);
      float c[NEQ];
#pragma unroll
      for (int e = 0; e < NEQ; ++e) {
        loss[1] += F[e] * F[e];
        c[e] = 2.f * nd.loss_w[1] * F[e] * inv_n;
      }
      Op<PDE>::residual_adj(u, c, ka.coef0, ub);
    } else if (it.kind == KIND_DATA || it.kind == KIND_AUX) {
#pragma unroll
      for (int c = 0; c < DO; ++c) {
        const float d = u[c][0] - tgt[c];
        loss[0] += d * d;
        ub[c][0] += 2.f * nd.loss_w[0] * d * inv_n;
      }
    } else if constexpr (PDE != PDE_INV) {
      const IfaceDesc ifd = ka.ifaces[it.iface];
      float ov[DO + NEQ];
      own_values(ifd.method, u, ifd.nx, ifd.ny, ka.coef0, ov);
#pragma unroll
      for (int c = 0; c < DO; ++c) {
        const float d = ov[c] - nb[c];
        loss[2] += 0.25f * d * d;
        ub[c][0] += 0.5f * nd.loss_w[2] * d * inv_n;
      }
      // the fourth term: residual continuity (XPINN) or flux matching (cPINN),
      // each equation's squared jump summed
      float c[NEQ];
#pragma unroll
      for (int e = 0; e < NEQ; ++e) {
        const float d = ov[DO + e] - nb[DO + e];
        loss[3] += d * d;
        c[e] = 2.f * nd.loss_w[3] * d * inv_n;
      }
      if (ifd.method == METHOD_XPINN) Op<PDE>::residual_adj(u, c, ka.coef0, ub);
      else Op<PDE>::flux_adj(u, ifd.nx, ifd.ny, ka.coef0, c, ub);
    }
  }

  // gradient / loss partial rows: written by the first tile of an item,
  // accumulated by the following ones (read at device scope, as for the stash)
  __device__ static void accum(float* dst, float v, bool first) {
    if (first) *dst = v;
    else *dst = __hip_atomic_load(dst, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + v;
  }
  // the value a partial-row entry holds before this tile (0 on an item's first
  // tile): loaded early into the accumulator, so the tile's sums add onto it
  // and the entry is then simply stored
  __device__ static float device_load(const float* src) {
    return __hip_atomic_load(src, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __device__ static float prior(const float* src, bool first) { return first ? 0.f : device_load(src); }

  // ------------------------------------------------------------------------
  // forward only, one tile starting at point t0 of the item, results written by
  // the first lane group of each point to dst (stride 3, or DO + NEQ for
  // VAL_OWN):
  //  VAL_OWN      the values this network contributes on an interface (u, then
  //               flux.n or L_x(u)) for the other side's loss -- the exchange of
  //               Algorithm 1 as an on-chip read;
  //  VAL_STREAMS  the output streams (value, d/dz0, d/dz1) of a one-output
  //               network (the K-network of the inverse problem);
  //  VAL_INV_NB   (u, K, L(u, K)) of a neighbour's u-network, with its K streams
  //               read from kin.
  // effective slope c_k = n a^k of hidden layer k (1 unless adaptive)
  __device__ static float slope(const NetDesc& nd, const float* K, const Layout& L, int k) {
    return nd.adaptive ? K[L.k_slope() + k - 1] : 1.f;
  }

  // GA: the general activation rule (any activation, trainable slopes);
  // for a tanh network without slopes it gives the plain rule's values
  template <int VMODE, bool GA>
  __device__ __forceinline__ static void values_tile(const KArgs& ka, const Item& it, const NetDesc& nd, float* lds,
                                                     float* dst, const float* kin, int t0) {
    char* sW = reinterpret_cast<char*>(lds);
    const int tid = item_tid();
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4, pc = lane & 15;
    const int tp = wave * 16 + pc;
    const Layout L(WP, nd.depth, DO);
    const float* K = ka.kparams + nd.koff;
    const float* xyv = it.kind == KIND_IFACE ? ka.if_xy : ka.res_xy;
    const bool valid = t0 + tp < it.count;
    const int gp = it.begin + t0 + tp;
    const float x = valid ? xyv[2 * (int64_t)gp] : 0.f;
    const float y = valid ? xyv[2 * (int64_t)gp + 1] : 0.f;
    if (nd.depth >= 2) fetch_wb(wbuf(sW, nd.depth, 2), K, L, 2, wave, lane);   // (the caller's barrier freed the buffers)
    Streams H;
    {
      Streams A;
      layer1(K, x, y, g, A);
      activate<GA>(A, H, nd.act, slope(nd, K, L, 1));
    }
    const __amdgpu_buffer_rsrc_t none = __builtin_amdgcn_make_buffer_rsrc(lds, 0, 0, 0x00020000);  // unused
    for (int k = 2; k <= nd.depth; ++k) {
      dma_landed();
      __syncthreads();
      if (k < nd.depth) fetch_wb(wbuf(sW, nd.depth, k + 1), K, L, k + 1, wave, lane);
      hidden_layer<false, GA>(wbuf(sW, nd.depth, k), g, H, none, k, wave, lane, nd, slope(nd, K, L, k));
    }
    float u[DO][4];
    out_fwd(K + L.k_out(), K + L.k_bout(), g, H, u);
    if (g != 0) return;
    if constexpr (VMODE == VAL_OWN) {
      const IfaceDesc ifd = ka.ifaces[it.iface];
      float ov[DO + NEQ];
      own_values(ifd.method, u, ifd.nx, ifd.ny, ka.coef0, ov);
#pragma unroll
      for (int v = 0; v < DO + NEQ; ++v) dst[tp * (DO + NEQ) + v] = ov[v];
    } else if constexpr (VMODE == VAL_STREAMS) {
#pragma unroll
      for (int s = 0; s < 3; ++s) dst[3 * tp + s] = u[0][s];
    } else {
      const float Kv = kin[3 * tp], Kx = kin[3 * tp + 1], Ky = kin[3 * tp + 2];
      dst[3 * tp] = u[0][0];
      dst[3 * tp + 1] = Kv;
      dst[3 * tp + 2] = fmaf(Kv, u[0][3], fmaf(Kx, u[0][1], Ky * u[0][2]));
    }
  }

  // ------------------------------------------------------------------------
  // forward, loss, adjoint and parameter-gradient partials of one item
  //
  // Tiles starting at t_lo .. t_hi - 1 (step TP) of the item; roff is the
  // offset of this network's part in the item's gradient row; MODE selects the
  // epilogue (sInv: the LDS exchange area of the inverse problem); PHASE the
  // parts run.  slot is this network's stash (slot_floats long).
  // Sum of dc over the wave's lanes into sSl[wave] (a fixed butterfly).
  __device__ static void slope_wave_sum(float dc, float* sSl, int lane, int wave) {
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) dc += __shfl_xor(dc, m);
    if (lane == 0) sSl[wave] = dc;
  }

  template <int MODE, int PHASE, bool GA>
  __device__ __forceinline__ static void run_train(const KArgs& ka, const Item& it, const NetDesc& nd, float* lds,
                                   float* slot, int64_t slot_floats, const float* sNb, float* sInv, float* sOW, int* sBad,
                                   int t_lo, int t_hi, int roff) {
    char* sW = reinterpret_cast<char*>(lds);
    float* sA = reinterpret_cast<float*>(sW + sums_offset(WP));   // sums of the output layer and of layer 1
    char* sS = sW + (stage_over_weights(WP) ? 0 : WBYTES);   // staging area of dW
    float* sRed = reinterpret_cast<float*>(sW + tile_bytes(WP, DO));   // [kWaves][kLossTerms]
    float* sSl = sRed + kWaves * kLossTerms;   // [kWaves] slope-gradient sums
    // the reverse pass follows the forward one here, and what it needs of the
    // last hidden layer is h^D, at hand, and a^D: of that layer, the value
    // stream alone is stashed.  (16 space-time boxes of 20 wide 147 -> 130
    // us a step, 50 wide 208 -> 203; a^D in registers as well spills and takes
    // that back.)
    constexpr bool HOLD = PHASE == PH_ALL && !GA;
    const int D = nd.depth;
    const Layout L(WP, D, DO);
    const float* K = ka.kparams + nd.koff;
    float* R = ka.partial + it.prow + roff;
    const float* xy = it.kind == KIND_RES    ? ka.res_xy
                      : it.kind == KIND_DATA ? ka.dat_xy
                      : it.kind == KIND_AUX  ? ka.aux_xy
                                             : ka.if_xy;
    const __amdgpu_buffer_rsrc_t rs =
        __builtin_amdgcn_make_buffer_rsrc(slot, 0, (int)(slot_floats * sizeof(float)), 0x00020000);

    for (int t0 = t_lo; t0 < t_hi; t0 += TP) {
      // lane indices re-derived per tile (see item_tid)
      int tid = item_tid();
      int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
      int g = lane >> 4, pc = lane & 15;
      int tp = wave * 16 + pc;
      const bool first = t0 == 0;
      const int pt = t0 + tp;
      const bool valid = pt < it.count;
      const int gp = it.begin + pt;
      const float x = valid ? xy[2 * (int64_t)gp] : 0.f;
      const float y = valid ? xy[2 * (int64_t)gp + 1] : 0.f;
      float tgt[NTGT] = {};
      if (valid && MODE != EPI_SEED && it.kind != KIND_IFACE) {
        const float* tg = it.kind == KIND_RES ? ka.res_f : it.kind == KIND_DATA ? ka.dat_g : ka.aux_g;
        const int nt = it.kind == KIND_RES ? NEQ : DO;
#pragma unroll
        for (int c = 0; c < NTGT; ++c)
          if (c < nt) tgt[c] = tg[(int64_t)gp * nt + c];
      }
      __syncthreads();  // previous tile done with LDS
      // the output layer's weights and the first hidden layer's stream in during layer 1
      dma_to_lds(sOW, K + L.k_out(), DO * WP / 4 + 1, wave, lane);
      if (PHASE != PH_BWD && D >= 2) fetch_wb(wbuf(sW, D, 2), K, L, 2, wave, lane);

      // ---- forward: Taylor streams through every layer, stashing what the
      // reverse pass needs (in PH_BWD only h^D is rebuilt, from the stash, or
      // from layer 1 if D = 1)
      Streams H;
      {
        Streams A;
        if (PHASE == PH_BWD && D >= 2) {
          stash_load(rs, D, wave, lane, A);
          const float cD = slope(nd, K, L, D);
#pragma unroll
          for (int s = 0; s < 4; ++s) h_stream<GA>(nd, s, cD, A, H[s]);
        } else {
          layer1(K, x, y, g, A);
          activate<GA>(A, H, nd.act, slope(nd, K, L, 1));
          if (D >= 2) stash_put_layer<GA>(nd, rs, 1, wave, lane, A, H);
        }
      }
      for (int k = 2; k <= (PHASE == PH_BWD ? 1 : D); ++k) {
        tid = item_tid();
        lane = tid & 63;
        wave = __builtin_amdgcn_readfirstlane(tid >> 6);
        g = lane >> 4;
        pc = lane & 15;
        tp = wave * 16 + pc;
        // W^k is in LDS (every wave's share landed) and every wave is done
        // with layer k - 1's buffer, which now receives W^{k+1}
        dma_landed();
        __syncthreads();
        if (k < D) fetch_wb(wbuf(sW, D, k + 1), K, L, k + 1, wave, lane);
        hidden_layer<true, GA>(wbuf(sW, D, k), g, H, rs, k, wave, lane, nd, slope(nd, K, L, k), HOLD && k == D);
      }
      if (PHASE == PH_BWD || D < 2) {   // else a hidden layer's barrier has published the output weights
        dma_landed();
        __syncthreads();
      }
      float u[DO][4];
      if constexpr (PHASE == PH_BWD) {
#pragma unroll
        for (int c = 0; c < DO; ++c) u[c][0] = u[c][1] = u[c][2] = u[c][3] = 0.f;   // seeds come from LDS
      } else {
        out_fwd(sOW, sOW + DO * WP, g, H, u);
      }
      if constexpr (PHASE == PH_FWD) {
        if (!finite_streams(u)) *sBad = 1;
        if (g == 0) {
#pragma unroll
          for (int s = 0; s < 3; ++s) sInv[3 * tp + s] = u[0][s];
        }
        continue;
      }

      // ---- loss terms and output seeds
      float ub[DO][4], loss[kLossTerms], kb[3];
      epilogue<MODE>(ka, it, nd, tp, valid, tgt, sNb + tp * (PDE == PDE_INV ? 3 : DO + NEQ), sInv, u, ub, loss, kb);
      if (!finite_streams(u) || !finite4(loss) || tiny_seeds(ub)) *sBad = 1;
#pragma unroll
      for (int t = 0; t < kLossTerms; ++t) {
        const float v = row_sum16(loss[t]);   // (the same in every lane group)
        if (lane == 0) sRed[wave * kLossTerms + t] = v;
      }
      if constexpr (MODE == EPI_INV_U) {
        if (g == 0) {
#pragma unroll
          for (int s = 0; s < 3; ++s) sInv[3 * TP + 3 * tp + s] = kb[s];
        }
      }

      // ---- output layer adjoint: g^D = W^{LT} ubar; dW^L, db^L
      // dW^L[c][n] = sum over points and streams of ubar_c h^D_n and db^L[c] =
      // sum over points of ubar_c (value stream): each lane's point term, summed
      // over the wave's 16 points by row_sum16 and over the waves through LDS
      {
        float* sOut = sA;                      // [kWaves][DO][WP], then [kWaves][DO] bias sums
        float* sOutB = sA + kWaves * DO * WP;
#pragma unroll
        for (int c = 0; c < DO; ++c) {
#pragma unroll
          for (int mb = 0; mb < MB; ++mb) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              float v = ub[c][0] * H[0][mb][i];
#pragma unroll
              for (int st = 1; st < 4; ++st) v = fmaf(ub[c][st], H[st][mb][i], v);
              v = row_sum16(v);
              if (pc == 0) sOut[(wave * DO + c) * WP + 16 * mb + 4 * g + i] = v;
            }
          }
          const float vb = row_sum16(ub[c][0]);
          if (lane == 0) sOutB[wave * DO + c] = vb;
        }
      }
      Streams G;
      __builtin_amdgcn_sched_barrier(0);
      {
        const float* WL = sOW;
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
          f4 wl[DO];
#pragma unroll
          for (int c = 0; c < DO; ++c) wl[c] = *reinterpret_cast<const f4*>(WL + c * WP + 16 * mb + 4 * g);
#pragma unroll
          for (int i = 0; i < 4; ++i) {
#pragma unroll
            for (int s = 0; s < 4; ++s) {
              float acc = 0.f;
#pragma unroll
              for (int c = 0; c < DO; ++c) acc = fmaf(wl[c][i], ub[c][s], acc);
              G[s][mb][i] = acc;
            }
          }
        }
      }
      __builtin_amdgcn_sched_barrier(0);
      // what was kept of layer k; what is not in registers (HOLD) of the last
      // layer's is loaded while the output layer's sums run
      Streams Sk;
      if constexpr (HOLD) {
        if (KEEP && D >= 2) stash_load_stream(rs, D, wave, lane, 0, Sk[0]);
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
#pragma unroll
          for (int s = 1; s < 4; ++s) Sk[s][mb] = H[s][mb];
        }
      } else if (KEEP && D >= 2) {
        stash_load(rs, D, wave, lane, Sk);
      }
      __syncthreads();
      // every wave is past the last forward layer: W^{D T} streams into the
      // first buffer (where the staging area of dW does not cover it)
      if (!stage_over_weights(WP) && D >= 2) fetch_wt(sW, K, L, D, wave, lane);
#pragma unroll
      for (int r = 0; r < KL; ++r) {
        const int t = tid + r * NT;
        if (t < DO * WP) {
          float v = prior(R + L.g_out() + t, first);
#pragma unroll
          for (int wv = 0; wv < kWaves; ++wv) v += sA[wv * DO * WP + t];
          R[L.g_out() + t] = v;
        }
      }
      if (tid < DO) {
        float v = prior(R + L.g_bout() + tid, first);
#pragma unroll
        for (int wv = 0; wv < kWaves; ++wv) v += sA[kWaves * DO * WP + wv * DO + tid];
        R[L.g_bout() + tid] = v;
      }
      if (MODE != EPI_SEED && tid < kLossTerms) {   // the u pass holds a paired item's loss
        float v = 0.f;
        for (int wv = 0; wv < kWaves; ++wv) v += sRed[wv * kLossTerms + tid];
        accum(ka.loss_part + (int64_t)it.lrow * kLossTerms + tid, v * it.inv_n, first);
      }

      // ---- hidden layers, top down.  G holds g^k on entry to layer k and is
      // turned into abar^k in place; then, stream by stream, abar^k and h^{k-1}
      // go through LDS for dW^k = sum_{points, streams} abar^k h^{k-1 T} and
      // db^k = sum_points abar^k_0, and last g^{k-1} = W^{kT} abar^k.  With dW
      // first, a pair of streams of g^{k-1} takes the registers its abar^k
      // leaves, so one layer of streams and one pair are live at most.
      for (int k = D; k >= 2; --k) {
        // and again per layer, so address arithmetic is not pinned across layers
        tid = item_tid();
        lane = tid & 63;
        wave = __builtin_amdgcn_readfirstlane(tid >> 6);
        g = lane >> 4;
        pc = lane & 15;
        tp = wave * 16 + pc;
        // dW^k / db^k accumulators start from the partial row
        float* Rw = R + L.g_w(k);
        float* Rb = R + L.g_b(k);
        // layer k - 1's share of the stash, for h^{k-1} here and for the next
        // layer's adjoint, takes the place of layer k's block by block (KEEP);
        // class 80 has no registers to hold it, loads h^{k-1} stream by
        // stream and the whole again at the end
        Streams Sp;
        if constexpr (!KEEP) {
          if (HOLD && k == D) stash_load_stream(rs, k, wave, lane, 0, Sk[0]);
          else stash_load(rs, k, wave, lane, Sk);
        }
        // abar^k from what was kept of layer k and the incoming g^k (in place of
        // g^k); with a general activation also the layer's slope gradient
        {
          const float ck = GA ? slope(nd, K, L, k) : 1.f;
          float dc = 0.f;
          const bool hk = h_form<GA>(nd);
#pragma unroll
          for (int mb = 0; mb < MB; ++mb) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              float a0, a1, a2, a3;
              if (hk)
                tanh_adj_h<S2>(Sk[0][mb][i], Sk[1][mb][i], Sk[2][mb][i], Sk[3][mb][i], G[0][mb][i], G[1][mb][i],
                               G[2][mb][i], G[3][mb][i], a0, a1, a2, a3);
              else
                act_adj<S2>(nd.act, ck, Sk[0][mb][i], Sk[1][mb][i], Sk[2][mb][i], Sk[3][mb][i], G[0][mb][i],
                            G[1][mb][i], G[2][mb][i], G[3][mb][i], a0, a1, a2, a3, dc);
              G[0][mb][i] = a0;
              G[1][mb][i] = a1;
              G[2][mb][i] = a2;
              G[3][mb][i] = a3;
            }
            if constexpr (MB >= 3) __builtin_amdgcn_sched_barrier(0);
            if constexpr (KEEP) {
#pragma unroll
              for (int s = 0; s < 4; ++s) stash_load_block(rs, k - 1, wave, lane, s, mb, Sp[s][mb]);
            }
          }
          if constexpr (GA) slope_wave_sum(dc, sSl, lane, wave);
        }
        pin(G);   // the adjoint is done here, not after the branches below
        if constexpr (PRIV) {
          // each wave on its own points, one stream after the other
          constexpr int NE = (MB * MB + kWaves - 1) / kWaves;   // sums of 4 entries per thread
          f4 before[NE];
          float bias_before = 0.f;
#pragma unroll
          for (int r = 0; r < NE; ++r) before[r] = f4{0.f, 0.f, 0.f, 0.f};
          if (!first) {
#pragma unroll
            for (int r = 0; r < NE; ++r) {
              const int b = min(wave + r * kWaves, MB * MB - 1);
#pragma unroll
              for (int i = 0; i < 4; ++i)
                before[r][i] = device_load(Rw + (16 * (b / MB) + 4 * g + i) * WP + 16 * (b % MB) + pc);
            }
            if (tid < WP) bias_before = device_load(Rb + tid);
          }
          char* my = sS + wave * (6 * PART);
          f4 dacc[MB][MB], dbias[MB];
#pragma unroll
          for (int mb = 0; mb < MB; ++mb) {
            dbias[mb] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int jb = 0; jb < MB; ++jb) dacc[mb][jb] = f4{0.f, 0.f, 0.f, 0.f};
          }
#pragma unroll
          for (int s = 0; s < 4; ++s) {
            f4 hs[MB];
            h_stream<GA>(nd, s, GA ? slope(nd, K, L, k - 1) : 1.f, Sp, hs);
            stage_put(my, pc, g, G[s]);
            stage_put(my + 3 * PART, pc, g, hs);
            wave_fence();
            b8 amh[MB], ahl[MB];
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) {
              const Frag16 a = stage_parts16(my, mb, lane);
              amh[mb] = join(a.m, a.h);
              ahl[mb] = join(a.h, a.l);
            }
#pragma unroll
            for (int jb = 0; jb < MB; ++jb) {
              const Frag16 h = stage_parts16(my + 3 * PART, jb, lane);
              const b8 hh = join(h.h, h.h), mm = join(h.m, h.m), lh = join(h.l, h.h);
#pragma unroll
              for (int mb = 0; mb < MB; ++mb) dacc[mb][jb] = mma(ahl[mb], lh, dacc[mb][jb]);
#pragma unroll
              for (int mb = 0; mb < MB; ++mb) dacc[mb][jb] = mma(amh[mb], mm, dacc[mb][jb]);
#pragma unroll
              for (int mb = 0; mb < MB; ++mb) dacc[mb][jb] = mma(amh[mb], hh, dacc[mb][jb]);
            }
            if (s == 0) {   // db^k: the rows times ones
              const __bf16 o = (__bf16)1.f, z = (__bf16)0.f;
#pragma unroll
              for (int mb = 0; mb < MB; ++mb)
                dbias[mb] = mma(amh[mb], b8{o, o, o, o, o, o, o, o}, mma(ahl[mb], b8{z, z, z, z, o, o, o, o}, dbias[mb]));
            }
            wave_fence();
          }
          // the wave's sums in place of its staging area, then their sum over the waves
          f4* red = reinterpret_cast<f4*>(my);
#pragma unroll
          for (int mb = 0; mb < MB; ++mb) {
#pragma unroll
            for (int jb = 0; jb < MB; ++jb) red[(mb * MB + jb) * 64 + lane] = dacc[mb][jb];
            if (pc == 0) red[MB * MB * 64 + 4 * mb + g] = dbias[mb];
          }
          dma_landed();
          __syncthreads();   // the sums are there, and W^{kT}
          if constexpr (GA) {
            if (nd.adaptive && tid == 0) accum(R + L.g_slope() + k - 1, (sSl[0] + sSl[1]) + (sSl[2] + sSl[3]), first);
          }
          const char* all = sS;
#pragma unroll
          for (int r = 0; r < NE; ++r) {
            const int b = wave + r * kWaves;
            if (b < MB * MB) {
              f4 v = before[r];
#pragma unroll
              for (int w = 0; w < kWaves; ++w) v += reinterpret_cast<const f4*>(all + w * (6 * PART))[b * 64 + lane];
#pragma unroll
              for (int i = 0; i < 4; ++i) Rw[(16 * (b / MB) + 4 * g + i) * WP + 16 * (b % MB) + pc] = v[i];
            }
          }
          if (tid < WP) {
            float v = bias_before;
#pragma unroll
            for (int w = 0; w < kWaves; ++w)
              v += reinterpret_cast<const float*>(all + w * (6 * PART))[MB * MB * 256 + tid];
            Rb[tid] = v;
          }
        } else {
          auto block_prior = [&](int mb, int jb) {
            f4 v;
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = device_load(Rw + (16 * mb + 4 * g + i) * WP + 16 * jb + pc);
            return v;
          };
          auto bias_prior = [&](int mb) {
            f4 v;
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = device_load(Rb + 16 * mb + 4 * g + i);
            return v;
          };
          // the wave's left-over block r (the last one again where there is none)
          auto left_over = [&](int r) { return min(wave + r * kWaves, REM - 1); };
          f4 dacc[ROWS][MB], drem[NREM + 1], dbias[ROWS], dbrem[NREM + 1];
          if (first) {
            const f4 zero = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int r = 0; r < ROWS; ++r) {
#pragma unroll
              for (int jb = 0; jb < MB; ++jb) dacc[r][jb] = zero;
              dbias[r] = zero;
            }
#pragma unroll
            for (int r = 0; r < NREM; ++r) drem[r] = dbrem[r] = zero;
          } else {
#pragma unroll
            for (int r = 0; r < ROWS; ++r) {
#pragma unroll
              for (int jb = 0; jb < MB; ++jb) dacc[r][jb] = block_prior(4 * r + wave, jb);
              dbias[r] = bias_prior(4 * r + wave);
            }
#pragma unroll
            for (int r = 0; r < NREM; ++r) {
              drem[r] = block_prior(4 * ROWS + left_over(r) / MB, left_over(r) % MB);
              dbrem[r] = bias_prior(4 * ROWS + left_over(r) / MB);
            }
          }
          f4 Hn[MB];
          const bool hf = h_form<GA>(nd);
          const int hlayer = k - 1 + (hf ? 0 : kMaxDepth);
          if constexpr (!KEEP) stash_load_stream(rs, hlayer, wave, lane, 0, Hn);
#pragma unroll
          for (int s = 0; s < 4; ++s) {
            __syncthreads();   // the previous stage's dW, or the last W^T abar, is done with the staging area
            if (s == 0) {      // (the barrier published the slope sums too)
              if constexpr (GA) {
                if (nd.adaptive && tid == 0)
                  accum(R + L.g_slope() + k - 1, (sSl[0] + sSl[1]) + (sSl[2] + sSl[3]), first);
              }
            }
            stage_put(sS, tp, g, G[s]);
            if constexpr (KEEP) {
              h_stream<GA>(nd, s, GA ? slope(nd, K, L, k - 1) : 1.f, Sp, Hn);
            } else if (s == 0 && hf) {
#pragma unroll
              for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                  float t, s1;
                  tanh_s1(Hn[mb][i], t, s1);
                  Hn[mb][i] = t;
                }
            }
            stage_put(sS + 3 * PART, tp, g, Hn);
            if constexpr (!KEEP) {
              if (s < 3) stash_load_stream(rs, hlayer, wave, lane, s + 1, Hn);
            }
            // every wave is past W^{k+1 T}: W^{kT} streams in during dW^k (issued here,
            // behind the waits for the stash)
            if (!stage_over_weights(WP) && s == 0 && k < D) fetch_wt(sW, K, L, k, wave, lane);
            __syncthreads();
            // fragments are read one block ahead of their MFMAs
            constexpr int NC = SROWS / 32;
#pragma unroll
            for (int r = 0; r < ROWS; ++r) {
              Frag a = stage_parts(sS, 0, 4 * r + wave, lane), h = stage_parts(sS + 3 * PART, 0, 0, lane);
#pragma unroll
              for (int c = 0; c < NC; ++c) {
                if (s == 0) dbias[r] = row_sums(a, dbias[r]);
#pragma unroll
                for (int jb = 0; jb < MB; ++jb) {
                  Frag an = a, hn = h;
                  if (jb + 1 < MB) {
                    hn = stage_parts(sS + 3 * PART, c, jb + 1, lane);
                  } else if (c + 1 < NC) {
                    an = stage_parts(sS, c + 1, 4 * r + wave, lane);
                    hn = stage_parts(sS + 3 * PART, c + 1, 0, lane);
                  }
                  __builtin_amdgcn_sched_barrier(0);
                  dacc[r][jb] = mma6(a, h, dacc[r][jb]);
                  a = an;
                  h = hn;
                }
              }
            }
            if constexpr (NREM > 0) {
              Frag a = stage_parts(sS, 0, 4 * ROWS + left_over(0) / MB, lane);
              Frag h = stage_parts(sS + 3 * PART, 0, left_over(0) % MB, lane);
#pragma unroll
              for (int t = 0; t < NREM * NC; ++t) {
                Frag an = a, hn = h;
                if (t + 1 < NREM * NC) {
                  const int b = left_over((t + 1) / NC);
                  an = stage_parts(sS, (t + 1) % NC, 4 * ROWS + b / MB, lane);
                  hn = stage_parts(sS + 3 * PART, (t + 1) % NC, b % MB, lane);
                }
                __builtin_amdgcn_sched_barrier(0);
                if (s == 0) dbrem[t / NC] = row_sums(a, dbrem[t / NC]);
                drem[t / NC] = mma6(a, h, drem[t / NC]);
                a = an;
                h = hn;
              }
            }
          }
          if constexpr (stage_over_weights(WP)) {
            __syncthreads();   // every wave is done with the staging area, which now receives W^{kT}
            fetch_wt(sW, K, L, k, wave, lane);
          }
          auto block_store = [&](int mb, int jb, f4 v) {
#pragma unroll
            for (int i = 0; i < 4; ++i) Rw[(16 * mb + 4 * g + i) * WP + 16 * jb + pc] = v[i];
          };
#pragma unroll
          for (int r = 0; r < ROWS; ++r) {
#pragma unroll
            for (int jb = 0; jb < MB; ++jb) block_store(4 * r + wave, jb, dacc[r][jb]);
            if (pc == 0) *reinterpret_cast<f4*>(Rb + 16 * (4 * r + wave) + 4 * g) = dbias[r];
          }
#pragma unroll
          for (int r = 0; r < NREM; ++r) {
            const int b = wave + r * kWaves;
            if (b < REM) {
              const int mb = 4 * ROWS + b / MB;
              block_store(mb, b % MB, drem[r]);
              if (b % MB == 0 && pc == 0) *reinterpret_cast<f4*>(Rb + 16 * mb + 4 * g) = dbrem[r];
            }
          }
          dma_landed();
          __syncthreads();   // W^{kT} is in LDS
        }
        {
          if constexpr (MB >= 4) pin(G);   // else the parts just staged are kept for W^T abar, half as many registers again
          Streams Gn;
#pragma unroll
          for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) Gn[s][mb] = f4{0.f, 0.f, 0.f, 0.f};
          if constexpr (KEEP) {
            contract4<MB <= 5>(sW, lane, G, Gn);
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
              for (int mb = 0; mb < MB; ++mb) Sk[s][mb] = Sp[s][mb];
          } else {
            contract<0, 2>(sW, lane, G, Gn);
            contract<2, 2>(sW, lane, G, Gn);
            if constexpr (HOLD) forget(Sk);   // loaded at the top, not carried there
          }
#pragma unroll
          for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) G[s][mb] = Gn[s][mb];
        }
        if constexpr (PRIV) {
          __syncthreads();   // every wave is done with W^{kT} and with the sums
          if (k > 2) fetch_wt(sW, K, L, k - 1, wave, lane);
        }
      }

      // ---- layer 1: abar^1 from a^1 and g^1; dW^1[n] = sum over points of
      // (abar^1_n z + d abar^1_n) and db^1[n] = sum of abar^1_n: each lane's
      // point terms, summed over the wave's 16 points by row_sum16 and over
      // the waves through LDS
      {
        float p0 = 0.f, p1 = 0.f, p2 = 0.f;
        if (tid < WP) {
          p0 = prior(R + 4 * tid, first);
          p1 = prior(R + 4 * tid + 1, first);
          p2 = prior(R + 4 * tid + 2, first);
        }
        Streams A1;
        layer1(K, x, y, g, A1);
        const float c1 = GA ? slope(nd, K, L, 1) : 1.f;
        float dc = 0.f;
        float* sOut = sA;   // [kWaves][3][WP]
        __syncthreads();    // every wave is done with LDS (the last W^T abar, or the output layer's sums)
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            float a0, a1, a2, a3;
            if constexpr (GA)
              act_adj<S2>(nd.act, c1, A1[0][mb][i], A1[1][mb][i], A1[2][mb][i], A1[3][mb][i], G[0][mb][i],
                          G[1][mb][i], G[2][mb][i], G[3][mb][i], a0, a1, a2, a3, dc);
            else
              tanh_adj<S2>(A1[0][mb][i], A1[1][mb][i], A1[2][mb][i], A1[3][mb][i], G[0][mb][i], G[1][mb][i],
                           G[2][mb][i], G[3][mb][i], a0, a1, a2, a3);
            const float r0 = row_sum16(fmaf(a0, x, a1));
            const float r1 = row_sum16(fmaf(a0, y, a2));
            const float r2 = row_sum16(a0);
            if (pc == 0) {
              const int n = 16 * mb + 4 * g + i;
              sOut[(wave * 3 + 0) * WP + n] = r0;
              sOut[(wave * 3 + 1) * WP + n] = r1;
              sOut[(wave * 3 + 2) * WP + n] = r2;
            }
          }
        }
        if constexpr (GA) slope_wave_sum(dc, sSl, lane, wave);
        __syncthreads();
        if constexpr (GA) {
          if (nd.adaptive && tid == 0) accum(R + L.g_slope(), (sSl[0] + sSl[1]) + (sSl[2] + sSl[3]), first);
        }
        if (tid < WP) {
          float dw0 = p0, dw1 = p1, db = p2;
#pragma unroll
          for (int wv = 0; wv < kWaves; ++wv) {
            dw0 += sOut[(wv * 3 + 0) * WP + tid];
            dw1 += sOut[(wv * 3 + 1) * WP + tid];
            db += sOut[(wv * 3 + 2) * WP + tid];
          }
          // whatever is not finite in the reverse pass arrives here
          if (!(fmaf(dw0, 0.f, fmaf(dw1, 0.f, db * 0.f)) == 0.f)) *sBad = 1;
          R[4 * tid] = dw0;
          R[4 * tid + 1] = dw1;
          R[4 * tid + 2] = db;
          if (first) R[4 * tid + 3] = 0.f;
        }
      }
    }
  }

};

// Whether the network's first hidden matrix begins with NaN, as all of a
// network's parameters are after one step on a gradient of NaN: every output
// and gradient entry is NaN in any arithmetic.
__device__ __forceinline__ bool nan_network(const KArgs& ka, const NetDesc& nd) {
  const Layout L(nd.wclass, nd.depth, nd.d_out);
  return nd.depth >= 2 && isnan((float)*reinterpret_cast<const __bf16*>(ka.kparams + nd.koff + L.k_w(2)));
}

// Whether the item's term has less than 2^-24 of the weight of another of its
// subdomain: its seeds may be tiny for that alone, and the last bits of its
// share are below those of the other's.  (A term weighted 1e-30 to leave it out
// would otherwise have its items run again at every step.)
__device__ __forceinline__ bool small_term(const Item& it, const NetDesc& nd) {
  const float wi = fmaxf(nd.loss_w[2], nd.loss_w[3]);
  const float w = it.kind == KIND_RES ? nd.loss_w[1] : it.kind == KIND_IFACE ? wi : nd.loss_w[0];
  return w < 0x1p-24f * fmaxf(fmaxf(nd.loss_w[0], nd.loss_w[1]), wi);
}

// ---------------------------------------------------------------------------
// The same item in float32 throughout, with sizes known at run time, for what
// is no sum of three bf16 parts: infinities (a split one is infinity and NaN,
// and the dot products of the split carry the NaN to the neuron beside it),
// values from 3.3961e38 on, and below 2^-109 the last bits.  Tile notes when a
// tile's outputs, losses or first-layer gradients are not finite, where all
// such values end up, or its output seeds are all below kTinySeed; the
// workgroup then runs the item again here, over the rows it has written.
//
// Rare, so short and light on registers rather than fast: a wave takes its 16
// points from layer to layer, pre-activations and adjoints through the stash
// slot (Tile's layout, layer 1's place taken by the adjoints), weights from the
// kernel copy in the L2 cache, contractions on the 16x16x4 float32 MFMA.
template <int PDE, bool GA>
struct Plain {
  using T = Tile<16, PDE>;   // for what does not depend on the width
  typedef __attribute__((address_space(4))) KArgs Args;   // the kernel's arguments where they lie
  typedef __attribute__((address_space(3))) float Lds;
  static constexpr int DO = Op<PDE>::DO, NEQ = Op<PDE>::NEQ;
  static constexpr bool S2 = Op<PDE>::S2;

  const KArgs& ka;
  const Item& it;
  const NetDesc& nd;
  float* st;        // the network's stash
  const int t0;     // the tile's first point
  const int WP, MB, D;
  const Layout L;
  const float* K;
  const float* xy;
  int tid, lane, wave, g, pc;

  __device__ Plain(const KArgs& ka_, const Item& it_, const NetDesc& nd_, float* st_, int t0_)
      : ka(ka_), it(it_), nd(nd_), st(st_), t0(t0_), WP(nd_.wclass), MB(nd_.wclass / 16), D(nd_.depth),
        L(nd_.wclass, nd_.depth, DO), K(ka_.kparams + nd_.koff) {
    xy = it.kind == KIND_RES ? ka.res_xy : it.kind == KIND_DATA ? ka.dat_xy : it.kind == KIND_AUX ? ka.aux_xy : ka.if_xy;
    tid = item_tid();
    lane = tid & 63;
    wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    g = lane >> 4;
    pc = lane & 15;
  }

  __device__ float coord(int p, int c) const { return t0 + p < it.count ? xy[2 * (int64_t)(it.begin + t0 + p) + c] : 0.f; }
  // place of (layer, wave, stream, block, lane) in the stash, 4 neurons each
  __device__ float* place(int layer, int wv, int s, int mb, int ln) const {
    return st + ((((int64_t)(layer - 1) * kWaves + wv) * 4 + s) * MB + mb) * 256 + 4 * ln;
  }
  __device__ f4 load4(int layer, int s, int mb) const {
    const float* p = place(layer, wave, s, mb, lane);
    f4 v;
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = T::device_load(p + i);
    return v;
  }
  __device__ void store4(int layer, int s, int mb, f4 v) const {
    *reinterpret_cast<f4*>(place(layer, wave, s, mb, lane)) = v;
  }
  // pre-activation streams of layer 1, neuron n, at (x, y)
  __device__ void first_layer(int n, float x, float y, float (&a)[4]) const {
    const f4 c = *reinterpret_cast<const f4*>(K + 4 * n);
    a[0] = fmaf(c[0], x, fmaf(c[1], y, c[2]));
    a[1] = c[0];
    a[2] = c[1];
    a[3] = 0.f;
  }
  // the lane's four neurons of block mb of layer k: pre-activation streams
  __device__ void pre(int k, int mb, float x, float y, f4 (&A)[4]) const {
    if (k == 1) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        float a[4];
        first_layer(16 * mb + 4 * g + i, x, y, a);
#pragma unroll
        for (int s = 0; s < 4; ++s) A[s][i] = a[s];
      }
    } else {
#pragma unroll
      for (int s = 0; s < 4; ++s) A[s] = load4(k, s, mb);
    }
  }
  __device__ void rule(float c, float a, float ax, float ay, float al, float (&h)[4]) const {
    if constexpr (GA) act_rule<S2>(nd.act, c, a, ax, ay, al, h[0], h[1], h[2], h[3]);
    else tanh_rule<S2>(a, ax, ay, al, h[0], h[1], h[2], h[3]);
  }
  __device__ void post(int k, int mb, float x, float y, f4 (&H)[4]) const {
    f4 A[4];
    pre(k, mb, x, y, A);
    const float c = T::slope(nd, K, L, k);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float h[4];
      rule(c, A[0][i], A[1][i], A[2][i], A[3][i], h);
#pragma unroll
      for (int s = 0; s < 4; ++s) H[s][i] = h[s];
    }
  }
  __device__ void adjoint(float c, float a, float ax, float ay, float al, f4 (&G)[4], int i, float& dc) const {
    float b[4];
    if constexpr (GA)
      act_adj<S2>(nd.act, c, a, ax, ay, al, G[0][i], G[1][i], G[2][i], G[3][i], b[0], b[1], b[2], b[3], dc);
    else
      tanh_adj<S2>(a, ax, ay, al, G[0][i], G[1][i], G[2][i], G[3][i], b[0], b[1], b[2], b[3]);
#pragma unroll
    for (int s = 0; s < 4; ++s) G[s][i] = b[s];
  }
  // acc_s += (rows of block rb) x (columns of block cb) of split matrix M times X_s
  __device__ void block(const float* M, int rb, int cb, const f4 (&X)[4], f4 (&acc)[4]) const {
    int ps;
    const __bf16* p = reinterpret_cast<const __bf16*>(M) + split_pos(WP, 16 * rb + pc, 16 * cb + 4 * g, ps);
    const b4 m = *reinterpret_cast<const b4*>(p), h = *reinterpret_cast<const b4*>(p + ps),
             l = *reinterpret_cast<const b4*>(p + 2 * ps);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float w = (float)h[i] + ((float)m[i] + (float)l[i]);
#pragma unroll
      for (int s = 0; s < 4; ++s) acc[s] = mma_f32(w, X[s][i], acc[s]);
    }
  }
  // the wave's own stores have arrived before its next loads
  __device__ void settle() const {
    wave_fence();
    dma_landed();
    wave_fence();
  }

  // hidden layers 2 .. D, pre-activations to the stash
  __device__ void forward(float x, float y) const {
#pragma unroll 1
    for (int k = 2; k <= D; ++k) {
#pragma unroll 1
      for (int mb = 0; mb < MB; ++mb) {
        f4 acc[4] = {};
        acc[0] = *reinterpret_cast<const f4*>(K + L.k_b(k) + 16 * mb + 4 * g);
#pragma unroll 1
        for (int jb = 0; jb < MB; ++jb) {
          f4 H[4];
          post(k - 1, jb, x, y, H);
          block(K + L.k_w(k), mb, jb, H, acc);
        }
#pragma unroll
        for (int s = 0; s < 4; ++s) store4(k, s, mb, acc[s]);
      }
      settle();
    }
  }
  __device__ void outputs(float x, float y, float (&u)[DO][4]) const {
    float acc[DO][4] = {};
#pragma unroll 1
    for (int mb = 0; mb < MB; ++mb) {
      f4 H[4];
      post(D, mb, x, y, H);
#pragma unroll
      for (int c = 0; c < DO; ++c) {
        const f4 w = *reinterpret_cast<const f4*>(K + L.k_out() + c * WP + 16 * mb + 4 * g);
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int s = 0; s < 4; ++s) acc[c][s] = fmaf(w[i], H[s][i], acc[c][s]);
      }
    }
#pragma unroll
    for (int c = 0; c < DO; ++c)
#pragma unroll
      for (int s = 0; s < 4; ++s) u[c][s] = group_sum(acc[c][s]) + (s == 0 ? K[L.k_bout() + c] : 0.f);
  }

  // values_tile
  template <int VMODE>
  __device__ void values(float* dst, const float* kin) const {
    const int tp = wave * 16 + pc;
    const float x = coord(tp, 0), y = coord(tp, 1);
    float u[DO][4];
    forward(x, y);
    outputs(x, y, u);
    if (g != 0) return;
    if constexpr (VMODE == VAL_OWN) {
      const IfaceDesc ifd = ka.ifaces[it.iface];
      float ov[DO + NEQ];
      T::own_values(ifd.method, u, ifd.nx, ifd.ny, ka.coef0, ov);
#pragma unroll
      for (int v = 0; v < DO + NEQ; ++v) dst[tp * (DO + NEQ) + v] = ov[v];
    } else if constexpr (VMODE == VAL_STREAMS) {
#pragma unroll
      for (int s = 0; s < 3; ++s) dst[3 * tp + s] = u[0][s];
    } else {
      const float Kv = kin[3 * tp], Kx = kin[3 * tp + 1], Ky = kin[3 * tp + 2];
      dst[3 * tp] = u[0][0];
      dst[3 * tp + 1] = Kv;
      dst[3 * tp + 2] = fmaf(Kv, u[0][3], fmaf(Kx, u[0][1], Ky * u[0][2]));
    }
  }

  // run_train on one tile (red: LDS for the sums over the waves)
  template <int MODE, int PHASE>
  __device__ void train(float* red, const float* sNb, float* sInv, int roff) const {
    const int tp = wave * 16 + pc;
    const bool first = t0 == 0, valid = t0 + tp < it.count;
    const float x = coord(tp, 0), y = coord(tp, 1);
    float* R = ka.partial + it.prow + roff;
    float* sSl = red;                                        // [kMaxDepth][kWaves] slope-gradient sums
    float* sLoss = sSl + kMaxDepth * kWaves;                 // [kWaves][kLossTerms]
    float* sOutB = sLoss + kWaves * kLossTerms;              // [kWaves][DO]
    float* sOut = sOutB + kWaves * DO;                       // [kWaves][DO or 3][WP]
    float u[DO][4] = {};
    if constexpr (PHASE != PH_BWD) {
      forward(x, y);
      outputs(x, y, u);
    }
    if constexpr (PHASE == PH_FWD) {
      if (g == 0) {
#pragma unroll
        for (int s = 0; s < 3; ++s) sInv[3 * tp + s] = u[0][s];
      }
      return;
    }
    __syncthreads();   // the K streams are there, and the sums' place is free
    float tgt[NTGT] = {};
    if (valid && MODE != EPI_SEED && it.kind != KIND_IFACE) {
      const float* tg = it.kind == KIND_RES ? ka.res_f : it.kind == KIND_DATA ? ka.dat_g : ka.aux_g;
      const int nt = it.kind == KIND_RES ? NEQ : DO;
#pragma unroll
      for (int c = 0; c < NTGT; ++c)
        if (c < nt) tgt[c] = tg[(int64_t)(it.begin + t0 + tp) * nt + c];
    }
    float ub[DO][4], loss[kLossTerms], kb[3];
    T::template epilogue<MODE>(ka, it, nd, tp, valid, tgt, sNb + tp * (PDE == PDE_INV ? 3 : DO + NEQ), sInv, u, ub, loss,
                               kb);
#pragma unroll
    for (int t = 0; t < kLossTerms; ++t) {
      const float v = row_sum16(loss[t]);
      if (lane == 0) sLoss[wave * kLossTerms + t] = v;
    }
    if constexpr (MODE == EPI_INV_U) {
      if (g == 0) {
#pragma unroll
        for (int s = 0; s < 3; ++s) sInv[3 * TP + 3 * tp + s] = kb[s];
      }
    }
    // output layer: its gradient, and g^D into layer 1's place
    int at = 1;
#pragma unroll 1
    for (int mb = 0; mb < MB; ++mb) {
      f4 H[4], G[4] = {};
      post(D, mb, x, y, H);
#pragma unroll
      for (int c = 0; c < DO; ++c) {
        const f4 w = *reinterpret_cast<const f4*>(K + L.k_out() + c * WP + 16 * mb + 4 * g);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          float v = ub[c][0] * H[0][i];
#pragma unroll
          for (int s = 1; s < 4; ++s) v = fmaf(ub[c][s], H[s][i], v);
          v = row_sum16(v);
          if (pc == 0) sOut[(wave * DO + c) * WP + 16 * mb + 4 * g + i] = v;
#pragma unroll
          for (int s = 0; s < 4; ++s) G[s][i] = fmaf(w[i], ub[c][s], G[s][i]);
        }
      }
#pragma unroll
      for (int s = 0; s < 4; ++s) store4(at, s, mb, G[s]);
    }
#pragma unroll
    for (int c = 0; c < DO; ++c) {
      const float v = row_sum16(ub[c][0]);
      if (lane == 0) sOutB[wave * DO + c] = v;
    }
    settle();
    __syncthreads();
    for (int t = tid; t < DO * WP; t += NT) {
      float v = T::prior(R + L.g_out() + t, first);
      for (int w = 0; w < kWaves; ++w) v += sOut[w * DO * WP + t];
      R[L.g_out() + t] = v;
    }
    if (tid < DO) {
      float v = T::prior(R + L.g_bout() + tid, first);
      for (int w = 0; w < kWaves; ++w) v += sOutB[w * DO + tid];
      R[L.g_bout() + tid] = v;
    }
    if (MODE != EPI_SEED && tid < kLossTerms) {
      float v = 0.f;
      for (int w = 0; w < kWaves; ++w) v += sLoss[w * kLossTerms + tid];
      T::accum(ka.loss_part + (int64_t)it.lrow * kLossTerms + tid, v * it.inv_n, first);
    }

    // hidden layers: the adjoint in place of g^k (place at), dW^k and db^k from
    // all waves' shares, then g^{k-1} in layer k's place
#pragma unroll 1
    for (int k = D; k >= 2; --k) {
      const float c = T::slope(nd, K, L, k);
      float dc = 0.f;
#pragma unroll 1
      for (int mb = 0; mb < MB; ++mb) {
        f4 A[4], G[4];
        pre(k, mb, x, y, A);
#pragma unroll
        for (int s = 0; s < 4; ++s) G[s] = load4(at, s, mb);
#pragma unroll
        for (int i = 0; i < 4; ++i) adjoint(c, A[0][i], A[1][i], A[2][i], A[3][i], G, i, dc);
#pragma unroll
        for (int s = 0; s < 4; ++s) store4(at, s, mb, G[s]);
      }
      if constexpr (GA) T::slope_wave_sum(dc, sSl + (k - 1) * kWaves, lane, wave);
      settle();
      __syncthreads();
      if constexpr (GA) {
        if (nd.adaptive && tid == 0) slope_grad(R, sSl, k, first);
      }
      const float c1 = T::slope(nd, K, L, k - 1);
#pragma unroll 1
      for (int b = wave; b < MB * MB; b += kWaves) {
        const int mb = b / MB, jb = b % MB;
        float* Rw = R + L.g_w(k) + (16 * mb + 4 * g) * WP + 16 * jb + pc;
        float* Rb = R + L.g_b(k) + 16 * mb + 4 * g;
        f4 acc, accb;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          acc[i] = T::prior(Rw + i * WP, first);
          accb[i] = T::prior(Rb + i, first);
        }
#pragma unroll 1
        for (int p = g; p < TP; p += 4) {   // neuron pc of the blocks at point p
          const int ln = 16 * (pc >> 2) + (p & 15), i = pc & 3;
          float a[4], h[4];
          if (k == 2) {
            first_layer(16 * jb + pc, coord(p, 0), coord(p, 1), a);
          } else {
#pragma unroll
            for (int s = 0; s < 4; ++s) a[s] = T::device_load(place(k - 1, p >> 4, s, jb, ln) + i);
          }
          rule(c1, a[0], a[1], a[2], a[3], h);
#pragma unroll
          for (int s = 0; s < 4; ++s) a[s] = T::device_load(place(at, p >> 4, s, mb, ln) + i);
#pragma unroll
          for (int s = 0; s < 4; ++s) acc = mma_f32(a[s], h[s], acc);
          accb = mma_f32(a[0], 1.f, accb);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) Rw[i * WP] = acc[i];
        if (jb == 0 && pc == 0) {
#pragma unroll
          for (int i = 0; i < 4; ++i) Rb[i] = accb[i];
        }
      }
#pragma unroll 1
      for (int jb = 0; jb < MB; ++jb) {
        f4 acc[4] = {};
#pragma unroll 1
        for (int mb = 0; mb < MB; ++mb) {
          f4 G[4];
#pragma unroll
          for (int s = 0; s < 4; ++s) G[s] = load4(at, s, mb);
          block(K + L.k_wt(k), jb, mb, G, acc);
        }
#pragma unroll
        for (int s = 0; s < 4; ++s) store4(k, s, jb, acc[s]);
      }
      at = k;
      settle();
    }

    // layer 1
    float dc = 0.f;
    const float c = T::slope(nd, K, L, 1);
    __syncthreads();   // the output layer's sums have been read
#pragma unroll 1
    for (int mb = 0; mb < MB; ++mb) {
      f4 A[4], G[4];
      pre(1, mb, x, y, A);
#pragma unroll
      for (int s = 0; s < 4; ++s) G[s] = load4(at, s, mb);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        adjoint(c, A[0][i], A[1][i], A[2][i], A[3][i], G, i, dc);
        const float r0 = row_sum16(fmaf(G[0][i], x, G[1][i])), r1 = row_sum16(fmaf(G[0][i], y, G[2][i])),
                    r2 = row_sum16(G[0][i]);
        if (pc == 0) {
          const int n = 16 * mb + 4 * g + i;
          sOut[(wave * 3 + 0) * WP + n] = r0;
          sOut[(wave * 3 + 1) * WP + n] = r1;
          sOut[(wave * 3 + 2) * WP + n] = r2;
        }
      }
    }
    if constexpr (GA) T::slope_wave_sum(dc, sSl, lane, wave);
    __syncthreads();
    if constexpr (GA) {
      if (nd.adaptive && tid == 0) slope_grad(R, sSl, 1, first);
    }
    if (tid < WP) {
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        float v = T::prior(R + 4 * tid + q, first);
        for (int w = 0; w < kWaves; ++w) v += sOut[(w * 3 + q) * WP + tid];
        R[4 * tid + q] = v;
      }
      if (first) R[4 * tid + 3] = 0.f;
    }
    __syncthreads();   // the sums have been read
  }
  static constexpr int NTGT = DO > NEQ ? DO : NEQ;
  __device__ void slope_grad(float* R, const float* sSl, int k, bool first) const {
    const float* v = sSl + (k - 1) * kWaves;
    T::accum(R + L.g_slope() + k - 1, (v[0] + v[1]) + (v[2] + v[3]), first);
  }

  // Whether the item's losses and first-layer gradients are finite: then it was
  // sent here for its tiny seeds.
  __device__ static bool finite_rows(const KArgs& ka, const Item& it, const NetDesc& nd, int* vote) {
    const int tid = (int)threadIdx.x;
    const bool pair = PDE == PDE_INV && nd.pair >= 0 && (it.kind == KIND_RES || it.kind == KIND_IFACE);
    const float* R = ka.partial + it.prow;
    float z = 0.f;
    for (int t = tid; t < 4 * nd.wclass; t += NT) z = fmaf(T::device_load(R + t), 0.f, z);
    if (pair)
      for (int t = tid; t < 4 * ka.nets[nd.pair].wclass; t += NT) z = fmaf(T::device_load(R + nd.gsize + t), 0.f, z);
    if (tid < kLossTerms) z = fmaf(T::device_load(ka.loss_part + (int64_t)it.lrow * kLossTerms + tid), 0.f, z);
    if (tid == 0) *vote = 0;
    __syncthreads();
    if (!(z == 0.f)) *vote = 1;
    __syncthreads();
    const int v = __builtin_amdgcn_readfirstlane(*vote);
    __syncthreads();
    return v == 0;
  }

  // dispatch of item idx (lds: the tile buffers; lds + nb_at: sNb and what
  // follows it as there).  Not inlined, and everything read again from the
  // kernel's arguments, for the registers of the path that matters: inlined a
  // step of 4 networks of 20 took 31.9 instead of 30.3 us, as a switch inside
  // Tile 32.6 (and 8 strips of 50 wide 275 instead of 216); so it takes 30.8
  // (and the strips 212).
  __device__ __attribute__((noinline, cold)) static void item(const Args* args, int index, Lds* lds, int nb_at,
                                                              float* slot) {
    const KArgs& ka = *(const KArgs*)args;
    const int idx = __builtin_amdgcn_readfirstlane(index);
    float* red = (float*)lds;
    float* sNb = (float*)(lds + nb_at);
    const Item& it = ka.items[idx];
    const NetDesc& nd = ka.nets[it.q];
    if (nan_network(ka, nd)) return;
    dma_landed();   // the rows are read, and written again, by other waves
    __syncthreads();
    if (small_term(it, nd) && finite_rows(ka, it, nd, reinterpret_cast<int*>(red))) return;
    float* sInv = sNb + 6 * TP;
    const IfaceDesc& ifd = ka.ifaces[it.kind == KIND_IFACE ? it.iface : 0];
    const NetDesc& nb = it.kind == KIND_IFACE ? ka.nets[it.side == 0 ? ifd.b_net : ifd.a_net] : nd;
#pragma unroll 1
    for (int t0 = 0; t0 < it.count; t0 += TP) {
      if constexpr (PDE == PDE_INV) {
        if (nd.pair >= 0 && (it.kind == KIND_RES || it.kind == KIND_IFACE)) {
          const NetDesc& ndk = ka.nets[nd.pair];
          const int64_t half = ka.scratch_slot / 2;
          if (it.kind == KIND_IFACE) {
            const NetDesc& nbk = ka.nets[nb.pair];
            Plain(ka, it, nbk, slot, t0).template values<VAL_STREAMS>(sInv + 6 * TP, nullptr);
            __syncthreads();
            Plain(ka, it, nb, slot, t0).template values<VAL_INV_NB>(sNb, sInv + 6 * TP);
          }
          const Plain k(ka, it, ndk, slot + half, t0);
          k.template train<EPI_SEED, PH_FWD>(red, sNb, sInv, nd.gsize);
          Plain(ka, it, nd, slot, t0).template train<EPI_INV_U, PH_ALL>(red, sNb, sInv, 0);
          k.template train<EPI_SEED, PH_BWD>(red, sNb, sInv, nd.gsize);
          continue;
        }
      } else if (it.kind == KIND_IFACE) {
        Plain(ka, it, nb, slot, t0).template values<VAL_OWN>(sNb, nullptr);
      }
      Plain(ka, it, nd, slot, t0).template train<EPI_OWN, PH_ALL>(red, sNb, sInv, 0);
    }
    __syncthreads();
  }
};

// LDS floats of a train kernel for classes up to WP: the tile buffers of
// Tile<WP> (weights and staging, sRed, sSl), then the neighbour values sNb (6
// per point), then for the inverse problem 9 per point: the own K streams,
// the K seeds, the neighbour's K streams.
template <int WP, int PDE>
constexpr int lds_tile_floats() {
  int n = 0;   // the largest need of the classes up to WP
  for (int w = 16; w <= WP; w += 16) n = tile_bytes(w, Op<PDE>::DO) > n ? tile_bytes(w, Op<PDE>::DO) : n;
  return n / 4 + kWaves * kLossTerms + kWaves;
}
template <int WP, int PDE>
constexpr int lds_train_floats() {
  return lds_tile_floats<WP, PDE>() + 6 * TP + (PDE == PDE_INV ? 9 * TP : 0) + Op<PDE>::DO * WP + 4;
}

// bytes of dynamic LDS the train kernel is launched with: the tile buffers and
// one 16-byte slot for the work-item broadcast
template <int WP, int PDE>
constexpr int lds_train_bytes() {
  return lds_train_floats<WP, PDE>() * 4 + 16;
}

// Run one item: for an interface item first evaluate the neighbour's network
// on the same tile (its width class may differ), then the item's own network.
// A paired item of the inverse problem goes tile by tile: the neighbour's K-
// and u-networks (interfaces), the own K-network's streams, the u-network's
// train pass (loss, u seeds, K seeds), then the K-network's train pass.
template <int WPMAX, int PDE, bool GA>
__device__ __forceinline__ void dispatch(const KArgs& ka, const Item& it, const NetDesc& nd, float* lds,
                                         float* slot, int* sBad) {
  float* sNb = lds + lds_tile_floats<WPMAX, PDE>();
  float* sInv = sNb + 6 * TP;
  float* sOW = sInv + (PDE == PDE_INV ? 9 * TP : 0);   // output-layer weights and biases of the network in training
#define DDP_CASE(WPV, ...)                                    \
  case WPV:                                                   \
    if constexpr (WPV <= WPMAX) Tile<WPV, PDE>::__VA_ARGS__;  \
    break;
#define DDP_SWITCH(CLS, ...)     \
  switch (CLS) {                 \
    DDP_CASE(16, __VA_ARGS__)    \
    DDP_CASE(32, __VA_ARGS__)    \
    DDP_CASE(48, __VA_ARGS__)    \
    DDP_CASE(64, __VA_ARGS__)    \
    DDP_CASE(80, __VA_ARGS__)    \
    DDP_CASE(96, __VA_ARGS__)    \
    DDP_CASE(112, __VA_ARGS__)   \
    default: break;              \
  }
  if constexpr (PDE == PDE_INV) {
    if (nd.pair >= 0 && (it.kind == KIND_RES || it.kind == KIND_IFACE)) {
      const NetDesc ndk = ka.nets[nd.pair];
      NetDesc nbu = nd, nbk = ndk;
      if (it.kind == KIND_IFACE) {
        const IfaceDesc ifd = ka.ifaces[it.iface];
        nbu = ka.nets[it.side == 0 ? ifd.b_net : ifd.a_net];
        nbk = ka.nets[nbu.pair];
      }
      // each network of the pair stashes into its own half of the slot: the
      // K-network's forward (its streams to LDS) comes first, its reverse pass
      // after the u-network's whole tile
      const int64_t half = ka.scratch_slot / 2;
      for (int t0 = 0; t0 < it.count; t0 += TP) {
        __syncthreads();
        if (it.kind == KIND_IFACE) {
          DDP_SWITCH(nbk.wclass,
                     template values_tile<VAL_STREAMS, GA>(ka, it, nbk, lds, sInv + 6 * TP, nullptr, t0))
          __syncthreads();
          DDP_SWITCH(nbu.wclass, template values_tile<VAL_INV_NB, GA>(ka, it, nbu, lds, sNb, sInv + 6 * TP, t0))
          __syncthreads();
        }
        DDP_SWITCH(ndk.wclass, template run_train<EPI_SEED, PH_FWD, GA>(ka, it, ndk, lds, slot + half, half,
                                                                            sNb, sInv, sOW, sBad, t0, t0 + 1, nd.gsize))
        DDP_SWITCH(nd.wclass,
                   template run_train<EPI_INV_U, PH_ALL, GA>(ka, it, nd, lds, slot, half, sNb, sInv, sOW, sBad, t0, t0 + 1,
                                                                 0))
        DDP_SWITCH(ndk.wclass, template run_train<EPI_SEED, PH_BWD, GA>(ka, it, ndk, lds, slot + half, half,
                                                                            sNb, sInv, sOW, sBad, t0, t0 + 1, nd.gsize))
      }
      return;
    }
  } else if (it.kind == KIND_IFACE) {
    const IfaceDesc ifd = ka.ifaces[it.iface];
    const NetDesc ndn = ka.nets[it.side == 0 ? ifd.b_net : ifd.a_net];
    __syncthreads();
    DDP_SWITCH(ndn.wclass, template values_tile<VAL_OWN, GA>(ka, it, ndn, lds, sNb, nullptr, 0))
    __syncthreads();
  }
  DDP_SWITCH(nd.wclass, template run_train<EPI_OWN, PH_ALL, GA>(ka, it, nd, lds, slot,
                                                       PDE == PDE_INV ? ka.scratch_slot / 2 : ka.scratch_slot, sNb,
                                                       sInv, sOW, sBad, 0, it.count, 0))
#undef DDP_SWITCH
#undef DDP_CASE
}

// What bounds it: for widths from 48 the matrix cores and the vector unit in
// turn (per hidden layer, wave and tile of class 64: 582 MFMAs of 16.8 cycles
// and 1960 vector instructions, a third of them splitting float32 into bf16
// parts; two waves share a SIMD and overlap only in part), for narrow networks
// the stash traffic (16 boxes of 20 wide: about 4 of the 5 TB/s a copy
// reaches) and latency, for a few tiles latency alone.  Train + reduce a step,
// with float32 MFMAs and everything stashed twice -> now: 16-subdomain mix of
// 143,157 points 720 -> 495 us, 9 subdomains of 60 wide 535 -> 363, 16 boxes of
// 20 184 -> 142, 4 of 20 38.5 -> 30.8.
//
// Persistent kernel: workgroup b starts with item b of the list (descending
// cost), then workgroups pull items from a device counter until it is drained;
// where every item has a workgroup the counter is not touched.  A first pull
// cost a round trip to memory (the counter is shared by all L2 caches) with
// nothing to hide it: 30.4 -> 29.2 us a step for 4 networks of 20 (one tile an
// item), 143 -> 142 for 16 of 20, 457 -> 453 for the 16-subdomain mix.
// Widths up to 80 fit two waves per SIMD (<= 256 registers); wider classes
// run one wave per SIMD.
template <int WPMAX>
constexpr int min_waves_per_eu() {
  return WPMAX <= 16 ? 4 : WPMAX <= 32 ? 3 : WPMAX <= 80 ? 2 : 1;
}

// GA: kernels with the general activation rule, launched for problems where a
// network uses another activation than tanh or trainable slopes (built for
// the class groups up to 80 and up to 112 only)
template <int WPMAX, int PDE, bool GA>
__global__ __launch_bounds__(NT, min_waves_per_eu<WPMAX>()) void k_train(KArgs ka) {
  // one 16-byte aligned dynamic LDS block: the tile buffers, then the slot
  // that broadcasts the next work item (no static LDS, so the float4
  // accesses of the tile buffers stay 16-byte aligned)
  extern __shared__ __attribute__((aligned(16))) float lds[];
  int& s_item = *reinterpret_cast<int*>(lds + lds_train_floats<WPMAX, PDE>());
  int& s_bad = *(&s_item + 1);   // the item has met values that Tile does not hold in full
  float* slot = ka.scratch + (int64_t)blockIdx.x * ka.scratch_slot;
  if (ka.prologue && blockIdx.x == 0 && threadIdx.x == 0) {
    // settle the Adam step counter of the previous update (k_reduce reads it)
    ka.tstate[0] += ka.tstate[1];
    ka.tstate[1] = 0;
  }
  for (int idx = blockIdx.x; idx < ka.n_items;) {
    const Item it = ka.items[idx];
    const NetDesc nd = ka.nets[it.q];
    if (threadIdx.x == 0) s_bad = 0;   // (set behind dispatch's first barrier)
    dispatch<WPMAX, PDE, GA>(ka, it, nd, lds, slot, &s_bad);
    __syncthreads();
    if (__builtin_expect(__builtin_amdgcn_readfirstlane(s_bad), 0)) {
      using P = Plain<PDE, GA>;
      P::item((const typename P::Args*)__builtin_amdgcn_kernarg_segment_ptr(), idx, (typename P::Lds*)lds,
              lds_tile_floats<WPMAX, PDE>(), slot);
    }
    if ((int)gridDim.x >= ka.n_items) break;
    if (threadIdx.x == 0) s_item = (int)gridDim.x + atomicAdd(ka.counter, 1);
    __syncthreads();
    idx = __builtin_amdgcn_readfirstlane(s_item);
  }
}

// A canonical parameter in its network's kernel-layout copy: a float at k1, or,
// for a hidden weight (k1 = -1), the three bf16 parts at bf16 positions w,
// w + ws, w + 2 ws of the weights and t, t + ts, t + 2 ts of the transposed
// copy.  sc: the kernel copy holds sc times the parameter and the partial rows
// hold the gradient divided by sc (n for a slope a^k, whose kernel copy is
// c_k = n a^k; 1 otherwise).
struct ParamPos {
  int k1, w, ws, t, ts;
  float sc;
};
__device__ __forceinline__ ParamPos float_pos(int k1, float sc = 1.f) { return ParamPos{k1, 0, 0, 0, 0, sc}; }
__device__ __forceinline__ ParamPos weight_pos(const Layout& L, int k, int m, int j) {
  ParamPos p{-1, 0, 0, 0, 0, 1.f};
  p.w = 2 * L.k_w(k) + split_pos(L.WP, m, j, p.ws);
  p.t = 2 * L.k_wt(k) + split_pos(L.WP, j, m, p.ts);
  return p;
}

// position of canonical parameter li
__device__ __forceinline__ ParamPos param_map(const NetDesc& nd, int li) {
  const int w = nd.width, D = nd.depth, DO = nd.d_out;
  const Layout L(nd.wclass, D, DO);
  if (li < 2 * w) return float_pos((li >> 1) * 4 + (li & 1));   // W^1[m][c]
  if (li < 3 * w) return float_pos((li - 2 * w) * 4 + 2);       // b^1[m]
  int r = li - 3 * w;
  const int per = w * w + w;
  const int h = r / per;
  if (h < D - 1) {                  // hidden layer k = h + 2
    const int rr = r - h * per;
    if (rr < w * w) return weight_pos(L, h + 2, rr / w, rr - (rr / w) * w);
    return float_pos(L.k_b(h + 2) + rr - w * w);
  }
  r -= (D - 1) * per;               // output layer, then the slopes a^k
  if (r < DO * w) return float_pos(L.k_out() + (r / w) * nd.wclass + r - (r / w) * w);
  if (r < DO * w + DO) return float_pos(L.k_bout() + r - DO * w);
  return float_pos(L.k_slope() + r - DO * w - DO, nd.slope_n);
}

// the canonical parameter of entry gi of a gradient partial row and its
// position, or -1 for padding
__device__ __forceinline__ int grad_map(const NetDesc& nd, int gi, ParamPos& p) {
  const int w = nd.width, WP = nd.wclass, D = nd.depth, DO = nd.d_out;
  const Layout L(WP, D, DO);
  if (gi < 4 * WP) {
    const int m = gi >> 2, c = gi & 3;
    p = float_pos(gi);
    return m >= w || c == 3 ? -1 : c == 2 ? 2 * w + m : 2 * m + c;
  }
  int r = gi - 4 * WP, base = 3 * w;
  const int per = WP * WP + WP;
  const int h = r / per;
  if (h < D - 1) {
    const int rr = r - h * per;
    base += h * (w * w + w);
    if (rr < WP * WP) {
      const int m = rr / WP, j = rr - (rr / WP) * WP;
      p = weight_pos(L, h + 2, m, j);
      return m >= w || j >= w ? -1 : base + m * w + j;
    }
    p = float_pos(L.k_b(h + 2) + rr - WP * WP);
    return rr - WP * WP >= w ? -1 : base + w * w + rr - WP * WP;
  }
  r -= (D - 1) * per;
  base += (D - 1) * (w * w + w);
  if (r < DO * WP) {
    const int c = r / WP, j = r - (r / WP) * WP;
    p = float_pos(L.k_out() + r);
    return j >= w ? -1 : base + c * w + j;
  }
  r -= DO * WP;
  if (r < 4) {
    p = float_pos(L.k_bout() + r);
    return r >= DO ? -1 : base + DO * w + r;
  }
  r -= 4;
  p = float_pos(L.k_slope() + r, nd.slope_n);
  return nd.adaptive && r < D ? base + DO * w + DO + r : -1;
}

// The split of one value over the whole range of float32: an infinite one is
// its first part alone, and one that rounds to infinity (from 3.3961e38) has the
// largest finite bf16 there, so the parts always add up to the value (down to
// the last bit of the smallest bf16, 2^-133).
__device__ __forceinline__ void split_any(float x, __bf16& h, __bf16& m, __bf16& l) {
  const float top = __uint_as_float(0x7f7f0000u);   // largest finite bf16
  const float hf = isinf(x) ? x : fminf(fmaxf(x, -top), top);
  h = (__bf16)(isnan(x) ? x : hf);
  const float r = isinf(x) ? 0.f : x - (float)h;
  m = (__bf16)r;
  l = (__bf16)(r - (float)m);
}

// write the kernel-layout copy of a parameter with value v
__device__ __forceinline__ void put_param(float* K, const ParamPos& p, float v) {
  if (p.k1 >= 0) {
    K[p.k1] = p.sc * v;
    return;
  }
  __bf16 h, m, l;
  split_any(v, h, m, l);
  __bf16* W = reinterpret_cast<__bf16*>(K) + p.w;
  __bf16* T = reinterpret_cast<__bf16*>(K) + p.t;
  W[0] = T[0] = m;
  W[p.ws] = T[p.ts] = h;
  W[2 * p.ws] = T[2 * p.ts] = l;
}

// network holding flat parameter i, searching upward from network n
__device__ __forceinline__ int find_net(const int64_t* net_poff, int n, int64_t i) {
  while (net_poff[n + 1] <= i) ++n;
  return n;
}

// The train kernels of each operator are compiled in a translation unit of
// their own (DDP_TRAIN_PDE set to the operator), so the build runs them in
// parallel; the unit without it holds the other kernels and the launchers.
#ifndef DDP_TRAIN_PDE

// Sum each network's gradient partial rows in a fixed order, then write the
// gradient and/or apply Adam (Kingma-Ba, bias corrected) and refresh the
// kernel-layout copy; the blocks behind those sum each subdomain's loss rows
// and flag non-finite losses.
//
// Bound by the latency of its chain (block description, network, row offsets,
// rows, Adam), not by bytes: the rows are a few MB and in cache.  A block owns kRedParams consecutive entries of one network's partial rows:
// wave w sums rows w, w + 4, ... four entries a lane and kRedRows rows at a
// time, then thread t takes entry t's four sums from LDS in order and updates
// its parameter.  The order does not depend on timing.  Against a thread per
// parameter that walks its rows one at a time, the offset of each found from
// the parameter's, and the loss sums in block 0 (us): 16 space-time boxes of 20
// 17.4 -> 10.6, 8 strips of 50 18.0 -> 13.5, 9 subdomains of 60 20.2 -> 12.7, the
// 16-subdomain Poisson mix 20.5 -> 15.9, 10 adaptive pairs of 80 30 -> 22, 10
// inverse pairs 28.7 -> 27.8 (99 with the autotuned plan, whose items are
// shorter), 4 of 20 6.7 -> 5.8.
constexpr int kRedRows = 8;

__global__ __launch_bounds__(kRedParams) void k_reduce(RArgs ra) {
  __shared__ f4 s_sum[kRedParams / 64][kRedParams / 4];
  const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  // the block's description and network are uniform across the block (scalar
  // loads); everything that waits for them is issued together
  const int bidx = (int)blockIdx.x, last = ra.n_blocks;
  if (bidx < last) {
    const RedBlock rb = ra.blocks[bidx];
    const NetDesc nd = ra.nets[rb.net];
    const int g0 = rb.begin;
    ParamPos pp = float_pos(0);
    const int gi = g0 + (int)threadIdx.x;
    const int li = gi < nd.gsize ? grad_map(nd, gi, pp) : -1;
    const int64_t i = nd.poff + li;
    // the optimiser's state is on its way while the rows are summed
    float m0 = 0.f, v0 = 0.f, th0 = 0.f;
    const float tstep = ra.do_adam ? (float)(ra.tstate[0] + 1) : 1.f;
    if (ra.do_adam && li >= 0) {
      m0 = ra.adam_m[i];
      v0 = ra.adam_v[i];
      th0 = ra.params[i];
    }
    const int n = rb.n;
    const int64_t* pr = ra.row_prow + rb.r0;
    const float* P = ra.partial + g0 + 4 * lane;
    f4 a[kRedRows];
#pragma unroll
    for (int j = 0; j < kRedRows; ++j) a[j] = f4{0.f, 0.f, 0.f, 0.f};
    if (g0 + 4 * lane < nd.gsize) {
      int r = wave;
      for (; r + 4 * (kRedRows - 1) < n; r += 4 * kRedRows) {
#pragma unroll
        for (int j = 0; j < kRedRows; ++j) a[j] += *reinterpret_cast<const f4*>(P + pr[r + 4 * j]);
      }
#pragma unroll
      for (int j = 0; j < kRedRows; ++j)
        if (r + 4 * j < n) a[j] += *reinterpret_cast<const f4*>(P + pr[r + 4 * j]);
    }
#pragma unroll
    for (int w = kRedRows / 2; w >= 1; w /= 2)
#pragma unroll
      for (int j = 0; j < w; ++j) a[j] += a[j + w];
    s_sum[wave][lane] = a[0];
    __syncthreads();
    if (li >= 0) {
      const float* S = reinterpret_cast<const float*>(s_sum) + threadIdx.x;
      const float s = pp.sc * ((S[0] + S[kRedParams]) + (S[2 * kRedParams] + S[3 * kRedParams]));
      if (ra.grad_out) ra.grad_out[i] = s;
      if (ra.do_adam) {
        const float bc1 = 1.f - powf(b1, tstep);
        const float bc2 = 1.f - powf(b2, tstep);
        const float m = b1 * m0 + (1.f - b1) * s;
        const float v = b2 * v0 + (1.f - b2) * s * s;
        ra.adam_m[i] = m;
        ra.adam_v[i] = v;
        const float mh = m / bc1;
        const float vh = v / bc2;
        const float th = th0 - nd.lr * mh / (sqrtf(vh) + eps);
        ra.params[i] = th;
        put_param(ra.kparams + nd.koff, pp, th);
      }
    }
  }
  // the blocks behind those: one wave per subdomain sums its loss rows (lane l
  // sums rows l, l + 64, ...; then a fixed butterfly across the wave).  As a
  // loop of the first block these sums outlasted the launch: 16 subdomains
  // took 16 of its 17 us.
  const int q = bidx >= last ? ra.sd_begin + (bidx - last) * (kRedParams / 64) + wave : ra.sd_end;
  if (q < ra.sd_end) {
    const NetDesc nd = ra.nets[ra.sd_net[q]];
    f4 t = {0.f, 0.f, 0.f, 0.f};
    for (int r = ra.sd_loss_ptr[q] + lane; r < ra.sd_loss_ptr[q + 1]; r += 64)
      t += *reinterpret_cast<const f4*>(ra.loss_part + (int64_t)ra.loss_rows[r] * kLossTerms);
    for (int m = 32; m >= 1; m >>= 1)
#pragma unroll
      for (int k = 0; k < kLossTerms; ++k) t[k] += __shfl_xor(t[k], m);
    if (lane == 0) {
      float J = 0.f;
#pragma unroll
      for (int k = 0; k < kLossTerms; ++k) J += nd.loss_w[k] * t[k];
      if (ra.loss_out) {
        ra.loss_out[q * 5] = J;
#pragma unroll
        for (int k = 0; k < kLossTerms; ++k) ra.loss_out[q * 5 + 1 + k] = t[k];
      }
      if (!isfinite(J)) ra.flags[0] = 1;
    }
  }
  if (blockIdx.x == 0) {
    if (ra.do_adam && threadIdx.x == 0) ra.tstate[1] = 1;
    // the train kernel of this step has finished: re-arm its work counter
    if (ra.counter_reset && (int)threadIdx.x < ra.n_counter_reset) ra.counter_reset[threadIdx.x] = 0;
  }
}

__global__ void k_reset_counter(int* c) { *c = 0; }

// Two streams meet: k_await polls w[0] for at most kAwaitPolls loads and
// leaves in w[1] what it saw; k_arrive sets w[0].  With k_arrive launched
// behind k_await on another stream, k_await sees it only if the two kernels
// can run at the same time; both end either way.
constexpr int kAwaitPolls = 512;   // about 0.3 ms

__global__ void k_await(int* w) {
  int seen = 0;
  for (int i = 0; i < kAwaitPolls && !seen; ++i)
    seen = __hip_atomic_load(w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  w[1] = seen;
}

__global__ void k_arrive(int* w) { __hip_atomic_store(w, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// Take the canonical parameters of networks [n_begin, n_end) from src (the
// caller's, or params itself) and write their kernel-layout copy: one launch
// per subdomain where a copy and a launch were two.
__global__ __launch_bounds__(256) void k_pack(const float* src, float* params, float* kparams, const NetDesc* nets,
                                              const int64_t* net_poff, int n_begin, int n_end) {
  const int64_t p0 = net_poff[n_begin], p1 = net_poff[n_end];
  for (int64_t i = p0 + (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < p1;
       i += (int64_t)gridDim.x * blockDim.x) {
    const int q = find_net(net_poff, n_begin, i);
    const NetDesc nd = nets[q];
    const float v = src[i - p0];
    params[i] = v;
    put_param(kparams + nd.koff, param_map(nd, (int)(i - net_poff[q])), v);
  }
}

// Stitched solution (Eq. FSol): average of the owning subdomains' outputs;
// the columns are the outputs of a subdomain's networks in order (u, or u
// then K for the inverse problem).
//
// A block takes pb consecutive points and sorts their (point, owner slot)
// pairs by subdomain in LDS; its waves then evaluate one network at 16, 32 or
// 64 of the pairs at once, the points being the columns of the contractions
// of Tile::contract, with the weights read in fragment order from the L2 cache.
// Each pair's outputs go to LDS and are summed in the order of the slots.
// (One thread a point, with the activations in scratch memory, took 3.6 ms for
// 40,401 points of 16 networks up to 80 wide and 11.1 ms for 10^6 points of 5 x
// 60, the copies to the device included; now 0.10 and 1.20 ms, mostly copies.)
constexpr int kEvalPts = 256;            // points per block at most

// Activations of the evaluation: sin and cos as in training (sin_cos), tanh
// without a branch: 1 - 2 / (exp(2|y|) + 1), and below 0.7, where that would
// cancel, y + y^3 P(y^2) with P fitted to (tanh(y)/y - 1)/y^2 (tanh to 2.0e-8 in
// exact arithmetic).  Largest relative error over every float from 2^-30 to
// 30: 8.8e-8 below 0.7, 1.58e-7 above (tanh_s1: 8.8e-8 and 2.04e-7).
__device__ __forceinline__ float tanh_value(float y) {
  const float a = fabsf(y), u = a * a;
  float p = -0.0051385928f;
  p = fmaf(p, u, 0.020091895f);
  p = fmaf(p, u, -0.053558834f);
  p = fmaf(p, u, 0.13329111f);
  p = fmaf(p, u, -0.33333191f);
  const float s = fmaf(a * u, p, a);
  const float r = __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(2.88539008f * a));
  return copysignf(a < 0.7f ? s : fmaf(-2.f, r, 1.f), y);
}

__device__ __forceinline__ float sin_cos_value(int act, float y) {
  float sn, cs;
  sin_cos(y, sn, cs);
  return act == ACT_SIN ? sn : cs;
}

// one network at up to 16 NG points: xs, ys the lane's points (16 i + pc of
// each of the NG groups), val(i, c, u) takes output c of group i's point.
// EXACT: contractions in float32, the padding's activations 0 whatever the
// point and the slope
template <int WP, int NG, bool EXACT, class F>
__device__ __forceinline__ void eval_net(const float* K, const NetDesc& nd, int lane, const float (&xs)[4],
                                         const float (&ys)[4], F val) {
  using T = Tile<WP, PDE_POISSON>;
  constexpr int MB = T::MB;
  const int g = lane >> 4;
  const Layout L(WP, nd.depth, nd.d_out);
  typename T::Streams H, A;
  for (int k = 1; k <= nd.depth; ++k) {
    const float c = nd.adaptive ? K[L.k_slope() + k - 1] : 1.f;
    if (k == 1) {
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const f4 w = *reinterpret_cast<const f4*>(K + (16 * mb + 4 * g + i) * 4);
#pragma unroll
          for (int j = 0; j < NG; ++j) A[j][mb][i] = fmaf(w[0], xs[j], fmaf(w[1], ys[j], w[2]));
        }
    } else {
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) {
        const f4 b = *reinterpret_cast<const f4*>(K + L.k_b(k) + 16 * mb + 4 * g);
#pragma unroll
        for (int j = 0; j < NG; ++j) A[j][mb] = b;
      }
      const char* w = reinterpret_cast<const char*>(K + L.k_w(k));
      if constexpr (EXACT) T::template contract_f32<0, NG>(w, lane, H, A);
      else T::template contract<0, NG>(w, lane, H, A);
    }
    if (nd.act == ACT_TANH) {
#pragma unroll
      for (int j = 0; j < NG; ++j)
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
          for (int i = 0; i < 4; ++i) H[j][mb][i] = tanh_value(c * A[j][mb][i]);
    } else {
#pragma unroll
      for (int j = 0; j < NG; ++j)
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
          for (int i = 0; i < 4; ++i) H[j][mb][i] = sin_cos_value(nd.act, c * A[j][mb][i]);
    }
    if constexpr (EXACT) {
#pragma unroll
      for (int j = 0; j < NG; ++j)
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
          for (int i = 0; i < 4; ++i) H[j][mb][i] = 16 * mb + 4 * g + i < nd.width ? H[j][mb][i] : 0.f;
    }
  }
  for (int o = 0; o < nd.d_out; ++o) {
    float acc[NG] = {};
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      const f4 w = *reinterpret_cast<const f4*>(K + L.k_out() + o * WP + 16 * mb + 4 * g);
#pragma unroll
      for (int j = 0; j < NG; ++j)
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[j] = fmaf(w[i], H[j][mb][i], acc[j]);
    }
#pragma unroll
    for (int j = 0; j < NG; ++j) val(j, o, group_sum(acc[j]) + K[L.k_bout() + o]);
  }
}

// two waves per SIMD: 64 points of up to 80 neurons fit the registers, 32 of
// the wider classes
// (activations: the library's tanhf, a branch for each, took 43 us of kernel
// for the 40,401 points and 446 for the 10^6; tanh_value 39 and 414)
__global__ __launch_bounds__(NT, 2) void k_eval(const float* kparams, const NetDesc* nets, const int* sd_net, int n_sd,
                                                int n, int pb, const float* xy, const int* owner, float* out,
                                                int n_cols) {
  __shared__ float s_xy[2 * kEvalPts];
  __shared__ int s_owner[4 * kEvalPts];            // per pair: subdomain, or -1
  __shared__ int s_order[4 * kEvalPts];            // pairs by subdomain
  __shared__ int s_seg[4 * kEvalPts][2];           // per subdomain met: its number, first pair
  __shared__ float s_val[4 * kEvalPts][kMaxOut];
  __shared__ int s_min[kWaves], s_cnt[kWaves];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int p0 = blockIdx.x * pb, np = min(pb, n - p0);
  for (int i = tid; i < 4 * np; i += NT) {
    const int q = owner[4 * (int64_t)p0 + i];
    s_owner[i] = q >= 0 && q < n_sd ? q : -1;
    if (i < 2 * np) s_xy[i] = xy[2 * (int64_t)p0 + i];
  }
  __syncthreads();
  // pairs by subdomain: the next number up, then its pairs in order
  int n_seg = 0, filled = 0;
  for (int last = -1;;) {
    int q = INT_MAX;
    for (int i = tid; i < 4 * np; i += NT)
      if (s_owner[i] > last) q = min(q, s_owner[i]);
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) q = min(q, __shfl_xor(q, m));
    if (lane == 0) s_min[wave] = q;
    __syncthreads();
    q = min(min(s_min[0], s_min[1]), min(s_min[2], s_min[3]));
    if (q == INT_MAX) break;
    if (tid == 0) {
      s_seg[n_seg][0] = q;
      s_seg[n_seg][1] = filled;
    }
    ++n_seg;
    last = q;
    for (int i0 = 0; i0 < 4 * np; i0 += NT) {
      const bool mine = i0 + tid < 4 * np && s_owner[i0 + tid] == q;
      const unsigned long long b = __ballot(mine);
      if (lane == 0) s_cnt[wave] = __popcll(b);
      __syncthreads();
      int at = filled + __popcll(b & ((1ull << lane) - 1));
      for (int w = 0; w < kWaves; ++w) {
        at += w < wave ? s_cnt[w] : 0;
        filled += s_cnt[w];
      }
      if (mine) s_order[at] = i0 + tid;
      __syncthreads();
    }
  }
  __syncthreads();
  // work units of up to 64 pairs of one subdomain, dealt out to the waves
  struct Seg {
    int q, b, e, step;
  };
  auto segment = [&](int sg) {
    Seg s;
    s.q = __builtin_amdgcn_readfirstlane(s_seg[sg][0]);
    s.b = __builtin_amdgcn_readfirstlane(s_seg[sg][1]);
    s.e = sg + 1 < n_seg ? __builtin_amdgcn_readfirstlane(s_seg[sg + 1][1]) : filled;
    const int groups = min(4, (s.e - s.b + 63) / 64);   // 16-point groups a unit: every wave gets a share first
    s.step = 16 * (groups == 3 ? 4 : groups);
    return s;
  };
  bool again = false;   // an output of this wave was not finite
  int unit = 0;
  for (int sg = 0; sg < n_seg; ++sg) {
    const auto [q, b, e, step] = segment(sg);
    for (int u0 = b; u0 < e; u0 += step, ++unit) {
      if ((unit & (kWaves - 1)) != wave) continue;
      const int end = min(e, u0 + step);
      int col = 0;
      for (int net = sd_net[q]; net < sd_net[q + 1]; ++net) {
        const NetDesc nd = nets[net];
        const float* K = kparams + nd.koff;
        const int most = nd.wclass > 80 ? 32 : 64;  // points at once
        for (int u1 = u0; u1 < end; u1 += most) {
          const int left = min(end - u1, most);
          float xs[4], ys[4];
          int pr[4];
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const int k = 16 * j + (lane & 15);
            pr[j] = s_order[u1 + min(k, left - 1)];
            xs[j] = s_xy[2 * (pr[j] >> 2)];
            ys[j] = s_xy[2 * (pr[j] >> 2) + 1];
          }
          bool finite = true;
          auto val = [&](int j, int o, float v) {
            finite = finite && fabsf(v) < INFINITY;
            if (lane < 16 && 16 * j + lane < left && col + o < n_cols) s_val[pr[j]][col + o] = v;
          };
#define DDP_EVAL(WPV, NGV) eval_net<WPV, NGV, false>(K, nd, lane, xs, ys, val)
#define DDP_EVAL_CASE(WPV, BIG)                \
  case WPV:                                    \
    if (left <= 16) DDP_EVAL(WPV, 1);          \
    else if (left <= 32) DDP_EVAL(WPV, 2);     \
    else DDP_EVAL(WPV, BIG);                   \
    break;
          switch (nd.wclass) {
            DDP_EVAL_CASE(16, 4)
            DDP_EVAL_CASE(32, 4)
            DDP_EVAL_CASE(48, 4)
            DDP_EVAL_CASE(64, 4)
            DDP_EVAL_CASE(80, 4)
            DDP_EVAL_CASE(96, 2)
            DDP_EVAL_CASE(112, 2)
            default: break;
          }
#undef DDP_EVAL_CASE
#undef DDP_EVAL
          again = again || __any(!finite);
        }
        col += nd.d_out;
      }
    }
  }
  // An infinite weight or point saturates its neurons, but is no sum of bf16
  // parts, and at an infinite point the padding's 0 times infinity reaches
  // every neuron: the wave's outputs that are not finite, and only they, are
  // computed again in float32, 16 points at a time.
  if (again) {
    wave_fence();
    unit = 0;
    for (int sg = 0; sg < n_seg; ++sg) {
      const auto [q, b, e, step] = segment(sg);
      for (int u0 = b; u0 < e; u0 += step, ++unit) {
        if ((unit & (kWaves - 1)) != wave) continue;
        for (int u1 = u0; u1 < min(e, u0 + step); u1 += 16) {
          const int k = u1 + (lane & 15), last = min(e, u0 + step) - 1;
          const int pr = s_order[min(k, last)];
          const float xs[4] = {s_xy[2 * (pr >> 2)]}, ys[4] = {s_xy[2 * (pr >> 2) + 1]};
          int col = 0;
          for (int net = sd_net[q]; net < sd_net[q + 1]; ++net) {
            const NetDesc nd = nets[net];
            const float* K = kparams + nd.koff;
            auto val = [&](int, int o, float v) {
              if (lane >= 16 || k > last || col + o >= n_cols) return;
              float& had = s_val[pr][col + o];
              if (!(fabsf(had) < INFINITY)) had = v;
            };
#define DDP_EVAL_CASE(WPV)                            \
  case WPV:                                           \
    eval_net<WPV, 1, true>(K, nd, lane, xs, ys, val); \
    break;
            switch (nd.wclass) {
              DDP_EVAL_CASE(16)
              DDP_EVAL_CASE(32)
              DDP_EVAL_CASE(48)
              DDP_EVAL_CASE(64)
              DDP_EVAL_CASE(80)
              DDP_EVAL_CASE(96)
              DDP_EVAL_CASE(112)
              default: break;
            }
#undef DDP_EVAL_CASE
            col += nd.d_out;
          }
        }
      }
    }
  }
  __syncthreads();
  for (int i = tid; i < np; i += NT) {
    float acc[kMaxOut] = {0.f, 0.f, 0.f};
    int cnt = 0;
    for (int o = 0; o < 4; ++o) {
      if (s_owner[4 * i + o] < 0) continue;
      ++cnt;
      for (int c = 0; c < n_cols; ++c) acc[c] += s_val[4 * i + o][c];
    }
    for (int c = 0; c < n_cols; ++c) out[(int64_t)(p0 + i) * n_cols + c] = cnt ? acc[c] / cnt : 0.f;
  }
}

#endif  // DDP_TRAIN_PDE

// ---------------------------------------------------------------------------
// host-side launchers

// One train kernel (operator, class group, activation rule) and the LDS bytes
// it is launched with.  A unit built with DDP_TRAIN_PDE defines the kernels
// of that operator for the class DDP_TRAIN_WP (0: those up to 64), with
// DDP_TRAIN_GA the general-activation one.
template <int PDE, int WPMAX, bool GA>
struct Kernel {
  static const void* fn;
  static int lds;
};
#ifdef DDP_TRAIN_PDE
#ifdef DDP_TRAIN_GA
#define DDP_GA true
#else
#define DDP_GA false
#endif
#define DDP_KERNEL(WPV)                                                                                            \
  template <> const void* Kernel<DDP_TRAIN_PDE, WPV, DDP_GA>::fn = (const void*)k_train<WPV, DDP_TRAIN_PDE, DDP_GA>; \
  template <> int Kernel<DDP_TRAIN_PDE, WPV, DDP_GA>::lds = lds_train_bytes<WPV, DDP_TRAIN_PDE>();
#if DDP_TRAIN_WP == 0
DDP_KERNEL(16)
DDP_KERNEL(32)
DDP_KERNEL(48)
DDP_KERNEL(64)
#else
DDP_KERNEL(DDP_TRAIN_WP)
#endif
#undef DDP_KERNEL
#undef DDP_GA
#else
// the kernels are defined in units of their own
#define DDP_DECL1(PDE, WPV, GA)                     \
  template <> const void* Kernel<PDE, WPV, GA>::fn; \
  template <> int Kernel<PDE, WPV, GA>::lds;
#define DDP_DECL(PDE)                                                                                     \
  DDP_DECL1(PDE, 16, false) DDP_DECL1(PDE, 32, false) DDP_DECL1(PDE, 48, false) DDP_DECL1(PDE, 64, false) \
  DDP_DECL1(PDE, 80, false) DDP_DECL1(PDE, 96, false) DDP_DECL1(PDE, 112, false)                          \
  DDP_DECL1(PDE, 80, true) DDP_DECL1(PDE, 112, true)
DDP_DECL(PDE_POISSON)
DDP_DECL(PDE_BURGERS)
DDP_DECL(PDE_NS)
DDP_DECL(PDE_INV)
#undef DDP_DECL
#undef DDP_DECL1

// the kernel of a class (general-activation kernels exist for the groups up
// to 80 and up to 112) and its LDS bytes
template <class K>
static const void* pick_kernel(int* lds) {
  *lds = K::lds;
  return K::fn;
}
template <int PDE>
static const void* pick_pde(int wpmax, bool ga, int* lds) {
  if (ga) {
    if (wpmax == 80) return pick_kernel<Kernel<PDE, 80, true>>(lds);
    if (wpmax == 112) return pick_kernel<Kernel<PDE, 112, true>>(lds);
    return nullptr;
  }
  switch (wpmax) {
    case 16: return pick_kernel<Kernel<PDE, 16, false>>(lds);
    case 32: return pick_kernel<Kernel<PDE, 32, false>>(lds);
    case 48: return pick_kernel<Kernel<PDE, 48, false>>(lds);
    case 64: return pick_kernel<Kernel<PDE, 64, false>>(lds);
    case 80: return pick_kernel<Kernel<PDE, 80, false>>(lds);
    case 96: return pick_kernel<Kernel<PDE, 96, false>>(lds);
    case 112: return pick_kernel<Kernel<PDE, 112, false>>(lds);
  }
  return nullptr;
}

static const void* pick(int pde, int wpmax, bool ga, int* lds) {
  switch (pde) {
    case PDE_POISSON: return pick_pde<PDE_POISSON>(wpmax, ga, lds);
    case PDE_BURGERS: return pick_pde<PDE_BURGERS>(wpmax, ga, lds);
    case PDE_NS: return pick_pde<PDE_NS>(wpmax, ga, lds);
    case PDE_INV: return pick_pde<PDE_INV>(wpmax, ga, lds);
  }
  return nullptr;
}

int64_t scratch_slot_floats(int pde, int wpmax, bool ga) {
  // four streams of up to kMaxDepth layers (the general-activation kernels
  // keep four more of an 80-wide network); the inverse problem keeps one such
  // stash per network of a pair
  const int64_t one = (int64_t)(ga ? 2 : 1) * kMaxDepth * kWaves * 4 * (wpmax / 16) * 64 * 4;
  return pde == PDE_INV ? 2 * one : one;
}

int kernel_wpmax(int wpmax, bool ga) { return ga ? (wpmax <= 80 ? 80 : 112) : wpmax; }

hipError_t launch_train(int pde, int wpmax, bool ga, const KArgs& ka, int grid, hipStream_t st) {
  int lds = 0;
  const void* fn = pick(pde, wpmax, ga, &lds);
  if (!fn) return hipErrorInvalidValue;
  KArgs a = ka;
  void* args[] = {&a};
  return hipLaunchKernel(fn, dim3(grid), dim3(NT), args, (size_t)lds, st);
}

hipError_t train_occupancy(int pde, int wpmax, bool ga, int* blocks_per_cu) {
  int lds = 0;
  const void* fn = pick(pde, wpmax, ga, &lds);
  if (!fn) return hipErrorInvalidValue;
  hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  if (e != hipSuccess) return e;
  return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, fn, NT, (size_t)lds);
}

hipError_t launch_reset_counter(int* c, hipStream_t st) {
  hipLaunchKernelGGL(k_reset_counter, dim3(1), dim3(1), 0, st, c);
  return hipGetLastError();
}

hipError_t launch_await(int* w, hipStream_t st) {
  hipLaunchKernelGGL(k_await, dim3(1), dim3(1), 0, st, w);
  return hipGetLastError();
}

hipError_t launch_arrive(int* w, hipStream_t st) {
  hipLaunchKernelGGL(k_arrive, dim3(1), dim3(1), 0, st, w);
  return hipGetLastError();
}

hipError_t launch_reduce(const RArgs& ra, int grid, hipStream_t st) {
  hipLaunchKernelGGL(k_reduce, dim3(grid), dim3(kRedParams), 0, st, ra);
  return hipGetLastError();
}

hipError_t launch_pack(const float* src, float* params, float* kparams, const NetDesc* nets, const int64_t* net_poff,
                       int n_begin, int n_end, int64_t n, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  const int grid = (int)std::min<int64_t>((n + 255) / 256, 4096);
  hipLaunchKernelGGL(k_pack, dim3(grid), dim3(256), 0, st, src, params, kparams, nets, net_poff, n_begin, n_end);
  return hipGetLastError();
}

hipError_t launch_eval(const float* kparams, const NetDesc* nets, const int* sd_net, int n_sd, int n, const float* xy,
                       const int* owner, float* out, int n_cols, int n_cu, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  // points per block: two blocks a compute unit before a block gets more than
  // 16, and at most what its LDS holds
  const int64_t share = ((int64_t)n + 2 * n_cu - 1) / (2 * n_cu);
  const int pb = (int)std::min<int64_t>(kEvalPts, (share + 15) / 16 * 16);
  hipLaunchKernelGGL(k_eval, dim3((n + pb - 1) / pb), dim3(NT), 0, st, kparams, nets, sd_net, n_sd, n, pb, xy, owner,
                     out, n_cols);
  return hipGetLastError();
}

#endif  // DDP_TRAIN_PDE
}  // namespace ddp
