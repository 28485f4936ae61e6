// m1_device.h -- device-side building blocks of the M1 step for gfx950:
// Levermore closure with the Sect. 2.6 signal speeds and the physical flux
// of one state, the HLL interface flux with the optical-depth limiter, the
// van Leer and LimO3 slopes and the face treatments (Eq. f_reconstruct and
// its alternatives).
// Templated on the working precision R (double or float).
#pragma once
#include <hip/hip_runtime.h>

#include "../../include/m1.h"

namespace m1 {

// Arithmetic primitives per precision.  FP64 refines the hardware estimates
// (good to 2^-24.4 for the reciprocal and 2^-23.2 for the reciprocal square
// root, measured) by one step of third order, which leaves 2^-70 and 2^-68 of
// relative error before rounding in one operation less (reciprocal) and three
// less (square roots) than two Newton steps, with a shorter chain:
//  * reciprocal: e = 1 - x r, r <- r (1 + e + e^2);
//  * reciprocal square root: e = 1 - x y^2, y <- y (1 + e / 2 + 3 e^2 / 8);
//  * square root: g = x y, h = y / 2, e = 1/2 - h g, g <- g (1 + e + 3 e^2 / 2),
//    and in sqrt_ one correction g <- g + (x - g^2) h and a select for zero.
// Arguments are positive normal numbers, or zero for sqrt_ (the callers pass
// no subnormal or infinite arguments).  All stay within an ulp or two, far
// inside the 1e-12 parity tolerance.  FP32: the hardware reciprocal, square
// root and reciprocal square root (about 1 ulp), inside 1e-5.
template <typename R> struct Num;
template <> struct Num<double> {
    static constexpr double tiny = __DBL_MIN__;      // smallest normal number
    static __device__ __forceinline__ double sqrt_(double x)
    {
        const double y = __builtin_amdgcn_rsq(x), h = 0.5 * y;
        double g = x * y;
        const double e = __builtin_fma(-h, g, 0.5);
        g = __builtin_fma(g, __builtin_fma(1.5 * e, e, e), g);
        g = __builtin_fma(__builtin_fma(-g, g, x), h, g);
        return x > 0.0 ? g : 0.0;
    }
    // x at least the smallest normal number
    static __device__ __forceinline__ double sqrt_pos(double x)
    {
        const double y = __builtin_amdgcn_rsq(x), h = 0.5 * y, g = x * y;
        const double e = __builtin_fma(-h, g, 0.5);
        return __builtin_fma(g, __builtin_fma(1.5 * e, e, e), g);
    }
    // the square root as above and the reciprocal square root, 1 <= x <= 4
    static __device__ __forceinline__ void sqrt_and_rsqrt(double x, double &s, double &is)
    {
        const double y = __builtin_amdgcn_rsq(x), g = x * y;
        const double e = __builtin_fma(-0.5 * y, g, 0.5), c = __builtin_fma(1.5 * e, e, e);
        s = __builtin_fma(g, c, g);
        is = __builtin_fma(y, c, y);
    }
    static __device__ __forceinline__ double rcp(double x)
    {
        const double r = __builtin_amdgcn_rcp(x);
        const double e = __builtin_fma(-x, r, 1.0);
        return __builtin_fma(r, __builtin_fma(e, e, e), r);
    }
    static __device__ __forceinline__ double rsqrt(double x)
    {
        const double y = __builtin_amdgcn_rsq(x);
        const double e = __builtin_fma(-x * y, y, 1.0);
        return __builtin_fma(y, e * __builtin_fma(0.375, e, 0.5), y);
    }
};
template <> struct Num<float> {
    static constexpr float tiny = __FLT_MIN__;
    static __device__ __forceinline__ float sqrt_(float x) { return __builtin_amdgcn_sqrtf(x); }
    static __device__ __forceinline__ float sqrt_pos(float x) { return __builtin_amdgcn_sqrtf(x); }
    static __device__ __forceinline__ float rcp(float x) { return __builtin_amdgcn_rcpf(x); }
    static __device__ __forceinline__ float rsqrt(float x) { return __builtin_amdgcn_rsqf(x); }
};

// The kernel's first argument, read anew from the argument segment at each
// use (scalar loads) through a pointer the compiler cannot follow back to the
// kernel's entry.  For arguments that a march uses in a small part of each
// plane: hoisted out of it, a large argument's pointers and constants exceed
// the scalar registers and are kept in vector lanes or scratch.
template <typename T>
__device__ __forceinline__ const T &first_argument()
{
    auto p = reinterpret_cast<__UINTPTR_TYPE__>(__builtin_amdgcn_kernarg_segment_ptr());
    asm("" : "+s"(p));
    return *(const T *)(const __attribute__((address_space(4))) T *)p;
}

// Adds to counter `which` the number of active lanes of the wavefront with
// hit set, by one atomic from the lowest such lane into the wavefront's slot
// of the counter (every active lane calls it).  Fix-up counters see up to
// millions of events per launch (a multigroup step clips several per cent of
// its cell-groups); atomics of every wavefront on one address serialised
// them and more than doubled the multigroup implicit step.
__device__ __forceinline__ void count_hits(unsigned long long *cnt, int which, bool hit)
{
    const unsigned long long m = __ballot(hit);
    if (m != 0ull && __lane_id() == unsigned(__ffsll((long long)m) - 1)) {
        const unsigned wave = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
        const unsigned slot = wave & (CNT_SLOTS - 1);
        atomicAdd(cnt + (size_t(which) * CNT_SLOTS + slot) * CNT_STRIDE, (unsigned long long)__popcll(m));
    }
}

// minimum / maximum as single instructions (finite arguments)
__device__ __forceinline__ float vmin(float a, float b) { return __builtin_fminf(a, b); }
__device__ __forceinline__ float vmax(float a, float b) { return __builtin_fmaxf(a, b); }
__device__ __forceinline__ double vmin(double a, double b) { return __builtin_fmin(a, b); }
__device__ __forceinline__ double vmax(double a, double b) { return __builtin_fmax(a, b); }

// f^2 = |F|^2 / E^2 of the state V with ie = 1 / E.  FP32 takes it from the
// components F / E (one operation more): |F|^2 leaves FP32's range for |F| below
// 1e-19, while radiation may be as low as the floor on E (1e-30 by default), and
// f^2 has to go with the closure's F_d / E: with f^2 = 0 beside F_d / E ~ 1 the
// pressure came out larger than E.  Steps became 0 to 0.8 % longer (256^3 second
// order 1041 -> 1049 us, 1000^2 cells 36.5 -> 36.7 us).
template <typename R>
__device__ __forceinline__ R f_squared(const R V[4], R ie)
{
    if constexpr (sizeof(R) == 8) return (V[1] * V[1] + V[2] * V[2] + V[3] * V[3]) * ie * ie;
    const R a = V[1] * ie, b = V[2] * ie, c = V[3] * ie;
    return a * a + b * b + c * c;
}

// Donor-cell quantities of the f-preserving fix, f_c^2 = |F_c|^2 / E_c^2 and
// 1 / E_c, computed once per cell and plane for all the faces the cell feeds.
template <typename R>
struct Centre {
    R f2, ie;
};
template <typename R>
__device__ __forceinline__ Centre<R> centre_of(const R C[4])
{
    const R ie = Num<R>::rcp(C[0]);
    return {f_squared(C, ie), ie};
}

// A face state after its face treatment, with the two quantities the
// treatment and the closure share: f^2 = |F|^2 / E^2 (not clamped) and 1 / E.
template <typename R>
struct Face {
    R E, F[3], f2, ie;
};

// f-preserving fix of a reconstructed face state U against its donor cell C
// (Eq. f_reconstruct): keep F_face iff f_face <= 1 and f_face > f_centre,
// else F_face = F_c E_f / E_c (E_face > 0).  The comparison is made on f^2, which the closure needs in either case (the
// rescaled state has the centre's), so it costs no operation of its own.
template <typename R>
__device__ __forceinline__ Face<R> ffix(const R U[4], const R C[4], Centre<R> cc)
{
    Face<R> s{U[0], {U[1], U[2], U[3]}, R(0), Num<R>::rcp(U[0])};
    s.f2 = f_squared(U, s.ie);
    if (!(s.f2 <= R(1) && s.f2 > cc.f2)) {
        const R r = s.E * cc.ie;
        s.F[0] = C[1] * r;
        s.F[1] = C[2] * r;
        s.F[2] = C[3] * r;
        s.f2 = cc.f2;
    }
    return s;
}

// The other face treatments, selected at run time: the "PLUTO" flat fallback
// or the simple clip (the alternatives of Sect. 2.5 and the beam comparison
// of Sect. 3.2); both act only when |R(F)| > R(E) and fall back to the flat
// state for R(E) <= 0.
template <typename R>
__device__ __forceinline__ Face<R> face_fix(int recon, const R U[4], const R C[4])
{
    R V[4] = {U[0], U[1], U[2], U[3]};
    const R Ff2 = U[1] * U[1] + U[2] * U[2] + U[3] * U[3];
    if (!(U[0] > R(0) && Ff2 <= U[0] * U[0])) {
        if (recon == M1_RECON_CLIP && U[0] > R(0)) {
            const R sc = U[0] * Num<R>::rsqrt(Ff2);
            V[1] *= sc;
            V[2] *= sc;
            V[3] *= sc;
        } else {
#pragma unroll
            for (int q = 0; q < 4; ++q) V[q] = C[q];
        }
    }
    const R ie = Num<R>::rcp(V[0]);
    return {V[0], {V[1], V[2], V[3]}, f_squared(V, ie), ie};
}

// component of (x, y, z) along d, by value (a conditional between members
// would select an address and keep the state in memory)
template <typename R>
__device__ __forceinline__ R along(int d, R x, R y, R z)
{
    return d == 0 ? x : (d == 1 ? y : z);
}

// Closure of a face state seen from direction d (Sect. 2.1, 2.6), all in units
// of c_hat: signal speeds lm <= lp and the flux as
//   Phi_0 = F_d,  Phi_q = c F_q + (q = d) iso / 3.
// With s = sqrt(4 - 3 f^2) Levermore's xi is (5 - 2 s) / 3, so that
// (1 - xi) / 2 = (s - 1) / 3 and (3 xi - 1) / 2 = 2 - s.  2 - s vanishes with
// f^2, as 3 f^2 / (2 + s), which takes 1 / |F|^2 out of every expression: with
// phi = F_d / E and m = 2 phi / (2 + s),
//   c      = (2 - s) E F_d / |F|^2      = 3 m / 2,
//   zeta^2 = (s - 1) (2 s / 3 - phi m)   (lambda_-+ = (phi -+ zeta) / s).
// No direction n = F / |F| is formed, so F = 0 and fluxes far below E need no
// case of their own (f^2 is then 0 or nearly, and phi as small; see f_squared for
// E itself that small), and the difference 2 - s
// of nearly equal numbers at small f is gone.  f > 1 (a centre state past the
// limit by a rounding, or a caller's) counts as f = 1: s = 1, phi = F_d / |F|
// and c = E F_d / |F|^2, a branch that no wavefront usually takes.
// FP64 takes s and 1 / s from one estimate y of the reciprocal square root: with
// g = s^2 y and e = (1 - g y) / 2 the corrections of Num's square root and
// reciprocal square root are the same, s = g (1 + e + 3 e^2 / 2) and
// 1 / s = y (1 + e + 3 e^2 / 2).  s taken as s^2 (1 / s) is half an ulp further
// off, and s - 1, a pressure's only factor beside E, three times that: the flux
// after a step in 2D was 5 % (1D 4 %) further from an 80-bit reference, for one
// operation less.  FP32 takes the hardware square root and reciprocal (the rsqrt
// form is two operations shorter, but
// raised the 100-step deviation of the flux from the FP64 form by a quarter).
template <typename R>
struct Wave {
    R lm, lp, c, iso;
};

template <typename R>
__device__ __forceinline__ void limit_f(Face<R> &u, R &k)
{
    const R y = u.f2 > R(1) ? Num<R>::rsqrt(u.f2) : R(1);
    u.ie *= y;
    k *= y;
    u.f2 = vmin(u.f2, R(1));
}

template <typename R>
__device__ __forceinline__ Wave<R> closure_of(const Face<R> &u, int d, R k)
{
    Wave<R> w;
    const R phi = along(d, u.F[0], u.F[1], u.F[2]) * u.ie;
    const R s2 = R(4) - R(3) * u.f2;               // in [1, 4]
    R s, is;
    if constexpr (sizeof(R) == 8) {
        Num<R>::sqrt_and_rsqrt(s2, s, is);
    } else {
        s = Num<R>::sqrt_(s2);
        is = Num<R>::rcp(s);
    }
    const R m = phi * Num<R>::rcp(R(1) + R(0.5) * s);
    const R g = s - R(1);
    // the lower bound keeps the FP64 square root's argument normal
    const R zeta = Num<R>::sqrt_pos(vmax(g * (R(2.0 / 3.0) * s - phi * m), Num<R>::tiny));
    w.lm = (phi - zeta) * is;
    w.lp = (phi + zeta) * is;
    w.c = k * m;
    w.iso = g * u.E;
    return w;
}

// Interface flux Phi* between two face states L | R (Sect. 2.5) in units of
// c_hat: HLL
// with lambda_L = min lambda_-, lambda_R = max lambda_+ clamped to -+4/(3 tau)
// (Sect. 2.6), S_L = min(lambda_L, 0), S_R = max(lambda_R, 0), the average flux
// for S_L = S_R = 0; or Lax-Friedrichs-Rusanov, which is HLL with S_R = -S_L
// the largest limited speed magnitude.  With k = 1 / (S_R - S_L),
// a = k S_R and b = -k S_L,
//   k (S_R Phi_L - S_L Phi_R + S_L S_R (U_R - U_L))
//     = a (c_L - S_L) F_L + b (c_R - S_R) F_R + (q = d) (a iso_L + b iso_R)
// for the flux components (two operations each instead of five), and for the
// energy a F_Ld + b F_Rd + a S_L (E_R - E_L), where the difference is kept: at
// small f its rounding must go with E_R - E_L, not with E.
// tau_sum is the sum of the two cells' optical depths: 4 / (3 tau) is
// 8 / (3 tau_sum), and as |lambda| <= 1 the limit is without effect for
// tau_sum below 1, which keeps the reciprocal finite at tau = 0.
template <typename R>
__device__ __forceinline__ void interface_flux(int d, Face<R> l, Face<R> r, R tau_sum, R out[4],
                                               int riemann)
{
    R kl = R(1.5), kr = R(1.5);
    if (vmax(l.f2, r.f2) > R(1)) {
        limit_f(l, kl);
        limit_f(r, kr);
    }
    const Wave<R> wl = closure_of(l, d, kl), wr = closure_of(r, d, kr);
    const R lim = R(8.0 / 3.0) * Num<R>::rcp(vmax(tau_sum, R(1)));
    R SL = vmax(vmin(vmin(wl.lm, wr.lm), R(0)), -lim);
    R SR = vmin(vmax(vmax(wl.lp, wr.lp), R(0)), lim);
    R a = R(0.5), b = a;
    if (riemann == M1_RIEMANN_LF) {
        const R lamL = vmax(vmin(wl.lm, wr.lm), -lim), lamR = vmin(vmax(wl.lp, wr.lp), lim);
        SR = vmax(__builtin_fabs(lamL), __builtin_fabs(lamR));
        SL = -SR;
    } else if (SR > SL) {
        const R k = Num<R>::rcp(SR - SL);
        a = k * SR;
        b = -(k * SL);
    }
    const R el = a * (wl.c - SL), er = b * (wr.c - SR);
    const R iso = R(1.0 / 3.0) * (a * wl.iso + b * wr.iso);
    const R Fl = along(d, l.F[0], l.F[1], l.F[2]), Fr = along(d, r.F[0], r.F[1], r.F[2]);
    out[0] = (a * SL) * (r.E - l.E) + (a * Fl + b * Fr);
#pragma unroll
    for (int q = 0; q < 3; ++q) out[1 + q] = el * l.F[q] + (er * r.F[q] + (d == q ? iso : R(0)));
}

// the hardware's legacy multiply, 0 x anything = 0 (through the compiler's
// intrinsic, so its scheduling and hazard rules apply)
extern "C" __device__ float amdgcn_fmul_legacy(float, float) __asm("llvm.amdgcn.fmul.legacy");

// van Leer limited slope without a branch: the harmonic mean
// 2 dl dr / (dl + dr) when the signs agree, zero when they differ or either
// is zero.  FP32: (dl |dr| + |dl| dr) / (|dl| + |dr|) with the legacy multiply
// (0 x inf = 0), so dl = dr = 0 gives 0 without a select (and a subnormal
// |dl| + |dr|, whose reciprocal overflows, has num = 0).  FP64: 2 u w (dl + dr)
// with the shares u = dl / (dl + dr) and w = dr / (dl + dr) clamped to
// [0, 1], which costs nothing (an output modifier): of opposite signs one
// share is negative, and of dl + dr = 0 both are NaN, which the clamp takes
// to 0; no compare and select, and no product of two small differences that
// could underflow.
template <typename R>
__device__ __forceinline__ R vanleer_fast(R dl, R dr);
template <>
__device__ __forceinline__ float vanleer_fast<float>(float dl, float dr)
{
    const float num = __builtin_fmaf(__builtin_fabsf(dl), dr, dl * __builtin_fabsf(dr));
    return amdgcn_fmul_legacy(num, __builtin_amdgcn_rcpf(__builtin_fabsf(dl) + __builtin_fabsf(dr)));
}
template <>
__device__ __forceinline__ double vanleer_fast<double>(double dl, double dr)
{
    const double den = dl + dr, t = Num<double>::rcp(den);
    const double u = __builtin_fmin(__builtin_fmax(dl * t, 0.0), 1.0);
    const double w = __builtin_fmin(__builtin_fmax(dr * t, 0.0), 1.0);
    return (u * w) * (den + den);
}

// Flux at the face between donor cells b (left) and c (right) along d from
// their states, slopes (sb, sc; per lower spacing) and f-fix quantities (cb,
// cc): face states q_b + s_b hp_b and q_c - s_c hm_c, the face treatment, both
// closures and the optical-depth-limited flux.
template <typename R>
__device__ __forceinline__ void face_flux_s(int d, const R qb[4], const R qc[4], const R sb[4], const R sc[4],
                                            Centre<R> cb, Centre<R> cc, R hpL, R hmR, R tau_sum,
                                            R out[4], int recon = M1_RECON_FPRESERVE,
                                            int riemann = M1_RIEMANN_HLL)
{
    R UL[4], UR[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        UL[v] = qb[v] + sb[v] * hpL;
        UR[v] = qc[v] - sc[v] * hmR;
    }
    Face<R> l, r;
    if (recon == M1_RECON_FPRESERVE) {
        // E_face <= 0 (no limited slope gives it on a positive field) falls
        // back to the centre state, which the fix then leaves as it is
        const bool pl = UL[0] > R(0), pr = UR[0] > R(0);
        if (!(vmin(UL[0], UR[0]) > R(0))) {
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                UL[v] = pl ? UL[v] : qb[v];
                UR[v] = pr ? UR[v] : qc[v];
            }
        }
        l = ffix(UL, qb, cb);
        r = ffix(UR, qc, cc);
    } else {
        l = face_fix(recon, UL, qb);
        r = face_fix(recon, UR, qc);
    }
    interface_flux(d, l, r, tau_sum, out, riemann);
}

// van Leer slopes of the four fields of cell m from cells m-1, m, m+1 and the
// ratio of its centre spacings (x_m - x_{m-1}) / (x_{m+1} - x_m); per lower
// spacing, as are the limiter's arguments (it is homogeneous of degree one).
template <typename R>
__device__ __forceinline__ void slopes4(const R qm[4], const R q0[4], const R qp[4], R rat, R s[4])
{
#pragma unroll
    for (int v = 0; v < 4; ++v) s[v] = vanleer_fast(q0[v] - qm[v], (qp[v] - q0[v]) * rat);
}

// LimO3 limited slope (Cada and Torrilhon 2009, the compact third-order
// reconstruction Sect. 2.5 names) of a cell for its face on the side of the
// divided difference dnear, dfar being the one on the other side:
// phi(theta) dnear with theta = dfar / dnear and
//   phi = max(0, min(p3, max(-theta/2, min(2 theta, p3, 3/2)))),
//   p3 = (2 + theta) / 3 (the unlimited third-order reconstruction).
// Evaluated without a division: with s = sign(dnear), a = s dfar and
// b = |dnear|, phi dnear = s b phi, and b >= 0 scales through every min and
// max, so phi dnear = s max(0, min(q, max(-a/2, min(2a, q, 3b/2)))) with
// q = (2b + a) / 3; dnear = 0 gives 0 (the limit of phi dnear).
template <typename R>
__device__ __forceinline__ R limo3(R dfar, R dnear)
{
    const R s = dnear < R(0) ? R(-1) : R(1);
    const R a = s * dfar, b = s * dnear;
    const R q = (R(2) * b + a) * R(1.0 / 3.0);
    const R inner = vmin(vmin(R(2) * a, q), R(1.5) * b);
    return s * vmax(R(0), vmin(q, vmax(R(-0.5) * a, inner)));
}

// LimO3 slopes of the four fields of cell m from cells m-1, m, m+1: lo for
// the lower face (near side m-1), hi for the upper face (near side m+1).
template <typename R>
__device__ __forceinline__ void limo3_slopes4(const R qm[4], const R q0[4], const R qp[4], R rat, R lo[4],
                                              R hi[4])
{
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const R dl = q0[v] - qm[v], dr = (qp[v] - q0[v]) * rat;
        hi[v] = limo3(dl, dr);
        lo[v] = limo3(dr, dl);
    }
}

} // namespace m1
