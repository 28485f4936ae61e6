// implicit_device.h -- one cell of the implicit radiation-matter step and its
// opacity-cache entry, shared by the implicit kernels and by the fused stages
// of the second-order step.
#pragma once
#include "m1_internal.h"
#include "m1_device.h"
#include "opacity_device.h"

namespace m1 {

template <typename R>
struct IArgs {
    R *E, *Fx, *Fy, *Fz;              // caller's radiation (written)
    const R *Es, *Fxs, *Fys, *Fzs;    // transported state
    const double *rho;
    double *mx, *my, *mz, *Eg;
    R *rkp, *tau;                     // opacity cache (read at T^n, written at T^{n+1})
    int n[3];
    int ndim;
    CellIndex ix;
    Metric<R> m;
    OpacityParams op;
    ImplicitConsts k;
    const double *irr;                // irradiation heating per cell, or null
    int absorb;                       // absorption without emission
    const double *gin[4];             // gas read (mx, my, mz, E_g); the written arrays in place
    const R *ravg[4];                 // second-order step: radiation written as (ravg + new) / 2, or null
    const double *gavg[4];            // and the gas likewise
    unsigned long long *cnt;
};

// largest cell extent over the active directions (optical depth of a cell)
template <typename R>
__device__ __forceinline__ R cell_hmax(const Metric<R> &m, int ndim, int i, int j, int k)
{
    R h = m.hd[0][i] * m.hI[0][i] * m.hJ[0][j];
    if (ndim >= 2) {
        const R h1 = m.hd[1][j] * m.hI[1][i] * m.hJ[1][j];
        h = h1 > h ? h1 : h;
    }
    if (ndim >= 3) {
        const R h2 = m.hd[2][k] * m.hI[2][i] * m.hJ[2][j];
        h = h2 > h ? h2 : h;
    }
    return h;
}

// Gas temperature with the reciprocal density supplied:
// T = (E_g - |m|^2 / (2 rho)) (gamma - 1) / rho.
// Written with explicit fused multiply-adds, so that every inlined copy
// rounds the same way whatever the compiler would contract around it.
__device__ __forceinline__ double gas_T_r(double inv_rho, double mx, double my, double mz, double Eg,
                                          double gm1)
{
    const double m2 = __builtin_fma(mx, mx, __builtin_fma(my, my, mz * mz));
    return __builtin_fma(-0.5 * inv_rho, m2, Eg) * (gm1 * inv_rho);
}

// Gas temperature of a stored state, in exactly the arithmetic the implicit
// step uses for the temperature at which it refreshes the opacity cache, so
// that a cache derived from a stored state (binding, refresh) equals the one
// the step left: a state saved and bound again continues bit for bit.
__device__ __forceinline__ double gas_T_stored(double rho, double mx, double my, double mz, double Eg, double gm1)
{
    return gas_T_r(Num<double>::rcp(rho), mx, my, mz, Eg, gm1);
}

// One opacity-cache entry: the absorption rate rho kappa_P and the cell's
// optical depth rho (kappa_R + sigma) h.  Contraction is off here, so the
// sum cannot fuse with the last product of the opacity evaluation in one
// kernel and not in another: the implicit step and the refresh from a stored
// state write the same bits, and a saved state bound again continues exactly.
template <typename R, typename K>
__device__ __forceinline__ void cache_entry(K rho, K kP, K kR, K sigma, R hm, R &rkp, R &tau)
{
#pragma clang fp contract(off)
    rkp = R(rho * kP);
    tau = R(rho * (kR + sigma)) * hm;
}

// Element t of the run of cells starting at base: the block's base offset is
// added to the array pointer on the scalar unit, so every access takes the
// scalar base and one shared 32-bit lane offset (no per-array 64-bit address
// arithmetic on the vector unit).
template <typename P>
__device__ __forceinline__ P &at(P *p, long base, unsigned t)
{
    return (p + base)[t];
}

// Read of element t of an input of the implicit step, which reads each
// input once per step.  NT: with the nontemporal hint, which streams past
// the caches (a probe of this kernel's read/write mix: 7.4 TB/s with it,
// 5.9 without) and leaves the last-level cache to the step's outputs, which
// the next transport reads; but inputs that are still in that cache (a
// working set within a few hundred MB, fresh from the transport) are then
// fetched from HBM again.  See NT_MIN_BYTES.
template <bool NT, typename P>
__device__ __forceinline__ P ld(const P *p, long base, unsigned t)
{
    if constexpr (NT)
        return __builtin_nontemporal_load(p + base + t);
    else
        return (p + base)[t];
}

// What one cell of the implicit step reads besides the transported state: gas
// and opacity cache (not with constant opacities).
template <typename R>
struct CellIn {
    double rho, mx, my, mz, Eg;
    R rkp, tau;
};

template <bool CONST_OPAC, bool NT, typename R>
__device__ __forceinline__ void load_cell(const IArgs<R> &a, long base, unsigned t, CellIn<R> &c)
{
    c.rho = ld<NT>(a.rho, base, t);
    c.mx = ld<NT>(a.gin[0], base, t);
    c.my = ld<NT>(a.gin[1], base, t);
    c.mz = ld<NT>(a.gin[2], base, t);
    c.Eg = ld<NT>(a.gin[3], base, t);
    if (!CONST_OPAC) {
        c.rkp = ld<NT>(a.rkp, base, t);
    }
}

// One cell of the implicit step (cell base + t) from its inputs and the
// transported state Er, Fr: writes the state and returns the new gas
// temperature.  Four FP64 reciprocals per cell (about 1 ulp): 1/rho, the
// determinant, the flux damping factor and the optical depth per length.
template <typename R, bool CONST_OPAC, bool NT>
__device__ __forceinline__ double solve_cell(const IArgs<R> &a, long base, unsigned t, R hmax, const CellIn<R> &c,
                                             R Er, const R Fr[3])
{
    const double rho = c.rho;
    double mx = c.mx, my = c.my, mz = c.mz, Eg = c.Eg;
    const double inv_rho = Num<double>::rcp(rho);
    const double Cv = rho * a.k.inv_gm1;
    const double T = gas_T_r(inv_rho, mx, my, mz, Eg, a.k.gm1);
    double rkP, rchi;
    if (CONST_OPAC) {
        rkP = rho * a.op.kP;
        rchi = rho * (a.op.kR + a.op.sigma);
    } else {
        rkP = double(c.rkp);
        rchi = double(c.tau) * Num<double>::rcp(double(hmax));
    }
    const double Es = double(Er);
    const double Fs[3] = {double(Fr[0]), double(Fr[1]), double(Fr[2])};
    // Eq. implicit_matrix with gamma_abs,red = dt c_hat kappa_P rho and
    // gamma_abs = dt c kappa_P rho, inverted by Cramer's rule in a
    // cancellation-free arrangement (det > 0)
    const double gr = a.k.dt_ch * rkP;
    const double g = a.k.dt_c * rkP;
    const double aT3 = a.k.a * T * T * T, aT4 = aT3 * T;
    const double det = Cv * (1.0 + gr) + 4.0 * g * aT3;
    // irradiation energy deposited in the step enters the S_1 row (Sect. 2.9)
    double S = 0.0;
    if (a.irr) S = ld<NT>(a.irr, base, t) * a.k.dt;
    // uniform branch: the absorption-only form costs the default path nothing
    double E1;
    if (a.absorb)
        E1 = Es / (1.0 + gr);
    else
        E1 = (Cv * (Es + gr * aT4) + 4.0 * aT3 * (g * Es + gr * S)) * Num<double>::rcp(det);
    const double inv_damp = Num<double>::rcp(1.0 + a.k.dt_ch * rchi);   // Eq. source_discrete2
    double F1[3] = {Fs[0] * inv_damp, Fs[1] * inv_damp, Fs[2] * inv_damp};
    // |F| > E is rare: its root is left to wavefronts with a cell near or past
    // the limit (the margin covers the rounding of the squares)
    const double F2 = F1[0] * F1[0] + F1[1] * F1[1] + F1[2] * F1[2];
    if (!(F2 < 0.9999 * E1 * E1)) {
        const double Fn = Num<double>::sqrt_(F2);
        const bool clipped = Fn > E1;
        if (clipped) {
            const double s = E1 / Fn;
            F1[0] *= s;
            F1[1] *= s;
            F1[2] *= s;
        }
        count_hits(a.cnt, 2, clipped);
    }
    // stored (possibly float) values define the exchanged amounts, so the
    // rescaled totals E_g + (c/c_hat) E and m + F/c_hat are conserved
    R E1r = R(E1), F1r[3] = {R(F1[0]), R(F1[1]), R(F1[2])};
    Eg += S - a.k.c_ratio * (double(E1r) - Es);
    mx -= (double(F1r[0]) - Fs[0]) * a.k.inv_ch;
    my -= (double(F1r[1]) - Fs[1]) * a.k.inv_ch;
    mz -= (double(F1r[2]) - Fs[2]) * a.k.inv_ch;
    if (a.ravg[0]) {
        // second-order step: U^{n+1} = (U^n + U2) / 2 (the averaging partner
        // is read before this cell is written)
        E1r = R(0.5 * (double(ld<NT>(a.ravg[0], base, t)) + double(E1r)));
        for (int v = 0; v < 3; ++v) F1r[v] = R(0.5 * (double(ld<NT>(a.ravg[1 + v], base, t)) + double(F1r[v])));
        mx = 0.5 * (ld<NT>(a.gavg[0], base, t) + mx);
        my = 0.5 * (ld<NT>(a.gavg[1], base, t) + my);
        mz = 0.5 * (ld<NT>(a.gavg[2], base, t) + mz);
        Eg = 0.5 * (ld<NT>(a.gavg[3], base, t) + Eg);
    }
    at(a.E, base, t) = E1r;
    at(a.Fx, base, t) = F1r[0];
    at(a.Fy, base, t) = F1r[1];
    at(a.Fz, base, t) = F1r[2];
    at(a.Eg, base, t) = Eg;
    at(a.mx, base, t) = mx;
    at(a.my, base, t) = my;
    at(a.mz, base, t) = mz;
    return gas_T_r(inv_rho, mx, my, mz, Eg, a.k.gm1);
}

// One cell of the implicit step, transported state and inputs read here;
// returns the new gas temperature and, in rho, the cell's density.
template <typename R, bool CONST_OPAC, bool NT>
__device__ __forceinline__ double implicit_cell(const IArgs<R> &a, long base, unsigned t, R hmax, double &rho)
{
    CellIn<R> c;
    load_cell<CONST_OPAC, NT>(a, base, t, c);
    if (!CONST_OPAC) c.tau = ld<NT>(a.tau, base, t);
    const R Er = ld<NT>(a.Es, base, t);
    const R Fr[3] = {ld<NT>(a.Fxs, base, t), ld<NT>(a.Fys, base, t), ld<NT>(a.Fzs, base, t)};
    rho = c.rho;
    return solve_cell<R, CONST_OPAC, NT>(a, base, t, hmax, c, Er, Fr);
}

// ---------------------------------------------------------------------------
// launch arguments
// ---------------------------------------------------------------------------

template <typename R>
inline void fill_args(m1_ctx *c, IArgs<R> &a, const Metric<R> &met, double dt)
{
    a.E = static_cast<R *>(c->f.E);
    a.Fx = static_cast<R *>(c->f.Fx);
    a.Fy = static_cast<R *>(c->f.Fy);
    a.Fz = static_cast<R *>(c->f.Fz);
    a.Es = static_cast<const R *>(c->star[0]);
    a.Fxs = static_cast<const R *>(c->star[1]);
    a.Fys = static_cast<const R *>(c->star[2]);
    a.Fzs = static_cast<const R *>(c->star[3]);
    a.rho = c->f.rho;
    a.mx = c->f.mx;
    a.my = c->f.my;
    a.mz = c->f.mz;
    a.Eg = c->f.Eg;
    a.rkp = static_cast<R *>(c->rkp);
    a.tau = static_cast<R *>(c->tau);
    for (int d = 0; d < 3; ++d) a.n[d] = c->n[d];
    a.ndim = c->ndim;
    a.ix.set(c->n[0], c->n[1]);
    a.m = met;
    a.op = c->op;
    a.k.dt = dt;
    a.k.c_hat = c->c_hat;
    a.k.c = c->par.c;
    a.k.a = c->par.a_rad;
    a.k.gamma = c->par.gamma;
    a.k.gm1 = c->par.gamma - 1.0;
    a.k.inv_gm1 = 1.0 / a.k.gm1;
    a.k.dt_ch = dt * c->c_hat;
    a.k.dt_c = dt * c->par.c;
    a.k.inv_ch = 1.0 / c->c_hat;
    a.k.c_ratio = c->par.c * a.k.inv_ch;
    a.irr = c->irr;
    a.absorb = c->par.absorb_only;
    a.gin[0] = a.mx;
    a.gin[1] = a.my;
    a.gin[2] = a.mz;
    a.gin[3] = a.Eg;
    for (int v = 0; v < 4; ++v) {
        a.ravg[v] = nullptr;
        a.gavg[v] = nullptr;
    }
    a.cnt = c->cnt;
}

// Stage of the second-order step (stage 0: an ordinary in-place step).
// Stage 1 reads the caller's gas and writes U1 (radiation and gas) to the
// save buffer; stage 2 reads U1's gas from there and writes (U^n + U2) / 2
// into the caller's arrays, the opacity cache following the written state.
// The buffer holds the four radiation fields of all groups (group-major, a
// field every rk2_rad_bytes) and then the four gas fields.
template <typename R>
inline void rk2_stage_args(m1_ctx *c, IArgs<R> &a, int stage)
{
    if (stage == 0) return;
    const long N = long(c->n[0]) * c->n[1] * c->n[2];
    unsigned char *sv = static_cast<unsigned char *>(c->rk2_save);
    R *srad[4];
    double *sgas[4];
    for (int v = 0; v < 4; ++v) {
        srad[v] = reinterpret_cast<R *>(sv + v * c->rk2_rad_bytes);
        sgas[v] = reinterpret_cast<double *>(sv + 4 * c->rk2_rad_bytes) + v * N;
    }
    if (stage == 1) {
        a.E = srad[0];
        a.Fx = srad[1];
        a.Fy = srad[2];
        a.Fz = srad[3];
        a.mx = sgas[0];
        a.my = sgas[1];
        a.mz = sgas[2];
        a.Eg = sgas[3];
        const double *g[4] = {c->f.mx, c->f.my, c->f.mz, c->f.Eg};
        for (int v = 0; v < 4; ++v) a.gin[v] = g[v];
    } else {
        const R *r[4] = {static_cast<const R *>(c->f.E), static_cast<const R *>(c->f.Fx),
                         static_cast<const R *>(c->f.Fy), static_cast<const R *>(c->f.Fz)};
        const double *g[4] = {c->f.mx, c->f.my, c->f.mz, c->f.Eg};
        for (int v = 0; v < 4; ++v) {
            a.gin[v] = sgas[v];
            a.ravg[v] = r[v];
            a.gavg[v] = g[v];
        }
    }
}

// Streaming reads in the implicit step above this many bytes per step.
// Measured on one box (A/B of both forms, 100-step runs): on the 256^3 box
// and the 192x96x192 grid in FP64 the hint made the whole step 1.6 % and
// 5.5 % faster (the next transport then finds the step's outputs in the
// 256 MB last-level cache), and the network form's 2 %; on the 128^3 box
// (285 MB FP64, 220 MB FP32) the inputs were still cached and the implicit
// kernel took 18-25 % longer with it.  The FP32 table form at 192x96x192
// (425 MB) came out 1 % slower, the one measured case above the line
// that did not gain.  The multigroup kernel follows the same rule (eight
// groups at 128^3: its launch 6-9 % faster, the step 1.3-1.4 %).
constexpr double NT_MIN_BYTES = 384.0 * (1 << 20);

// whether the implicit step of a context streams its reads (m1_params.stream_reads)
inline bool stream_reads(const m1_ctx *c, double bytes)
{
    if (c->par.stream_reads == M1_STREAM_ON) return true;
    if (c->par.stream_reads == M1_STREAM_OFF) return false;
    return bytes >= NT_MIN_BYTES;
}

} // namespace m1
