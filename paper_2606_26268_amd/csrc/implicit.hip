// implicit.hip -- implicit radiation-matter step and the opacity cache.
//
// Per cell (Sect. 2.8): T^n from the gas energy, the 2x2 backward-Euler
// system of Eq. implicit_matrix solved analytically in FP64, flux damping of
// Eq. source_discrete2, the gas total energy and momentum from the rescaled
// conservation laws (Sect. 2.7), f <= 1, and the opacity cache (rho kappa_P,
// optical depth rho chi h_max) re-evaluated at the new temperature for the
// next transport and implicit steps.
#include "m1_internal.h"
#include "implicit_device.h"
#include "mlp_device.h"

namespace m1 {

template <typename R, int OPK, bool NT>
__global__ void __launch_bounds__(256) k_implicit(IArgs<R> a)
{
    const int n0 = a.n[0], n1 = a.n[1];
    const int N = n0 * n1 * a.n[2];
    const long base = long(blockIdx.x) * blockDim.x;
    const unsigned t = threadIdx.x;
    const int id = int(base) + int(t);
    if (id >= N) return;
    int i, j, k;
    a.ix.split(id, i, j, k);
    // the cell extent serves both the optical depth read and the one written
    const R hm = OPK == OPK_CONST ? R(0) : cell_hmax(a.m, a.ndim, i, j, k);
    double rho_d;
    const double T1 = implicit_cell<R, OPK == OPK_CONST, NT>(a, base, t, hm, rho_d);
    if (OPK != OPK_CONST) {
        const R rho = R(rho_d);
        R kP, kR;
        opacity_analytic<R, OPK>(a.op, rho, R(T1), kP, kR);
        cache_entry(rho, kP, kR, R(a.op.sigma), hm, at(a.rkp, base, t), at(a.tau, base, t));
    }
}

// MLP opacity: every lane of a wavefront takes part in the network
// evaluation (one 64-cell chunk per wavefront), so lanes past the last cell
// compute on a clamped index instead of exiting early.  The cell update runs
// before the weights are staged into LDS: its many array pointers are then
// dead during the staging, which keeps the kernel within the scalar register
// file (staged first, the pointers were spilled to vector lanes).
template <typename R, bool NT>
__global__ void __launch_bounds__(256, 4) k_implicit_mlp(IArgs<R> a)
{
    const int n0 = a.n[0], n1 = a.n[1];
    const int N = n0 * n1 * a.n[2];
    const int lane = threadIdx.x & 63;
    __shared__ MlpShared sh;
    {
        const long base = long(blockIdx.x) * blockDim.x;
        const unsigned t = threadIdx.x;
        const int id = int(base) + int(t);
        const bool live = id < N;
        const int idc = live ? id : N - 1;
        int i, j, k;
        a.ix.split(idc, i, j, k);
        const R hm = cell_hmax(a.m, a.ndim, i, j, k);
        // lanes past the last cell evaluate the network at rho = T = 1
        double T1 = 1.0, rho_d = 1.0;
        if (live) T1 = implicit_cell<R, false, NT>(a, base, t, hm, rho_d);
        const float rho = float(rho_d);
        mlp_stage(a.op.mlp, sh, threadIdx.x, blockDim.x);
        __syncthreads();
        float kP, kR;
        mlp_opacity_shared(a.op, sh, rho, float(T1), lane, kP, kR);
        if (live) {
            cache_entry(rho, kP, kR, a.op.f32.sigma, hm, at(a.rkp, base, t), at(a.tau, base, t));
        }
    }
}

template <typename R>
static hipError_t launch_i(m1_ctx *c, double dt, const Metric<R> &met, int stage = 0)
{
    IArgs<R> a;
    fill_args(c, a, met, dt);
    rk2_stage_args(c, a, stage);
    const int N = c->n[0] * c->n[1] * c->n[2];
    dim3 block(256), grid((N + 255) / 256);
    // the step's bytes: E*, F* in, E, F out, the gas in and out, the
    // opacity cache in and out
    const double bytes = double(N) * (8.0 * sizeof(R) + 72.0 + (c->op.kind == OPK_CONST ? 0.0 : 4.0 * sizeof(R)));
    if (stream_reads(c, bytes)) {
        switch (c->op.kind) {
        case OPK_CONST: hipLaunchKernelGGL((k_implicit<R, OPK_CONST, true>), grid, block, 0, c->stream, a); break;
        case OPK_POWERLAW: hipLaunchKernelGGL((k_implicit<R, OPK_POWERLAW, true>), grid, block, 0, c->stream, a); break;
        case OPK_TABLE: hipLaunchKernelGGL((k_implicit<R, OPK_TABLE, true>), grid, block, 0, c->stream, a); break;
        default: hipLaunchKernelGGL((k_implicit_mlp<R, true>), grid, block, 0, c->stream, a); break;
        }
    } else {
        switch (c->op.kind) {
        case OPK_CONST: hipLaunchKernelGGL((k_implicit<R, OPK_CONST, false>), grid, block, 0, c->stream, a); break;
        case OPK_POWERLAW: hipLaunchKernelGGL((k_implicit<R, OPK_POWERLAW, false>), grid, block, 0, c->stream, a); break;
        case OPK_TABLE: hipLaunchKernelGGL((k_implicit<R, OPK_TABLE, false>), grid, block, 0, c->stream, a); break;
        default: hipLaunchKernelGGL((k_implicit_mlp<R, false>), grid, block, 0, c->stream, a); break;
        }
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// multigroup (one gray fluid per frequency group, (m+1)^2 implicit system)
// ---------------------------------------------------------------------------

// Fraction of the Planck energy density below x = h nu / k T,
// (15 / pi^4) int_0^x t^3 / (e^t - 1) dt.  Below x = 5/2: the power series
// of t^3 / (e^t - 1) integrated term by term, coefficients B_k / ((k + 3) k!)
// with B_k the Bernoulli numbers, through k = 42 (the series converges for
// x < 2 pi; at x = 5/2 the omitted terms are below 2e-18 of the sum); above:
// 1 minus the tail sum_n e^{-n x} (x^3/n + 3 x^2/n^2 + 6 x/n^3 + 6/n^4),
// summed until its terms drop below double precision (at most 17 of them
// above 5/2).  The split at 5/2 rather than 1 bounds the tail loop, whose
// length otherwise grows as 1/x and dominated the multigroup implicit step.
__device__ double planck_fraction(double x)
{
    constexpr double NORM = 0.15398973382026503;   // 15 / pi^4
    if (x <= 0.0) return 0.0;
    if (x < 2.5) {
        // B_k / ((k + 3) k!) for k = 2, 4, ..., 42 (odd B_k > 1 vanish)
        constexpr double C[21] = {
            0.016666666666666666, -0.00019841269841269841, 3.6743092298647855e-06, -7.5156325156325161e-08,
            1.6059043836821615e-09, -3.5227934257916621e-11, 7.8720803121674577e-13, -1.7840422612224122e-14,
            4.0886009791799258e-16, -9.4559508632959214e-18, 2.2036011313440918e-19, -5.1683202540046385e-21,
            1.2188644964239542e-22, -2.8882314280766281e-24, 6.8725831889020704e-26, -1.641368762534915e-27,
            3.9328985827428784e-29, -9.451269078629001e-31, 2.2772522578280597e-32, -5.5000521295363484e-34,
            1.3312603916626966e-35};
        const double x2 = x * x;
        // x^3 (1/3 - x/8 + x^2 (C_2 + C_4 x^2 + ...))
        double p = C[20];
        for (int j = 19; j >= 0; --j) p = __builtin_fma(p, x2, C[j]);
        const double series = (1.0 / 3.0) + x * (-0.125) + x2 * p;
        return NORM * x * x2 * series;
    }
    // 1/n, n = 1 .. 17 (the most terms the tail takes above 5/2)
    constexpr double RN[18] = {0.0, 1.0, 1.0 / 2, 1.0 / 3, 1.0 / 4, 1.0 / 5, 1.0 / 6, 1.0 / 7, 1.0 / 8, 1.0 / 9,
                               1.0 / 10, 1.0 / 11, 1.0 / 12, 1.0 / 13, 1.0 / 14, 1.0 / 15, 1.0 / 16, 1.0 / 17};
    const double e1 = exp(-x);
    const double x2 = x * x, x3 = x2 * x;
    double e = e1, tail = 0.0;
    for (int n = 1; n <= 17 && e > 1e-18 * e1; ++n) {
        const double rn = RN[n];
        tail += e * rn * (x3 + rn * (3.0 * x2 + rn * (6.0 * x + rn * 6.0)));
        e *= e1;
    }
    return 1.0 - NORM * tail;
}

template <typename R>
struct MgArgs {
    GroupParams gp;
    long N;
    size_t plane;                     // bytes between scratch fields
    const unsigned char *star;        // transported group states
};

// Optical depth of every group from the gas density (constant opacities).
template <typename R>
__global__ void __launch_bounds__(256) k_tau_mg(IArgs<R> a, MgArgs<R> g, unsigned char *tau)
{
    const int id = blockIdx.x * blockDim.x + threadIdx.x;
    if (id >= g.N) return;
    int i, j, k;
    a.ix.split(id, i, j, k);
    const R h = cell_hmax(a.m, a.ndim, i, j, k);
    const double rho = a.rho[id];
    for (int q = 0; q < g.gp.m; ++q)
        reinterpret_cast<R *>(tau + q * g.plane)[id] = R(rho * (g.gp.kR[q] + g.gp.sigma)) * h;
}

// One cell of the multigroup implicit step.  The (m+1)^2 system
//   (1 + gr_g) E'_g - 4 gr_g b_g a T^3 T' = E*_g - 3 gr_g b_g a T^4
//   -sum_g g_g E'_g + (C_v + 4 sum_g g_g b_g a T^3) T' = C_v T + 3 sum_g g_g b_g a T^4 + S
// is an arrowhead matrix: eliminating the group rows leaves one equation
// for T' whose coefficients are sums of positive terms,
//   D  = C_v + sum_g 4 g_g b_g a T^3 / (1 + gr_g),
//   L  = a (4 T^3 T' - 3 T^4) = a T^3 (C_v T + 4 S + 4 sum_g g_g E*_g / (1 + gr_g)) / D,
//   E'_g = (E*_g + gr_g b_g L) / (1 + gr_g),
// O(m) work and no cancellation.
template <typename R, int MG, bool NT>
__global__ void __launch_bounds__(256) k_implicit_mg(IArgs<R> a, MgArgs<R> g)
{
    const int id = blockIdx.x * blockDim.x + threadIdx.x;
    if (id >= g.N) return;
    const int m = g.gp.m;
    const double rho = ld<NT>(a.rho, 0, id);
    double mx = ld<NT>(a.gin[0], 0, id), my = ld<NT>(a.gin[1], 0, id), mz = ld<NT>(a.gin[2], 0, id);
    double Eg = ld<NT>(a.gin[3], 0, id);
    const double inv_rho = Num<double>::rcp(rho);
    const double Cv = rho * a.k.inv_gm1;
    const double T = gas_T_r(inv_rho, mx, my, mz, Eg, a.k.gm1);
    const double S = a.irr ? ld<NT>(a.irr, 0, id) * a.k.dt : 0.0;
    const double aT3 = a.k.a * T * T * T;
    const double iT = Num<double>::rcp(T);
    // pass 1: group fractions, transported energies and the reduced equation
    // for the temperature (per-group values stay in registers: MG >= m)
    double b[MG], Es[MG], inv1[MG];
    double D = Cv, Lnum = Cv * T + 4.0 * S, lo = 0.0;
#pragma unroll
    for (int q = 0; q < MG; ++q) {
        if (q < m) {
            const double hi = q + 1 < m ? planck_fraction(g.gp.edges[q] * iT) : 1.0;
            b[q] = hi - lo;
            lo = hi;
            Es[q] = double(ld<NT>(reinterpret_cast<const R *>(g.star + 4 * q * g.plane), 0, id));
            const double kr = rho * g.gp.kP[q];
            inv1[q] = Num<double>::rcp(1.0 + a.k.dt_ch * kr);
            const double gg = a.k.dt_c * kr;
            D += 4.0 * gg * b[q] * aT3 * inv1[q];
            Lnum += 4.0 * gg * Es[q] * inv1[q];
        }
    }
    const double L = aT3 * Lnum * Num<double>::rcp(D);
    // pass 2: group energies, damped fluxes, rescaled totals
    double dE = 0.0, dF[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int q = 0; q < MG; ++q) {
        if (q < m) {
            const double gr = a.k.dt_ch * rho * g.gp.kP[q];
            const double E1 = a.absorb ? Es[q] * inv1[q] : (Es[q] + gr * b[q] * L) * inv1[q];
            const double inv_damp = Num<double>::rcp(1.0 + a.k.dt_ch * rho * (g.gp.kR[q] + g.gp.sigma));
            double F1[3], Fs[3];
            for (int v = 0; v < 3; ++v) {
                Fs[v] = double(ld<NT>(reinterpret_cast<const R *>(g.star + (4 * q + 1 + v) * g.plane), 0, id));
                F1[v] = Fs[v] * inv_damp;
            }
            const double Fn = Num<double>::sqrt_(F1[0] * F1[0] + F1[1] * F1[1] + F1[2] * F1[2]);
            const bool clipped = Fn > E1;
            if (clipped) {
                const double sc = E1 / Fn;
                F1[0] *= sc;
                F1[1] *= sc;
                F1[2] *= sc;
            }
            count_hits(a.cnt, 2, clipped);
            R E1r = R(E1), F1r[3] = {R(F1[0]), R(F1[1]), R(F1[2])};
            dE += double(E1r) - Es[q];
            for (int v = 0; v < 3; ++v) dF[v] += double(F1r[v]) - Fs[v];
            const long o = q * g.N + id;
            if (a.ravg[0]) {
                // second-order step: (U^n + U2) / 2, the partner read before
                // this cell is written
                E1r = R(0.5 * (double(ld<NT>(a.ravg[0], o, 0)) + double(E1r)));
                for (int v = 0; v < 3; ++v) F1r[v] = R(0.5 * (double(ld<NT>(a.ravg[1 + v], o, 0)) + double(F1r[v])));
            }
            a.E[o] = E1r;
            a.Fx[o] = F1r[0];
            a.Fy[o] = F1r[1];
            a.Fz[o] = F1r[2];
        }
    }
    Eg += S - a.k.c_ratio * dE;
    mx -= dF[0] * a.k.inv_ch;
    my -= dF[1] * a.k.inv_ch;
    mz -= dF[2] * a.k.inv_ch;
    if (a.ravg[0]) {
        mx = 0.5 * (ld<NT>(a.gavg[0], 0, id) + mx);
        my = 0.5 * (ld<NT>(a.gavg[1], 0, id) + my);
        mz = 0.5 * (ld<NT>(a.gavg[2], 0, id) + mz);
        Eg = 0.5 * (ld<NT>(a.gavg[3], 0, id) + Eg);
    }
    a.Eg[id] = Eg;
    a.mx[id] = mx;
    a.my[id] = my;
    a.mz[id] = mz;
}

template <typename R>
static MgArgs<R> mg_args(m1_ctx *c)
{
    MgArgs<R> g;
    g.gp = c->grp;
    g.N = long(c->n[0]) * c->n[1] * c->n[2];
    g.plane = c->plane_bytes;
    g.star = static_cast<const unsigned char *>(c->star[0]);
    return g;
}

template <typename R, bool NT>
static void launch_mg_kernel(m1_ctx *c, dim3 grid, dim3 block, const IArgs<R> &a, const MgArgs<R> &g)
{
    if (g.gp.m <= 4)
        hipLaunchKernelGGL((k_implicit_mg<R, 4, NT>), grid, block, 0, c->stream, a, g);
    else if (g.gp.m <= 8)
        hipLaunchKernelGGL((k_implicit_mg<R, 8, NT>), grid, block, 0, c->stream, a, g);
    else if (g.gp.m <= 16)
        hipLaunchKernelGGL((k_implicit_mg<R, 16, NT>), grid, block, 0, c->stream, a, g);
    else
        hipLaunchKernelGGL((k_implicit_mg<R, 32, NT>), grid, block, 0, c->stream, a, g);
}

template <typename R>
static hipError_t launch_i_mg(m1_ctx *c, double dt, const Metric<R> &met, int stage = 0)
{
    IArgs<R> a;
    fill_args(c, a, met, dt);
    rk2_stage_args(c, a, stage);
    const MgArgs<R> g = mg_args<R>(c);
    const dim3 grid(unsigned((g.N + 255) / 256)), block(256);
    const double bytes = double(g.N) * (8.0 * sizeof(R) * g.gp.m + 72.0);
    if (stream_reads(c, bytes))
        launch_mg_kernel<R, true>(c, grid, block, a, g);
    else
        launch_mg_kernel<R, false>(c, grid, block, a, g);
    return hipGetLastError();
}

hipError_t launch_implicit_rk2(m1_ctx *c, double dt, int stage)
{
    if (c->grp.m > 1) {
        if (c->par.precision == M1_F32) return launch_i_mg<float>(c, dt, c->met32, stage);
        return launch_i_mg<double>(c, dt, c->met64, stage);
    }
    if (c->par.precision == M1_F32) return launch_i<float>(c, dt, c->met32, stage);
    return launch_i<double>(c, dt, c->met64, stage);
}

hipError_t launch_implicit(m1_ctx *c, double dt)
{
    if (c->grp.m > 1) {
        if (c->par.precision == M1_F32) return launch_i_mg<float>(c, dt, c->met32);
        return launch_i_mg<double>(c, dt, c->met64);
    }
    if (c->par.precision == M1_F32) return launch_i<float>(c, dt, c->met32);
    return launch_i<double>(c, dt, c->met64);
}

// ---------------------------------------------------------------------------
// opacity cache from the current gas state
// ---------------------------------------------------------------------------

template <typename R, int OPK>
__global__ void __launch_bounds__(256) k_opacity_init(IArgs<R> a)
{
    const int n0 = a.n[0], n1 = a.n[1];
    const int N = n0 * n1 * a.n[2];
    const int id = blockIdx.x * blockDim.x + threadIdx.x;
    if (id >= N) return;
    int i, j, k;
    a.ix.split(id, i, j, k);
    const double T = gas_T_stored(a.rho[id], a.mx[id], a.my[id], a.mz[id], a.Eg[id], a.k.gm1);
    const R rho = R(a.rho[id]);
    R kP, kR;
    opacity_analytic<R, OPK>(a.op, rho, R(T), kP, kR);
    cache_entry(rho, kP, kR, R(a.op.sigma), cell_hmax(a.m, a.ndim, i, j, k), a.rkp[id], a.tau[id]);
}

template <typename R>
__global__ void __launch_bounds__(256) k_opacity_init_mlp(IArgs<R> a)
{
    const int n0 = a.n[0], n1 = a.n[1];
    const int N = n0 * n1 * a.n[2];
    const int lane = threadIdx.x & 63;
    __shared__ MlpShared sh;
    mlp_stage(a.op.mlp, sh, threadIdx.x, blockDim.x);
    __syncthreads();
    {
        const int id = blockIdx.x * blockDim.x + threadIdx.x;
        const bool live = id < N;
        const int idc = live ? id : N - 1;
        int i, j, k;
        a.ix.split(idc, i, j, k);
        const double T = gas_T_stored(a.rho[idc], a.mx[idc], a.my[idc], a.mz[idc], a.Eg[idc], a.k.gm1);
        const float rho = float(a.rho[idc]);
        float kP, kR;
        mlp_opacity_shared(a.op, sh, rho, float(T), lane, kP, kR);
        if (live) {
            cache_entry(rho, kP, kR, a.op.f32.sigma, cell_hmax(a.m, a.ndim, i, j, k), a.rkp[id], a.tau[id]);
        }
    }
}

template <typename R>
static hipError_t launch_init(m1_ctx *c, const Metric<R> &met)
{
    IArgs<R> a;
    fill_args(c, a, met, 0.0);
    const int N = c->n[0] * c->n[1] * c->n[2];
    dim3 block(256), grid((N + 255) / 256);
    switch (c->op.kind) {
    case OPK_CONST: hipLaunchKernelGGL((k_opacity_init<R, OPK_CONST>), grid, block, 0, c->stream, a); break;
    case OPK_POWERLAW: hipLaunchKernelGGL((k_opacity_init<R, OPK_POWERLAW>), grid, block, 0, c->stream, a); break;
    case OPK_TABLE: hipLaunchKernelGGL((k_opacity_init<R, OPK_TABLE>), grid, block, 0, c->stream, a); break;
    default:
        hipLaunchKernelGGL((k_opacity_init_mlp<R>), grid, block, 0, c->stream, a);
        break;
    }
    return hipGetLastError();
}

template <typename R>
static hipError_t launch_init_mg(m1_ctx *c, const Metric<R> &met)
{
    IArgs<R> a;
    fill_args(c, a, met, 0.0);
    const MgArgs<R> g = mg_args<R>(c);
    hipLaunchKernelGGL((k_tau_mg<R>), dim3(unsigned((g.N + 255) / 256)), dim3(256), 0, c->stream, a, g,
                       static_cast<unsigned char *>(c->tau));
    return hipGetLastError();
}

hipError_t launch_opacity_init(m1_ctx *c)
{
    if (c->grp.m > 1) {
        if (c->par.precision == M1_F32) return launch_init_mg<float>(c, c->met32);
        return launch_init_mg<double>(c, c->met64);
    }
    if (c->par.precision == M1_F32) return launch_init<float>(c, c->met32);
    return launch_init<double>(c, c->met64);
}

// ---------------------------------------------------------------------------
// pointwise evaluation of the active opacity source (tests, tools)
// ---------------------------------------------------------------------------

template <int OPK>
__global__ void __launch_bounds__(256) k_opacity_eval(OpacityParams op, long n, const double *rho,
                                                      const double *T, double *kP, double *kR)
{
    const long id = blockIdx.x * (long)blockDim.x + threadIdx.x;
    if (id >= n) return;
    double a, b;
    opacity_analytic<double, OPK>(op, rho[id], T[id], a, b);
    kP[id] = a;
    kR[id] = b;
}

__global__ void __launch_bounds__(256) k_opacity_eval_mlp(OpacityParams op, long n, const double *rho,
                                                          const double *T, double *kP, double *kR)
{
    const int lane = threadIdx.x & 63;
    __shared__ MlpShared sh;
    mlp_stage(op.mlp, sh, threadIdx.x, blockDim.x);
    __syncthreads();
    {
        const long id = blockIdx.x * (long)blockDim.x + threadIdx.x;
        const bool live = id < n;
        const long idc = live ? id : n - 1;
        float a, b;
        mlp_opacity_shared(op, sh, float(rho[idc]), float(T[idc]), lane, a, b);
        if (live) {
            kP[id] = a;
            kR[id] = b;
        }
    }
}

hipError_t launch_opacity_eval(m1_ctx *c, long n, const double *rho, const double *T, double *kP,
                               double *kR)
{
    if (n <= 0) return hipSuccess;
    dim3 block(256);
    dim3 grid((unsigned)((n + 255) / 256));
    switch (c->op.kind) {
    case OPK_CONST: hipLaunchKernelGGL((k_opacity_eval<OPK_CONST>), grid, block, 0, c->stream, c->op, n, rho, T, kP, kR); break;
    case OPK_POWERLAW: hipLaunchKernelGGL((k_opacity_eval<OPK_POWERLAW>), grid, block, 0, c->stream, c->op, n, rho, T, kP, kR); break;
    case OPK_TABLE: hipLaunchKernelGGL((k_opacity_eval<OPK_TABLE>), grid, block, 0, c->stream, c->op, n, rho, T, kP, kR); break;
    default:
        hipLaunchKernelGGL(k_opacity_eval_mlp, grid, block, 0, c->stream, c->op, n, rho, T, kP, kR);
        break;
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// RK2 averaging: U <- (U_saved + U) / 2 for E, F (form precision) and m, E_g
// ---------------------------------------------------------------------------

} // namespace m1

