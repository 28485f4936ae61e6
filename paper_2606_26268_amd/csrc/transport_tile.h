// transport_tile.h -- the transport of one cell column (1D, 2D) and of one
// 3D tile, for the transport kernels (which store the transported state) and
// the fused stages of the second-order step (which solve the implicit step on
// it in registers).  What happens to a finished cell is a functor:
//   struct Fin {
//       struct In;                                  // what it reads per cell
//       void load(long base, unsigned c, In &in);   // cell base + c
//       void operator()(In &in, const R Us[4], R tau, int i, int j, int k, long base, unsigned c);
//   };
#pragma once
#include <mutex>

#include "m1_internal.h"
#include "m1_device.h"

namespace m1 {

// (the first argument of every kernel that runs transport_tile)
template <typename R>
struct TArgs {
    const R *U[4];
    const R *tau;
    R *out;                    // transported fields, a field every out_fs elements
    long out_fs;
    int n[3];
    int bc[3][2];
    int ign[3];
    Metric<R> m;
    R dt, c_hat, e_floor;
    int recon, riemann;
    int limo3;                 // LimO3 slopes instead of PLM van Leer
    int special;               // some side is reflective or fixed
    R bcs[3][2][4];            // ghost state of fixed sides
    long gs_in, gs_out, gs_tau; // element strides between frequency groups
    unsigned long long *cnt;
};

// Frequency group of this block (grid y): offset the group's arrays.
template <typename R>
__device__ __forceinline__ void select_group(TArgs<R> &a)
{
    const long g = blockIdx.y;
    if (g == 0) return;
#pragma unroll
    for (int v = 0; v < 4; ++v) a.U[v] += g * a.gs_in;
    a.out += g * a.gs_out;
    a.tau += g * a.gs_tau;
}

// index along one direction after applying the boundary condition: periodic
// wrap, mirror image (reflective), or the edge cell (outflow and fixed,
// whose ghost state is replaced by ghost_fix).  Mirror indices past the
// interior (cells no face uses, in ragged tiles) are clamped.
__device__ __forceinline__ int map_index(int t, int n, int lo, int hi)
{
    if (t < 0) {
        if (lo == M1_BC_PERIODIC) { while (t < 0) t += n; return t; }
        if (lo == M1_BC_REFLECT) return min(-1 - t, n - 1);
        return 0;
    }
    if (t >= n) {
        if (hi == M1_BC_PERIODIC) { while (t >= n) t -= n; return t; }
        if (hi == M1_BC_REFLECT) return max(2 * n - 1 - t, 0);
        return n - 1;
    }
    return t;
}

// State of a ghost cell of direction d at index t (t outside [0, n)): a
// reflective side reverses the flux component normal to it, a fixed side
// supplies its given state.  Interior indices are left alone.
template <typename R>
__device__ __forceinline__ void ghost_fix(const TArgs<R> &a, int d, int t, int n, R q[4])
{
    if (t >= 0 && t < n) return;
    const int side = t < 0 ? 0 : 1;
    const int bc = a.bc[d][side];
    if (bc == M1_BC_REFLECT) {
        if (d == 0) q[1] = -q[1];
        else if (d == 1) q[2] = -q[2];
        else q[3] = -q[3];
    } else if (bc == M1_BC_FIXED) {
#pragma unroll
        for (int v = 0; v < 4; ++v) q[v] = a.bcs[d][side][v];
    }
}

template <typename R>
__device__ __forceinline__ void load4(const TArgs<R> &a, int lin, R q[4])
{
    q[0] = a.U[0][lin];
    q[1] = a.U[1][lin];
    q[2] = a.U[2][lin];
    q[3] = a.U[3][lin];
}

// Whether the two faces of a cell along D carry the same area factor A / V:
// every Cartesian direction, the azimuthal and axial directions of the
// cylindrical grid and the azimuthal direction of the spherical grid.
template <int GEOM, int D>
constexpr bool same_area = GEOM == M1_CARTESIAN || (GEOM == M1_CYLINDRICAL && D > 0) ||
                           (GEOM == M1_SPHERICAL && D == 2);

// A_hi/V Phi_hi - A_lo/V Phi_lo of one direction, from the lower area factor and the
// difference of the two, da.  Equal face fluxes of equal areas (a uniform state)
// cancel exactly: the contracted a Phi_hi - a Phi_lo would leave the
// rounding error of one product behind in every cell.  Where the areas differ, da is
// the factor of the geometric sources (area_step), and the pressure on the
// wider face meets its source in the same factor: with
// a_hi Phi_hi - a_lo Phi_lo the roundings of two area factors, each times dt c_hat,
// are left behind, many times da P on a grid of thin rings or shells.  (An isotropic
// field at rest on 3000 rings between R = 1 and 2 moved by up to 6000 u da E in a step,
// by 3500 with dt c_hat applied after the difference, and by less than 5 so; u is the unit
// roundoff.)
template <int GEOM, int D, typename R>
__device__ __forceinline__ R face_diff(R al, R da, R flo, R fhi)
{
    const R d = al * (fhi - flo);
    return same_area<GEOM, D> ? d : d + da * fhi;
}

// A_hi/V - A_lo/V of a cell (times dt c_hat, as tr1): radial (b - a) / ring on the
// cylindrical and (b^2 - a^2) / shell on the spherical grid, once and twice the radius
// factor tr1 of the other directions; polar cot(theta)_eff times it.
template <int GEOM, int D, typename R>
__device__ __forceinline__ R area_step(R tr1, R ct)
{
    if (same_area<GEOM, D>) return R(0);
    return D == 1 ? ct * tr1 : (GEOM == M1_SPHERICAL ? tr1 + tr1 : tr1);
}

// Contribution of direction D to the flux divergence of the cell at index t
// along D (row base `base`, stride `stride`): reconstruct cells t-1, t, t+1
// (stencil t-2 .. t+2), take HLL fluxes at both faces of cell t and add
// A_hi/V * Phi_hi - A_lo/V * Phi_lo to acc (tr: dt c_hat times the direction's
// factors of the other coordinates).
template <typename R, int D, int GEOM>
__device__ __forceinline__ void direction_div(const TArgs<R> &a, int base, int stride, int t,
                                              R tr, Centre<R> c0, R acc[4])
{
    const int n = a.n[D], lo = a.bc[D][0], hi = a.bc[D][1];
    R q[5][4];
    int li[5];
#pragma unroll
    for (int s = 0; s < 5; ++s) {
        li[s] = base + map_index(t - 2 + s, n, lo, hi) * stride;
        load4(a, li[s], q[s]);
        if (a.special) ghost_fix(a, D, t - 2 + s, n, q[s]);
    }
    const R *rat = a.m.rat[D], *hp = a.m.hp[D], *hm = a.m.hm[D];
    // slopes: cell t-1 for its upper face, cell t for its lower and upper
    // faces, cell t+1 for its lower face
    R sm[4], slo[4], shi[4], sp[4];
    if (a.limo3) {
        R other[4];
        limo3_slopes4(q[0], q[1], q[2], rat[t + 1], other, sm);
        limo3_slopes4(q[1], q[2], q[3], rat[t + 2], slo, shi);
        limo3_slopes4(q[2], q[3], q[4], rat[t + 3], sp, other);
    } else {
        slopes4(q[0], q[1], q[2], rat[t + 1], sm);
        slopes4(q[1], q[2], q[3], rat[t + 2], slo);
        slopes4(q[2], q[3], q[4], rat[t + 3], sp);
#pragma unroll
        for (int v = 0; v < 4; ++v) shi[v] = slo[v];
    }
    const R tm = a.tau[li[1]], t0 = a.tau[li[2]], tp = a.tau[li[3]];
    const Centre<R> cm = centre_of(q[1]), cp = centre_of(q[3]);
    R flo[4], fhi[4];
    face_flux_s<R>(D, q[1], q[2], sm, slo, cm, c0, hp[t + 1], hm[t + 2], tm + t0, flo, a.recon, a.riemann);
    face_flux_s<R>(D, q[2], q[3], shi, sp, c0, cp, hp[t + 2], hm[t + 3], t0 + tp, fhi, a.recon, a.riemann);
    const R al = a.m.alo[D][t] * tr;                     // tr carries dt c_hat
    const R da = area_step<GEOM, D>(D == 0 ? a.m.inv_reff[t] * tr : tr, GEOM == M1_SPHERICAL && D == 1 ? a.m.cot_eff[t] : R(0));
#pragma unroll
    for (int v = 0; v < 4; ++v) acc[v] += face_diff<GEOM, D>(al, da, flo[v], fhi[v]);
}

template <typename R, int D>
__device__ __forceinline__ void ignorable_div(const TArgs<R> &a, const R U[4], Centre<R> c0, R tr, R acc[4])
{
    Face<R> u{U[0], {U[1], U[2], U[3]}, c0.f2, c0.ie};
    R k = R(1.5);
    limit_f(u, k);
    const Wave<R> w = closure_of(u, D, k);
    const R dA = (a.m.ahi[D][0] - a.m.alo[D][0]) * tr;
    acc[0] += dA * U[1 + D];
#pragma unroll
    for (int q = 0; q < 3; ++q) acc[1 + q] += dA * (w.c * U[1 + q] + (q == D ? R(1.0 / 3.0) * w.iso : R(0)));
}

// U* = U - acc + dt c_hat S_geo(U), acc = dt div(Phi) (the fluxes come in units
// of c_hat and the area factors carry dt c_hat; k_ = dt c_hat / r_eff, the same
// number as dt c_hat times the radius factor of the transverse area factors in
// both curvilinear geometries), then E >= floor and f <= 1
// (counted).
template <typename R, int GEOM>
__device__ __forceinline__ void finish_cell(const TArgs<R> &a, const R U[4], Centre<R> cu, const R acc[4], R k_, R ct,
                                            R Us[4])
{
#pragma unroll
    for (int v = 0; v < 4; ++v) Us[v] = U[v] - acc[v];

    if (GEOM != M1_CARTESIAN) {
        // geometric sources from the cell-centre pressure tensor
        // P_ij = an F_i F_j + delta_ij iso, an = (2 - s) E / |F|^2
        // = 3 / ((2 + s) E) and iso = (s - 1) E / 3 (closure_of), from the
        // cell's f^2 and 1 / E; f > 1 counts as f = 1
        const R f2 = vmin(cu.f2, R(1));
        const R s = Num<R>::sqrt_pos(R(4) - R(3) * f2);
        R an = R(3) * cu.ie * Num<R>::rcp(R(2) + s);
        if (cu.f2 > R(1)) an *= Num<R>::rcp(cu.f2);
        const R iso = (s - R(1)) * (R(1) / R(3)) * U[0];
        if (GEOM == M1_CYLINDRICAL) {           // (R, phi, z)
            const R Ppp = an * U[2] * U[2] + iso, PRp = an * U[1] * U[2];
            Us[1] += k_ * Ppp;
            Us[2] -= k_ * PRp;
        } else {                                 // (r, theta, phi)
            const R Ptt = an * U[2] * U[2] + iso, Ppp = an * U[3] * U[3] + iso;
            const R Prt = an * U[1] * U[2], Prp = an * U[1] * U[3], Ptp = an * U[2] * U[3];
            Us[1] += k_ * (Ptt + Ppp);
            Us[2] += k_ * (ct * Ppp - Prt);
            Us[3] -= k_ * (Prp + ct * Ptp);
        }
    }

    // positivity floor on E, then f <= 1 at the cell centre
    const bool floored = Us[0] < a.e_floor;
    if (floored) Us[0] = a.e_floor;
    count_hits(a.cnt, 0, floored);
    // |F| > E is rare: its square root and reciprocal are left to wavefronts
    // with a cell near or past the limit (the margin covers the rounding of
    // the squares, the comparison itself is that of |F| with E)
    const R F2 = Us[1] * Us[1] + Us[2] * Us[2] + Us[3] * Us[3];
    if (!(F2 < R(0.9999) * Us[0] * Us[0])) {
        const R Fn = Num<R>::sqrt_(F2);
        const bool clipped = Fn > Us[0];
        if (clipped) {
            const R sc = Us[0] * Num<R>::rcp(Fn);
            Us[1] *= sc;
            Us[2] *= sc;
            Us[3] *= sc;
        }
        count_hits(a.cnt, 1, clipped);
    }
}

// the transport step's functor: store the transported state
template <typename R>
struct StoreCell {
    struct In {};
    R *out;
    long fs;
    __device__ __forceinline__ void load(long, unsigned, In &) const {}
    __device__ __forceinline__ void operator()(In &, const R Us[4], R, int, int, int, long base, unsigned c) const
    {
#pragma unroll
        for (int v = 0; v < 4; ++v) (out + v * fs + base)[c] = Us[v];
    }
};

// One cell of a 1D grid, or of a 2D grid too thin for the tiles (tiled_2d), per
// thread (blocks of 256 threads).
template <typename R, int NDIM, int GEOM, class Fin>
__device__ __forceinline__ void transport_cell(const TArgs<R> &a, const Fin &fin)
{
    const int n0 = a.n[0], n1 = a.n[1];
    const long base = long(blockIdx.x) * blockDim.x;
    const int id = int(base) + int(threadIdx.x);
    if (id >= n0 * n1) return;
    typename Fin::In in;
    fin.load(base, threadIdx.x, in);
    const int i = id % n0, j = id / n0;
    R U[4];
    load4(a, id, U);
    R acc[4] = {R(0), R(0), R(0), R(0)};
    const Centre<R> c0 = centre_of(U);

    const R dtc = a.dt * a.c_hat;
    direction_div<R, 0, GEOM>(a, id - i, 1, i, dtc, c0, acc);
    if (NDIM >= 2) {
        const R tr = a.m.trA[1][i] * dtc;
        direction_div<R, 1, GEOM>(a, id - j * n0, n0, j, tr, c0, acc);
    } else if (a.ign[1]) {
        ignorable_div<R, 1>(a, U, c0, a.m.trA[1][i] * dtc, acc);
    }
    if (a.ign[2]) ignorable_div<R, 2>(a, U, c0, a.m.trA[2][i] * a.m.trB[2][j] * dtc, acc);

    R Us[4];
    finish_cell<R, GEOM>(a, U, c0, acc, GEOM == M1_CARTESIAN ? R(0) : a.m.inv_reff[i] * dtc,
                         GEOM == M1_SPHERICAL ? a.m.cot_eff[j] : R(0), Us);
    fin(in, Us, a.tau[id], i, j, 0, base, threadIdx.x);
}

// ---------------------------------------------------------------------------
// Tiled kernels.  3D: a block owns a TX x TY column of cells (Tile below) and
// marches along z
// over a chunk of planes.  Per plane: (1) the state with a two-cell halo in
// x and y (cross-shaped, no corners) is staged in LDS; (2) van Leer slopes
// of every cell that donates to a face of the tile are computed once per
// direction (x: columns -1 .. TX, y: rows -1 .. TY) into LDS; (3) every x
// and y face of the tile is computed once from the two donor states and
// slopes (faces of both directions in one flat pass, direction chosen at run
// time), and the z face above the plane from a per-thread register window
// of four planes and the z slopes of planes k and k+1; (4) the update.  2D: a
// block owns one tile and takes it through the same steps without the z part.
// ---------------------------------------------------------------------------
// Tile of a block: TX x TY cells, one thread per cell, TY = 8 (256 threads)
// or 16 (512 threads).  The taller tile computes 4 % fewer halo faces and
// slopes per cell; FP32 blocks of it take 47 KB of LDS (two per CU, four
// waves per SIMD).  FP64 and general kernels have only the 32 x 8 tile; an FP64
// block takes 52.6 KB, and three share a CU (LDS is dealt out in steps of 1280
// bytes, so a block may take 53,760).
template <int TY_>
struct Tile {
    static constexpr int TX = 32, TY = TY_, HX = TX + 4, HY = TY + 4, NT = TX * TY;
    static constexpr int NHALO = 2 * (2 * TY + 2 * TX);
    // x slots (slopes of the cells of columns -1 .. TX; later x fluxes) and y
    // slots (slopes of the cells of rows -1 .. TY), each row by row
    static constexpr int XS = TX + 2, NXS = TY * XS, NYS = (TY + 2) * TX;
    // Task passes of the slope and face stages: in pass 0 thread (lx, ly) takes
    // the slope of column lx - 1 and the face left of column lx, in pass 1 the
    // slope of row ly - 1 and the face below row ly (their direction is fixed
    // at compile time); pass 2 takes what is left, x first: the slopes of two
    // columns and two rows, the faces right of the last column and above the
    // last row.
    static constexpr int S2X = 2 * TY, S2 = S2X + 2 * TX, F2X = TY, F2 = F2X + TX;
    static_assert(S2 <= NT && F2 <= NT && NHALO <= NT, "one task per thread in pass 2, one halo cell at most");
};

template <typename R, int NDIM, int GEOM, bool GENERAL, int TYB, bool LIMO3, class Fin>
__device__ __forceinline__ void transport_tile(const TArgs<R> &a, int nz_chunk, int tiles_x, int tiles_y, int nblocks,
                                               int cus, const Fin &fin)
{
    using T = Tile<TYB>;
    constexpr int TX = T::TX, TY = T::TY, HX = T::HX, HY = T::HY, NT = T::NT;
    constexpr int NHALO = T::NHALO, XS = T::XS, NXS = T::NXS, NYS = T::NYS;
    // the default scheme (f-preserving fix + HLL, periodic / outflow sides)
    // is compiled without the variant and ghost-state code
    const int recon = GENERAL ? a.recon : int(M1_RECON_FPRESERVE);
    const int riemann = GENERAL ? a.riemann : int(M1_RIEMANN_HLL);
    __shared__ R sq[4][HY][HX];
    // optical depth, f^2 and 1 / E of the staged cells a face can have as a
    // donor: rows -1 .. TY (the outermost rows only enter slopes)
    __shared__ R st[HY - 2][HX];
    __shared__ R scf[2][HY - 2][HX];
    static_assert(GENERAL || !LIMO3, "LimO3 only in the general kernel");
    // Slopes, x slots then y slots (LimO3: upper-face slopes).  The x fluxes
    // take the place of the x slopes: the face left of column c is computed by
    // the wavefront that owns its row, which has read every slope of the row
    // but the last two by then (a wave barrier stands between its reads and its
    // stores), and goes to the slot of column c - 1; the face
    // right of the last column reads the last two slots and goes to the last,
    // which only it reads.
    static_assert(64 % TX == 0, "a row's faces belong to one wavefront");
    __shared__ R ss[4][NXS + NYS];
    __shared__ R ssl[LIMO3 ? 4 : 1][LIMO3 ? NXS + NYS : 1];   // LimO3: lower-face slopes
    __shared__ R sfy[4][TY + 1][TX];
    // spacing ratio and the two centre-to-face offsets of the cells of columns
    // -1 .. TX and rows -1 .. TY
    __shared__ R smx[3][TX + 2], smy[3][TY + 2];
    __shared__ R sux[2][TX], suy[GEOM == M1_SPHERICAL ? 3 : 1][TY];
    R *const sqf = &sq[0][0][0];
    // of the cell at flat index b of sq
    const auto depth = [&](int b) { return (&st[0][0])[b - HX]; };
    const auto centre = [&](int b) { return Centre<R>{(&scf[0][0][0])[b - HX], (&scf[1][0][0])[b - HX]}; };
    constexpr int QS = HY * HX;

    // consecutive logical tiles share an XCD (blocks are dealt to XCDs round-robin)
    const int per = (nblocks + 7) / 8;
    const int L = (blockIdx.x % 8) * per + blockIdx.x / 8;
    if (L >= nblocks) return;
    const int n0 = a.n[0], n1 = a.n[1], n2 = a.n[2];
    const int tx_i = L % tiles_x, rest = L / tiles_x;
    const int x0 = tx_i * TX, y0 = (rest % tiles_y) * TY, z0 = (rest / tiles_y) * nz_chunk;
    const int z1 = min(z0 + nz_chunk, n2);
    const int tid = threadIdx.x, lx = tid % TX, ly = tid / TX;
    const int i = x0 + lx, j = y0 + ly;
    const bool live = i < n0 && j < n1;
    const int mi = map_index(i, n0, a.bc[0][0], a.bc[0][1]);
    const int mj = map_index(j, n1, a.bc[1][0], a.bc[1][1]);
    const int plane = n0 * n1;
    const int col = mj * n0 + mi;

    // halo cell of this thread (tid < NHALO): cross-shaped, no corners; its
    // index in sq, and whether it is also in st and scf
    int hx = 0, hy = 0, hcol = 0;
    if (tid < NHALO) {
        if (tid < 2 * TX) { hy = tid / TX; hx = 2 + tid % TX; }
        else if (tid < 4 * TX) { hy = TY + 2 + (tid - 2 * TX) / TX; hx = 2 + (tid - 2 * TX) % TX; }
        else if (tid < 4 * TX + 2 * TY) { hx = (tid - 4 * TX) / TY; hy = 2 + (tid - 4 * TX) % TY; }
        else { hx = TX + 2 + (tid - 4 * TX - 2 * TY) / TY; hy = 2 + (tid - 4 * TX - 2 * TY) % TY; }
        const int gi = map_index(x0 - 2 + hx, n0, a.bc[0][0], a.bc[0][1]);
        const int gj = map_index(y0 - 2 + hy, n1, a.bc[1][0], a.bc[1][1]);
        hcol = gj * n0 + gi;
    }
    const int hq = hy * HX + hx;
    const bool donor = tid >= TX && (tid < 3 * TX || tid >= 4 * TX);
    // ghost transformation of a state in this thread's column (x, y ghosts)
    // and in plane kk (z ghosts); halo cells are ghosts in x or y only
    auto fix_col = [&](int kk, R q[4]) {
        if (!GENERAL || !a.special) return;
        const TArgs<R> &g = first_argument<TArgs<R>>();
        ghost_fix(g, 0, i, n0, q);
        ghost_fix(g, 1, j, n1, q);
        if (NDIM == 3) ghost_fix(g, 2, kk, n2, q);
    };
    auto fix_halo = [&](R q[4]) {
        if (!GENERAL || !a.special) return;
        const TArgs<R> &g = first_argument<TArgs<R>>();
        ghost_fix(g, 0, x0 - 2 + hx, n0, q);
        ghost_fix(g, 1, y0 - 2 + hy, n1, q);
    };

    // Every task's cells and slots lie at fixed offsets from the thread's own
    // cell in passes 0 and 1, so one address serves them all.  Cells past the
    // last ghost feed no face that is used: passes 0 and 1 run them along (on
    // staged cells and a zero ratio) rather than split the code into one block
    // per pass, pass 2 is left to the wavefronts that have tasks in it.
    const int own = ly * HX + lx, xs = ly * XS + lx;
    const bool s_on = tid < T::S2, f_on = tid < T::F2;
    // The thread's index as pass 2 decodes it: FP64 and LimO3 kernels hide it
    // from the compiler, which otherwise keeps the decoded words through the
    // march (10 registers: the third wave per SIMD in FP64, the fourth in FP32
    // with LimO3; the other kernels have them to spare and are 2-3 % faster with
    // the words kept).
    const auto task = [&] {
        int t = tid;
        if constexpr (sizeof(R) == 8 ? !GENERAL : LIMO3) asm("" : "+v"(t));
        return t;
    };
    // metric of the tile's columns and rows (read after the first barrier)
    if (tid < TX + 2) {
        const int m = x0 + tid - 1;
        smx[0][tid] = m <= n0 ? a.m.rat[0][m + 2] : R(0);
        smx[1][tid] = m <= n0 ? a.m.hp[0][m + 2] : R(0);
        smx[2][tid] = m <= n0 ? a.m.hm[0][m + 2] : R(0);
    } else if (tid >= 64 && tid < 64 + TY + 2) {
        const int q = tid - 64, m = y0 + q - 1;
        smy[0][q] = m <= n1 ? a.m.rat[1][m + 2] : R(0);
        smy[1][q] = m <= n1 ? a.m.hp[1][m + 2] : R(0);
        smy[2][q] = m <= n1 ? a.m.hm[1][m + 2] : R(0);
    }
    // Update factors of the tile's columns (the lower area factor of x, dt c_hat
    // in it, and the radius factor of the other directions, which is also
    // that of the geometric sources) and rows (the lower area factor of y, the
    // sine factor of z and cot theta); the upper faces' follow (area_step).
    if (tid >= 128 && tid < 128 + TX) {
        const int c = tid - 128, m = x0 + c;
        const R dtc = m < n0 ? a.dt * a.c_hat : R(0);
        const int mm = min(m, n0 - 1);
        sux[0][c] = a.m.alo[0][mm] * dtc;
        sux[1][c] = a.m.trA[1][mm] * dtc;
    } else if (tid >= 192 && tid < 192 + TY) {
        const int q = tid - 192, mm = min(y0 + q, n1 - 1);
        suy[0][q] = a.m.alo[1][mm];
        if (GEOM == M1_SPHERICAL) {
            suy[1][q] = a.m.trB[2][mm];
            suy[2][q] = a.m.cot_eff[mm];
        }
    }
    const R dtc = a.dt * a.c_hat;

    const int bz0 = a.bc[2][0], bz1 = a.bc[2][1];
    // cell c of plane kk (mapped) and its optical depth
    auto loadp = [&](int kk, int c, R q[4], R &t) {
        const int lin = NDIM == 3 ? map_index(kk, n2, bz0, bz1) * plane + c : c;
        load4(a, lin, q);
        t = a.tau[lin];
    };
    const R *rz = a.m.rat[2], *hpz = a.m.hp[2], *hmz = a.m.hm[2];

    // register window of the thread's column: planes k-1 .. k+2, z slope of
    // plane k.  Plane k+2 is loaded at the top of iteration k and first used
    // after the x/y slopes: the neighbouring tiles read a plane's
    // edge lines as their halo two planes after it was loaded, and those
    // lines are still in L2.  Loaded a plane earlier (k+3 in iteration k),
    // the halo read came three planes later and often missed: on the
    // 192x96x192 grid the kernel fetched 136 MB per launch instead of
    // 99 MB, and ran 1-2 % slower.
    // Halo cells are loaded one plane ahead: issued after the staging of plane
    // k, they arrive while its faces are computed.
    R W0[4], W1[4], T0, T1, Fz0[4], Fz1[4], Sz0[4], Sz1[4], Hq[4], Ht = R(0);
    Centre<R> C0, C1;                   // f-fix quantities of plane k and k + 1
    if constexpr (NDIM == 2) {
        loadp(0, col, W0, T0);
        if (tid < NHALO) loadp(0, hcol, Hq, Ht);
        fix_col(0, W0);
        C0 = centre_of(W0);
    } else {
        R Q0[4], Qm[4], Szm[4], Tm, Tx;
        loadp(z0 - 2, col, Q0, Tx);
        loadp(z0 - 1, col, Qm, Tm);
        loadp(z0, col, W0, T0);
        loadp(z0 + 1, col, W1, T1);
        if (tid < NHALO) loadp(z0, hcol, Hq, Ht);
        fix_col(z0 - 2, Q0);
        fix_col(z0 - 1, Qm);
        fix_col(z0, W0);
        fix_col(z0 + 1, W1);
        C0 = centre_of(W0);
        if constexpr (LIMO3) {
            // the face below plane z0 takes the upper-face slope of plane
            // z0 - 1 and the lower-face slope of plane z0; Sz0 carries the
            // upper-face slope of the current plane
            R lo_m[4], lo_0[4];
            limo3_slopes4(Q0, Qm, W0, rz[z0 + 1], lo_m, Szm);
            limo3_slopes4(Qm, W0, W1, rz[z0 + 2], lo_0, Sz0);
            face_flux_s<R>(2, Qm, W0, Szm, lo_0, centre_of(Qm), C0, hpz[z0 + 1], hmz[z0 + 2], Tm + T0, Fz0, recon,
                           riemann);
        } else {
            slopes4(Q0, Qm, W0, rz[z0 + 1], Szm);
            slopes4(Qm, W0, W1, rz[z0 + 2], Sz0);
            face_flux_s<R>(2, Qm, W0, Szm, Sz0, centre_of(Qm), C0, hpz[z0 + 1], hmz[z0 + 2], Tm + T0, Fz0, recon,
                           riemann);
        }
    }

    // Default kernels: blocks b and b + cus share a compute unit (each XCD
    // hands out its blocks in order, one per compute unit before the
    // second), and the wave arbiter favours the older block: left alone, the
    // first block on a unit finished its chunk in 70 % of the second's time
    // (FP32, measured on the 192x96x192 grid), and the second then ran alone
    // at half occupancy.  The two alternate their wave priority every plane
    // and stay level (FP32: 3-4 % faster transport with one round of blocks,
    // 1 % with several; FP64, measured with two blocks per unit: 1-1.5 %).  The
    // general kernels run other block counts per unit; for them the
    // alternation did not pay (1-6 % slower).
    constexpr bool ALTERNATE = NDIM == 3 && !GENERAL;
    const int prio_grp = (int(blockIdx.x) / cus) & 1;
    // One plane: Wa, Wb are planes k and k + 1 of the window, Wc takes k + 2;
    // Fa, Fb the fluxes below and above, Sa, Sb the (upper-face) z slopes of
    // planes k and k + 1.  In 2D the one plane there is, without window or z faces.
    auto step = [&](int k, const R (&Wa)[4], const R (&Wb)[4], R (&Wc)[4], const R (&Fa)[4], R (&Fb)[4],
                    const R (&Sa)[4], R (&Sb)[4], const Centre<R> &Ca, Centre<R> &Cb, R Ta, R Tb, R &Tc) {
        if constexpr (ALTERNATE) {
            if (((k - z0) ^ prio_grp) & 1)
                __builtin_amdgcn_s_setprio(1);
            else
                __builtin_amdgcn_s_setprio(0);
        }
        // the plane entering the window
        if constexpr (NDIM == 3) {
            loadp(k + 2, col, Wc, Tc);
            fix_col(k + 2, Wc);
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) sq[v][ly + 2][lx + 2] = Wa[v];
        st[ly + 1][lx + 2] = Ta;
        scf[0][ly + 1][lx + 2] = Ca.f2;
        scf[1][ly + 1][lx + 2] = Ca.ie;
        if (tid < NHALO) {
            fix_halo(Hq);
#pragma unroll
            for (int v = 0; v < 4; ++v) sqf[v * QS + hq] = Hq[v];
            if (donor) {
                (&st[0][0])[hq - HX] = Ht;
                const Centre<R> ch = centre_of(Hq);
                (&scf[0][0][0])[hq - HX] = ch.f2;
                (&scf[1][0][0])[hq - HX] = ch.ie;
            }
            if (NDIM == 3 && k + 1 < z1) loadp(k + 1, hcol, Hq, Ht);
        }
        __syncthreads();

        // slopes of the x and y donor cells
#pragma unroll
        for (int p = 0; p < 3; ++p) {
            if (p == 2 && !s_on) continue;

            R qm[4], q0[4], qp[4], sl[4], rat;
            bool y = p == 1;
            int ctr, slot;                  // centre cell and slope slot
            if (p == 0) {
                ctr = own + 2 * HX + 1;
                slot = xs;
                rat = smx[0][lx];
            } else if (p == 1) {
                ctr = own + HX + 2;
                slot = NXS + tid;
                rat = smy[0][ly];
            } else {
                const int t2 = task();
                y = t2 >= T::S2X;
                const int q = t2 - T::S2X;
                const int r = y ? TY + q / TX : t2 >> 1, c = y ? q % TX : TX + (t2 & 1);
                ctr = (r + (y ? 1 : 2)) * HX + c + (y ? 2 : 1);
                slot = y ? NXS + r * TX + c : r * XS + c;
                rat = y ? smy[0][r] : smx[0][c];
            }
            const int str = y ? HX : 1;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                qm[v] = sqf[v * QS + ctr - str];
                q0[v] = sqf[v * QS + ctr];
                qp[v] = sqf[v * QS + ctr + str];
            }
            if constexpr (LIMO3) {
                R lo[4];
                limo3_slopes4(qm, q0, qp, rat, lo, sl);
#pragma unroll
                for (int v = 0; v < 4; ++v) ssl[v][slot] = lo[v];
            } else {
                slopes4(qm, q0, qp, rat, sl);
            }
#pragma unroll
            for (int v = 0; v < 4; ++v) ss[v][slot] = sl[v];
        }

        // z slope(s) of plane k+1 (LimO3: Sb its upper-face slope, Sl its
        // lower-face one)
        R Sl[4];
        if constexpr (NDIM == 2)
            ;
        else if constexpr (LIMO3)
            limo3_slopes4(Wa, Wb, Wc, rz[k + 3], Sl, Sb);
        else
            slopes4(Wa, Wb, Wc, rz[k + 3], Sb);
        __syncthreads();

        // x faces (left face of a column) and y faces (lower face of a row)
#pragma unroll
        for (int p = 0; p < 3; ++p) {
            if (p == 2 && !f_on) continue;

            bool y = p == 1;
            int b, sb, fo;                  // left donor, its slope's slot, flux slot
            R hp, hm;
            if (p == 0) {
                b = own + 2 * HX + 1;
                sb = fo = xs;
                hp = smx[1][lx];
                hm = smx[2][lx + 1];
            } else if (p == 1) {
                b = own + HX + 2;
                sb = NXS + tid;
                fo = tid;
                hp = smy[1][ly];
                hm = smy[2][ly + 1];
            } else {
                const int t2 = task();
                y = t2 >= T::F2X;
                const int c = t2 - T::F2X;
                b = y ? (TY + 1) * HX + c + 2 : (t2 + 2) * HX + TX + 1;
                sb = y ? NXS + TY * TX + c : t2 * XS + TX;
                fo = y ? NT + c : sb + 1;
                hp = y ? smy[1][TY] : smx[1][TX];
                hm = y ? smy[2][TY + 1] : smx[2][TX + 1];
            }
            const int qst = y ? HX : 1, sst = y ? TX : 1;
            R qb[4], qc[4], slb[4], slc[4], fl[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                qb[v] = sqf[v * QS + b];
                qc[v] = sqf[v * QS + b + qst];
                slb[v] = ss[v][sb];
                slc[v] = LIMO3 ? ssl[v][sb + sst] : ss[v][sb + sst];
            }
            face_flux_s<R>(p == 2 ? int(y) : p, qb, qc, slb, slc, centre(b), centre(b + qst), hp, hm,
                           depth(b) + depth(b + qst), fl, recon, riemann);
            // a lane's x flux takes the slot its left neighbour read as slc
            // (with LimO3 slc is in an array of its own): every lane's reads
            // come before any lane's stores
            if (p == 0 && !LIMO3) {
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                __builtin_amdgcn_wave_barrier();
            }
            R *dst = y ? &sfy[0][0][0] : &ss[0][0];
            const int fs = y ? (TY + 1) * TX : NXS + NYS;
#pragma unroll
            for (int v = 0; v < 4; ++v) dst[v * fs + fo] = fl[v];
        }

        // z face above the plane from the register window
        if constexpr (NDIM == 3) {
            Cb = centre_of(Wb);
            face_flux_s<R>(2, Wa, Wb, Sa, LIMO3 ? Sl : Sb, Ca, Cb, hpz[k + 2], hmz[k + 3], Ta + Tb, Fb, recon, riemann);
        }
        // The empty statement hides that the cell's index is the same in every
        // plane: the compiler otherwise hoists a 64-bit lane address for each
        // of the cell's arrays out of the loop and spills.
        unsigned cell = unsigned(col);
        asm("" : "+v"(cell));
        const long base = long(k) * plane;
        typename Fin::In in;
        if (live) fin.load(base, cell, in);
        __syncthreads();

        if (live) {
            R acc[4], Us[4];
            const int xr = xs + 1 + (lx == TX - 1);      // slot of the flux right of the cell
            const R axl = sux[0][lx];
            const R tr1 = GEOM == M1_CARTESIAN ? dtc : sux[1][lx];
            const R ayl = suy[0][ly] * tr1;
            const R tr2 = GEOM == M1_SPHERICAL ? suy[1][ly] * tr1 : dtc;
            const R azl = NDIM == 3 ? a.m.alo[2][k] * tr2 : R(0);
            const R ct = GEOM == M1_SPHERICAL ? suy[2][ly] : R(0);
            const R dax = area_step<GEOM, 0>(tr1, ct), day = area_step<GEOM, 1>(tr1, ct);
#pragma unroll
            for (int v = 0; v < 4; ++v)
                acc[v] = face_diff<GEOM, 0>(axl, dax, ss[v][xs], ss[v][xr]) +
                         face_diff<GEOM, 1>(ayl, day, sfy[v][ly][lx], sfy[v][ly + 1][lx]) +
                         (NDIM == 3 ? face_diff<GEOM, 2>(azl, R(0), Fa[v], Fb[v]) : R(0));
            if (NDIM == 2 && a.ign[2]) ignorable_div<R, 2>(a, Wa, Ca, tr2, acc);
            finish_cell<R, GEOM>(a, Wa, Ca, acc, tr1, ct, Us);
            fin(in, Us, Ta, i, j, k, base, cell);
        }
    };
    if constexpr (NDIM == 2) {
        R Wn[4], Tn;
        step(0, W0, W1, Wn, Fz0, Fz1, Sz0, Sz1, C0, C1, T0, T1, Tn);
        return;
    }
    for (int k = z0; k < z1; ++k) {
        R Wn[4], Tn;
        step(k, W0, W1, Wn, Fz0, Fz1, Sz0, Sz1, C0, C1, T0, T1, Tn);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            Fz0[v] = Fz1[v];
            Sz0[v] = Sz1[v];
            W0[v] = W1[v];
            W1[v] = Wn[v];
        }
        C0 = C1;
        T0 = T1;
        T1 = Tn;
    }
}

// ---------------------------------------------------------------------------
// launch shape and arguments
// ---------------------------------------------------------------------------

// Blocks of a kernel the whole device holds at once (occupancy per compute
// unit times the compute units), cached per kernel and device in a fixed
// table (no heap allocation on any launch path; a full table just stops
// caching).
inline int resident_blocks(const void *kern, int block)
{
    struct Entry {
        const void *kern;
        int dev, block, blocks;
    };
    static std::mutex mu;
    static Entry cache[256];
    static int used = 0;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 1024;
    std::lock_guard<std::mutex> lock(mu);
    for (int e = 0; e < used; ++e)
        if (cache[e].kern == kern && cache[e].dev == dev && cache[e].block == block) return cache[e].blocks;
    int cus = 0, per = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1) cus = 256;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, kern, block, 0) != hipSuccess || per < 1) per = 1;
    if (used < 256) cache[used++] = Entry{kern, dev, block, per * cus};
    return per * cus;
}

// Shape of a tiled 3D launch.  The planes per block (z chunk) minimise rounds x
// (planes + 1): blocks run in rounds of the resident block count, and each
// chunk also pays about one plane of start-up (its first z face and slopes),
// so a chunk that fills the last round evenly beats one that leaves a
// mostly idle tail.  Chunks are kept to at most 16 planes: measured over the
// 128^3, 256^3, 192x96x192 and eight-group workloads (chunks of 4 to 64
// planes), the 28-64-plane chunks this cost picks without the cap were 4-6 %
// slower than 16 (fewer blocks to balance, more halo misses in L2); with the
// cap it lands on the fastest chunk measured or within 3 % of it.
struct TileShape {
    int tiles_x, tiles_y, nz, nblocks, launched;
    long rounds;
};
template <int TYB>
inline TileShape tile_shape(const m1_ctx *c, const void *kern, unsigned ngrp)
{
    using T = Tile<TYB>;
    TileShape s;
    s.tiles_x = (c->n[0] + T::TX - 1) / T::TX;
    s.tiles_y = (c->n[1] + T::TY - 1) / T::TY;
    const long slots = resident_blocks(kern, T::NT);
    double best = 1e300;
    s.nz = 8;
    s.rounds = 1;
    for (int z = 2; z <= 16; ++z) {
        const long nb = long(s.tiles_x) * s.tiles_y * ((c->n[2] + z - 1) / z) * ngrp;
        const long r = (nb + slots - 1) / slots;
        const double cost = double(r) * (z + 1);
        if (cost < best) {
            best = cost;
            s.nz = z;
            s.rounds = r;
        }
    }
    s.nblocks = s.tiles_x * s.tiles_y * ((c->n[2] + s.nz - 1) / s.nz);
    s.launched = ((s.nblocks + 7) / 8) * 8;
    return s;
}

// 2D: one 32 x 8 tile a block.
inline TileShape tile_shape_2d(const m1_ctx *c)
{
    using T = Tile<8>;
    TileShape s;
    s.tiles_x = (c->n[0] + T::TX - 1) / T::TX;
    s.tiles_y = (c->n[1] + T::TY - 1) / T::TY;
    s.nz = 1;
    s.rounds = 0;
    s.nblocks = s.tiles_x * s.tiles_y;
    s.launched = ((s.nblocks + 7) / 8) * 8;
    return s;
}

// Whether a 2D grid takes the tiles: where more than half of their threads own
// a cell.  A tile computes each face and slope once (a thread per cell computes
// two faces and three slopes per direction), so the sides meet at half its
// threads idle.  Transport, a thread per cell -> tiles, FP32 and FP64: 20 x
// 200,000 cells (0.63 of the threads) 115 -> 91 and 258 -> 224 us, 16 x 200,000
// (0.5) 93 -> 91 and 199 -> 214 us, 200,000 x 3 (0.38) 22 -> 25 and 45 -> 56 us.
inline bool tiled_2d(const m1_ctx *c)
{
    if (c->ndim != 2) return false;
    const TileShape s = tile_shape_2d(c);
    return 2.0 * c->n[0] * c->n[1] > 256.0 * s.tiles_x * s.tiles_y;
}

// Transport arguments for the radiation arrays rad (the bound state's if null)
// and the optical depths tau.  Group arrays of the caller start at
// g n0 n1 n2; the scratch arrays are laid out per group (transported fields
// 4 g + v, optical depth of group g).
template <typename R>
inline void fill_targs(m1_ctx *c, TArgs<R> &a, const Metric<R> &met, double dt, const void *const rad[4],
                       const void *tau)
{
    const long N = long(c->n[0]) * c->n[1] * c->n[2];
    a.out = static_cast<R *>(c->star[0]);
    a.out_fs = long(c->plane_bytes / sizeof(R));
    const void *src[4] = {c->f.E, c->f.Fx, c->f.Fy, c->f.Fz};
    for (int v = 0; v < 4; ++v) a.U[v] = static_cast<const R *>(rad ? rad[v] : src[v]);
    a.tau = static_cast<const R *>(tau);
    a.gs_in = N;
    a.gs_out = long(4 * c->plane_bytes / sizeof(R));
    a.gs_tau = long(c->plane_bytes / sizeof(R));
    for (int d = 0; d < 3; ++d) {
        a.n[d] = c->n[d];
        a.bc[d][0] = c->bc[d][0];
        a.bc[d][1] = c->bc[d][1];
        a.ign[d] = c->ign[d];
    }
    a.m = met;
    a.dt = R(dt);
    a.c_hat = R(c->c_hat);
    a.e_floor = R(c->par.e_floor);
    a.recon = c->par.recon;
    a.riemann = c->par.riemann;
    a.limo3 = c->par.limiter == M1_LIMITER_LIMO3;
    a.special = 0;
    for (int d = 0; d < 3; ++d)
        for (int sd = 0; sd < 2; ++sd) {
            if (c->bc[d][sd] == M1_BC_REFLECT || c->bc[d][sd] == M1_BC_FIXED) a.special = 1;
            for (int v = 0; v < 4; ++v) a.bcs[d][sd][v] = R(c->bc_state[d][sd][v]);
        }
    a.cnt = c->cnt;
}

// whether the run needs the general tiled kernel (face treatment, Riemann
// solver, ghost states)
template <typename R>
inline bool general_transport(const m1_ctx *c, const TArgs<R> &a)
{
    return c->par.recon != M1_RECON_FPRESERVE || c->par.riemann != M1_RIEMANN_HLL || a.special;
}

} // namespace m1
