// transport.hip -- explicit M1 transport step on gfx950.
//
// One Euler stage of the hyperbolic part (Sect. 2.4-2.6): boundary values
// by index mapping in the loader (periodic wrap / outflow copy), PLM van
// Leer reconstruction of (E, F) on faces with the f-preserving fix, the
// Levermore closure and signal speeds of both face states, the HLL flux with
// the optical-depth limiter, and the conservative update with the geometric
// sources of the flux equation in cylindrical / spherical coordinates.
#include "transport_tile.h"

namespace m1 {

template <typename R, int NDIM, int GEOM>
__global__ void __launch_bounds__(256) k_transport(TArgs<R> a)
{
    select_group(a);
    transport_cell<R, NDIM, GEOM>(a, StoreCell<R>{a.out, a.out_fs});
}

// FP32 instantiations ask for four waves per SIMD (the second argument of the
// bound), i.e. at most 128 VGPRs; the FP64 ones for three (default, at most 168)
// and two (general, at most 256).
// LIMO3 (general kernel only): each donor cell keeps two slopes per
// direction, one for its lower and one for its upper face, and takes the
// 32 x 8 tile in FP64 (the 512-thread block spilled).
//
// What bounds it: vector issue, in FP32 (about 640 instructions a cell, 57 of
// them transcendental at two slots and a third; 80 % of the cycles issue on the
// 192x96x192 grid, the rest is ramp, tail and barriers) and in FP64 (about 970,
// 69 % of the cycles).  A step of the 128^3 box went from 99 to 92.9 us (FP32) and
// 176 to 153.8 us (FP64) with the closure without 1 / |F|^2, the face fix on
// f^2 and the regrouped Riemann flux of m1_device.h, on to 88.5 and 143.5 us
// with one spacing factor per slope, dt c_hat in the area factors, one code
// block for the first two task passes and the halo loaded a plane ahead, and
// to 86.5 and 140 us with tasks at fixed offsets of the thread's own cell, the
// metric and update factors in LDS and the x fluxes in the slopes' place
// (fewer registers and 13 % less LDS: three waves per SIMD in FP64, four in
// the general FP32 kernels); 192x96x192 with the table in FP64 330 -> 290 -> 270
// us and, the last step on another card, 262 -> 251 us; eight groups on the
// 128^3 box 536 -> 495 -> 460 us and 467 -> 462 us; the transport of the FP32
// box with a lit and a mirror side 55.4 -> 48.3 us in the last step.  Tried and not kept: two or
// three planes per turn of the loop (no register moves; the FP32 kernels
// spilled and ran 15 % slower, FP64 was equal); scalar bases with a 32-bit lane
// offset for the plane loads and stores (4 % slower); selects in place of the
// branches of the face fix and the Riemann flux (equal); five waves per SIMD
// in FP32 (2 % faster on 256^3, 7 % slower on 128^3, a few spills); scheduling
// barriers between the directions (2 % slower in FP64).
template <typename R, int GEOM, bool GENERAL, int TYB, bool LIMO3 = false>
__global__ void __launch_bounds__((Tile<TYB>::NT),
                                  (sizeof(R) == 4 ? 4 : (GENERAL ? 2 : 3)))
    k_transport3d(TArgs<R> a, int nz_chunk, int tiles_x, int tiles_y, int nblocks, int cus)
{
    select_group(a);
    transport_tile<R, 3, GEOM, GENERAL, TYB, LIMO3>(a, nz_chunk, tiles_x, tiles_y, nblocks, cus, StoreCell<R>{a.out, a.out_fs});
}

// 2D: one 32 x 8 tile a block.  What bounds it: the chain load - slopes - faces -
// update behind three barriers, which the six FP32 blocks on a compute unit overlap in
// part (1000^2 cells: 18-20 us, where a large copy takes 7.5 us for their 36 bytes a
// cell); in FP64 that chain and issue, three blocks on a unit (52.6 KB of LDS
// each).  Against a thread per cell, which computed every
// face twice and every slope three times: 1000^2 cells FP32 30.3 -> 18.4 us, FP64
// 66.6 -> 38 us, LimO3 FP32 33.1 -> 25.9 us; 300 x 200 FP32 6.1 -> 5.3 us, FP64
// 7.8 -> 6.3 us.
template <typename R, int GEOM, bool GENERAL, bool LIMO3>
__global__ void __launch_bounds__(256, (sizeof(R) == 4 ? 4 : (LIMO3 ? 2 : 3)))
    k_transport2d(TArgs<R> a, int tiles_x, int tiles_y, int nblocks)
{
    select_group(a);
    transport_tile<R, 2, GEOM, GENERAL, 8, LIMO3>(a, 1, tiles_x, tiles_y, nblocks, 1, StoreCell<R>{a.out, a.out_fs});
}

// Launch with tile height TYB; with max_rounds > 0, only if the launch then
// takes at most that many rounds of resident blocks (returns whether it
// launched).
template <typename R, int GEOM, bool GENERAL, int TYB, bool LIMO3 = false>
static bool launch_tile(m1_ctx *c, const TArgs<R> &a, unsigned ngrp, long max_rounds)
{
    const TileShape s =
        tile_shape<TYB>(c, reinterpret_cast<const void *>(&k_transport3d<R, GEOM, GENERAL, TYB, LIMO3>), ngrp);
    if (max_rounds > 0 && s.rounds > max_rounds) return false;
    hipLaunchKernelGGL((k_transport3d<R, GEOM, GENERAL, TYB, LIMO3>), dim3(s.launched, ngrp), dim3(Tile<TYB>::NT), 0,
                       c->stream, a, s.nz, s.tiles_x, s.tiles_y, s.nblocks, c->cus);
    return true;
}

// Default FP32 kernel: the 32 x 16 tile where its launch takes at most two
// rounds of resident blocks (the 192x96x192 and 128^3 grids: 1.5 % faster
// transport than 32 x 8), else 32 x 8 (on the 256^3 grid and eight groups
// at 128^3, launches of four to sixteen rounds, the taller blocks were
// 2-4 % slower).  FP64 takes 32 x 8 everywhere (three blocks share a compute
// unit; two sharing one beat one 32 x 16 block by 1-1.5 %).
template <typename R, int GEOM, bool GENERAL, bool LIMO3 = false>
static void launch_tiled(m1_ctx *c, const TArgs<R> &a, unsigned ngrp)
{
    if constexpr (sizeof(R) == 4 && !GENERAL && !LIMO3) {
        if (launch_tile<R, GEOM, GENERAL, 16, LIMO3>(c, a, ngrp, 2)) return;
    }
    launch_tile<R, GEOM, GENERAL, 8, LIMO3>(c, a, ngrp, 0);
}

// One transport launch for every frequency group (grid y = group; one group
// for gray states).
template <typename R>
static hipError_t launch_t(m1_ctx *c, double dt, const Metric<R> &met, const void *const rad[4] = nullptr)
{
    TArgs<R> a;
    fill_targs(c, a, met, dt, rad, c->tau);
    const long N = long(c->n[0]) * c->n[1] * c->n[2];
    const unsigned ngrp = unsigned(c->grp.m);
    if (c->ndim == 3) {
        const bool var = general_transport(c, a);
#define M1_T3D(GM, V, L) launch_tiled<R, GM, V, L>(c, a, ngrp)
#define M1_T3D_ANY(GM)                  \
    if (a.limo3) M1_T3D(GM, true, true);  \
    else if (var) M1_T3D(GM, true, false); \
    else M1_T3D(GM, false, false)
        switch (c->geom) {
        case M1_CARTESIAN: M1_T3D_ANY(M1_CARTESIAN); break;
        case M1_CYLINDRICAL: M1_T3D_ANY(M1_CYLINDRICAL); break;
        default: M1_T3D_ANY(M1_SPHERICAL); break;
        }
#undef M1_T3D_ANY
#undef M1_T3D
        return hipGetLastError();
    }
    if (tiled_2d(c)) {
        const bool var = general_transport(c, a);
        const TileShape s = tile_shape_2d(c);
#define M1_T2D(GM, V, L) \
    hipLaunchKernelGGL((k_transport2d<R, GM, V, L>), dim3(s.launched, ngrp), dim3(256), 0, c->stream, a, s.tiles_x, s.tiles_y, s.nblocks)
#define M1_T2D_ANY(GM)                  \
    if (a.limo3) M1_T2D(GM, true, true);  \
    else if (var) M1_T2D(GM, true, false); \
    else M1_T2D(GM, false, false)
        switch (c->geom) {
        case M1_CARTESIAN: M1_T2D_ANY(M1_CARTESIAN); break;
        case M1_CYLINDRICAL: M1_T2D_ANY(M1_CYLINDRICAL); break;
        default: M1_T2D_ANY(M1_SPHERICAL); break;
        }
#undef M1_T2D_ANY
#undef M1_T2D
        return hipGetLastError();
    }
    dim3 block(256), grid(unsigned((N + 255) / 256), ngrp);
#define M1_LAUNCH(ND, G) \
    hipLaunchKernelGGL((k_transport<R, ND, G>), grid, block, 0, c->stream, a)
#define M1_GEOMS(ND)                                                      \
    switch (c->geom) {                                                    \
    case M1_CARTESIAN: M1_LAUNCH(ND, M1_CARTESIAN); break;                \
    case M1_CYLINDRICAL: M1_LAUNCH(ND, M1_CYLINDRICAL); break;            \
    default: M1_LAUNCH(ND, M1_SPHERICAL); break;                          \
    }
    if (c->ndim == 1) {
        M1_GEOMS(1);
    } else {
        M1_GEOMS(2);
    }
#undef M1_GEOMS
#undef M1_LAUNCH
    return hipGetLastError();
}

hipError_t launch_transport(m1_ctx *c, double dt)
{
    if (c->par.precision == M1_F32) return launch_t<float>(c, dt, c->met32);
    return launch_t<double>(c, dt, c->met64);
}

// transport of a state held elsewhere (the second-order step's U1)
hipError_t launch_transport_from(m1_ctx *c, double dt, const void *const rad[4])
{
    if (c->par.precision == M1_F32) return launch_t<float>(c, dt, c->met32, rad);
    return launch_t<double>(c, dt, c->met64, rad);
}

} // namespace m1
