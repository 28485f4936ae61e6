// stage.hip -- the fused stages of the second-order step: transport and
// implicit step of a cell in one kernel.
//
// m1_step_rk2 runs U1 = S(T(U^n)), U2 = S(T(U1)) and writes (U^n + U2) / 2.  Both
// stages write elsewhere than where their transport reads its neighbours (U1
// to the library's buffer, the average to the bound arrays while the second
// transport reads U1), so the implicit step can take the transported cell from
// registers: the four transported fields are neither written nor read back
// (64 of 328 bytes a cell and step in FP32, 128 of 480 in FP64, with constant
// opacities), and the
// implicit step's loads overlap the transport's arithmetic.  Where opacities
// depend on temperature a stage writes the optical depths of its new state to
// another array than the one neighbouring cells still read: stage 1 to the
// first transported field (unused here), stage 2 back to the cache.
//
// What bounds it: vector issue in 3D (transport and solve are about 800 FP32
// operations a cell and stage), where the split step alternated between an
// issue-bound and a memory-bound kernel.  A second-order step, split -> fused:
// 256^3 FP32 1363 -> 1025 us, 128^3 FP32 166 -> 114 us and FP64 304 -> 220 us,
// 192x96x192 FP32 298 -> 241 us (constant opacities) and 310 -> 289 us (table),
// 128^3 FP32 power law 185 -> 147 us, 1D 2000 cells FP64 17.3 -> 13.3 us, 2D 1000^2 FP64
// 187 -> 153 us and in tiles 92 us, 300x200 shell with the table, FP32, 24.0 ->
// 19.8 and in tiles 16.7 us, 300^2 beam with LimO3 in FP64 38 -> 33 -> 24.8 us.
//
// Covers gray states with constant, power-law and tabulated opacities, in 1D
// and 2D with every variant, in 3D with the default scheme and, in FP64 with
// temperature-dependent opacities, up to FUSED_P64_CELLS.  The split kernels
// stay for the network (a wavefront-wide product with its own registers and
// LDS), frequency groups (the solve needs every group of a cell) and the
// general 3D kernels (at the edge of their registers).
#include "transport_tile.h"
#include "implicit_device.h"

namespace m1 {

// Argument of a fused stage.  The implicit step's two dozen array pointers and
// two dozen constants are read where they are used (first_argument).
template <typename R>
struct StageArgs {
    TArgs<R> t;
    IArgs<R> i;
    int nt;                       // stream the inputs past the caches
    int nz_chunk, tiles_x, tiles_y, nblocks, cus;
};

template <typename R, bool CONST_OPAC>
struct SolveCell {
    using In = CellIn<R>;
    __device__ __forceinline__ void load(long base, unsigned c, In &in) const
    {
        const StageArgs<R> &sa = first_argument<StageArgs<R>>();
        const IArgs<R> &ia = sa.i;
        if (sa.nt)
            load_cell<CONST_OPAC, true>(ia, base, c, in);
        else
            load_cell<CONST_OPAC, false>(ia, base, c, in);
    }
    __device__ __forceinline__ void operator()(In &in, const R Us[4], R tau, int i, int j, int k, long base,
                                               unsigned c) const
    {
        const IArgs<R> &ia = first_argument<StageArgs<R>>().i;
        const R hm = CONST_OPAC ? R(0) : cell_hmax(ia.m, ia.ndim, i, j, k);
        in.tau = tau;
        const double T1 = solve_cell<R, CONST_OPAC, false>(ia, base, c, hm, in, Us[0], Us + 1);
        if (!CONST_OPAC) {
            const R rho = R(in.rho);
            R kP, kR;
            if (ia.op.kind == OPK_POWERLAW)
                opacity_analytic<R, OPK_POWERLAW>(ia.op, rho, R(T1), kP, kR);
            else
                opacity_analytic<R, OPK_TABLE>(ia.op, rho, R(T1), kP, kR);
            cache_entry(rho, kP, kR, R(ia.op.sigma), hm, at(ia.rkp, base, c), at(ia.tau, base, c));
        }
    }
};

template <typename R, int NDIM, int GEOM, bool CONST_OPAC>
__global__ void __launch_bounds__(256) k_stage(StageArgs<R> a)
{
    transport_cell<R, NDIM, GEOM>(a.t, SolveCell<R, CONST_OPAC>{});
}

template <typename R, int GEOM, int TYB, bool CONST_OPAC>
__global__ void __launch_bounds__((Tile<TYB>::NT), (sizeof(R) == 4 ? 4 : (CONST_OPAC ? 3 : 2))) k_stage3d(StageArgs<R> a)
{
    transport_tile<R, 3, GEOM, false, TYB, false>(a.t, a.nz_chunk, a.tiles_x, a.tiles_y, a.nblocks, a.cus,
                                               SolveCell<R, CONST_OPAC>{});
}

template <typename R, int GEOM, bool GENERAL, bool LIMO3, bool CONST_OPAC>
__global__ void __launch_bounds__(256, (sizeof(R) == 4 ? 4 : 2)) k_stage2d(StageArgs<R> a)
{
    transport_tile<R, 2, GEOM, GENERAL, 8, LIMO3>(a.t, 1, a.tiles_x, a.tiles_y, a.nblocks, 1, SolveCell<R, CONST_OPAC>{});
}

template <typename R, int GEOM, int TYB, bool CONST_OPAC>
static bool launch_tile(m1_ctx *c, StageArgs<R> &a, long max_rounds)
{
    const TileShape s = tile_shape<TYB>(c, reinterpret_cast<const void *>(&k_stage3d<R, GEOM, TYB, CONST_OPAC>), 1);
    if (max_rounds > 0 && s.rounds > max_rounds) return false;
    a.nz_chunk = s.nz;
    a.tiles_x = s.tiles_x;
    a.tiles_y = s.tiles_y;
    a.nblocks = s.nblocks;
    hipLaunchKernelGGL((k_stage3d<R, GEOM, TYB, CONST_OPAC>), dim3(s.launched), dim3(Tile<TYB>::NT), 0, c->stream, a);
    return true;
}

template <typename R, int GEOM, bool CONST_OPAC>
static void launch_geom(m1_ctx *c, StageArgs<R> &a)
{
    if (c->ndim == 3) {
        if constexpr (sizeof(R) == 4) {
            if (launch_tile<R, GEOM, 16, CONST_OPAC>(c, a, 2)) return;
        }
        launch_tile<R, GEOM, 8, CONST_OPAC>(c, a, 0);
        return;
    }
    if (tiled_2d(c)) {
        const TileShape s = tile_shape_2d(c);
        a.tiles_x = s.tiles_x;
        a.tiles_y = s.tiles_y;
        a.nblocks = s.nblocks;
        const dim3 grid(s.launched), block(256);
        if (a.t.limo3)
            hipLaunchKernelGGL((k_stage2d<R, GEOM, true, true, CONST_OPAC>), grid, block, 0, c->stream, a);
        else if (general_transport(c, a.t))
            hipLaunchKernelGGL((k_stage2d<R, GEOM, true, false, CONST_OPAC>), grid, block, 0, c->stream, a);
        else
            hipLaunchKernelGGL((k_stage2d<R, GEOM, false, false, CONST_OPAC>), grid, block, 0, c->stream, a);
        return;
    }
    const long N = long(c->n[0]) * c->n[1];
    const dim3 grid(unsigned((N + 255) / 256)), block(256);
    if (c->ndim == 1)
        hipLaunchKernelGGL((k_stage<R, 1, GEOM, CONST_OPAC>), grid, block, 0, c->stream, a);
    else
        hipLaunchKernelGGL((k_stage<R, 2, GEOM, CONST_OPAC>), grid, block, 0, c->stream, a);
}

template <typename R>
static hipError_t launch_s(m1_ctx *c, double dt, const Metric<R> &met, int stage)
{
    const bool con = c->op.kind == OPK_CONST;
    StageArgs<R> a;
    fill_args(c, a.i, met, dt);
    rk2_stage_args(c, a.i, stage);
    // optical depths: stage 1 reads the cache and writes the spare array,
    // stage 2 the other way round (constant opacities: only read)
    R *const cache = static_cast<R *>(c->tau), *const spare = static_cast<R *>(c->star[0]);
    a.i.tau = stage == 1 ? spare : cache;
    const R *const tau_in = con || stage == 1 ? cache : spare;
    const unsigned char *sv = static_cast<const unsigned char *>(c->rk2_save);
    const size_t per = c->rk2_rad_bytes;
    const void *const u1[4] = {sv, sv + per, sv + 2 * per, sv + 3 * per};
    fill_targs(c, a.t, met, dt, stage == 1 ? nullptr : u1, tau_in);
    a.cus = c->cus;
    // A stage's own inputs (the gas and the opacity cache) are streamed past the caches only
    // where the caller asks for it: its reads wait behind issue, not behind
    // memory.  A step with streaming reads and without: 128^3 118.0 and 117.2 us,
    // 192^3 510.6 and 510.7, 256^3 1060 and 1047 (FP32, constant opacities);
    // 160x144x128 323.8 and 322.7, 192^3 737 and 739 (FP64); 192x96x192 290 and
    // 289, 256x192x192 750 and 741 (FP32, table).
    a.nt = c->par.stream_reads == M1_STREAM_ON;
#define M1_STAGE(G)                                  \
    if (con) launch_geom<R, G, true>(c, a);           \
    else launch_geom<R, G, false>(c, a)
    switch (c->geom) {
    case M1_CARTESIAN: M1_STAGE(M1_CARTESIAN); break;
    case M1_CYLINDRICAL: M1_STAGE(M1_CYLINDRICAL); break;
    default: M1_STAGE(M1_SPHERICAL); break;
    }
#undef M1_STAGE
    return hipGetLastError();
}

// Temperature-dependent opacities in 3D in FP64 step split above half a million
// cells.  The line was drawn with the fused kernel at two waves per SIMD, where the
// logarithms, powers and exponentials (about 250 FP64 operations a cell) cost more
// than the transported state's way through memory.  At today's three waves the
// fused stages are shorter on either side of it (split, fused: 154,000 cells, power
// law, 53.7 and 47.2 us; 885,000 151.6 and 132.7; 128^3 330 and 296; 192x96x192
// with the table 536 and 486); the split step stays above it because it stores the
// transported state, which m1_transported then answers.
constexpr long FUSED_P64_CELLS = 1L << 19;

bool fused_stages(const m1_ctx *c)
{
    if (c->grp.m > 1 || c->op.kind == OPK_MLP) return false;
    if (c->ndim < 3) return true;
    if (c->op.kind != OPK_CONST && c->par.precision == M1_P64 &&
        long(c->n[0]) * c->n[1] * c->n[2] > FUSED_P64_CELLS)
        return false;
    bool special = false;
    for (int d = 0; d < 3; ++d)
        for (int s = 0; s < 2; ++s)
            special = special || c->bc[d][s] == M1_BC_REFLECT || c->bc[d][s] == M1_BC_FIXED;
    return c->par.limiter == M1_LIMITER_PLM && c->par.recon == M1_RECON_FPRESERVE &&
           c->par.riemann == M1_RIEMANN_HLL && !special;
}

hipError_t launch_stage(m1_ctx *c, double dt, int stage)
{
    if (c->par.precision == M1_F32) return launch_s<float>(c, dt, c->met32, stage);
    return launch_s<double>(c, dt, c->met64, stage);
}

} // namespace m1
