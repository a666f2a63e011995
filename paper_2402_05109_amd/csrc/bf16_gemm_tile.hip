// bf16 storage family: shapes, planning and launches of the many-rows GEMM (kernel in gemm_tile.h).
#include <stdlib.h>

#include <hip/hip_ext.h>

#include <algorithm>
#include <cmath>
#include <type_traits>

#include "gemm_epilogues.h"
#include "gemm_tile.h"
#include "internal.h"

namespace hydra {

// The tiles that are built.  Eight waves (two per SIMD) where the tile divides among them, four otherwise.  What each is for:
//   256 x 192, 256 x 256  wide matrices at many rows
//   256 x 160  one group of 256 rows against a wide matrix: as many columns as 256 CUs can take in one round
//   256 x 128  d-wide matrices from 160 rows on, K split two to eight ways
//   128 x 192, 128 x 128, 128 x 96  up to 128 rows and small matrices, K split over workgroups
// `eff` is the time per multiplication relative to 256 x 192 (smaller tiles read more of LDS per multiplication).
enum { TILE_NONE = 0, TILE_256x256, TILE_256x192, TILE_256x160, TILE_256x128, TILE_128x192, TILE_128x128, TILE_128x96, TILE_COUNT };
typedef TileShape<4, 2, 2, 4, 4> Tile256x256;
typedef TileShape<4, 2, 2, 3, 5> Tile256x192;
typedef TileShape<4, 1, 2, 5, 5> Tile256x160;
typedef TileShape<4, 2, 2, 2, 6> Tile256x128;
typedef TileShape<4, 2, 1, 3, 7> Tile128x192;
typedef TileShape<4, 2, 1, 2, 8> Tile128x128;
typedef TileShape<4, 1, 1, 3, 10> Tile128x96;
struct TileInfo { int rows, cols, slots; double eff; };
template <class S> static constexpr TileInfo tile_of(double eff) { return TileInfo{32 * S::XB, 32 * S::WB, S::SLOTS, eff}; }
static TileInfo tile_info(int id) {
    switch (id) {
        case TILE_256x256: return tile_of<Tile256x256>(0.99);
        case TILE_256x192: return tile_of<Tile256x192>(1.0);
        case TILE_256x160: return tile_of<Tile256x160>(1.11);
        case TILE_256x128: return tile_of<Tile256x128>(1.03);
        case TILE_128x192: return tile_of<Tile128x192>(1.17);
        case TILE_128x128: return tile_of<Tile128x128>(1.27);
        default:           return tile_of<Tile128x96>(1.33);
    }
}

// The cheapest tile and K split for an M x N x K product; false where none applies.  `forced` (tests): HYDRA_PLAN_TILE_ID names
// the tile and HYDRA_PLAN_TILE_SPLITS the K splits of plain outputs, and a product that cannot have them gets a plan that
// launch_tile refuses, never another one; splits of a residual's product are then always taken, and whole K never instead of
// the fused epilogue.
//
// The estimate was fitted to 3658 timings (14 matrices of the 7B, 13B-like, 33B and a 2048-wide shape, 72 to 1024 rows, all
// tiles, 1 to 8 splits; 7 % root mean square error, the tile it picks is 1.4 % off the best on average).  A workgroup's
// k-step takes its multiplications at the CU's share of 1200 TFLOP/s (at most 6 per CU) and its operands at 86 GB/s (107
// where several row groups share the weights in L2), combined as the cube root of the cubes' sum because the two overlap in
// part; rounds of 256 workgroups follow one another; the weights need HBM at 5.3 TB/s; and the output is written at 4.3 TB/s
// once per split.  Splits are chosen with the consumer's reading of the partial sums (5 TB/s) in mind, which is not part
// of cost_us.
bool plan_tile(int M, int N, int K, int kind, bool forced, GemmPlan *p) {
    const bool may_split = kind == GEMM_KIND_PLAIN;
    const int KT = K / 16, bands = ceil_div(N, 32);
    // up to 64 rows the register-streaming kernels win: at 72 rows this one takes 23.1 against 29.9 us (12288 x 4096), at 64
    // those take 24.9 with the epilogue fused
    if (M <= 64 || KT % 2 != 0) return false;
    const char *only_s = forced ? getenv("HYDRA_PLAN_TILE_ID") : nullptr, *splits_s = only_s ? getenv("HYDRA_PLAN_TILE_SPLITS") : nullptr;
    const int only = only_s ? atoi(only_s) : 0, only_splits = may_split && splits_s ? atoi(splits_s) : 0;
    const double hbm = (double)N * K * 2 / 5.3e6;
    double best = 1e30;
    for (int id = TILE_256x256; id < TILE_COUNT; ++id) {
        const TileInfo ti = tile_info(id);
        if (only && id != only) continue;
        if (ti.rows == 256 && M <= 128) continue;
        const int gx = ceil_div(bands, ti.cols / 32), gz = ceil_div(M, ti.rows);
        const double by = (std::min(ti.rows, ceil_div(M, 32) * 32) + ti.cols) * 32 / (gz > 1 ? 107e3 : 86e3);
        double step_few = 0.0, step_all = 0.0;                         // a k-step with up to 200 workgroups and with 256: the same for every split
        auto step_us = [&](int active) {
            double &known = active <= 200 ? step_few : step_all;
            if ((active <= 200 || active == 256) && known > 0.0) return known;
            const double fl = 32.0 * ti.rows * ti.cols / std::min(6.0e6, 1200e6 / active);
            const double us = std::cbrt(fl * fl * fl + by * by * by);
            if (active <= 200 || active == 256) known = us;
            return us;
        };
        for (int s = 1; s <= (may_split ? 8 : 1); ++s) {
            const int kps = ceil_div(ceil_div(KT, s), 2) * 2, wgs = gx * gz * s;
            if ((s > 1 || !only) && kps < 2 * ti.slots) break;             // fewer slots than are in flight
            if (s > 1 && wgs > 640 && !only_splits) break;                 // the chip is full
            if (ceil_div(KT, kps) != s || (only_splits && s != only_splits)) continue;
            auto round_us = [&](int active) { return kps * ti.eff * step_us(active); };
            double run = (wgs >= 256 ? (wgs / 256) * round_us(256) : 0.0) + (wgs % 256 ? round_us(wgs % 256) : 0.0);
            run = std::sqrt(std::sqrt(run * run * run * run + hbm * hbm * hbm * hbm));
            const double out = (double)M * N * (may_split ? 4.0 * s : 2.0);
            const double cost = 2.8 + run + out / 4.3e6 + (may_split ? 0.0 : 2.0);
            const double read = s > 1 ? out / 5e6 : 0.0;
            if (cost + read < best) {
                best = cost + read;
                p->tile = id; p->splits = s; p->kpw = kps; p->cost_us = (float)cost;
                p->mb = ti.rows / 32; p->nt = ti.cols / 32; p->nw = 1; p->kw = 1; p->shared_x = 0;
            }
        }
    }
    if (only) {
        if (best == 1e30) *p = GemmPlan{8, 1, 1, 1, 1, 0, 0, only, 0.f};       // kpw = 0
        else if (may_split) p->cost_us = p->splits > 1 ? 0.f : 1e6f;
        return true;
    }
    return best < 1e30;
}

template <class S, class Epi>
static void launch_shape(dim3 grid, hipStream_t s, const GemmGeom &g, const Epi &epi, hipEvent_t e0, hipEvent_t e1) {
    if (e0) hipExtLaunchKernelGGL((gemm_tile_kernel<S, Epi>), grid, dim3(S::WAVES * 64), S::LDS, s, e0, e1, 0, GEMM_GEOM_ARGS(g), epi);
    else    hipLaunchKernelGGL((gemm_tile_kernel<S, Epi>), grid, dim3(S::WAVES * 64), S::LDS, s, GEMM_GEOM_ARGS(g), epi);
}

// 128 x 128: does the kernel of bf16_gemm_halves.hip take it?  Where the reads of LDS are the bound: from three row groups on, with
// enough workgroups that the chip is busy.  Both kernels over 2048 to 6656 columns, K from 1024 to 17920, 160 to 1024 rows (us):
//   three and more row groups, 192 workgroups and more   1.5 to 15 % faster (4096 x 11008, 1024 rows 124.8 -> 116.4; 2048 x 5504, 384 rows
//                                                        17.8 -> 17.0; 5120 x 17920, 288 rows 26.5 -> 25.7), 3 % slower at worst (4096 x 4096,
//                                                        384 rows 23.7 -> 24.4)
//   two row groups, where cold weights are the bound     1 to 20 % slower (4096 x 11008, 224 rows 32.8 -> 36.6; 6656 x 6656, 256 rows
//                                                        37.2 -> 38.6; 5120 x 5504, 224 rows 23.1 -> 24.8)
//   up to 112 workgroups                                 4 to 9 % slower (64 x 2048, 896 rows 6.0 -> 6.4)
//   K split with every CU taken                          slower (2048 x 5504, 480 rows, 4 splits 19.4 -> 22.7)
// Tests that name the tile get it for any number of row groups.
static bool takes_halves(const GemmGeom &g) {
    if (getenv("HYDRA_PLAN_TILE_ID")) return g.gz > 1;
    const int wgs = g.gx * g.gy * g.gz;
    return g.gz > 2 && wgs >= 160 && (g.gy == 1 || wgs < 256);
}

template <class Epi>
int launch_tile(hydra_ctx *c, hipStream_t s, const void *X, const void *W, int M, int N, int K, const GemmPlan &p, const Epi &epi, hipEvent_t e0,
                hipEvent_t e1) {
    if (p.tile <= TILE_NONE || p.tile >= TILE_COUNT || M < 1 || K % 32 != 0 || p.kpw < 2 || p.kpw % 2 != 0 || (p.splits > 1 && !std::is_same<Epi, EpiPlain>::value))
        return fail(HYDRA_E_UNSUPPORTED, "gemm: inconsistent tile plan");
    const TileInfo ti = tile_info(p.tile);
    GemmGeom g;
    g.X = (const u32x4_t *)X; g.W = (const u32x4_t *)W;
    g.M = M; g.NTiles = ceil_div(N, 32); g.KT = K / 16; g.kpw = p.kpw; g.NW = 1; g.KW = 1;
    g.gx = ceil_div(g.NTiles, ti.cols / 32); g.gy = p.splits; g.gz = ceil_div(M, ti.rows);
    dim3 grid(g.gx, g.gy, 1);
    if (g.gz > 1) grid = dim3((unsigned)(ceil_div(g.gx * g.gy, 8) * 8 * g.gz), 1, 1);          // see gemm_block()
    switch (p.tile) {
        case TILE_256x256: launch_shape<Tile256x256>(grid, s, g, epi, e0, e1); break;
        case TILE_256x192: launch_shape<Tile256x192>(grid, s, g, epi, e0, e1); break;
        case TILE_256x160: launch_shape<Tile256x160>(grid, s, g, epi, e0, e1); break;
        case TILE_256x128: launch_shape<Tile256x128>(grid, s, g, epi, e0, e1); break;
        case TILE_128x192: launch_shape<Tile128x192>(grid, s, g, epi, e0, e1); break;
        case TILE_128x128:
            if (takes_halves(g)) launch_tile_halves(grid, s, g, epi, e0, e1);
            else                 launch_shape<Tile128x128>(grid, s, g, epi, e0, e1);
            break;
        default:           launch_shape<Tile128x96>(grid, s, g, epi, e0, e1); break;
    }
    HYDRA_LAUNCH_CHECK("gemm_tile_kernel");
    return HYDRA_OK;
}
#define TILE_FOR(Epi) template int launch_tile<Epi>(hydra_ctx *, hipStream_t, const void *, const void *, int, int, int, const GemmPlan &, const Epi &, hipEvent_t, hipEvent_t)
TILE_FOR(EpiPlain);
TILE_FOR(EpiResidStaged);
TILE_FOR(EpiSilu);
#undef TILE_FOR

template <class S, class Epi>
static hipError_t tile_attr() { return hipFuncSetAttribute((const void *)gemm_tile_kernel<S, Epi>, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024); }
template <class Epi>
static hipError_t tile_attr_all() {
    hipError_t e = tile_attr<Tile256x256, Epi>();
    if (e == hipSuccess) e = tile_attr<Tile256x192, Epi>();
    if (e == hipSuccess) e = tile_attr<Tile256x160, Epi>();
    if (e == hipSuccess) e = tile_attr<Tile256x128, Epi>();
    if (e == hipSuccess) e = tile_attr<Tile128x192, Epi>();
    if (e == hipSuccess) e = tile_attr<Tile128x128, Epi>();
    if (e == hipSuccess) e = tile_attr<Tile128x96, Epi>();
    return e;
}
int gemm_tile_max_dynamic_lds() {
    hipError_t e = tile_attr_all<EpiPlain>();
    if (e == hipSuccess) e = tile_attr_all<EpiResidStaged>();
    if (e == hipSuccess) e = tile_attr_all<EpiSilu>();
    if (e == hipSuccess) e = tile_halves_attr();
    if (e != hipSuccess) return hip_fail(e, "hipFuncSetAttribute(gemm_tile_kernel)");
    return HYDRA_OK;
}

}  // namespace hydra
