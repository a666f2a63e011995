// The bf16-family GEMM for many rows: both operands through LDS (device code; the kernel for up to 64 rows, the operand
// tile order and the epilogue interface are in gemm_bf16.h).
//
// From about a hundred rows on, what a CU pulls per output column is the activations as much as the weights, and from a
// few hundred on the matrix cores are the limit.  Here a workgroup computes a tile of 32 MB WM rows x 32 NT WN columns
// for its whole share of K: the 1 KiB operand tiles of U k-steps at a time (a slot) are brought into LDS by the LDS DMA
// (global_load_lds, 16 bytes per lane: the tile order in memory is the order the matrix cores read, so a tile is copied
// as it lies and read back lane by lane without bank conflicts), every wave fetching an equal share, and each wave
// multiplies MB x NT of them out of LDS.  No registers hold data in flight: of a ring of up to 140 KB (five slots of 28 or ten
// of 14) all but two slots are under way in the steady state, 84 KB for 256 x 192 and 112 KB for 128 x 96, all but one at the start.
//
// One workgroup barrier per slot.  Slot j + 1 is awaited in front of the last k-step of slot j, so that the reads of its
// first k-step overlap the multiplications of that last one:
//   own DMA of slot j + 1 has landed (vmcnt), own reads of slot j - 1 are done (lgkmcnt: the reads of slot j may be under way) |
//   barrier: everybody's has and are |
//   request slot j + SLOTS - 1 into the place of slot j - 1 | read the first operands of slot j + 1 | multiply.
// Every wave issues the same number of loads per slot, past the end too (the last k-step again), so the counts that
// vmcnt waits for are exact and every wave meets the same number of barriers.
//
// Measured alone (plain output, weights of three matrices in turn; the kernels that hold operands in registers -> this one):
// 1024 x 12288 x 4096 129 -> 107 us (0.97 PFLOP/s, where the library's 8192^3 product reaches 1.13), 1024 x 22016 x 4096
// 221 -> 193, 768 x 4096 x 11008 103 -> 76, 256 x 35840 x 6656 173 -> 153, 128 x 22016 x 4096 53 -> 44, 96 x 4096 x 4096
// 15.5 -> 11.3.  Eight waves of 2 x 3 tiles and four of 4 x 3 tie; explicit scheduling barriers or groups around the LDS
// reads change nothing; three slots of four k-steps instead of six of two are 15 % slower (less in flight).
#pragma once

#include "gemm_bf16.h"

namespace hydra {

// KG: groups of WM x WN waves that take the k-steps of a slot in turn (1, or U with one k-step each)
template <int WM_, int WN_, int MB_, int NT_, int SLOTS_, int KG_ = 1>
struct TileShape {
    static constexpr int WM = WM_, WN = WN_, MB = MB_, NT = NT_, SLOTS = SLOTS_, U = 2, KG = KG_;
    static constexpr int WAVES = WM * WN * KG, XB = MB * WM, WB = NT * WN, PER_STEP = XB + WB, PER_SLOT = U * PER_STEP;
    static constexpr int SHARE = (PER_SLOT + WAVES - 1) / WAVES;                    // tiles of a slot that each wave fetches
    static constexpr int TABLE_FLOATS = 11 * GemmTile<MB, NT, XB>::ROWS;            // in front of the slots: see GemmTile
    static constexpr size_t LDS = (size_t)TABLE_FLOATS * 4 + (size_t)SLOTS * PER_SLOT * 1024;
    static_assert(KG == 1 || (KG == U && MB % KG == 0), "a group finishes its share of the row blocks");
    static_assert(KG == 1 || (size_t)WAVES * (GEMM_LDS_STAGE_WAVE * 4 + MB / KG * NT * 4096) <= (size_t)SLOTS * PER_SLOT * 1024, "LDS of the exchange");
    static_assert(SLOTS >= 3 && LDS <= 160 * 1024 && (size_t)WAVES * GEMM_LDS_STAGE_WAVE * 4 <= (size_t)SLOTS * PER_SLOT * 1024, "LDS");
};

// the 128 x 128 tile of several row groups (bf16_gemm_halves.hip)
template <class Epilogue>
void launch_tile_halves(dim3 grid, hipStream_t s, const GemmGeom &g, const Epilogue &epi, hipEvent_t e0, hipEvent_t e1);
hipError_t tile_halves_attr();

// one KiB: lane l's 16 bytes at src go to LDS byte address dst + 16 l
__device__ __forceinline__ void tile_dma(const u32x4_t *src, uint32_t dst) {
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)src,
                                     (__attribute__((address_space(3))) void *)(uintptr_t)dst, 16, 0, 0);
}
template <int N> __device__ __forceinline__ void wait_loads() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }
// and at most L reads of LDS still under way
template <int N, int L> __device__ __forceinline__ void wait_loads_and_reads() {
    static_assert(L <= 15, "the counter's range");
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(%1)" ::"n"(N), "n"(L) : "memory");
}

template <class S, class Epilogue>
__global__ __launch_bounds__(S::WAVES * 64) void gemm_tile_kernel(GEMM_GEOM_PARAMS, Epilogue epi) {
    const GemmGeom g = GEMM_GEOM_OF_PARAMS;
    static_assert(!Epilogue::PAIRED, "the waves' tiles need not hold whole band pairs");
    constexpr int MB = S::MB, NT = S::NT, XB = S::XB, WB = S::WB, U = S::U, SLOTS = S::SLOTS, SHARE = S::SHARE;
    extern __shared__ float lds[];                     // [tables] + SLOTS x [U][XB + WB] tiles of 1 KiB
    u32x4_t *ring = reinterpret_cast<u32x4_t *>(lds + S::TABLE_FLOATS);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int bx, by, bz;
    if (!gemm_block(g, bx, by, bz)) return;
    constexpr int KG = S::KG;
    const int kg = wave / (S::WM * S::WN), wm = wave / S::WN % S::WM, wn = wave % S::WN;
    GemmTile<MB, NT, XB> t;
    t.tile0 = bx * WB + wn * NT;
    t.wg_mb0 = bz * XB;
    t.mb0 = t.wg_mb0 + wm * MB;
    t.row_off = wm * MB * 32;
    t.lane = lane;
    t.wave = wave;
    t.split = by;
    t.lds = lds;
    t.stage = reinterpret_cast<float *>(ring);         // the slots are free once the last one is multiplied

    const int k0 = by * g.kpw, k1 = min(g.KT, k0 + g.kpw);             // kpw: k-steps per split, whole slots
    const int nblk = (k1 - k0 + U - 1) / U;
    // this wave's tiles of a slot: number id = k-step * (XB + WB) + (row block, or XB + band); past the last row block or
    // band, and past the last tile where the waves do not divide a slot evenly, the last one again
    const uint32_t ring_at = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void *)ring;
    const int row_blocks = (g.M + 31) >> 5;
    const u32x4_t *src[SHARE];
    int ku[SHARE], at[SHARE];
#pragma unroll
    for (int e = 0; e < SHARE; ++e) {
        const int id = min(wave * SHARE + e, S::PER_SLOT - 1), u = id / S::PER_STEP, r = id % S::PER_STEP;
        at[e] = id * 1024;
        ku[e] = u;
        src[e] = r < XB ? g.X + (size_t)min(t.wg_mb0 + r, row_blocks - 1) * g.KT * 64 + lane
                        : g.W + (size_t)min(bx * WB + (r - XB), g.NTiles - 1) * g.KT * 64 + lane;
    }
    auto request = [&](int j, int slot) {
#pragma unroll
        for (int e = 0; e < SHARE; ++e) {
            const int k = min(k0 + j * U + ku[e], g.KT - 1);
            tile_dma(src[e] + (size_t)k * 64, ring_at + (uint32_t)(slot * (S::PER_SLOT * 1024) + at[e]));
        }
    };
    auto pre = epi.issue(t, g);
#pragma unroll
    for (int s = 0; s < SLOTS - 1; ++s) request(s, s);
    auto carry = epi.prologue(pre, t, g);

    f32x16_t acc[MB][NT];
#pragma unroll
    for (int a = 0; a < MB; ++a)
#pragma unroll
        for (int i = 0; i < NT; ++i)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[a][i][v] = 0.f;
    u32x4_t fx[2][MB], fw[2][NT];
    auto read = [&](int slot, int u, int p) {
        const u32x4_t *b = ring + ((size_t)slot * S::PER_SLOT + u * S::PER_STEP) * 64 + lane;
#pragma unroll
        for (int a = 0; a < MB; ++a) fx[p][a] = b[(wm * MB + a) * 64];
#pragma unroll
        for (int i = 0; i < NT; ++i) fw[p][i] = b[(XB + wn * NT + i) * 64];
    };
    auto meet = [&] { __builtin_amdgcn_s_barrier(); asm volatile("" ::: "memory"); };
    const bool live = t.mb0 * 32 < g.M && t.tile0 < g.NTiles;          // the others only fetch
    wait_loads<(SLOTS - 2) * SHARE>();
    meet();
    int slot = 0;
    auto sweep = [&](auto LIVE) {
        constexpr bool on = decltype(LIVE)::value;
        auto multiply = [&](int p) {
#pragma unroll
            for (int a = 0; a < MB; ++a)
#pragma unroll
                for (int i = 0; i < NT; ++i)
                    acc[a][i] = HYDRA_MFMA16(__builtin_bit_cast(a16x8_t, fx[p][a]), __builtin_bit_cast(a16x8_t, fw[p][i]), acc[a][i]);
        };
        if constexpr (on) read(0, kg, 0);
        // KG == U: this group's k-step of slot j, out of register set p; its reads may be under way, those of slot j - 1 are done
        auto one = [&](int j, int p) {
            const int next = slot + 1 == SLOTS ? 0 : slot + 1, prev = slot == 0 ? SLOTS - 1 : slot - 1;
            wait_loads_and_reads<(SLOTS - 3) * SHARE, MB + NT>();
            meet();
            request(j + SLOTS - 1, prev);
            if constexpr (on) read(next, kg, p ^ 1);
            if constexpr (on) multiply(p);
            slot = next;
        };
        if constexpr (KG > 1) {
            for (int j = 0; j + 1 < nblk; j += 2) { one(j, 0); one(j + 1, 1); }
            if (nblk & 1) one(nblk - 1, 0);
            return;
        }
        for (int j = 0; j < nblk; ++j) {
            const int next = slot + 1 == SLOTS ? 0 : slot + 1, prev = slot == 0 ? SLOTS - 1 : slot - 1;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (u == U - 1) {
                    wait_loads_and_reads<(SLOTS - 3) * SHARE, U * (MB + NT)>();
                    meet();
                    request(j + SLOTS - 1, prev);
                    if constexpr (on) read(next, 0, (u + 1) & 1);
                } else {
                    if constexpr (on) read(slot, u + 1, (u + 1) & 1);
                }
                if constexpr (on) multiply(u & 1);
            }
            slot = next;
        }
    };
    if (live) sweep(std::true_type{});
    else      sweep(std::false_type{});

    wait_loads<0>();                                   // nothing may land in the slots any more: the epilogue stages there
    epi.before_barrier(carry, t, g);
    __syncthreads();
    if constexpr (KG > 1) {
        // each group finishes half of the row blocks: the other half of its sums goes to the wave of the same tile in the other group
        constexpr int HB = MB / KG;
        f32x4_t *give = reinterpret_cast<f32x4_t *>(t.stage + S::WAVES * GEMM_LDS_STAGE_WAVE) + lane;
        const int peer = wave ^ (S::WM * S::WN);
        if (live)
            static_for<HB * NT>([&](auto J) {
                constexpr int b = decltype(J)::value / NT, i = decltype(J)::value % NT;
                const f32x16_t out = kg == 0 ? acc[HB + b][i] : acc[b][i];
#pragma unroll
                for (int q = 0; q < 4; ++q) give[((wave * HB * NT + decltype(J)::value) * 4 + q) * 64] = f32x4_t{out[4 * q], out[4 * q + 1], out[4 * q + 2], out[4 * q + 3]};
            });
        __syncthreads();
        if (!live) return;
        epi.begin(t, g);
        static_for<HB * NT>([&](auto J) {
            constexpr int b = decltype(J)::value / NT, i = decltype(J)::value % NT;
            f32x16_t own = kg == 0 ? acc[b][i] : acc[HB + b][i];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const f32x4_t got = give[((peer * HB * NT + decltype(J)::value) * 4 + q) * 64];
#pragma unroll
                for (int e = 0; e < 4; ++e) own[4 * q + e] += got[e];
            }
            epi.tile(own, kg * HB + b, i, t, g);
        });
        return;
    }
    if (!live) return;
    epi.begin(t, g);
    static_for<MB * NT>([&](auto J) {
        constexpr int a = decltype(J)::value / NT, i = decltype(J)::value % NT;
        const f32x16_t tile_acc = acc[a][i];
        epi.tile(tile_acc, a, i, t, g);
    });
}

}  // namespace hydra
