// bf16 storage family: tree attention on MFMA.
//
// Per (row b, head h) the T tree queries attend to slots [0, L) of the paged
// cache and to the tree slots allowed by each query's ancestor bitmask (paper,
// section 2, "Tree decoding").  All T queries share every K/V byte, so the cache
// is streamed once per (b, h) and both contractions run on the matrix cores:
//
//   S^T[key][query] = K[key][:] . Q[query][:]         A = K tile, B = Q^T
//   O^T[dim][query] += V^T[dim][key] * P^T[key][query] A = V^T tile, B = P^T
//
// Working with the transposes makes a query a COLUMN of every accumulator, so
// its softmax statistics, its ancestor mask and its rescale factor are per-lane
// scalars, and the exponentiated scores are already in the register order the
// second contraction needs for its B operand: no LDS and no shuffles in the
// loop except one exchange between the two half-waves.  The in-page placement
// of K and V (device_common.h) makes both A operands single coalesced
// 16-byte-per-lane loads straight from the cache pages.
//
// A workgroup works on one (b, h).  Launch shapes:
//   short contexts (up to 1280 keys, and no more workgroups than CUs): attn_short_kernel,
//     one workgroup per 32-query tile and share of the head's dims; its 8 waves split the keys and
//     the result goes straight out as the next GEMM's input: one kernel, no
//     partial records;
//   longer contexts, or more rows: attn_bf16_kernel up to 32 queries (and where its
//     waves with a query tile each fill the chip better), attn_pair_kernel beyond (two
//     query tiles to a wave).  The waves of a workgroup split the keys, and
//     so do several workgroups per (b, h) while the chip has room; each of those leaves
//     a (max, sum, O) record that attn_merge_kernel combines.
#include <algorithm>

#include "attn_bf16.h"
#include "device_common.h"
#include "internal.h"

namespace hydra {

typedef __attribute__((ext_vector_type(4))) float f32x4_t;

// QW: query tiles of a workgroup, one or two, each with 8 / QW waves that split the keys
template <int DH, int QW, bool PACKED>
__global__ __launch_bounds__(ATTN_WAVES * 64) void attn_bf16_kernel(
    const u32x4_t *__restrict__ qbuf, const a16_t *__restrict__ kpages, const a16_t *__restrict__ vpages,
    const int32_t *__restrict__ page_table, int max_pages, int n_pages, int layer, const int32_t *__restrict__ seq_len,
    const TreeDev *__restrict__ tree, int T, int H, float scale, float *__restrict__ apart, void *out, int32_t *flags) {
    extern __shared__ float lds[];
    attn_bf16_body<DH, QW, PACKED, false>(qbuf, kpages, vpages, page_table, max_pages, n_pages, layer, seq_len, tree, T, H, 0,
                                          scale, apart, out, flags, (int)blockIdx.x, (int)gridDim.x, (int)blockIdx.y, (int)blockIdx.z, lds, (int)threadIdx.x);
}

// Short contexts: a workgroup takes one 32-query tile of one (row, head) and 1 / DS of the head's dims; its eight waves split
// the keys and meet in LDS, and the result goes straight out as the next GEMM's input.  The key loop does what attn_bf16_body does,
// sum for sum.
//
// Bound by a chain: launch and row length 2.0 us, K/V 3.2 (memory-side cache), three to four tiles of 0.7, merge and store 1.1
// (in-kernel clocks, 64 queries, 840 keys, 32 heads).  A workgroup's requests go through its CU at 64 bytes a cycle, so a head is shared
// out over as many workgroups as the chip takes in one round: with all of K and 1 / DS of V each one asks for less (430 KB ->
// 270 with DS = 4) and holds more tiles at once (RING; the accumulators and V tiles shrink with DS).  The scores are computed
// DS times over, which idle CUs do for nothing.  The workgroups of a head sit on one XCD (workgroup i runs on XCD i % 8),
// whose L2 then fetches K and V once.  64 x 840: 10.9 / 10.2 / 9.7 us with DS = 1 / 2 / 4, 12.5 before; on the whole
// verification call of 32 layers 3769 -> 3687 us, one node behind 701 tokens 797 -> 775 (8 layers).
template <int DH, int DS>
struct ShortTile { u32x4_t k[DH / 16]; u32x4_t v[2][DH / 32 / DS]; };
static constexpr float LOG2E = 1.44269504f;
enum { ATTN_SHORT_TILES = 5 };                              // 32-key tiles per wave up to which the launch rule takes this kernel

template <int DH, int DS, bool STREAM, bool PACKED>
__global__ __launch_bounds__(ATTN_WAVES * 64) void attn_short_kernel(
    const u32x4_t *__restrict__ qbuf, const a16_t *__restrict__ kpages, const a16_t *__restrict__ vpages,
    const int32_t *__restrict__ page_table, int max_pages, int n_pages, int layer, const int32_t *__restrict__ seq_len,
    const TreeDev *__restrict__ tree, int T, int H, int groups, float scale, void *out, int32_t *flags) {
    constexpr int KS = DH / 16, DT = DH / 32 / DS, RING = DS == 4 ? 4 : DS == 2 ? 3 : 2, NW = ATTN_WAVES;
    extern __shared__ float lds[];                          // [NW][2][32] maxima and sums, then the query tile and later O[NW][DT * 16][64]
    const int tid = (int)threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int hl = lane >> 5, col = lane & 31;
    const int QTtot = (T + 31) >> 5, per = QTtot * DS;
    const int seq = (int)blockIdx.x >> 3;
    const int group = seq / per * 8 + ((int)blockIdx.x & 7), j = seq % per;
    if (group >= groups) return;
    const int b = group / H, h = group - b * H, qtile = j / DS, ds = j % DS;
    const int32_t *pt = page_table + (size_t)b * max_pages;
    // everything whose address does not depend on the row's length is requested before the length is known: the queries (each
    // wave brings a share of the tile), the ancestor masks, and the page ids of this wave's tiles (the table has max_pages
    // entries for every row; entries past the row's pages are not used)
    u32x4_t *qs = reinterpret_cast<u32x4_t *>(lds + NW * 64);
    const int query = qtile * 32 + col;
    uint64_t anc0 = 0ull, anc1 = 0ull;
    if (query < T) { anc0 = tree->anc[query][0]; anc1 = tree->anc[query][1]; }
    int pg[ATTN_SHORT_TILES][2];
#pragma unroll
    for (int i = 0; i < ATTN_SHORT_TILES; ++i) {
        const int t = wave + i * NW;
        pg[i][0] = pt[min(2 * t, max_pages - 1)];
        pg[i][1] = pt[min(2 * t + 1, max_pages - 1)];
    }
    const int L = seq_len[b];
    if (wave < KS) qs[wave * 64 + lane] = qbuf[((((size_t)b * H + h) * QTtot + qtile) * KS + wave) * 64 + lane];
    if (L < 0 || L + T > max_pages * 16) {                  // uniform over the workgroup
        if (tid == 0 && j == 0 && h == 0) atomicOr(flags, FLAG_CAPACITY);
        return;
    }
    const int total = L + T, n_tiles = (total + 31) >> 5, row_pages = (total + 15) >> 4;
    const int mine_n = wave < n_tiles ? (n_tiles - wave + NW - 1) / NW : 0;     // this wave's tiles: wave, wave + NW, ...

    // Loads are never behind a condition (the compiler then knows how many are younger than the ones it waits for): a tile past
    // the last one reads one and the same piece of page 0 in every lane.
    auto load = [&](ShortTile<DH, DS> &kv, int it, int p0, int p1) {
        const int t = wave + it * NW;
        const bool live = t < n_tiles;
        if (2 * t + 1 >= row_pages) p1 = p0;                // second page of a tile: absent when the row ends inside the first
        p0 = live ? checked_page(p0, n_pages, flags) : 0;
        p1 = live ? checked_page(p1, n_pages, flags) : 0;
        const int ln = live ? lane : 0, lh = ln >> 5, lc = ln & 31;
        const u32x4_t *kp = reinterpret_cast<const u32x4_t *>(kpages + kv_block_base(layer, n_pages, (lc >> 4) ? p1 : p0, H, h, DH));
#pragma unroll
        for (int s = 0; s < KS; ++s) kv.k[s] = load_kv<STREAM>(kp + (2 * s + lh) * 16 + (lc & 15));
#pragma unroll
        for (int g = 0; g < 2; ++g) {
            const u32x4_t *vp = reinterpret_cast<const u32x4_t *>(vpages + kv_block_base(layer, n_pages, g ? p1 : p0, H, h, DH));
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) kv.v[g][dt] = load_kv<STREAM>(vp + (32 * (ds * DT + dt) + lc) * 2 + lh);
        }
    };
    f32x16_t o[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int v = 0; v < 16; ++v) o[dt][v] = 0.f;
    float m_run = -INFINITY, l_run = 0.f;
    auto step = [&](ShortTile<DH, DS> &kv, int it) {
        const int slot0 = (wave + it * NW) * 32;
        if (slot0 + 32 > total) {       // zero V of slots >= total (stale or never written): 0 * garbage must not appear
#pragma unroll
            for (int g = 0; g < 2; ++g)
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    // dword w holds keys i = 2w, 2w+1 of this half-wave: token = 8*(i/4) + 4*hl + i%4
                    const int i0 = 2 * w, i1 = 2 * w + 1;
                    const int s0 = slot0 + 16 * g + 8 * (i0 >> 2) + 4 * hl + (i0 & 3);
                    const int s1 = slot0 + 16 * g + 8 * (i1 >> 2) + 4 * hl + (i1 & 3);
                    const uint32_t keep = (s0 < total ? 0x0000ffffu : 0u) | (s1 < total ? 0xffff0000u : 0u);
#pragma unroll
                    for (int dt = 0; dt < DT; ++dt) kv.v[g][dt][w] &= keep;
                }
        }
        f32x16_t sc;
#pragma unroll
        for (int v = 0; v < 16; ++v) sc[v] = 0.f;
        int qoff = lane;
        asm volatile("" : "+v"(qoff));                       // keeps the reads of the queries here (hoisted, they are registers)
#pragma unroll
        for (int s = 0; s < KS; ++s)
            sc = HYDRA_MFMA16(__builtin_bit_cast(a16x8_t, kv.k[s]), __builtin_bit_cast(a16x8_t, qs[qoff + s * 64]), sc);
        bool moved;
        const float alpha = softmax_tile(sc, scale, slot0 + 32 > L, slot0, L, anc0, anc1, hl, m_run, l_run, moved);
        // the accumulators are rescaled only where some query's maximum moved (a factor of one otherwise; the first tile has
        // nothing to rescale)
        if (it > 0 && moved) {
#pragma unroll
            for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                for (int v = 0; v < 16; ++v) o[dt][v] *= alpha;
        }
        // P^T operands: page g uses accumulator registers 8g .. 8g+7 in order
#pragma unroll
        for (int g = 0; g < 2; ++g) {
            u32x4_t pb;
#pragma unroll
            for (int w = 0; w < 4; ++w) pb[w] = half_pack(sc[8 * g + 2 * w], sc[8 * g + 2 * w + 1]);
#pragma unroll
            for (int dt = 0; dt < DT; ++dt)
                o[dt] = HYDRA_MFMA16(__builtin_bit_cast(a16x8_t, kv.v[g][dt]), __builtin_bit_cast(a16x8_t, pb), o[dt]);
        }
    };
    ShortTile<DH, DS> ring[RING];
#pragma unroll
    for (int i = 0; i < RING; ++i) load(ring[i], i, pg[i][0], pg[i][1]);
    __syncthreads();                                         // the query tile is in LDS
    int it = 0;
    for (; it + RING < mine_n; it += RING)                   // all of the ring's tiles exist
#pragma unroll
        for (int i = 0; i < RING; ++i) {
            const int next = it + i + RING, t = wave + next * NW;
            int p0, p1;
            if (next < ATTN_SHORT_TILES) {                   // wave-uniform
                p0 = pg[ATTN_SHORT_TILES - 1][0]; p1 = pg[ATTN_SHORT_TILES - 1][1];
#pragma unroll
                for (int q = RING; q + 1 < ATTN_SHORT_TILES; ++q)
                    if (next == q) { p0 = pg[q][0]; p1 = pg[q][1]; }
            } else {                                         // a row longer than the host's hint
                p0 = pt[min(2 * t, max_pages - 1)];
                p1 = pt[min(2 * t + 1, max_pages - 1)];
            }
            step(ring[i], it + i);
            load(ring[i], next, p0, p1);
        }
#pragma unroll
    for (int i = 0; i < RING; ++i)
        if (it + i < mine_n) step(ring[i], it + i);

    // ---- merge the waves through LDS: ml[NW][2][32], then O[NW][DT * 16][64] where the queries were
    float *ml = lds, *ob = lds + NW * 64;
    if (hl == 0) {
        ml[(wave * 2 + 0) * 32 + col] = m_run;
        ml[(wave * 2 + 1) * 32 + col] = l_run;
    }
    __syncthreads();
    float m_tot = -INFINITY;
#pragma unroll
    for (int w = 0; w < NW; ++w) m_tot = fmaxf(m_tot, ml[(w * 2 + 0) * 32 + col]);
    float l_tot = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) l_tot += __expf(ml[(w * 2 + 0) * 32 + col] - (m_tot == -INFINITY ? 0.f : m_tot)) * ml[(w * 2 + 1) * 32 + col];
    const float mine = __expf(m_run - (m_tot == -INFINITY ? 0.f : m_tot));
    {
        float *dst = ob + (size_t)wave * DT * 16 * 64 + lane;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int v = 0; v < 16; ++v) dst[(dt * 16 + v) * 64] = o[dt][v] * mine;
    }
    __syncthreads();
    // the (band, group of 4 registers = 4 consecutive dims) items are shared out over the waves
    const float inv = 1.0f / l_tot;
    for (int id = wave; id < DT * 4; id += NW) {
        const int dt = id >> 2, g4 = id & 3;
        float acc[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const float *src = ob + (size_t)w * DT * 16 * 64 + lane;
#pragma unroll
            for (int q = 0; q < 4; ++q) acc[q] += src[(dt * 16 + 4 * g4 + q) * 64];
        }
        if (query >= T) continue;
        const int dim = 32 * (ds * DT + dt) + 8 * g4 + 4 * hl, m = b * T + query;
        if (PACKED) {
            const u32x2_t pk = {f2a_pack(acc[0] * inv, acc[1] * inv), f2a_pack(acc[2] * inv, acc[3] * inv)};
            *reinterpret_cast<u32x2_t *>(reinterpret_cast<a16_t *>(out) + x_index<true>(m, h * DH + dim, H * DH)) = pk;
        } else {
            *reinterpret_cast<f32x4_t *>(reinterpret_cast<float *>(out) + ((size_t)m * H + h) * DH + dim) = f32x4_t{acc[0] * inv, acc[1] * inv, acc[2] * inv, acc[3] * inv};
        }
    }
}

// More rows, or longer ones, with more than 32 queries per row: a wave holds TWO query tiles, so that a CU asks for every byte of
// K and V once (a wave per query tile asked twice, and what a CU can ask for is the bound: 33B shape, 4 rows of 2048 keys: 63 us a
// launch, 45 now; 7B, 16 rows of 1024: 67, 51 now).  There is no room for K and V tiles in registers next to two sets of accumulators
// (128 of them), so each wave has a tile of its own in LDS that the LDS DMA fills: K is requested again as soon as the scores
// are computed, V as soon as it is used, and no wave waits for another before the end.
// STREAM (up to 64 queries, every byte of K and V read once on the chip): nontemporal requests, 47.1 -> 43.8 us on the same shape; with
// a second workgroup on the same bytes 62.9 -> 65.3.
// NW waves split the keys: eight where the workgroups fit one round of the chip, four, two workgroups to a CU, beyond.
//
// Softmax in powers of two: maxima of the unscaled scores, and the scale as a factor of the exponent 2^((s - max) c).  The largest
// probability has to be exactly one, since the sums take it as it is and the products rounded to half.  With c in a multiply-add,
// 2^(s c - max c), it was off by the rounding of max c: scores of 200 and more cost that much (64 queries behind 3900 keys, scores of
// deviation 50 / 100: error 6.0e-6 / 1.03e-5 of the result's 2-norm, 3.3e-6 / 2.9e-6 now; the loop takes 0.5 to 2.5 % longer).  A reference that trails the maximum by up to 2^8 saves
// most of the rescaling and costs far more (sharp rows 5e-5 -> 1.6e-4); nothing is gained either, since the loads alone take as long.
template <int DH, int NW, bool STREAM>
__global__ __launch_bounds__(NW * 64, 2) void attn_pair_kernel(
    const u32x4_t *__restrict__ qbuf, const a16_t *__restrict__ kpages, const a16_t *__restrict__ vpages,
    const int32_t *__restrict__ page_table, int max_pages, int n_pages, int layer, const int32_t *__restrict__ seq_len,
    const TreeDev *__restrict__ tree, int T, int H, int groups, int key_wgs, float scale, float *__restrict__ apart, void *out, int packed,
    int32_t *flags) {
    constexpr int KS = DH / 16, DT = DH / 32, TILE = KS + 2 * DT;    // KiB of a K and V tile
    extern __shared__ float lds[];                          // queries [2][KS] and tiles [NW][TILE] of 1 KiB; then maxima and sums, O of one query tile
    const int tid = (int)threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int hl = lane >> 5, col = lane & 31;
    const int QTtot = (T + 31) >> 5, QG = (QTtot + 1) >> 1, per = QG * key_wgs;
    const int seq = (int)blockIdx.x >> 3;
    const int group = seq / per * 8 + ((int)blockIdx.x & 7), j = seq % per;
    if (group >= groups) return;
    const int b = group / H, h = group - b * H, qg = j % QG, key_wg = j / QG;
    const int units = key_wgs * NW, unit = key_wg * NW + wave;
    const int32_t *pt = page_table + (size_t)b * max_pages;
    u32x4_t *qs = reinterpret_cast<u32x4_t *>(lds);
    const u32x4_t *ql = qs + lane;
    uint64_t anc[2][2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int query = (qg * 2 + q) * 32 + col;
        anc[q][0] = anc[q][1] = 0ull;
        if (query < T) { anc[q][0] = tree->anc[query][0]; anc[q][1] = tree->anc[query][1]; }
    }
    // page ids of this wave's next 32 tiles, two per tile, one per lane
    auto page_ids = [&](int first) { return pt[min(2 * (unit + (first + (lane >> 1)) * units) + (lane & 1), max_pages - 1)]; };
    int pgs = page_ids(0);
    const int L = seq_len[b];
    // the second query tile of the last group may lie behind the last query: the first one again, which nobody stores
    const size_t qblk = (((size_t)b * H + h) * QTtot + qg * 2) * KS;
    const int second = qg * 2 + 1 < QTtot ? KS : 0;
    for (int i = wave; i < 2 * KS; i += NW) qs[i * 64 + lane] = qbuf[(qblk + (i < KS ? i : second + i - KS)) * 64 + lane];
    __syncthreads();
    if (L < 0 || L + T > max_pages * 16) {                  // uniform over the workgroup
        if (tid == 0 && j == 0 && h == 0) atomicOr(flags, FLAG_CAPACITY);
        return;
    }
    const int total = L + T, n_tiles = (total + 31) >> 5, row_pages = (total + 15) >> 4;
    const int mine_n = unit < n_tiles ? (n_tiles - unit + units - 1) / units : 0;      // this wave's tiles: unit, unit + units, ...

    u32x4_t *mine = qs + (2 * KS + wave * TILE) * 64;       // this wave's tile: K blocks, then V blocks [page][dims / 32]
    const uint32_t mine_at = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void *)mine;
    auto dma = [&](const u32x4_t *src, int block) {
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)src,
                                         (__attribute__((address_space(3))) void *)(uintptr_t)(mine_at + (uint32_t)block * 1024u), 16, 0, STREAM ? 2 : 0);      // 2: nontemporal
    };
    int p0 = 0, p1 = 0;                                     // pages of the tile that is requested next
    auto next_pages = [&](int it) {
        if (it > 0 && (it & 31) == 0) { pgs = page_ids(it); asm volatile("" : "+v"(pgs)); }      // awaited in here, not behind the branch
        p0 = checked_page(__builtin_amdgcn_readlane(pgs, 2 * (it & 31)), n_pages, flags);
        // second page of a tile: absent when the row ends inside the first one (its keys are masked; any valid page will do)
        p1 = 2 * (unit + it * units) + 1 < row_pages ? checked_page(__builtin_amdgcn_readlane(pgs, 2 * (it & 31) + 1), n_pages, flags) : p0;
    };
    auto request_k = [&] {
        const u32x4_t *kp = reinterpret_cast<const u32x4_t *>(kpages + kv_block_base(layer, n_pages, (col >> 4) ? p1 : p0, H, h, DH)) + hl * 16 + (col & 15);
#pragma unroll
        for (int s = 0; s < KS; ++s) dma(kp + s * 32, s);
    };
    auto request_v = [&] {
#pragma unroll
        for (int g = 0; g < 2; ++g) {
            const u32x4_t *vp = reinterpret_cast<const u32x4_t *>(vpages + kv_block_base(layer, n_pages, g ? p1 : p0, H, h, DH)) + col * 2 + hl;
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) dma(vp + dt * 64, KS + g * DT + dt);
        }
    };
    f32x16_t o[2][DT];
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int v = 0; v < 16; ++v) o[q][dt][v] = 0.f;
    float m_run[2] = {-INFINITY, -INFINITY}, l_run[2] = {0.f, 0.f};
    const float c = scale * LOG2E;
    // these have arrived: nothing in the loop is to wait for an ordinary load, which would be a wait for the DMA as well
    asm volatile("" : "+v"(pgs), "+v"(anc[0][0]), "+v"(anc[0][1]), "+v"(anc[1][0]), "+v"(anc[1][1]));
    if (mine_n > 0) { next_pages(0); request_k(); request_v(); }
    for (int it = 0; it < mine_n; ++it) {
        const bool more = it + 1 < mine_n;
        const int slot0 = (unit + it * units) * 32;
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * DT) : "memory");             // K has landed: of what was asked for only V may be missing
        f32x16_t sc[2];
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int v = 0; v < 16; ++v) sc[q][v] = 0.f;
        int at = 0;
        asm volatile("" : "+v"(at));                        // keeps the reads of the queries inside the loop
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            const a16x8_t k = __builtin_bit_cast(a16x8_t, mine[s * 64 + lane]);
#pragma unroll
            for (int q = 0; q < 2; ++q) sc[q] = HYDRA_MFMA16(k, __builtin_bit_cast(a16x8_t, ql[at + (q * KS + s) * 64]), sc[q]);
        }
        if (more) {
            next_pages(it + 1);
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");                    // K is read
            request_k();
        }
        u32x4_t pb[2][2];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            if (slot0 + 32 > L) {                           // uniform: the tiles that hold tree slots or end the row
                const uint32_t seen = keys_seen(slot0, L, anc[q][0], anc[q][1]) >> (4 * hl);
#pragma unroll
                for (int v = 0; v < 16; ++v) sc[q][v] = (seen >> (8 * (v >> 2) + (v & 3))) & 1u ? sc[q][v] : -INFINITY;
            }
            float cmax = -INFINITY;
#pragma unroll
            for (int v = 0; v < 16; ++v) cmax = fmaxf(cmax, sc[q][v]);
            const HalfWaves cm = half_waves(cmax);
            cmax = fmaxf(cm.lo, cm.hi);
            if (__any(cmax > m_run[q])) {                                          // always on the first visible tile
                const float m_new = fmaxf(m_run[q], cmax);
                const float alpha = m_new == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((m_run[q] - m_new) * c);
                m_run[q] = m_new;
                l_run[q] *= alpha;
#pragma unroll
                for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                    for (int v = 0; v < 16; ++v) o[q][dt][v] *= alpha;
            }
            const float ref = m_run[q] == -INFINITY ? 0.f : m_run[q];
            float rs = 0.f;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const float p = __builtin_amdgcn_exp2f((sc[q][v] - ref) * c);     // 0 for masked keys, exactly 1 for the largest
                sc[q][v] = p;
                rs += p;
            }
            const HalfWaves rh = half_waves(rs);
            l_run[q] += rh.lo + rh.hi;
            // P^T operands: page g uses accumulator registers 8g .. 8g+7 in order
#pragma unroll
            for (int g = 0; g < 2; ++g)
#pragma unroll
                for (int w = 0; w < 4; ++w) pb[q][g][w] = half_pack(sc[q][8 * g + 2 * w], sc[q][8 * g + 2 * w + 1]);
        }
        if (more) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(KS) : "memory");       // V has landed: only the next K may be missing
        else      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        if (slot0 + 32 > total) {       // zero V of slots >= total (stale or never written): 0 * garbage must not appear
#pragma unroll
            for (int g = 0; g < 2; ++g) {
                u32x4_t keep;
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    // dword w holds keys i = 2w, 2w+1 of this half-wave: token = 8*(i/4) + 4*hl + i%4
                    const int i0 = 2 * w, i1 = 2 * w + 1;
                    const int s0 = slot0 + 16 * g + 8 * (i0 >> 2) + 4 * hl + (i0 & 3);
                    const int s1 = slot0 + 16 * g + 8 * (i1 >> 2) + 4 * hl + (i1 & 3);
                    keep[w] = (s0 < total ? 0x0000ffffu : 0u) | (s1 < total ? 0xffff0000u : 0u);
                }
#pragma unroll
                for (int dt = 0; dt < DT; ++dt) mine[(KS + g * DT + dt) * 64 + lane] &= keep;      // each lane its own 16 bytes
            }
        }
#pragma unroll
        for (int g = 0; g < 2; ++g)
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) {
                const a16x8_t v = __builtin_bit_cast(a16x8_t, mine[(KS + g * DT + dt) * 64 + lane]);
#pragma unroll
                for (int q = 0; q < 2; ++q) o[q][dt] = HYDRA_MFMA16(v, __builtin_bit_cast(a16x8_t, pb[q][g]), o[q][dt]);
            }
        if (more) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");                    // V is read
            request_v();
        }
    }

    // ---- merge the waves through LDS, one query tile after the other: ml[2][NW][2][32], then O[NW][DT * 16][64]
    __syncthreads();                                         // every wave is done with queries and tiles
    float *ml = lds, *ob = lds + NW * 128;
    if (hl == 0) {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            ml[((q * NW + wave) * 2 + 0) * 32 + col] = m_run[q];
            ml[((q * NW + wave) * 2 + 1) * 32 + col] = l_run[q];
        }
    }
    __syncthreads();
    const int Tq = QTtot * 32;
    float *rec = apart + (((size_t)b * H + h) * key_wgs + key_wg) * apart_record(Tq, DH);
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int qtile = qg * 2 + q, query = qtile * 32 + col;
        if (qtile >= QTtot) break;                           // uniform over the workgroup
        const float *mq = ml + q * NW * 64;
        float m_tot = -INFINITY;
#pragma unroll
        for (int w = 0; w < NW; ++w) m_tot = fmaxf(m_tot, mq[w * 64 + col]);
        const float m_safe = m_tot == -INFINITY ? 0.f : m_tot;
        float l_tot = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) l_tot += __builtin_amdgcn_exp2f((mq[w * 64 + col] - m_safe) * c) * mq[w * 64 + 32 + col];
        const float f = __builtin_amdgcn_exp2f((m_run[q] - m_safe) * c);
        float *dst = ob + (size_t)wave * DT * 16 * 64 + lane;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int v = 0; v < 16; ++v) dst[(dt * 16 + v) * 64] = o[q][dt][v] * f;
        __syncthreads();
        // the (band, group of 4 registers = 4 consecutive dims) items are shared out over the waves
        const float inv = key_wgs == 1 ? 1.0f / l_tot : 1.0f;
        for (int id = wave; id < DT * 4; id += NW) {
            const int dt = id >> 2, g4 = id & 3;
            float acc[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                const float *src = ob + (size_t)w * DT * 16 * 64 + lane;
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[e] += src[(dt * 16 + 4 * g4 + e) * 64];
            }
            const int dim = 32 * dt + 8 * g4 + 4 * hl, m = b * T + query;
            if (key_wgs > 1) {
                *reinterpret_cast<f32x4_t *>(rec + (size_t)query * DH + dim) = f32x4_t{acc[0], acc[1], acc[2], acc[3]};
            } else if (query < T) {
                if (packed) {
                    const u32x2_t pk = {f2a_pack(acc[0] * inv, acc[1] * inv), f2a_pack(acc[2] * inv, acc[3] * inv)};
                    *reinterpret_cast<u32x2_t *>(reinterpret_cast<a16_t *>(out) + x_index<true>(m, h * DH + dim, H * DH)) = pk;
                } else {
                    *reinterpret_cast<f32x4_t *>(reinterpret_cast<float *>(out) + ((size_t)m * H + h) * DH + dim) = f32x4_t{acc[0] * inv, acc[1] * inv, acc[2] * inv, acc[3] * inv};
                }
            }
        }
        if (key_wgs > 1 && wave == 0 && hl == 0) {
            rec[(size_t)Tq * DH + query] = m_tot;
            rec[(size_t)Tq * DH + Tq + query] = l_tot;
        }
        if (q == 0) __syncthreads();                         // the second query tile's sums go where these were
    }
}

// out[b, n, h, :] = sum_u w_u O_u[n] / sum_u w_u l_u,  w_u = exp(m_u - max_u m_u), or 2^(c (m_u - max_u m_u)) where the records hold
// unscaled maxima (RAW: attn_pair_kernel).
// One workgroup per (row, head, 8 queries), one thread per (query, 4 dims); all loads of a thread are
// independent of each other and of the row length, so they make one round trip.
enum { MERGE_MAX_UNITS = 16 };
template <bool PACKED, bool RAW>
__global__ __launch_bounds__(256) void attn_merge_kernel(const float *__restrict__ apart, const int32_t *__restrict__ seq_len,
                                                          int T, int H, int Dh, int units, int max_pages, float c, void *out) {
    const int h = blockIdx.y, b = blockIdx.z;
    const int per_q = Dh >> 2;                              // threads per query
    const int n = blockIdx.x * (256 / per_q) + threadIdx.x / per_q;
    const int dim = (threadIdx.x % per_q) * 4;
    const int Tq = ((T + 31) >> 5) * 32;
    const size_t recsz = apart_record(Tq, Dh);
    const float *base = apart + (((size_t)b * H + h) * units) * recsz;
    const bool live = n < T;
    float mu[MERGE_MAX_UNITS], lu[MERGE_MAX_UNITS];
    f32x4_t ou[MERGE_MAX_UNITS];
#pragma unroll
    for (int u = 0; u < MERGE_MAX_UNITS; ++u) {
        mu[u] = -INFINITY; lu[u] = 0.f; ou[u] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        if (u < units && live) {
            const float *r = base + u * recsz;
            mu[u] = r[(size_t)Tq * Dh + n];
            lu[u] = r[(size_t)Tq * Dh + Tq + n];
            ou[u] = *reinterpret_cast<const f32x4_t *>(r + (size_t)n * Dh + dim);
        }
    }
    const int L = seq_len[b];
    if (L < 0 || L + T > max_pages * 16 || !live) return;
    float mt = -INFINITY;
#pragma unroll
    for (int u = 0; u < MERGE_MAX_UNITS; ++u) mt = fmaxf(mt, mu[u]);
    float den = 0.f;
    f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int u = 0; u < MERGE_MAX_UNITS; ++u) {
        const float w = u < units ? (RAW ? __builtin_amdgcn_exp2f((mu[u] - mt) * c) : __expf(mu[u] - mt)) : 0.f;
        den += w * lu[u];
        acc += ou[u] * w;
    }
    const float inv = 1.0f / den;
    const int m = b * T + n;
    if (PACKED) {
        u32x2_t pk = {f2a_pack(acc[0] * inv, acc[1] * inv), f2a_pack(acc[2] * inv, acc[3] * inv)};
        *reinterpret_cast<u32x2_t *>(reinterpret_cast<a16_t *>(out) + x_index<true>(m, h * Dh + dim, H * Dh)) = pk;
    } else {
        *reinterpret_cast<f32x4_t *>(reinterpret_cast<float *>(out) + ((size_t)m * H + h) * Dh + dim) = acc * inv;
    }
}

// upper bound of workgroups per (b, h) that the partial buffer is sized for
int attn_units(const hydra_ctx *c, int B) {
    int u = 512 / (B * c->m.n_heads);
    if (u < 1) u = 1;
    if (u > MERGE_MAX_UNITS) u = MERGE_MAX_UNITS;
    return u;
}

int launch_attention_f32(hydra_ctx *c, hipStream_t s, int B, int layer, const float *q, const int32_t *seq_len,
                         const hydra_kv *kv, float *out, int32_t *flags);

static size_t attn_lds_bytes(int Dh) { return ((size_t)ATTN_WAVES * 64 + (size_t)ATTN_WAVES * (Dh / 32) * 16 * 64) * 4; }

static size_t attn_short_lds_bytes(int Dh, int ds) {
    return ((size_t)ATTN_WAVES * 64 + std::max((size_t)ATTN_WAVES * (Dh / 32 / ds) * 16 * 64, (size_t)Dh * 16)) * 4;       // O, or the query tile
}

static size_t attn_pair_lds_bytes(int Dh, int nw) { return ((size_t)2 * (Dh / 16) + (size_t)nw * (Dh / 8)) * 1024; }

int attn_max_dynamic_lds(hydra_ctx *c) {
    (void)c;
    hipError_t e = hipSuccess;
#define ATTR(DHv, QWv) \
    if (e == hipSuccess) e = hipFuncSetAttribute((const void *)attn_bf16_kernel<DHv, QWv, true>, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024); \
    if (e == hipSuccess) e = hipFuncSetAttribute((const void *)attn_bf16_kernel<DHv, QWv, false>, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024)
    ATTR(128, 1); ATTR(128, 2); ATTR(64, 1); ATTR(64, 2);
#undef ATTR
#define ATTR(DHv, DSv, STv) \
    if (e == hipSuccess) e = hipFuncSetAttribute((const void *)attn_short_kernel<DHv, DSv, STv, true>, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024); \
    if (e == hipSuccess) e = hipFuncSetAttribute((const void *)attn_short_kernel<DHv, DSv, STv, false>, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024)
    ATTR(128, 1, false); ATTR(128, 1, true); ATTR(128, 2, false); ATTR(64, 1, false); ATTR(64, 1, true);
#undef ATTR
#define ATTR(DHv, NWv, Pv) if (e == hipSuccess) e = hipFuncSetAttribute((const void *)attn_pair_kernel<DHv, NWv, Pv>, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024)
    ATTR(128, 8, true); ATTR(128, 8, false); ATTR(64, 8, true); ATTR(64, 8, false); ATTR(128, 4, true); ATTR(128, 4, false);
#undef ATTR
    if (e != hipSuccess) return hip_fail(e, "hipFuncSetAttribute(attention kernels)");
    return HYDRA_OK;
}

// x_out != NULL: result as the next GEMM's input; plain_out != NULL: fp32 [B,T,H,Dh].
int launch_attention(hydra_ctx *c, hipStream_t s, int B, int layer, const void *qbuf, const int32_t *seq_len,
                     const hydra_kv *kv, float *apart, int units_max, void *x_out, float *plain_out, int32_t *flags) {
    if (!c->bf16) {
        float *dst = plain_out ? plain_out : (float *)x_out;     // the fp32 GEMM input order is [B,T,H,Dh] itself
        return launch_attention_f32(c, s, B, layer, (const float *)qbuf, seq_len, kv, dst, flags);
    }
    const int T = c->tree.T, H = c->m.n_heads, Dh = c->m.head_dim;
    const int QTtot = ceil_div(T, 32);
    const int len = kv->seq_len_hint > 0 ? kv->seq_len_hint : c->m.max_pos;
    const int tiles = ceil_div(len + T, 32);
    const float scale = 1.0f / sqrtf((float)Dh);
    void *out = x_out ? x_out : (void *)plain_out;
    const bool packed = x_out != nullptr;
    // Short contexts, up to five key tiles per wave, while a workgroup per (row, head, 32-query tile) fits one round of the chip: the
    // result goes straight out, without records and merge.  The head's dims are shared out over more workgroups while those still fit the
    // round.  (More rows than that: a workgroup that holds all query tiles of its head and reads each K/V byte once is 2-3 % faster on the whole
    // verification call at batch 8 and 16.)
    if (tiles <= ATTN_WAVES * ATTN_SHORT_TILES && QTtot * H * B <= 256) {
        int ds = Dh / 32;
        while (ds > 1 && QTtot * H * B * ds > 256) ds >>= 1;
        const dim3 sgrid(ceil_div(H * B, 8) * 8 * QTtot * ds), sblock(ATTN_WAVES * 64);
#define SHORT(DHv, DSv, STv, Pv)                                                                                                                  \
    hipLaunchKernelGGL((attn_short_kernel<DHv, DSv, STv, Pv>), sgrid, sblock, attn_short_lds_bytes(DHv, DSv), s, (const u32x4_t *)qbuf,           \
                       (const a16_t *)kv->k_pages, (const a16_t *)kv->v_pages, kv->page_table, kv->max_pages, kv->n_pages, layer, seq_len,        \
                       tree_dev(c), T, H, H * B, scale, out, flags)
#define SHORT_DS(DHv, DSv, STv) do { if (packed) SHORT(DHv, DSv, STv, true); else SHORT(DHv, DSv, STv, false); } while (0)
        if (Dh == 128) {
            if (ds == 4) SHORT_DS(128, 4, false);
            else if (ds == 2) SHORT_DS(128, 2, false);
            else if (QTtot > 1) SHORT_DS(128, 1, false);
            else SHORT_DS(128, 1, true);
        } else {
            if (ds == 2) SHORT_DS(64, 2, false);
            else if (QTtot > 1) SHORT_DS(64, 1, false);
            else SHORT_DS(64, 1, true);
        }
#undef SHORT_DS
#undef SHORT
        HYDRA_LAUNCH_CHECK("attn_short_kernel");
        return HYDRA_OK;
    }
    // Longer contexts, or more rows: a CU streams at most ~45 GB/s, so the keys of one head are spread over several workgroups, two tiles per
    // wave or more, whose partial records attn_merge_kernel combines.  Never more of them than one round of the chip: a workgroup
    // holds a CU by itself (registers), so a second round only repeats the fixed cost of a workgroup (first round trips, LDS merge,
    // partial record).  Measured best at about 200 workgroups in all: 7B at 2066 / 4114 keys 4.30 -> 4.01 / 4.63 -> 4.30 ms per verify.
    //
    // More than 32 queries: two query tiles to a wave (attn_pair_kernel), eight waves to a workgroup, or four where two workgroups fit a
    // CU and all have work (more groups than CUs).  With 33 to 64 queries in all it has half as many waves as tiles to hand
    // out, which a single short row does not make up for (attention call in us, cold, 64 queries):
    //   up to 52 tiles (1664 keys), eight waves on no more than half of the chip (a quarter with 64 dims): a wave per query tile, as
    //     many waves again (attn_bf16_kernel with two tiles; 16 heads behind 1250 / 1500 keys 17.1 / 18.2 against 18.9 / 19.2, 32
    //     heads 19.6 / 20.0 against 20.2 / 20.9, 40 heads behind 1250 20.6 against 21.1; beyond: 40 heads behind 1500 22.9 against 22.2,
    //     32 heads behind 1600 22.1 against 20.8; 32 heads of 64 dims behind 1250 15.2 against 14.5)
    //   more tiles, eight waves on less than half of the chip, 128 dims: twice the workgroups of four waves (16 heads behind 2100 / 3200
    //     keys 20.4 / 20.6 -> 17.8 / 20.0; with 64 dims it gains nothing, 13.9 against 14.0)
    const int qgroups = (QTtot + 1) / 2, hb = H * B * qgroups;
    const int eight = hb * ceil_div(tiles, ATTN_WAVES * 2);          // workgroups of eight waves with two tiles each
    const bool apart_tiles = QTtot == 2 && tiles <= 52 && eight <= Dh;
    const bool pair = QTtot > 1 && !apart_tiles, few = QTtot == 2 && Dh == 128 && eight < 128;
    const int nw = pair ? (hb > 256 || few ? 4 : 8) : apart_tiles ? ATTN_WAVES / 2 : ATTN_WAVES;       // waves that split a workgroup's keys
    const int wgs = pair && hb > 256 ? 1 : std::max(1, std::min({ceil_div(tiles, nw * 2), std::max(1, 208 / hb), units_max}));
    if (pair) {
        const dim3 pgrid(ceil_div(H * B, 8) * 8 * qgroups * wgs);
#define PAIR(DHv, NWv, STv)                                                                                                                       \
    hipLaunchKernelGGL((attn_pair_kernel<DHv, NWv, STv>), pgrid, dim3(NWv * 64), attn_pair_lds_bytes(DHv, NWv), s, (const u32x4_t *)qbuf,          \
                       (const a16_t *)kv->k_pages, (const a16_t *)kv->v_pages, kv->page_table, kv->max_pages, kv->n_pages, layer, seq_len,        \
                       tree_dev(c), T, H, H * B, wgs, scale, apart, out, packed ? 1 : 0, flags)
#define PAIR_NW(DHv, NWv) do { if (qgroups == 1) PAIR(DHv, NWv, true); else PAIR(DHv, NWv, false); } while (0)
        if (Dh == 128) { if (nw == 8) PAIR_NW(128, 8); else PAIR_NW(128, 4); }
        else           { if (nw == 8) PAIR_NW(64, 8); else PAIR_NW(64, 4); }
#undef PAIR_NW
#undef PAIR
        HYDRA_LAUNCH_CHECK("attn_pair_kernel");
    } else {
        dim3 grid(wgs, H, B), block(ATTN_WAVES * 64);
        const size_t lds = attn_lds_bytes(Dh);
#define ATTN_CASE(DHv, QWv, Pv)                                                                                      \
        hipLaunchKernelGGL((attn_bf16_kernel<DHv, QWv, Pv>), grid, block, lds, s, (const u32x4_t *)qbuf,                       \
                           (const a16_t *)kv->k_pages, (const a16_t *)kv->v_pages, kv->page_table, kv->max_pages,      \
                           kv->n_pages, layer, seq_len, tree_dev(c), T, H, scale, apart, out, flags)
#define ATTN_QW(DHv, QWv) do { if (packed) ATTN_CASE(DHv, QWv, true); else ATTN_CASE(DHv, QWv, false); } while (0)
        if (Dh == 128) { if (apart_tiles) ATTN_QW(128, 2); else ATTN_QW(128, 1); }
        else           { if (apart_tiles) ATTN_QW(64, 2); else ATTN_QW(64, 1); }
#undef ATTN_QW
#undef ATTN_CASE
        HYDRA_LAUNCH_CHECK("attn_bf16_kernel");
    }
    if (wgs > 1) {
        const int q_per_wg = 256 / (Dh / 4);
        dim3 mgrid(ceil_div(T, q_per_wg), H, B), mblock(256);
#define MERGE(Pv, RAWv) hipLaunchKernelGGL((attn_merge_kernel<Pv, RAWv>), mgrid, mblock, 0, s, apart, seq_len, T, H, Dh, wgs, kv->max_pages, scale * LOG2E, out)
        if (pair) { if (packed) MERGE(true, true); else MERGE(false, true); }
        else      { if (packed) MERGE(true, false); else MERGE(false, false); }
#undef MERGE
        HYDRA_LAUNCH_CHECK("attn_merge_kernel");
    }
    return HYDRA_OK;
}

}  // namespace hydra
