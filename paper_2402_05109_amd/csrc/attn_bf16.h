// Tree attention on MFMA, 16-bit family: the body of one workgroup (see bf16_attn.hip for the method and the
// launch shapes).  Shared by the stand-alone kernel and by the persistent layer kernel (bf16_layers.hip).
#pragma once

#include "device_common.h"
#include "internal.h"

namespace hydra {

typedef __attribute__((ext_vector_type(16))) float f32x16_t;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4_t;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2_t;
typedef __attribute__((ext_vector_type(4))) float f32x4_t;


// record of one workgroup in the partial buffer: O[Tq][Dh], m[Tq], l[Tq]   (Tq = 32 * ceil(T/32))
__host__ __device__ inline size_t apart_record(int Tq, int Dh) { return (size_t)Tq * Dh + 2 * (size_t)Tq; }

enum { ATTN_WAVES = 8 };

// two probabilities rounded to half: nothing to saturate, so without the four clamps per pair of f2a_pack
__device__ __forceinline__ uint32_t half_pack(float lo, float hi) {
    typedef __attribute__((ext_vector_type(2))) float f2;
    typedef __attribute__((ext_vector_type(2))) _Float16 h2;
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((f2{lo, hi}), h2));
}

// Which of the 32 keys at slot0 .. slot0 + 31 a query sees, one bit each: every cached slot, and the tree slots that its ancestor
// mask names (no bit of it is set from node T on).  Written without a branch per key: with `slot < L ? .. : mask bit` per score
// the compiler made two nested branches of each of the 16 scores of a lane, also for tiles that need no mask, and they were
// a fifth of a tile's time (0.9 us per 32-key tile with two waves to a SIMD, 0.7 now).
__device__ __forceinline__ uint32_t keys_seen(int slot0, int L, uint64_t anc0, uint64_t anc1) {
    const int rel = slot0 - L;                             // node of the first key; negative: cached slots first
    if (rel < 0) {
        const int n = -rel;                                // cached slots among the 32 (uniform)
        return n >= 32 ? 0xffffffffu : ((1u << n) - 1u) | ((uint32_t)anc0 << n);
    }
    if (rel >= 64) return rel >= 128 ? 0u : (uint32_t)(anc1 >> (rel - 64));
    return (uint32_t)(anc0 >> rel) | (rel > 32 ? (uint32_t)(anc1 << (64 - rel)) : 0u);
}

// One 32-key tile's scores, S^T = K Q^T as the matrix cores leave it -> probabilities, in place, and the running maximum and sum
// of the lane's query.  Returns the factor by which what was accumulated before has to be scaled.
__device__ __forceinline__ float softmax_tile(f32x16_t &sc, float scale, bool need_mask, int slot0, int L, uint64_t anc0, uint64_t anc1, int hl,
                                              float &m_run, float &l_run, bool &moved) {
#pragma unroll
    for (int v = 0; v < 16; ++v) sc[v] *= scale;
    if (need_mask) {                                       // uniform: the tiles that hold tree slots or end the row
        const uint32_t seen = keys_seen(slot0, L, anc0, anc1) >> (4 * hl);
#pragma unroll
        for (int v = 0; v < 16; ++v) sc[v] = (seen >> (8 * (v >> 2) + (v & 3))) & 1u ? sc[v] : -INFINITY;
    }
    float cmax = -INFINITY;
#pragma unroll
    for (int v = 0; v < 16; ++v) cmax = fmaxf(cmax, sc[v]);
    const HalfWaves cm = half_waves(cmax);
    cmax = fmaxf(cm.lo, cm.hi);
    const float m_new = fmaxf(m_run, cmax);
    const float m_safe = (m_new == -INFINITY) ? 0.f : m_new;
    const float alpha = __expf(m_run - m_safe);
    moved = __any(m_new != m_run);
    float rs = 0.f;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const float p = __expf(sc[v] - m_safe);            // exp(-inf) = 0 for masked keys
        sc[v] = p;
        rs += p;
    }
    const HalfWaves rh = half_waves(rs);
    rs = rh.lo + rh.hi;
    l_run = l_run * alpha + rs;
    m_run = m_new;
    return alpha;
}

template <int DH>
struct KVTile { u32x4_t k[DH / 16]; u32x4_t v[2][DH / 32]; };

// STREAM: nontemporal, for K and V that one workgroup alone reads (16 rows x 64 queries, 1000 keys: 58.8 -> 54.8 us; where the
// workgroups of two query tiles read the same bytes it costs time)
template <bool STREAM>
__device__ __forceinline__ u32x4_t load_kv(const u32x4_t *p) {
    if (STREAM) return __builtin_nontemporal_load(p);
    return *p;
}
template <int DH, bool STREAM>
__device__ __forceinline__ void load_k_tile(KVTile<DH> &kv, const a16_t *kpages, int p0, int p1, int layer, int n_pages, int H, int h, int lane) {
    const int hl = lane >> 5, col = lane & 31;
    const u32x4_t *kp = reinterpret_cast<const u32x4_t *>(kpages + kv_block_base(layer, n_pages, (col >> 4) ? p1 : p0, H, h, DH));
#pragma unroll
    for (int s = 0; s < DH / 16; ++s) kv.k[s] = load_kv<STREAM>(kp + (2 * s + hl) * 16 + (col & 15));
}
template <int DH, bool STREAM>
__device__ __forceinline__ void load_v_tile(KVTile<DH> &kv, const a16_t *vpages, int p0, int p1, int layer, int n_pages, int H, int h, int lane) {
    const int hl = lane >> 5, col = lane & 31;
#pragma unroll
    for (int g = 0; g < 2; ++g) {
        const u32x4_t *vp = reinterpret_cast<const u32x4_t *>(vpages + kv_block_base(layer, n_pages, g ? p1 : p0, H, h, DH));
#pragma unroll
        for (int dt = 0; dt < DH / 32; ++dt) kv.v[g][dt] = load_kv<STREAM>(vp + (32 * dt + col) * 2 + hl);
    }
}

// One workgroup of tree attention: (bx of nbx, h, b) are its coordinates in the launch shape described at the top of
// bf16_attn.hip, lds its ATTN_WAVES * 64 + ATTN_WAVES * (DH / 32) * 1024 floats of shared memory.  DEV: the final
// output is written with device-scope stores (the reader is another workgroup of the same kernel).  The function
// contains two workgroup barriers that every wave reaches unless the row is over capacity (uniform early return).
// tid: the thread's index in the workgroup.  The row has QW query tiles, or qsplit (QW = 1) hands each workgroup one of
// them.  The query tiles are kept in LDS, which takes 8 * DH / 32 registers per lane off a kernel that sits at the limit
// of 256.  They lie in the space of the O merge buffers (QW * DH * 64 bytes, never more than those), which are first
// written behind the barrier that follows the key loops of all waves.
template <int DH, int QW, bool PACKED, bool DEV>
__device__ __forceinline__ void attn_bf16_body(
    const u32x4_t *__restrict__ qbuf, const a16_t *__restrict__ kpages, const a16_t *__restrict__ vpages,
    const int32_t *__restrict__ page_table, int max_pages, int n_pages, int layer, const int32_t *__restrict__ seq_len,
    const TreeDev *__restrict__ tree, int T, int H, int qsplit, float scale, float *__restrict__ apart, void *out,
    int32_t *flags, int bx, int nbx, int h, int b, float *lds, int tid) {
    constexpr int KS = DH / 16, DT = DH / 32;
    constexpr bool STREAM = !DEV && QW == 1;               // with two query tiles to a workgroup two of its waves read the same bytes
    const int lane = tid & 63, wave = QW > 1 ? __builtin_amdgcn_readfirstlane(tid >> 6) : tid >> 6;      // a scalar: two query tiles are at the limit of registers
    const int hl = lane >> 5, col = lane & 31;
    constexpr int KWV = ATTN_WAVES / QW;
    const int qw = wave % QW, kwv = wave / QW;
    const int QTtot = (T + 31) >> 5;
    const int Tq = QTtot * 32;
    // qsplit: the workgroups of a (row, head) take different 32-query tiles and each sees all keys (no partial
    // records, no merge kernel); otherwise they split the keys and every workgroup holds all query tiles
    const int qtile = qsplit ? bx * QW + qw : qw;
    const int key_wgs = qsplit ? 1 : nbx;
    const int units = key_wgs * KWV;
    const int unit = (qsplit ? 0 : bx) * KWV + kwv;
    // true in every launch; kept because without the branch the compiler lays the layer kernel out differently, and a verification call
    // through it takes 1.3 % longer (7B, 64 rows 3827 -> 3875 us)
    const bool active = qtile < QTtot;
    const int32_t *pt = page_table + (size_t)b * max_pages;
    // Everything whose address does not depend on the row's length is requested before the length is known:
    // the queries, the ancestor masks and the page-table entries of this wave's first key tiles (the table
    // has max_pages entries for every row, so the reads are in bounds; entries past the row's pages are not used).
    enum { PG_AHEAD = 5 };                                 // page ids of this many key tiles per wave are fetched up front
    u32x4_t qreg[KS];
    uint64_t anc0 = 0ull, anc1 = 0ull;
    int pg[PG_AHEAD][2];
    if (active) {
        const size_t blk = (((size_t)b * H + h) * QTtot + qtile) * KS;
#pragma unroll
        for (int s = 0; s < KS; ++s) qreg[s] = qbuf[(blk + s) * 64 + lane];
        if (kwv == 0) {                            // one copy per query tile, written by the first wave of its key split
            u32x4_t *qs = reinterpret_cast<u32x4_t *>(lds + ATTN_WAVES * 64) + (size_t)qw * KS * 64;
#pragma unroll
            for (int s = 0; s < KS; ++s) qs[s * 64 + lane] = qreg[s];
        }
        const int query = qtile * 32 + col;
        if (query < T) { anc0 = tree->anc[query][0]; anc1 = tree->anc[query][1]; }
#pragma unroll
        for (int j = 0; j < PG_AHEAD; ++j) {
            const int t = unit + j * units;
            pg[j][0] = pt[min(2 * t, max_pages - 1)];             // checked below, where they are used
            pg[j][1] = pt[min(2 * t + 1, max_pages - 1)];
        }
    }
    const int L = seq_len[b];
    __syncthreads();                                       // the query tiles are in LDS (before any early return: every wave reaches it)
    const u32x4_t *qlds = reinterpret_cast<const u32x4_t *>(lds + ATTN_WAVES * 64) + (size_t)qw * KS * 64 + lane;
    if (L < 0 || L + T > max_pages * 16) {                 // uniform over the workgroup
        if (tid == 0 && bx == 0 && h == 0) atomicOr(flags, FLAG_CAPACITY);
        return;
    }
    const int total = L + T;
    const int n_tiles = (total + 31) >> 5;
    const int row_pages = (total + 15) >> 4;

    f32x16_t o[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int v = 0; v < 16; ++v) o[dt][v] = 0.f;
    float m_run = -INFINITY, l_run = 0.f;

    if (active && unit < n_tiles) {
        KVTile<DH> cur, nxt;
        // second page of a tile: absent when the row ends inside the first one (its keys are masked; any valid page will do)
        {
            const int p0 = checked_page(pg[0][0], n_pages, flags);
            const int p1 = (2 * unit + 1 < row_pages) ? checked_page(pg[0][1], n_pages, flags) : p0;
            load_k_tile<DH, STREAM>(cur, kpages, p0, p1, layer, n_pages, H, h, lane);
            load_v_tile<DH, STREAM>(cur, vpages, p0, p1, layer, n_pages, H, h, lane);
        }
        int it = 0;                                        // index of tile t among this wave's tiles
        for (int t = unit; t < n_tiles; t += units, ++it) {
            const bool more = t + units < n_tiles;
            int p0 = 0, p1 = 0;                            // pages of the next tile
            if (more) {
                const int tn = t + units;
                switch (it + 1) {                          // wave-uniform; keeps the page ids in scalar registers
                    case 1: p0 = pg[1][0]; p1 = pg[1][1]; break;
                    case 2: p0 = pg[2][0]; p1 = pg[2][1]; break;
                    case 3: p0 = pg[3][0]; p1 = pg[3][1]; break;
                    case 4: p0 = pg[4][0]; p1 = pg[4][1]; break;
                    default: p0 = pt[2 * tn]; p1 = (2 * tn + 1 < row_pages) ? pt[2 * tn + 1] : p0; break;
                }
                if (2 * tn + 1 >= row_pages) p1 = p0;
                p0 = checked_page(p0, n_pages, flags);                  // wave-uniform
                p1 = checked_page(p1, n_pages, flags);
                if (!DEV) {
                    load_k_tile<DH, STREAM>(nxt, kpages, p0, p1, layer, n_pages, H, h, lane);
                    load_v_tile<DH, STREAM>(nxt, vpages, p0, p1, layer, n_pages, H, h, lane);
                }
            }
            const int slot0 = t * 32;
            if (slot0 + 32 > total) {   // zero V of slots >= total (stale or never written): 0 * garbage must not appear
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
                        for (int dt = 0; dt < DT; ++dt) cur.v[g][dt][w] &= keep;
                    }
            }
            f32x16_t sc;
#pragma unroll
            for (int v = 0; v < 16; ++v) sc[v] = 0.f;
            int qoff = 0;
            asm volatile("" : "+v"(qoff));           // keeps the LDS reads of the queries inside the loop (hoisted, they are registers again)
#pragma unroll
            for (int s = 0; s < KS; ++s)
                sc = HYDRA_MFMA16(__builtin_bit_cast(a16x8_t, cur.k[s]), __builtin_bit_cast(a16x8_t, qlds[qoff + s * 64]), sc);
            // the layer kernel, whose waves hold weights as well, has one tile's registers: the next K comes once K is used
            if (DEV && more) load_k_tile<DH, STREAM>(cur, kpages, p0, p1, layer, n_pages, H, h, lane);
            bool moved;
            const float alpha = softmax_tile(sc, scale, slot0 + 32 > L, slot0, L, anc0, anc1, hl, m_run, l_run, moved);
            // the accumulators are rescaled only where some query's maximum moved (a factor of one otherwise; the first tile
            // has nothing to rescale).  Always in the layer kernel, where the branch costs registers that it lacks.
            if (DEV || (it > 0 && moved)) {
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
                    o[dt] = HYDRA_MFMA16(__builtin_bit_cast(a16x8_t, cur.v[g][dt]), __builtin_bit_cast(a16x8_t, pb), o[dt]);
            }
            if (DEV && more) load_v_tile<DH, STREAM>(cur, vpages, p0, p1, layer, n_pages, H, h, lane);
            if (!DEV && more) cur = nxt;
        }
    }

    // ---- merge the KWV key-split waves of each query tile through LDS
    // layout: ml[QW][KWV][2][32] then O[QW][KWV][DT*16][64]
    float *ml = lds;
    float *ob = lds + ATTN_WAVES * 64;
    if (hl == 0) {
        ml[((qw * KWV + kwv) * 2 + 0) * 32 + col] = m_run;
        ml[((qw * KWV + kwv) * 2 + 1) * 32 + col] = l_run;
    }
    __syncthreads();
    float m_tot = -INFINITY;
    for (int w = 0; w < KWV; ++w) m_tot = fmaxf(m_tot, ml[((qw * KWV + w) * 2 + 0) * 32 + col]);
    float l_tot = 0.f;
    for (int w = 0; w < KWV; ++w) {
        const float mw = ml[((qw * KWV + w) * 2 + 0) * 32 + col];
        l_tot += __expf(mw - (m_tot == -INFINITY ? 0.f : m_tot)) * ml[((qw * KWV + w) * 2 + 1) * 32 + col];
    }
    const float mine = __expf(m_run - (m_tot == -INFINITY ? 0.f : m_tot));
    {
        float *dst = ob + (size_t)(qw * KWV + kwv) * DT * 16 * 64 + lane;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int v = 0; v < 16; ++v) dst[(dt * 16 + v) * 64] = o[dt][v] * mine;
    }
    __syncthreads();
    if (!active) return;
    // the (band, group of 4 registers = 4 consecutive dims) items are shared out over the KWV waves of the query tile
    const int query = qtile * 32 + col;
    const bool final_out = key_wgs == 1;
    const float inv = final_out ? 1.0f / l_tot : 1.0f;
    float *rec = apart + ((((size_t)b * H + h) * nbx) + bx) * apart_record(Tq, DH);
    for (int id = kwv; id < DT * 4; id += KWV) {
        const int dt = id >> 2, g4 = id & 3;
        float acc[4] = {0.f, 0.f, 0.f, 0.f};
        for (int w = 0; w < KWV; ++w) {
            const float *src = ob + (size_t)(qw * KWV + w) * DT * 16 * 64 + lane;
#pragma unroll
            for (int q = 0; q < 4; ++q) acc[q] += src[(dt * 16 + 4 * g4 + q) * 64];
        }
        const int dim = 32 * dt + 8 * g4 + 4 * hl;
        if (final_out) {
            if (query < T) {
                const int m = b * T + query;
                if (PACKED) {
                    st_dev64<DEV>(reinterpret_cast<a16_t *>(out) + x_index<true>(m, h * DH + dim, H * DH),
                                  f2a_pack(acc[0] * inv, acc[1] * inv), f2a_pack(acc[2] * inv, acc[3] * inv));
                } else {
                    f32x4_t v4 = {acc[0] * inv, acc[1] * inv, acc[2] * inv, acc[3] * inv};
                    *reinterpret_cast<f32x4_t *>(reinterpret_cast<float *>(out) + ((size_t)m * H + h) * DH + dim) = v4;
                }
            }
        } else {
            f32x4_t v4 = {acc[0], acc[1], acc[2], acc[3]};
            *reinterpret_cast<f32x4_t *>(rec + (size_t)query * DH + dim) = v4;
        }
    }
    if (!final_out && kwv == 0 && hl == 0) {
        rec[(size_t)Tq * DH + query] = m_tot;
        rec[(size_t)Tq * DH + Tq + query] = l_tot;
    }
}

}  // namespace hydra
