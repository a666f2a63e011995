// Kernels of the draft phases (gather/concat, bias + SiLU, wave-level top-k)
// and of the integer tail of a step (greedy acceptance, cache compaction,
// state update).
#include <type_traits>

#include "device_common.h"
#include "internal.h"

namespace hydra {

// tree_tokens[b, 0] = root[b]   (node 0 is x_t); for trees of one node, otherwise the first phase's gather does it
__global__ void draft_root_kernel(const int32_t *root, int32_t *tree_tokens, int B, int T) {
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b < B) tree_tokens[(size_t)b * T] = root[b];
}

int launch_draft_root(hydra_ctx *c, hipStream_t s, int B, const int32_t *root, int32_t *tree_tokens) {
    hipLaunchKernelGGL(draft_root_kernel, dim3(ceil_div(B, 64)), dim3(64), 0, s, root, tree_tokens, B, c->tree.T);
    HYDRA_LAUNCH_CHECK("draft_root_kernel");
    return HYDRA_OK;
}

// ---------------------------------------------------------------------------
// Head input (paper, section 3): for expanding node n of phase i (depth i-1),
//   u = [h_last ; E[tok(p_0)] ; ... ; E[tok(p_{i-1})]],  p_0 = root, p_{i-1} = n,
// concatenated on the feature axis.  Row r = b * n_expand + j.
// grid = (rows, segments); segment 0 copies h_last, segment s >= 1 one embedding.
// Medusa-style heads (section 2) have segment 0 only; z_out then also receives
// h_last in fp32, the residual term of their first layer.  Phase 1 also writes the root token into the tree (node 0 is the
// only node that expands then, so segment 0 of its row does) and takes it from `root`: a kernel of its own for that cost
// 4.4 us of a draft.
// ---------------------------------------------------------------------------
template <bool BF>
__global__ void draft_gather_kernel(const TreeDev *tree, int phase, int include_root, const float *h_last, const int32_t *root,
                                    int32_t *tree_tokens, const typename Elem<BF>::type *E, int d, int V,
                                    int Kin, typename Act<BF>::type *out, float *z_out, int32_t *flags) {
    const int ne = tree->n_expand[phase];
    const int r = blockIdx.x, seg = blockIdx.y;
    const int b = r / ne, j = r - b * ne;
    const int n = tree->expand_nodes[tree->expand_off[phase] + j];
    typedef __attribute__((ext_vector_type(4))) uint32_t u4;
    typedef __attribute__((ext_vector_type(4))) float f4;
    if (seg == 0) {
        if (phase == 1 && threadIdx.x == 0) tree_tokens[(size_t)b * tree->T] = root[b];
        if (BF) {                                               // 8 columns per thread: one 16-byte store into the operand tile
            for (int k = threadIdx.x * 8; k < d; k += blockDim.x * 8) {
                const f4 v0 = *reinterpret_cast<const f4 *>(h_last + (size_t)b * d + k);
                const f4 v1 = *reinterpret_cast<const f4 *>(h_last + (size_t)b * d + k + 4);
                const u4 pk = {f2a_pack(v0[0], v0[1]), f2a_pack(v0[2], v0[3]), f2a_pack(v1[0], v1[1]), f2a_pack(v1[2], v1[3])};
                *reinterpret_cast<u4 *>(reinterpret_cast<a16_t *>(out) + x_index<true>(r, k, Kin)) = pk;
                if (z_out) {
                    *reinterpret_cast<f4 *>(z_out + (size_t)r * d + k) = v0;
                    *reinterpret_cast<f4 *>(z_out + (size_t)r * d + k + 4) = v1;
                }
            }
            return;
        }
        for (int k = threadIdx.x; k < d; k += blockDim.x) {
            const float v = h_last[(size_t)b * d + k];
            Act<BF>::st(out, x_index<BF>(r, k, Kin), v);
            if (z_out) z_out[(size_t)r * d + k] = v;
        }
        return;
    }
    // embedding of the path node at depth dd; n itself has depth phase-1
    const int dd = seg - 1 + (include_root ? 0 : 1);
    int a = n;
    for (int up = (phase - 1) - dd; up > 0; --up) a = tree->parent[a];
    int tok = phase == 1 ? root[b] : tree_tokens[(size_t)b * tree->T + a];
    if (tok < 0 || tok >= V) {
        if (threadIdx.x == 0) atomicOr(flags, FLAG_BAD_TOKEN);
        tok = 0;
    }
    if (BF) {
        for (int k = threadIdx.x * 8; k < d; k += blockDim.x * 8) {
            const u4 raw = *reinterpret_cast<const u4 *>(reinterpret_cast<const bf16_t *>(E) + (size_t)tok * d + k);     // 8 bfloat16
            u4 pk;
#pragma unroll
            for (int q = 0; q < 4; ++q) pk[q] = f2a_pack(__uint_as_float(raw[q] << 16), __uint_as_float(raw[q] & 0xffff0000u));
            *reinterpret_cast<u4 *>(reinterpret_cast<a16_t *>(out) + x_index<true>(r, seg * d + k, Kin)) = pk;
        }
        return;
    }
    for (int k = threadIdx.x; k < d; k += blockDim.x)
        Act<BF>::st(out, x_index<BF>(r, seg * d + k, Kin), Elem<BF>::ld(E, (size_t)tok * d + k));
}

int launch_draft_gather(hydra_ctx *c, hipStream_t s, int B, int phase, const float *h_last, const int32_t *root,
                        int32_t *tree_tokens, void *x_out, float *z_out, int32_t *flags) {
    const int ne = c->tree.n_expand[phase];
    const int inc = c->h.include_root_embedding ? 1 : 0;
    const int nseg = c->h.medusa ? 1 : 1 + (inc ? phase : phase - 1);
    const int Kin = nseg * c->m.d;
    dim3 grid(B * ne, nseg), block(256);
    const void *E = c->arena + c->off_embed;
    if (c->bf16) hipLaunchKernelGGL(draft_gather_kernel<true>, grid, block, 0, s, tree_dev(c), phase, inc, h_last, root, tree_tokens, (const bf16_t *)E, c->m.d, c->m.vocab, Kin, (a16_t *)x_out, z_out, flags);
    else         hipLaunchKernelGGL(draft_gather_kernel<false>, grid, block, 0, s, tree_dev(c), phase, inc, h_last, root, tree_tokens, (const float *)E, c->m.d, c->m.vocab, Kin, (float *)x_out, z_out, flags);
    HYDRA_LAUNCH_CHECK("draft_gather_kernel");
    return HYDRA_OK;
}

// z <- (residual ? z : 0) + SiLU(W u + b);  also written as the next GEMM input (16-bit family, where the product's K is split)
__global__ void bias_silu_kernel(const float *part, int S, int part_ld, size_t split_stride, const float *bias,
                                 float *z, int residual, int d, a16_t *out) {
    const int m = blockIdx.y;
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= d) return;
    float a = silu_f(part_sum(part, S, split_stride, (size_t)m * part_ld + k) + bias[k]);
    if (residual) a += z[(size_t)m * d + k];
    z[(size_t)m * d + k] = a;
    out[x_index<true>(m, k, d)] = f2a(a);
}

int launch_bias_silu(hydra_ctx *c, hipStream_t s, const float *part, int S, int part_ld, size_t split_stride,
                     const float *bias, float *z, bool residual, void *x_out, int M) {
    dim3 grid(ceil_div(c->m.d, 256), M), block(256);
    hipLaunchKernelGGL(bias_silu_kernel, grid, block, 0, s, part, S, part_ld, split_stride, bias, z, residual ? 1 : 0, c->m.d, (a16_t *)x_out);
    HYDRA_LAUNCH_CHECK("bias_silu_kernel");
    return HYDRA_OK;
}

// ---------------------------------------------------------------------------
// Top-k per row, ordered by (logit descending, token id ascending) (paper,
// section 2: children are the m most likely tokens, sorted).  The helpers come
// first (order, monotone keys, wave-wide reductions); the two kernels that use
// them, one wave per 1024-id chunk and one wave per row for the merge, are
// described above topk_chunk_kernel.
// ---------------------------------------------------------------------------
struct Cand { float v; int id; };
__device__ __forceinline__ bool better(float v, int id, float w, int jd) { return v > w || (v == w && id < jd); }

// Monotone 32-bit key of a float: a > b <=> key(a) > key(b).  -0 shares the key of +0 (they compare equal, so the
// token id decides between them) and a NaN gets the key of -infinity (it never wins, as with float comparisons).
__device__ __forceinline__ uint32_t order_key(float v) {
    uint32_t b = __float_as_uint(v);
    if ((b & 0x7fffffffu) > 0x7f800000u) b = 0xff800000u;
    if (b == 0x80000000u) b = 0u;
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}
__device__ __forceinline__ float key_value(uint32_t k) { return __uint_as_float((k & 0x80000000u) ? (k ^ 0x80000000u) : ~k); }

// Wave-wide max / min of a 32-bit unsigned value, the same in every lane: four cross-lane steps inside each row of
// 16 lanes (swap neighbours, swap pairs, mirror halves of 8, mirror the row), then the four rows meet in scalars.
template <bool MAX>
__device__ __forceinline__ uint32_t wave_reduce_u32(uint32_t x) {
    auto op = [](uint32_t a, uint32_t b) { return MAX ? (a > b ? a : b) : (a < b ? a : b); };
    x = op(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0xB1, 0xf, 0xf, false));    // quad_perm [1,0,3,2]
    x = op(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x4E, 0xf, 0xf, false));    // quad_perm [2,3,0,1]
    x = op(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x141, 0xf, 0xf, false));   // row_half_mirror
    x = op(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x140, 0xf, 0xf, false));   // row_mirror
    const uint32_t r0 = (uint32_t)__builtin_amdgcn_readlane((int)x, 0), r1 = (uint32_t)__builtin_amdgcn_readlane((int)x, 16);
    const uint32_t r2 = (uint32_t)__builtin_amdgcn_readlane((int)x, 32), r3 = (uint32_t)__builtin_amdgcn_readlane((int)x, 48);
    return op(op(r0, r1), op(r2, r3));
}

// best candidate of the wave in the (value descending, id ascending) order; every lane must be active
__device__ __forceinline__ Cand wave_best(Cand c) {
    const uint32_t key = order_key(c.v);
    const uint32_t kmax = wave_reduce_u32<true>(key);
    const uint32_t idmin = wave_reduce_u32<false>(key == kmax ? (uint32_t)c.id : 0xffffffffu);
    return Cand{key_value(kmax), (int)idmin};
}

// Top-k of a logits row in two kernels.  One workgroup on 32000 logits is bound by its own instruction issue (every
// wave rescans its registers once per extracted entry, and the waves of a workgroup share four SIMDs), so the row is
// cut into chunks of 1024 ids, one workgroup of four waves each, spread over the chip: lane l of a wave holds four ids
// base + l, base + 64 + l, ... as monotone keys (order_key; key 0 is below every real key and marks an absent or
// already extracted entry), k rounds leave the wave's k best, in order, as (key, id) pairs, and the first wave picks the
// chunk's k best of those.  The second kernel, one wave per row, picks the k best of the at most 32 * k survivors of the
// chunks in the same (value descending, id ascending) order.
enum { TOPK_CHUNK = 1024, TOPK_MAX_CHUNKS = 32 };

// lane's share of a chunk: ids base + i * 64 + lane
template <int N>
__device__ __forceinline__ void topk_load(uint32_t (&key)[N], const float *part, int S, size_t split_stride, size_t row, int base, int V, int lane) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const int id = base + i * 64 + lane;
        key[i] = id < V ? order_key(part_sum(part, S, split_stride, row + id)) : 0u;
    }
}
// the k best of a wave's 64 N ids, best first, entry t at out[t * stride]; key 0: the wave ran out of entries
template <int N>
__device__ __forceinline__ void topk_rounds(uint32_t (&key)[N], int k, int base, int lane, uint2 *out, int stride) {
    for (int t = 0; t < k; ++t) {
        // the lane's best: the first maximum in slot order is also its lowest id
        uint32_t bk = 0u, bs = 0u;
#pragma unroll
        for (int i = 0; i < N; ++i)
            if (key[i] > bk) { bk = key[i]; bs = (uint32_t)i; }
        const uint32_t kmax = wave_reduce_u32<true>(bk);
        const uint32_t idmin = wave_reduce_u32<false>(bk == kmax && kmax != 0u ? (uint32_t)base + bs * 64u + (uint32_t)lane : 0xffffffffu);
        if (idmin != 0xffffffffu) {                                   // wave-uniform; the winner's owner retires it
            const uint32_t off = idmin - (uint32_t)base;
            const uint32_t slot = off >> 6;
            const bool owner = (off & 63u) == (uint32_t)lane;
#pragma unroll
            for (int i = 0; i < N; ++i)
                if ((uint32_t)i == slot && owner) key[i] = 0u;
        }
        if (lane == 0) out[t * stride] = make_uint2(kmax, idmin);
    }
}

// The k best of the entries that a wave's lanes hold, without k rounds (the second step of every kernel here): any entry among them is at least
// as large as the k-th largest of the 64 lane maxima, so the lanes rank their maxima against each other (64 scalar broadcasts), drop
// everything below that bound, put what is left (a little over k entries) one per lane through LDS and rank those the same
// way; ranks follow the order, ids break ties, so nothing has to be extracted in turn.  The bound is as good as the maxima are: the
// callers deal the sorted lists of their first step out so that the lanes hold the heads of all lists (a list per group of lanes,
// its ranks in turn), not one rank of two lists each.  More than 64 entries at or above the bound (many equal logits) go back to k
// rounds of a maximum over the wave, as do one or two children.  Draft of one head, rounds against ranking: one child 15.4 / 16.0 / 22.5 us
// against 16.9 / 17.5 / 25.8 (1000 / 4000 / 32000 ids), two 15.7 / 16.8 / 23.2 against 17.2 / 18.0 / 26.2; three 16.1 / 17.6 / 23.7 against
// 17.4 / 18.3 / 26.4, five 17.1 / 19.1 / 25.5 against 18.0 / 19.1 / 27.0: with the few entries that a lane holds now the line could lie higher.

// key[i] (0: no entry) with id[i]; put(t, key, id) is called for t < k by one lane each: key 0 and id ~0 past the last entry.
// list: 64 entries of LDS.
template <int N, class Put>
__device__ __forceinline__ void wave_top_k(uint32_t (&key)[N], const uint32_t (&id)[N], int k, uint2 *list, int lane, Put put) {
    if (k > 2) {
        uint32_t best = 0u;
#pragma unroll
        for (int i = 0; i < N; ++i) best = max(best, key[i]);
        int rank = 0;                                                     // of this lane's maximum; equal ones by lane number
#pragma unroll 8
        for (int l = 0; l < 64; ++l) {
            const uint32_t o = (uint32_t)__builtin_amdgcn_readlane((int)best, l);
            rank += (o > best || (o == best && l < lane)) ? 1 : 0;
        }
        const uint64_t at = __ballot(rank == k - 1);                      // k <= HYDRA_MAX_TOPK = 32: exactly one lane
        const uint32_t bound = max((uint32_t)__builtin_amdgcn_readlane((int)best, __builtin_ctzll(at)), 1u);
        int count = 0;
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const uint64_t has = __ballot(key[i] >= bound);
            if (key[i] >= bound) {
                const int pos = count + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(has >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)has, 0u));
                if (pos < 64) list[pos] = make_uint2(key[i], id[i]);
            }
            count += __popcll(has);
        }
        if (count <= 64) {                                                // wave-uniform
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");         // LDS is in order within a wave; keep the compiler from reordering
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            const uint2 e = lane < count ? list[lane] : make_uint2(0u, 0xffffffffu);
            int r = 0;
            for (int l = 0; l < count; ++l) {
                const uint32_t ok = (uint32_t)__builtin_amdgcn_readlane((int)e.x, l), oi = (uint32_t)__builtin_amdgcn_readlane((int)e.y, l);
                r += (ok > e.x || (ok == e.x && oi < e.y)) ? 1 : 0;
            }
            if (lane < count && r < k) put(r, e.x, e.y);
            if (lane >= count && lane < k) put(lane, 0u, 0xffffffffu);     // fewer entries than k
            return;
        }
    }
    for (int t = 0; t < k; ++t) {
        uint32_t bk = 0u, bi = 0xffffffffu;
#pragma unroll
        for (int i = 0; i < N; ++i)
            if (key[i] > bk || (key[i] == bk && bk != 0u && id[i] < bi)) { bk = key[i]; bi = id[i]; }
        const uint32_t kmax = wave_reduce_u32<true>(bk);
        const uint32_t idmin = wave_reduce_u32<false>(bk == kmax && kmax != 0u ? bi : 0xffffffffu);
#pragma unroll
        for (int i = 0; i < N; ++i)
            if (id[i] == idmin) key[i] = 0u;                          // ids are unique
        if (lane == 0) put(t, kmax, idmin);
    }
}

// A chunk of 1024 ids: four waves find the k best of 256 each (four entries to a lane: rescanning them is what a round costs), the
// first one picks from those.  One wave with sixteen entries to a lane took 10.4 us a launch (7B, up to 10 children), this 6.9.
__global__ __launch_bounds__(TOPK_CHUNK / 4) void topk_chunk_kernel(const float *part, int S, int part_ld, size_t split_stride, int V,
                                                                     const TreeDev *tree, int ne, int expand_off, uint2 *surv) {
    constexpr int WAVES = TOPK_CHUNK / 256;
    __shared__ uint2 best[WAVES * HYDRA_MAX_TOPK];
    __shared__ uint2 list[64];
    const int r = blockIdx.y, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int base = blockIdx.x * TOPK_CHUNK + wave * 256;
    // the logits first: their addresses need nothing from the tree tables, whose dependent lookups follow
    uint32_t key[4];
    topk_load(key, part, S, split_stride, (size_t)r * part_ld, base, V, lane);
    const int k = tree->expand_k[expand_off + r % ne];
    topk_rounds(key, k, base, lane, best + wave, WAVES);
    __syncthreads();
    if (wave > 0) return;
    uint2 *out = surv + ((size_t)r * gridDim.x + blockIdx.x) * HYDRA_MAX_TOPK;
    uint32_t mk[WAVES * HYDRA_MAX_TOPK / 64], mi[WAVES * HYDRA_MAX_TOPK / 64];
#pragma unroll
    for (int i = 0; i < WAVES * HYDRA_MAX_TOPK / 64; ++i) {
        const int q = i * 64 + lane;
        const uint2 e = q < WAVES * k ? best[q] : make_uint2(0u, 0xffffffffu);
        mk[i] = e.x; mi[i] = e.y;
    }
    wave_top_k(mk, mi, k, list, lane, [&](int t, uint32_t kk, uint32_t ii) { out[t] = make_uint2(kk, ii); });
}

__global__ __launch_bounds__(64) void topk_merge_kernel(const uint2 *surv, int chunks, int share_log2, const TreeDev *tree, int ne,
                                                         int expand_off, int32_t *tree_tokens) {
    __shared__ uint2 list[64];
    const int r = blockIdx.x, lane = threadIdx.x;
    const int b = r / ne, j = r - b * ne;
    const int k = tree->expand_k[expand_off + j];
    const int first = tree->expand_first[expand_off + j];
    // 64 lanes over the chunks, at most 32 of them: 1 << share_log2 lanes to a chunk, which take its survivors in turn: an address without a
    // division, and no more entries per lane than there have to be.  (Two lanes to a chunk whatever their number: five chunks kept ten
    // lanes busy, no bound came out of their maxima and 12 and more children went back to rounds: one row of 5000 logits, 16 / 32
    // children, a draft of one head 31.3 / 48.0 us, 20.3 / 26.0 now.)
    const int chunk = lane >> share_log2, part = lane & ((1 << share_log2) - 1);
    const uint2 *in = surv + ((size_t)r * chunks + chunk) * HYDRA_MAX_TOPK;
    int32_t *out = tree_tokens + (size_t)b * tree->T + first;
    auto merge = [&](auto N) {
        uint32_t mk[decltype(N)::value], mi[decltype(N)::value];
#pragma unroll
        for (int i = 0; i < decltype(N)::value; ++i) {
            const int q = (i << share_log2) + part;
            uint2 e = make_uint2(0u, 0xffffffffu);
            if (q < k && chunk < chunks) e = in[q];
            mk[i] = e.x; mi[i] = e.y;
        }
        wave_top_k(mk, mi, k, list, lane, [&](int t, uint32_t, uint32_t ii) { out[t] = (int32_t)ii; });
    };
    if (k <= 2 << share_log2) merge(std::integral_constant<int, 2>{});
    else if (k <= 6 << share_log2) merge(std::integral_constant<int, 6>{});
    else merge(std::integral_constant<int, HYDRA_MAX_TOPK / 2>{});
}

// Small vocabularies: both kernels in one, a wave per 256 ids (four to a lane: rescanning the lane's entries is what a round
// costs) and the survivors in LDS, at most 16 * 32.  One row of 1000 logits took 7.9 + 3.8 us with the pair of kernels; a draft of
// one head at 4096 ids takes 10.8 / 15.6 / 25.4 us for 1 / 8 / 32 children, with the pair 12.7 / 18.5 / more.
enum { TOPK_ROW_PART = 256, TOPK_ROW_WAVES = 16 };
template <int WAVES>
__global__ __launch_bounds__(64 * WAVES) void topk_row_kernel(const float *part, int S, int part_ld, size_t split_stride, int V,
                                                               const TreeDev *tree, int ne, int expand_off, int32_t *tree_tokens) {
    __shared__ uint2 surv[WAVES * HYDRA_MAX_TOPK];
    __shared__ uint2 list[64];
    const int r = blockIdx.x, b = r / ne, lane = threadIdx.x & 63, wave = threadIdx.x >> 6, waves = blockDim.x >> 6;
    uint32_t key[TOPK_ROW_PART / 64];
    topk_load(key, part, S, split_stride, (size_t)r * part_ld, wave * TOPK_ROW_PART, V, lane);
    const int at = expand_off + r - b * ne, k = tree->expand_k[at];
    int32_t *out = tree_tokens + (size_t)b * tree->T + tree->expand_first[at];
    topk_rounds(key, k, wave * TOPK_ROW_PART, lane, surv + wave, waves);
    __syncthreads();
    if (wave > 0) return;
    uint32_t mk[WAVES * HYDRA_MAX_TOPK / 64], mi[WAVES * HYDRA_MAX_TOPK / 64];
#pragma unroll
    for (int i = 0; i < WAVES * HYDRA_MAX_TOPK / 64; ++i) {
        const int q = i * 64 + lane;
        const uint2 e = q < waves * k ? surv[q] : make_uint2(0u, 0xffffffffu);
        mk[i] = e.x; mi[i] = e.y;
    }
    wave_top_k(mk, mi, k, list, lane, [&](int t, uint32_t, uint32_t ii) { out[t] = (int32_t)ii; });
}

// Any-V fallback: k rounds over memory, each picking the best entry that comes
// strictly after the previous winner in the (value desc, id asc) order.
__global__ __launch_bounds__(256) void topk_scan_kernel(const float *part, int S, int part_ld, size_t split_stride,
                                                         int V, const TreeDev *tree, int phase, int32_t *tree_tokens) {
    const int ne = tree->n_expand[phase];
    const int r = blockIdx.x;
    const int b = r / ne, j = r - b * ne;
    const int n = tree->expand_nodes[tree->expand_off[phase] + j];
    const int k = tree->n_children[n];
    __shared__ Cand red[4];
    __shared__ Cand prev;
    if (threadIdx.x == 0) { prev.v = INFINITY; prev.id = -1; }
    __syncthreads();
    for (int t = 0; t < k; ++t) {
        const Cand p = prev;
        Cand c = {-INFINITY, 0x7fffffff};
        for (int id = threadIdx.x; id < V; id += 256) {
            const float v = part_sum(part, S, split_stride, (size_t)r * part_ld + id);
            const bool after = better(p.v, p.id, v, id);
            if (after && better(v, id, c.v, c.id)) { c.v = v; c.id = id; }
        }
        c = wave_best(c);
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = c;
        __syncthreads();
        if (threadIdx.x == 0) {
            Cand w = red[0];
            for (int i = 1; i < 4; ++i) if (better(red[i].v, red[i].id, w.v, w.id)) w = red[i];
            prev = w;
            tree_tokens[(size_t)b * tree->T + tree->first_child[n] + t] = w.id;
        }
        __syncthreads();
    }
}

size_t topk_scratch_bytes(const hydra_ctx *c, int rows) {
    return (size_t)rows * TOPK_MAX_CHUNKS * HYDRA_MAX_TOPK * sizeof(uint2);
}

int launch_topk(hydra_ctx *c, hipStream_t s, const float *part, int S, int part_ld, size_t split_stride, int B,
                int phase, int32_t *tree_tokens, void *scratch) {
    const int ne = c->tree.n_expand[phase], eoff = c->tree.expand_off[phase];
    const int rows = B * ne;
    const int chunks = ceil_div(c->m.vocab, TOPK_CHUNK);
    if (const int waves = ceil_div(c->m.vocab, TOPK_ROW_PART); waves <= TOPK_ROW_WAVES) {
        if (waves <= 4) hipLaunchKernelGGL(topk_row_kernel<4>, dim3(rows), dim3(64 * waves), 0, s, part, S, part_ld, split_stride, c->m.vocab, tree_dev(c), ne, eoff, tree_tokens);
        else            hipLaunchKernelGGL(topk_row_kernel<TOPK_ROW_WAVES>, dim3(rows), dim3(64 * waves), 0, s, part, S, part_ld, split_stride, c->m.vocab, tree_dev(c), ne, eoff, tree_tokens);
        HYDRA_LAUNCH_CHECK("topk_row_kernel");
    } else if (chunks <= TOPK_MAX_CHUNKS) {
        hipLaunchKernelGGL(topk_chunk_kernel, dim3(chunks, rows), dim3(TOPK_CHUNK / 4), 0, s, part, S, part_ld, split_stride, c->m.vocab, tree_dev(c), ne, eoff, (uint2 *)scratch);
        HYDRA_LAUNCH_CHECK("topk_chunk_kernel");
        int share_log2 = 1;                                    // lanes of the merge's wave per chunk
        while (2 * chunks << share_log2 <= 64) ++share_log2;
        hipLaunchKernelGGL(topk_merge_kernel, dim3(rows), dim3(64), 0, s, (const uint2 *)scratch, chunks, share_log2, tree_dev(c), ne, eoff, tree_tokens);
        HYDRA_LAUNCH_CHECK("topk_merge_kernel");
    } else {
        hipLaunchKernelGGL(topk_scan_kernel, dim3(rows), dim3(256), 0, s, part, S, part_ld, split_stride, c->m.vocab, tree_dev(c), phase, tree_tokens);
        HYDRA_LAUNCH_CHECK("topk_scan_kernel");
    }
    return HYDRA_OK;
}

// ---------------------------------------------------------------------------
// Greedy acceptance (paper, section 2): walk down from the root while some
// child carries the base model's most likely token.  One thread per row.
// ---------------------------------------------------------------------------
__global__ void accept_kernel(const TreeDev *tree, int B, const int32_t *tree_tokens, const int32_t *argmax,
                              int32_t *n_acc, int32_t *path, int32_t *next_root, int32_t *last_node) {
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= B) return;
    const int T = tree->T, plen = tree->max_depth + 1;
    const int32_t *tok = tree_tokens + (size_t)b * T;
    const int32_t *am = argmax + (size_t)b * T;
    int32_t *p = path + (size_t)b * plen;
    int cur = 0, len = 1;
    p[0] = 0;
    for (;;) {
        const int g = am[cur];
        const int fc = tree->first_child[cur], nc = tree->n_children[cur];
        int nxt = -1;
        for (int i = 0; i < nc; ++i)
            if (tok[fc + i] == g) { nxt = fc + i; break; }
        if (nxt < 0) break;
        cur = nxt;
        p[len++] = cur;
    }
    for (int i = len; i < plen; ++i) p[i] = -1;
    n_acc[b] = len;
    next_root[b] = am[cur];
    last_node[b] = cur;
}

int launch_accept(hydra_ctx *c, hipStream_t s, int B, const int32_t *tree_tokens, const int32_t *argmax,
                  int32_t *n_acc, int32_t *path, int32_t *next_root, int32_t *last_node) {
    hipLaunchKernelGGL(accept_kernel, dim3(ceil_div(B, 64)), dim3(64), 0, s, tree_dev(c), B, tree_tokens, argmax, n_acc, path, next_root, last_node);
    HYDRA_LAUNCH_CHECK("accept_kernel");
    return HYDRA_OK;
}

// ---------------------------------------------------------------------------
// Typical acceptance (paper, section 6.3): the child c of node n passes if
//   p(tok[c]) > min(eps, alpha * exp(-H)),  p = softmax(logits[n] / tau), H = entropy(p).
// Kernel 1, one workgroup per (row, node with children): max, Z = sum exp(z - max),
// S = sum exp(z - max) (z - max) with z = logit / tau, so H = ln Z - S / Z; then the
// test for each child.  Kernel 2, one workgroup per row: the deepest node whose whole
// path passes (lowest id among equally deep ones), and the next root: the most likely
// token of that node, or the token at which the cumulative distribution of
// softmax(logits / tau), taken in id order, first exceeds u.
//
// Both are one workgroup on one row of logits, bound by the round trips to memory and the
// reductions between them.  A thread therefore takes 32 logits of a row of up to 32768 into
// registers at once (TypRow: 16-byte loads) and everything after that runs from there; longer
// rows go through in pieces of that size.  At 1024 threads a wave has 128 registers: nothing
// but the 32 logits may live across the steps.  Reading the row once per pass, four bytes at a
// time, and walking the tree in one thread took 17.3 us and 40.1 us (4 rows x 64 nodes, V = 32000).
// ---------------------------------------------------------------------------
enum { TYP_THREADS = 1024, TYP_GROUPS = 8, TYP_STRIPE = TYP_THREADS * 4, TYP_PIECE = TYP_STRIPE * TYP_GROUPS };

// One piece of a row in registers: thread t holds groups of four consecutive ids, group i at (i * 1024 + t) * 4, so that the
// ids ascend with i first and with the thread second.  Rows start wherever V puts them: the loads ask for no more than float
// alignment.  Groups past V4 = V rounded down to 4 are -infinity: never a maximum, and of weight exp(-inf / tau) = 0, except that
// an infinite temperature makes that exp(-inf * 0), not a number: then (PAD) their weight is 0 by their id.  A comparison per
// entry at every temperature cost typical_stats_kernel 0.5 of 6.7 us.
// The up to three entries behind V4 (TypTail) are the same loads in every thread.  Letting the group that V cuts take them, entry
// by entry, puts branches between the loads: the stats of 4 rows took 6.9 us at V = 32000 and 12.1 at 50257, so 6.7 and 10.8.
struct TypTail { float x[3]; };
__device__ __forceinline__ TypTail typ_tail(const float *__restrict__ row, int V, int V4) {
    TypTail t;
#pragma unroll
    for (int k = 0; k < 3; ++k) t.x[k] = V4 + k < V ? row[V4 + k] : -INFINITY;
    return t;
}
struct TypRow {
    float x[TYP_GROUPS][4];
    __device__ __forceinline__ int id(int piece, int i) const { return piece * TYP_PIECE + i * TYP_STRIPE + (int)threadIdx.x * 4; }
    // the same, worked out where it is used: the id of every group kept across the steps costs more registers than there are
    __device__ __forceinline__ int id_here(int piece, int i) const {
        int t = (int)threadIdx.x;
        asm volatile("" : "+v"(t));
        return piece * TYP_PIECE + i * TYP_STRIPE + t * 4;
    }
    __device__ __forceinline__ void load(const float *__restrict__ row, int V4, int piece) {
        typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));
#pragma unroll
        for (int i = 0; i < TYP_GROUPS; ++i) {
            const int v = id(piece, i);
            f4u t = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
            if (v < V4) t = *reinterpret_cast<const f4u *>(row + v);
#pragma unroll
            for (int e = 0; e < 4; ++e) x[i][e] = t[e];
        }
    }
    __device__ __forceinline__ float largest() const {
        float m = -INFINITY;
#pragma unroll
        for (int i = 0; i < TYP_GROUPS; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) m = fmaxf(m, x[i][e]);
        return m;
    }
};

// over the workgroup in a fixed order; every thread gets the result
__device__ __forceinline__ float block_reduce(float v, float *sh, bool is_max) {
    v = is_max ? wave_max(v) : wave_sum(v);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    __syncthreads();
    if (lane == 0) sh[wave] = v;
    __syncthreads();
    float r = sh[0];
    for (int w = 1; w < (int)(blockDim.x >> 6); ++w) r = is_max ? fmaxf(r, sh[w]) : r + sh[w];   // fixed order
    return r;
}

__global__ __launch_bounds__(TYP_THREADS) void typical_stats_kernel(const float *__restrict__ logits, int V,
                                                                     const TreeDev *tree, const int32_t *__restrict__ tree_tokens,
                                                                     float inv_tau, float eps, float alpha,
                                                                     int32_t *__restrict__ ok, int32_t *flags, int T) {
    __shared__ float sh[16];
    __shared__ float2 sh2[16];
    const int n = blockIdx.x, b = blockIdx.y;
    const float *row = logits + ((size_t)b * T + n) * V;
    const int nc = tree->n_children[n], first = tree->first_child[n], V4 = V & ~3;
    if (nc == 0) return;                                            // uniform over the workgroup
    TypRow r;
    r.load(row, V4, 0);
    const TypTail tail = typ_tail(row, V, V4);
    int tok = 0;
    float xt = 0.f;
    if ((int)threadIdx.x < nc) {                                    // at most 32 children; their logits are fetched with the row
        tok = tree_tokens[(size_t)b * T + first + threadIdx.x];
        if (tok < 0 || tok >= V) { atomicOr(flags, FLAG_BAD_TOKEN); tok = 0; }
        xt = row[tok];
    }
    const int pieces = (V + TYP_PIECE - 1) / TYP_PIECE;
    float m = fmaxf(fmaxf(r.largest(), tail.x[0]), fmaxf(tail.x[1], tail.x[2]));
    for (int pc = 1; pc < pieces; ++pc) { TypRow q; q.load(row, V4, pc); m = fmaxf(m, q.largest()); }
    m = block_reduce(m, sh, true);
    float z = 0.f, sz = 0.f;
    auto one = [&](float x, bool in) {
        const float t = (x - m) * inv_tau;                          // <= 0
        const float ex = in ? __expf(t) : 0.f;
        z += ex;
        sz += ex > 0.f ? ex * t : 0.f;                              // exp underflow: 0 * (-inf) must not appear
    };
    auto add = [&](auto PAD, int pc) {
#pragma unroll
        for (int i = 0; i < TYP_GROUPS; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) one(r.x[i][e], !decltype(PAD)::value || r.id(pc, i) < V4);
    };
    for (int pc = 0; pc < pieces; ++pc) {
        if (pieces > 1) r.load(row, V4, pc);
        if (inv_tau > 0.f) add(std::false_type{}, pc);
        else               add(std::true_type{}, pc);
    }
    if (threadIdx.x == 0) {
#pragma unroll
        for (int k = 0; k < 3; ++k) one(tail.x[k], V4 + k < V);
    }
    z = wave_sum(z);
    sz = wave_sum(sz);
    if ((threadIdx.x & 63) == 0) sh2[threadIdx.x >> 6] = float2{z, sz};
    __syncthreads();
    if ((int)threadIdx.x >= nc) return;
    z = 0.f; sz = 0.f;
    for (int w = 0; w < 16; ++w) { z += sh2[w].x; sz += sh2[w].y; }
    const float H = __logf(z) - sz / z;
    const float th = fminf(eps, alpha * __expf(-H));
    const float p = __expf((xt - m) * inv_tau) / z;
    ok[(size_t)b * T + first + threadIdx.x] = p > th ? 1 : 0;
}

// next_root by u: a stripe is the 4096 ids that the workgroup holds side by side.  Every stripe is reduced to one sum per
// wave; the stripe in which the cumulative mass exceeds u times the total, the wave inside it, and then lane and id inside
// that wave follow from prefix sums of ever smaller pieces, each starting from the very number at which the piece before it
// ended, and only pieces that hold any mass are taken: the token drawn always has a positive weight.  4 rows: 7.4 us at
// V = 32000, 7.3 at 32003, 15.0 at 50257.  A scan of every stripe over the lanes instead of the one that matters keeps a
// prefix sum per group alive (16 registers spilled, 192 where V ruled out 16-byte loads) and took 16.2, 28.6 and 75.3.
__global__ __launch_bounds__(TYP_THREADS) void typical_select_kernel(const float *__restrict__ logits, int V, const TreeDev *tree,
                                                                      const int32_t *__restrict__ ok, float inv_tau,
                                                                      const float *__restrict__ u, int32_t *n_acc,
                                                                      int32_t *path, int32_t *next_root, int32_t *last_node, int T) {
    __shared__ float sh[16];
    __shared__ uint64_t pass[2];
    __shared__ int bestw[2];
    const int b = blockIdx.x, plen = tree->max_depth + 1, V4 = V & ~3;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    // Waves 0 and 1 hold one node per lane (T <= 128): a node is accepted if its own test and those of all its ancestors
    // passed, which its ancestor mask says; the winner is the deepest, then the lowest id.
    const int c = threadIdx.x;
    int dep = 0;
    uint64_t anc0 = 0ull, anc1 = 0ull;
    if (wave < 2) {
        bool okc = false;
        if (c < T) {
            okc = c == 0 || ok[(size_t)b * T + c] != 0;
            dep = tree->depth[c]; anc0 = tree->anc[c][0]; anc1 = tree->anc[c][1];
        }
        const uint64_t bits = __ballot(okc);
        if (lane == 0) pass[wave] = bits;
    }
    __syncthreads();
    if (wave < 2) {
        const bool reach = c < T && (anc0 & ~pass[0]) == 0ull && (anc1 & ~pass[1]) == 0ull;
        const uint32_t key = reach ? ((uint32_t)dep << 8 | (uint32_t)(255 - c)) : 0u;
        const uint32_t kmax = wave_reduce_u32<true>(key);
        if (lane == 0) bestw[wave] = (int)kmax;
    }
    __syncthreads();
    const uint32_t kbest = (uint32_t)__builtin_amdgcn_readfirstlane(max(bestw[0], bestw[1]));      // node 0 always counts: never 0; scalar, and with it the row's address
    const int best = 255 - (int)(kbest & 255u);
    const float *row = logits + ((size_t)b * T + best) * V;
    TypRow r;
    r.load(row, V4, 0);                                             // requested before the path is written out
    const TypTail tail = typ_tail(row, V, V4);
    if (threadIdx.x == 0) {
        const int len = (int)(kbest >> 8) + 1;
        int32_t *p = path + (size_t)b * plen;
        int cur = best;
        for (int j = len - 1; j >= 0; --j) { p[j] = cur; cur = tree->parent[cur]; }
        n_acc[b] = len;
        last_node[b] = best;
    }
    for (int j = (int)(kbest >> 8) + 1 + threadIdx.x; j < plen; j += TYP_THREADS) path[(size_t)b * plen + j] = -1;
    const int pieces = (V + TYP_PIECE - 1) / TYP_PIECE;
    if (!u) {
        // most likely token, lowest id at ties
        float bv = -INFINITY; int bi = 0x7fffffff;
        for (int pc = 0; pc < pieces; ++pc) {
            if (pc) r.load(row, V4, pc);
#pragma unroll
            for (int i = 0; i < TYP_GROUPS; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (r.x[i][e] > bv) { bv = r.x[i][e]; bi = r.id(pc, i) + e; }      // ascending ids per thread: first maximum kept
        }
        if (threadIdx.x == 0) {
#pragma unroll
            for (int k = 0; k < 3; ++k)
                if (tail.x[k] > bv) { bv = tail.x[k]; bi = V4 + k; }
        }
        Cand cnd = wave_best(Cand{bv, bi});
        __shared__ Cand red[16];
        if (lane == 0) red[wave] = cnd;
        __syncthreads();
        if (threadIdx.x == 0) {
            Cand w = red[0];
            for (int i = 1; i < 16; ++i) if (better(red[i].v, red[i].id, w.v, w.id)) w = red[i];
            next_root[b] = w.id;
        }
        return;
    }
    float m = fmaxf(fmaxf(r.largest(), tail.x[0]), fmaxf(tail.x[1], tail.x[2]));
    for (int pc = 1; pc < pieces; ++pc) { TypRow q; q.load(row, V4, pc); m = fmaxf(m, q.largest()); }
    m = block_reduce(m, sh, true);
    __shared__ float part[16][TYP_GROUPS];                          // [wave][stripe] of one piece
    float sum_a = 0.f, sum_b = 0.f;                                  // lane l: the sums of stripes l / 16 and 4 + l / 16
    auto stripes = [&](int pc) {                                     // piece pc: its weights in place of the logits, part, sum_a, sum_b
        if (pieces > 1) r.load(row, V4, pc);
        auto weights = [&](auto PAD) {
#pragma unroll
            for (int i = 0; i < TYP_GROUPS; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) r.x[i][e] = !decltype(PAD)::value || r.id_here(pc, i) < V4 ? __expf((r.x[i][e] - m) * inv_tau) : 0.f;
        };
        if (inv_tau > 0.f) weights(std::false_type{});
        else               weights(std::true_type{});
        float s[TYP_GROUPS];
#pragma unroll
        for (int i = 0; i < TYP_GROUPS; ++i) s[i] = (r.x[i][0] + r.x[i][1]) + (r.x[i][2] + r.x[i][3]);
        // all stripes together: each step a lane keeps the ones that agree with one bit of its number and hands the others over
#pragma unroll
        for (int hf = TYP_GROUPS / 2; hf > 0; hf >>= 1) {
            const bool up = (lane & hf) != 0;
#pragma unroll
            for (int q = 0; q < hf; ++q) {
                const float keep = up ? s[q + hf] : s[q], give = up ? s[q] : s[q + hf];
                s[q] = keep + __shfl_xor(give, hf, 64);
            }
        }
#pragma unroll
        for (int o = TYP_GROUPS; o < 64; o <<= 1) s[0] += __shfl_xor(s[0], o, 64);
        __syncthreads();                                             // every reader of the last piece's part is done
        if (lane < TYP_GROUPS) part[wave][lane] = s[0];
        __syncthreads();
        sum_a = part[lane & 15][lane >> 4];
        sum_b = part[lane & 15][4 + (lane >> 4)];
#pragma unroll
        for (int o = 1; o < 16; o <<= 1) { sum_a += __shfl_xor(sum_a, o, 64); sum_b += __shfl_xor(sum_b, o, 64); }
    };
    auto stripe = [&](int i) { return __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(i < 4 ? sum_a : sum_b), (i & 3) * 16)); };
    auto prefix = [&](float v, int width) {                          // inclusive, over lanes 0 .. width - 1
        for (int o = 1; o < width; o <<= 1) {
            const float t = __shfl_up(v, o, 64);
            if (lane >= o) v += t;
        }
        return v;
    };
    // the first of the lanes that hold mass whose prefix, on top of `from`, exceeds the target; the last of them where rounding leaves none
    auto crossing = [&](float v, float incl, float from, float target, bool in) {
        const uint64_t has = __ballot(in && v > 0.f), hit = __ballot(in && v > 0.f && from + incl > target);
        return hit ? __builtin_ctzll(hit) : 63 - __builtin_clzll(has);
    };
    float total = 0.f;
    for (int pc = 0; pc < pieces; ++pc) {
        stripes(pc);
#pragma unroll
        for (int i = 0; i < TYP_GROUPS; ++i) total += stripe(i);     // the same in every thread
    }
    float wt[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        wt[k] = V4 + k < V ? __expf((tail.x[k] - m) * inv_tau) : 0.f;
        total += wt[k];
    }
    const float target = u[b] * total;
    float cum = 0.f;
    int at = -1, pc = 0;
    for (; pc < pieces && target >= 0.f; ++pc) {                     // a negative u ends at the last token, as one of 1 or more and NaN do
        if (pieces > 1) stripes(pc);
#pragma unroll
        for (int i = 0; i < TYP_GROUPS; ++i) {
            if (at >= 0) continue;
            if (cum + stripe(i) > target) at = i;                    // cum <= target: the stripe holds mass
            else cum += stripe(i);
        }
        if (at >= 0) break;
    }
    if (at < 0) {
        int pick = V - 1;                                            // no token's cumulative mass exceeds the target
#pragma unroll
        for (int k = 2; k >= 0; --k)                                 // the tail's entries, the first that does last
            if (target >= 0.f && wt[k] > 0.f && cum + (k > 0 ? wt[0] : 0.f) + (k > 1 ? wt[1] : 0.f) + wt[k] > target) pick = V4 + k;
        if (threadIdx.x == 0) next_root[b] = pick;
        return;
    }
    const float wsum = part[lane & 15][at], wincl = prefix(wsum, 16);
    const int wv = crossing(wsum, wincl, cum, target, lane < 16);
    if (wave != wv) return;
    const float wfrom = wv ? cum + __shfl(wincl, wv - 1, 64) : cum;
    float w[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < TYP_GROUPS; ++i)
        if (i == at)
#pragma unroll
            for (int e = 0; e < 4; ++e) w[e] = r.x[i][e];
    const float mass = (w[0] + w[1]) + (w[2] + w[3]), incl = prefix(mass, 64);
    const int ln = crossing(mass, incl, wfrom, target, true);
    const float before = __shfl_up(incl, 1, 64);
    if (lane != ln) return;
    float sum = lane ? wfrom + before : wfrom;
    int pick = -1, held = 0;                                         // held: the last id of the group with any mass
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        sum += w[e];
        if (w[e] > 0.f) held = e;
        if (pick < 0 && w[e] > 0.f && sum > target) pick = e;
    }
    next_root[b] = pc * TYP_PIECE + at * TYP_STRIPE + (int)threadIdx.x * 4 + (pick < 0 ? held : pick);
}

int launch_accept_typical(hydra_ctx *c, hipStream_t s, int B, const int32_t *tree_tokens, const float *logits, float tau,
                          float eps, float alpha, const float *u, int32_t *ok_scratch, int32_t *flags, int32_t *n_acc,
                          int32_t *path, int32_t *next_root, int32_t *last_node) {
    const int T = c->tree.T, V = c->m.vocab;
    const float inv_tau = 1.0f / tau;
    hipLaunchKernelGGL(typical_stats_kernel, dim3(T, B), dim3(TYP_THREADS), 0, s, logits, V, tree_dev(c), tree_tokens, inv_tau, eps, alpha, ok_scratch, flags, T);
    HYDRA_LAUNCH_CHECK("typical_stats_kernel");
    hipLaunchKernelGGL(typical_select_kernel, dim3(B), dim3(TYP_THREADS), 0, s, logits, V, tree_dev(c), ok_scratch, inv_tau, u, n_acc, path, next_root, last_node, T);
    HYDRA_LAUNCH_CHECK("typical_select_kernel");
    return HYDRA_OK;
}

// ---------------------------------------------------------------------------
// Cache compaction: slot L + path[j] -> slot L + j for j < n_acc, every layer.
// A workgroup owns 256 (head, dim) columns of one layer of one row; no two threads touch the same element.  Its waves
// look at 64 entries of the path at once, one per lane, so the chain is row length -> path -> page table -> source ->
// destination however long the path is, and a path that moves nothing (a prompt chunk accepted whole) ends after the
// second of these.  The moved entries are then taken eight at a time, all sources before the first destination:
// path[j] >= j and strictly increasing, so within the eight every source is read before it can be overwritten, and no
// later source lies at or below an earlier destination.  Walking j in every thread, one dependent chain per entry, took
// 27.3 us for 4 rows of 1..5 accepted tokens in 32 layers of 4096 columns and 28.5 us for the identity path of a
// 128-token chunk in two.
// A path that is not strictly increasing inside [0, T) (only a caller's own
// path can be: accept_greedy and accept_typical always produce one) ends the
// walk at the offending entry and is reported (FLAG_BAD_PATH); page ids outside
// the cache are reported (FLAG_BAD_PAGE) and their copies skipped.
// ---------------------------------------------------------------------------
enum { COMPACT_THREADS = 256, COMPACT_AT_ONCE = 8 };
template <bool BF>
__global__ __launch_bounds__(COMPACT_THREADS) void compact_kernel(const int32_t *n_acc, const int32_t *path, const int32_t *seq_len,
                               const int32_t *page_table, int max_pages, int n_pages,
                               typename Act<BF>::type *kpages, typename Act<BF>::type *vpages, int H, int Dh, int T, int plen, int32_t *flags) {
    typedef typename Act<BF>::type elem;
    typedef uint32_t u4 __attribute__((ext_vector_type(4), aligned(2)));        // the caller's pages: no more than element alignment is known
    const int layer = blockIdx.y, b = blockIdx.z;
    const int lane = threadIdx.x & 63;
    const int col = blockIdx.x * COMPACT_THREADS + threadIdx.x;                  // this thread's (head, dim) of V (and K in the fp32 family)
    const bool vcol = col < H * Dh;
    const int h = col / Dh, dim = col - h * Dh;
    // 16-bit K: eight dims of a token lie together, so an eighth of the threads move them, 16 bytes each
    const int kcol = blockIdx.x * COMPACT_THREADS + (int)threadIdx.x * 8;
    const bool kown = BF && threadIdx.x < COMPACT_THREADS / 8 && kcol < H * Dh;
    const int kh = kcol / Dh, kdim = kcol - kh * Dh;
    const bool report = threadIdx.x == 0 && blockIdx.x == 0 && layer == 0;
    const int L = seq_len[b];
    int na = n_acc[b];
    const int32_t *pr = path + (size_t)b * plen;
    const int32_t *pt = page_table + (size_t)b * max_pages;
    for (int j0 = 0; j0 < plen; j0 += 64) {
        const int j = j0 + lane;
        const int n = j < plen ? pr[j] : -1, prev = j > 0 && j < plen ? pr[j - 1] : -1;
        if (L < 0 || L + T > max_pages * 16) return;       // row was skipped by the verify kernels (the same for every thread)
        na = na < 0 ? 0 : (na > plen ? plen : na);
        const bool in = j < na;
        const uint64_t bad = __ballot(in && (n <= prev || n < j || n >= T));
        const uint64_t good = bad ? (bad & (0ull - bad)) - 1ull : ~0ull;          // entries in front of the first offending one
        const bool move = in && n != j && ((good >> lane) & 1ull);
        int sp = 0, dp = 0;
        if (move) { sp = pt[(L + n) >> 4]; dp = pt[(L + j) >> 4]; }
        const bool bad_page = move && ((unsigned)sp >= (unsigned)n_pages || (unsigned)dp >= (unsigned)n_pages);
        if (__ballot(bad_page) && report) atomicOr(flags, FLAG_BAD_PAGE);
        uint64_t todo = __ballot(move && !bad_page);
        while (todo) {
            elem vv[COMPACT_AT_ONCE], kk[COMPACT_AT_ONCE];
            u4 k8[COMPACT_AT_ONCE];
            uint64_t rest = todo;
#pragma unroll
            for (int q = 0; q < COMPACT_AT_ONCE; ++q) {
                if (!rest) continue;                        // wave-uniform
                const int l = __builtin_ctzll(rest);
                rest &= rest - 1ull;
                const int ss = L + __builtin_amdgcn_readlane(n, l), page = __builtin_amdgcn_readlane(sp, l);
                if (vcol) {
                    const size_t sb = kv_block_base(layer, n_pages, page, H, h, Dh);
                    vv[q] = vpages[sb + v_in_block<BF>(ss & 15, dim, Dh)];
                    if (!BF) kk[q] = kpages[sb + k_in_block<BF>(ss & 15, dim, Dh)];
                }
                if (kown) k8[q] = *reinterpret_cast<const u4 *>(kpages + kv_block_base(layer, n_pages, page, H, kh, Dh) + k_in_block<BF>(ss & 15, kdim, Dh));
            }
            asm volatile("" ::: "memory");                  // every source of the eight is requested before the first destination is written
#pragma unroll
            for (int q = 0; q < COMPACT_AT_ONCE; ++q) {
                if (!todo) continue;
                const int l = __builtin_ctzll(todo);
                todo &= todo - 1ull;
                const int ds = L + j0 + l, page = __builtin_amdgcn_readlane(dp, l);
                if (vcol) {
                    const size_t db = kv_block_base(layer, n_pages, page, H, h, Dh);
                    vpages[db + v_in_block<BF>(ds & 15, dim, Dh)] = vv[q];
                    if (!BF) kpages[db + k_in_block<BF>(ds & 15, dim, Dh)] = kk[q];
                }
                if (kown) *reinterpret_cast<u4 *>(kpages + kv_block_base(layer, n_pages, page, H, kh, Dh) + k_in_block<BF>(ds & 15, kdim, Dh)) = k8[q];
            }
        }
        if (bad) {
            if (report) atomicOr(flags, FLAG_BAD_PATH);
            return;
        }
        if (j0 + 64 >= na) return;
    }
}

// h_last <- hidden[last accepted node]; root <- next_root; seq_len += n_acc;
// kv_index[j] = (physical page, offset) of slot L + j.  Runs after compact_kernel.
// A row that the verify kernels skipped for lack of cache capacity keeps its state
// (seq_len, h_last, root) and gets kv_index = -1: its n_acc, last_node and hidden
// were computed from nothing.
__global__ void state_update_kernel(const TreeDev *tree, const int32_t *n_acc, const int32_t *next_root,
                                    const int32_t *last_node, const float *hidden, const int32_t *page_table,
                                    int max_pages, int d, int32_t *seq_len, float *h_last, int32_t *root,
                                    int32_t *kv_index) {
    const int b = blockIdx.x;
    const int T = tree->T, plen = tree->max_depth + 1;
    const int L = seq_len[b];
    const bool ok = L >= 0 && L + T <= max_pages * 16;     // uniform over the workgroup
    int na = n_acc[b];
    na = na < 0 ? 0 : (na > plen ? plen : na);
    int last = last_node[b];
    last = last < 0 ? 0 : (last >= T ? T - 1 : last);
    if (ok)
        for (int k = threadIdx.x; k < d; k += blockDim.x) h_last[(size_t)b * d + k] = hidden[((size_t)b * T + last) * d + k];
    if (kv_index)                                           // one entry per thread: a chunk of 128 tokens has 128 of them
        for (int j = threadIdx.x; j < plen; j += blockDim.x) {
            const bool in = ok && j < na;
            kv_index[((size_t)b * plen + j) * 2 + 0] = in ? page_table[(size_t)b * max_pages + ((L + j) >> 4)] : -1;
            kv_index[((size_t)b * plen + j) * 2 + 1] = in ? ((L + j) & 15) : -1;
        }
    __syncthreads();                                        // every thread has read seq_len[b]
    if (threadIdx.x == 0 && ok) {
        root[b] = next_root[b];
        seq_len[b] = L + na;
    }
}

int launch_compact(hydra_ctx *c, hipStream_t s, int B, const int32_t *n_acc, const int32_t *path,
                   const int32_t *next_root, const int32_t *last_node, const float *hidden, const hydra_kv *kv,
                   int32_t *seq_len, float *h_last, int32_t *root, int32_t *kv_index) {
    dim3 grid(ceil_div(c->m.d, COMPACT_THREADS), c->m.n_layers, B), block(COMPACT_THREADS);
    const int T = c->tree.T, plen = c->tree.max_depth + 1;
    if (c->bf16) hipLaunchKernelGGL(compact_kernel<true>, grid, block, 0, s, n_acc, path, seq_len, kv->page_table, kv->max_pages, kv->n_pages, (a16_t *)kv->k_pages, (a16_t *)kv->v_pages, c->m.n_heads, c->m.head_dim, T, plen, flags_dev(c));
    else         hipLaunchKernelGGL(compact_kernel<false>, grid, block, 0, s, n_acc, path, seq_len, kv->page_table, kv->max_pages, kv->n_pages, (float *)kv->k_pages, (float *)kv->v_pages, c->m.n_heads, c->m.head_dim, T, plen, flags_dev(c));
    HYDRA_LAUNCH_CHECK("compact_kernel");
    hipLaunchKernelGGL(state_update_kernel, dim3(B), dim3(1024), 0, s, tree_dev(c), n_acc, next_root, last_node, hidden, kv->page_table, kv->max_pages, c->m.d, seq_len, h_last, root, kv_index);
    HYDRA_LAUNCH_CHECK("state_update_kernel");
    return HYDRA_OK;
}

// ---------------------------------------------------------------------------
// accept_typical for callers that cannot allocate or pass a workspace (HIP graph capture, tight serving loops):
// the per-candidate pass flags that typical_stats_kernel hands to typical_select_kernel live in a fixed array
// in device memory that belongs to the library.  Each GPU has its own copy of the array at its own address; the
// address is looked up once per device (scratch_pointer) and only that pointer is ever given to kernels or
// memory calls, never the array's name.
// ---------------------------------------------------------------------------
enum { TYP_STATIC_MAX_NODES = 16384, TYP_MAX_DEVICES = 64 };          // B * T <= 16384: 64 KiB per device
static __device__ __align__(256) int32_t scratch[TYP_STATIC_MAX_NODES];
static int32_t *g_scratch_ptr[TYP_MAX_DEVICES];                        // per device; NULL until looked up

// the current device's copy of `scratch`; looked up on first use on that device (hydra_bind_weights does it at set-up)
int typical_static_scratch(int32_t **out) {
    int dev = -1;
    HYDRA_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= TYP_MAX_DEVICES) return fail(HYDRA_E_UNSUPPORTED, "accept_typical_static: device index beyond 63");
    int32_t *p = __atomic_load_n(&g_scratch_ptr[dev], __ATOMIC_ACQUIRE);
    if (!p) {
        void *sym = nullptr;
        HYDRA_HIP(hipGetSymbolAddress(&sym, HIP_SYMBOL(scratch)));
        if (!sym) return fail(HYDRA_E_HIP, "accept_typical_static: no device address for the scratch array");
        p = static_cast<int32_t *>(sym);
        __atomic_store_n(&g_scratch_ptr[dev], p, __ATOMIC_RELEASE);    // every thread that races here stores the same address
    }
    *out = p;
    return HYDRA_OK;
}

}  // namespace hydra

extern "C" int accept_typical_static(hydra_ctx *c, void *stream, int B, const int32_t *tree_tokens, const float *logits, float tau,
                                     float eps, float alpha, const float *u, int32_t *n_acc, int32_t *path, int32_t *next_root,
                                     int32_t *last_node) {
    using namespace hydra;
    if (!c) return fail(HYDRA_E_INVALID_ARG, "ctx is NULL");
    if (B < 1 || B > c->max_batch) return fail(HYDRA_E_CAPACITY, "B outside [1, max_batch]");
    if (!c->arena) return fail(HYDRA_E_STATE, "no weight arena bound (hydra_bind_weights)");
    if (!tree_tokens || !logits || !n_acc || !path || !next_root || !last_node)
        return fail(HYDRA_E_INVALID_ARG, "accept_typical_static: NULL argument");
    if (!(tau > 0.f) || !(eps >= 0.f) || !(alpha >= 0.f)) return fail(HYDRA_E_INVALID_ARG, "accept_typical_static: need tau > 0, eps >= 0, alpha >= 0");
    if ((int64_t)B * c->tree.T > TYP_STATIC_MAX_NODES)
        return fail(HYDRA_E_CAPACITY, "accept_typical_static: B * T exceeds the 16384 tree nodes its fixed buffer holds; use accept_typical with a workspace");
    int32_t *ok = nullptr;
    int rc = typical_static_scratch(&ok);
    if (rc) return rc;
    int32_t *flags = reinterpret_cast<int32_t *>(c->arena + c->off_tables + (size_t)c->table_slot * TABLE_SLOT_BYTES + FLAGS_OFF_IN_SLOT);
    // typical_stats_kernel writes the flag of every non-root node before typical_select_kernel reads it, so nothing
    // in the buffer has to start at zero
    return launch_accept_typical(c, (hipStream_t)stream, B, tree_tokens, logits, tau, eps, alpha, u, ok, flags, n_acc, path, next_root, last_node);
}
