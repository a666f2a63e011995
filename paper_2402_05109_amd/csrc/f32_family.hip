// fp32 storage family: a GEMM on the fp32 matrix instruction and a tree attention.  Used by fp32 models (small, launch-bound), where what a
// kernel costs is its chain of dependent memory round trips and cross-lane steps, not bandwidth.
#include "device_common.h"
#include "internal.h"

namespace hydra {

typedef __attribute__((ext_vector_type(4))) float f32x4_t;
typedef float f32x4_u __attribute__((ext_vector_type(4), aligned(4)));      // the caller's pages: no more than float alignment is known

// part[m][n] = sum_k X[m][k] W[n][k] on the fp32 matrix instruction (16 x 16 x 4, fp32 products and sums).  A workgroup
// computes 16 rows x 16 features; its four waves take the 16-long pieces of K in turn and meet in LDS.
// Lane (r, g) loads four consecutive k of row r and of feature r at piece + 4 g, and instruction e of a piece multiplies the
// k of every lane's element e: the four lane groups hold different k, the same ones on both sides, so no data is moved
// between lanes.  Bound by one round of loads (four pieces in flight per wave) and the meeting.  With a feature per wave, 16
// rows per lane and a reduction over the lanes a launch of the tiny shape (16 rows, K = 256 or 688) took 8.3 us on average,
// 8.9 with a shared reduction and 16-byte loads.
// Rows and features past the end repeat the last one and are not stored; k past K is zero on both sides.
template <bool VEC>
__global__ __launch_bounds__(256) void gemm_f32_kernel(const float *__restrict__ X, const float *__restrict__ W,
                                                        float *__restrict__ part, int M, int N, int K, int ld) {
    __shared__ f32x4_t red[4][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, r = lane & 15, g = lane >> 4;
    const int n0 = blockIdx.x * 16, m0 = blockIdx.y * 16;
    const float *xr = X + (size_t)min(m0 + r, M - 1) * K + 4 * g, *wr = W + (size_t)min(n0 + r, N - 1) * K + 4 * g;
    auto four = [&](const float *p, int k) {
        f32x4_t v = {0.f, 0.f, 0.f, 0.f};
        if (VEC) {
            if (k + 4 * g < K) v = *reinterpret_cast<const f32x4_t *>(p + k);       // K % 4 == 0: all four or none
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (k + 4 * g + e < K) v[e] = p[k + e];
        }
        return v;
    };
    f32x4_t part_acc[4][4];                                            // a sum per (piece, element): chains of K / 256 products, added as a tree
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int e = 0; e < 4; ++e) part_acc[u][e] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    for (int k0 = wave * 16; k0 < K; k0 += 256) {
        f32x4_t a[4], b[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) { a[u] = four(xr, k0 + 64 * u); b[u] = four(wr, k0 + 64 * u); }
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int e = 0; e < 4; ++e) part_acc[u][e] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[u][e], b[u][e], part_acc[u][e], 0, 0, 0);
    }
    f32x4_t by_piece[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) by_piece[u] = (part_acc[u][0] + part_acc[u][1]) + (part_acc[u][2] + part_acc[u][3]);
    const f32x4_t acc = (by_piece[0] + by_piece[1]) + (by_piece[2] + by_piece[3]);
    red[wave][lane] = acc;                                            // acc[v]: row 4 g + v, feature r
    __syncthreads();
    const int m = threadIdx.x >> 4, n = threadIdx.x & 15;
    const int from = (m >> 2) * 16 + n;
    const float s = (red[0][from][m & 3] + red[1][from][m & 3]) + (red[2][from][m & 3] + red[3][from][m & 3]);
    if (m0 + m < M && n0 + n < N) part[(size_t)(m0 + m) * ld + n0 + n] = s;
}

int launch_gemm_f32(hydra_ctx *c, hipStream_t s, const float *X, const float *W, float *part, int M, int N, int K) {
    (void)c;
    // K % 4 == 0: X and W start at 256-byte boundaries of the workspace and the arena, so every row is 16-byte aligned
    dim3 grid(ceil_div(N, 16), ceil_div(M, 16)), block(256);
    if (K % 4 == 0) hipLaunchKernelGGL(gemm_f32_kernel<true>, grid, block, 0, s, X, W, part, M, N, K, N);
    else            hipLaunchKernelGGL(gemm_f32_kernel<false>, grid, block, 0, s, X, W, part, M, N, K, N);
    HYDRA_LAUNCH_CHECK("gemm_f32_kernel");
    return HYDRA_OK;
}

// ---------------------------------------------------------------------------
// Tree attention (paper, section 2): node n of row b attends to cache slots
// [0, L) and to the tree nodes named by its ancestor bitmask (slots L + a).
// One workgroup per (node, head, row); its four waves take the 64-key chunks in turn and meet in LDS at the end.
// Per chunk: lane = key, its whole K row in 16-byte loads, mask, online softmax; then the wave turns round: DH / 4 lanes
// span the dims of one key, 64 / (DH / 4) keys at a time, 16-byte loads of V that are all in flight together.
// Keys that are masked (or whose weight underflows) are never read: their lanes read slot 0 instead, which every query
// sees (the first prefix token, or the root where nothing is cached), and multiply it by nothing.
// Bound by the chain page table -> K -> softmax -> V.  One wave per query, a scalar dot product per lane and one key of
// V per step took 48.6 us a launch (16 nodes, 4 heads, 144 keys of the tiny shape).
// ---------------------------------------------------------------------------
enum { ATTN_F32_WAVES = 4 };
template <int DH>
__global__ __launch_bounds__(ATTN_F32_WAVES * 64) void attn_f32_kernel(
    const float *__restrict__ q, const float *__restrict__ kpages, const float *__restrict__ vpages, const int32_t *page_table,
    int max_pages, int n_pages, int layer, const int32_t *seq_len, const TreeDev *tree, int H, float scale, float *out, int32_t *flags) {
    constexpr int DL = DH / 4, KG = 64 / DL, NW = ATTN_F32_WAVES;    // lanes across the dims, keys per V step
    const int n = blockIdx.x, h = blockIdx.y, b = blockIdx.z;
    const int T = tree->T;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int L = seq_len[b];
    if (L < 0 || L + T > max_pages * 16) {                           // uniform over the workgroup
        if (threadIdx.x == 0) atomicOr(flags, FLAG_CAPACITY);
        return;
    }
    __shared__ f32x4_t qs[DL];
    __shared__ float ps[NW][64];
    __shared__ size_t offs[NW][64];
    __shared__ f32x4_t os[NW][DL];
    __shared__ float ms[NW], ls[NW];
    const size_t qoff = (((size_t)b * T + n) * H + h) * DH;
    for (int i = threadIdx.x; i < DH; i += NW * 64) reinterpret_cast<float *>(qs)[i] = q[qoff + i] * scale;
    const uint64_t anc0 = tree->anc[n][0], anc1 = tree->anc[n][1];
    const int32_t *pt = page_table + (size_t)b * max_pages;
    const size_t off0 = kv_block_base(layer, n_pages, checked_page(pt[0], n_pages, flags), H, h, DH);
    const int total = L + T;
    float m_run = -INFINITY, l_run = 0.f;
    f32x4_t o = {0.f, 0.f, 0.f, 0.f};
    __syncthreads();
    for (int base = wave * 64; base < total; base += NW * 64) {
        const int key = base + lane;
        bool valid = key < total;
        if (valid && key >= L) {
            const int a = key - L;
            valid = ((a < 64 ? anc0 >> a : anc1 >> (a - 64)) & 1ull) != 0;
        }
        size_t off = off0;
        if (valid) off = kv_block_base(layer, n_pages, checked_page(pt[key >> 4], n_pages, flags), H, h, DH) + (size_t)(key & 15) * DH;
        const f32x4_u *kp = reinterpret_cast<const f32x4_u *>(kpages + off);
        float a4[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < DL; ++i) {
            const f32x4_t kv = kp[i], qv = qs[i];
#pragma unroll
            for (int e = 0; e < 4; ++e) a4[e] = fmaf(qv[e], kv[e], a4[e]);
        }
        const float sc = valid ? (a4[0] + a4[1]) + (a4[2] + a4[3]) : -INFINITY;
        const float m_new = fmaxf(m_run, wave_max(sc));
        // nothing visible yet (wave-uniform).  A chunk of nothing but NaN scores has no maximum either, but must not be left out.
        if (m_new == -INFINITY && !__any(sc != sc)) continue;
        const float p = valid ? __expf(sc - m_new) : 0.f;
        const float alpha = __expf(m_run - m_new);                   // exp(-inf) = 0 on the first visible chunk
        l_run = l_run * alpha + wave_sum(p);
        o *= alpha;
        m_run = m_new;
        ps[wave][lane] = p;
        offs[wave][lane] = p == 0.f ? off0 : off;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");       // LDS is in order within a wave; keep the compiler from reordering
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll 8
        for (int kk = lane / DL; kk < 64; kk += KG) {
            const float pk = ps[wave][kk];
            const f32x4_t vv = reinterpret_cast<const f32x4_u *>(vpages + offs[wave][kk])[lane % DL];
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = fmaf(pk, pk == 0.f ? 0.f : vv[e], o[e]);
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
#pragma unroll
    for (int s = DL; s < 64; s <<= 1)                                 // the key groups of the wave
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] += __shfl_xor(o[e], s, 64);
    if (lane < DL) os[wave][lane] = o;
    if (lane == 0) { ms[wave] = m_run; ls[wave] = l_run; }
    __syncthreads();
    if (threadIdx.x >= DL) return;
    float mt = ms[0], lt = 0.f;                                       // wave 0 holds slot 0, which every query sees: finite
#pragma unroll
    for (int w = 1; w < NW; ++w) mt = fmaxf(mt, ms[w]);
    f32x4_t r = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        const float f = __expf(ms[w] - mt);
        lt += f * ls[w];
        r += os[w][lane] * f;
    }
    const float inv = 1.0f / lt;
#pragma unroll
    for (int e = 0; e < 4; ++e) out[qoff + lane * 4 + e] = r[e] * inv;
}

int launch_attention_f32(hydra_ctx *c, hipStream_t s, int B, int layer, const float *q, const int32_t *seq_len,
                         const hydra_kv *kv, float *out, int32_t *flags) {
    dim3 grid(c->tree.T, c->m.n_heads, B), block(ATTN_F32_WAVES * 64);
    const float scale = 1.0f / sqrtf((float)c->m.head_dim);
#define ATTN_F32(DHv)                                                                                                 \
    hipLaunchKernelGGL(attn_f32_kernel<DHv>, grid, block, 0, s, q, (const float *)kv->k_pages, (const float *)kv->v_pages,  \
                       kv->page_table, kv->max_pages, kv->n_pages, layer, seq_len, tree_dev(c), c->m.n_heads, scale, out, flags)
    if (c->m.head_dim == 128) ATTN_F32(128); else ATTN_F32(64);
#undef ATTN_F32
    HYDRA_LAUNCH_CHECK("attn_f32_kernel");
    return HYDRA_OK;
}

}  // namespace hydra
