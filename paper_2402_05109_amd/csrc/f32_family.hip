// fp32 storage family: a GEMM on the fp32 matrix instruction and a tree attention.  Used by fp32 models (small, launch-bound), where what a
// kernel costs is its chain of dependent memory round trips and cross-lane steps, not bandwidth.
#include "device_common.h"
#include "internal.h"

namespace hydra {

typedef __attribute__((ext_vector_type(4))) float f32x4_t;
typedef float f32x4_u __attribute__((ext_vector_type(4), aligned(4)));      // the caller's pages: no more than float alignment is known

// sum_k X[m][k] W[n][k] on the fp32 matrix instruction (16 x 16 x 4, fp32 products and sums).  A workgroup
// computes 16 rows x 16 features; its four waves take the 16-long pieces of K in turn and meet in LDS.
// Lane (r, g) loads four consecutive k of row r and of feature r at piece + 4 g, and instruction e of a piece multiplies the
// k of every lane's element e: the four lane groups hold different k, the same ones on both sides, so no data is moved
// between lanes.  Bound by one round of loads (four pieces in flight per wave, the next four requested before these are
// multiplied) and the meeting.  With a feature per wave, 16 rows per lane and a reduction over the lanes a launch of the tiny
// shape (16 rows, K = 256 or 688) took 8.3 us on average, 8.9 with a shared reduction and 16-byte loads.
// Rows and features past the end repeat the last one and are not stored; k past K is zero on both sides.
//
// A launch of these models costs 2 to 5 us whatever it does, so what stands in front of and behind a product is part of it:
//   NORM      X is the residual stream: x * gain is multiplied, and 1 / rms(x), whose sum of squares the lanes collect on the
//             way, scales the sums (it commutes with the contraction)
//   ADD       out (the residual stream) += sums
//   BIAS_SILU z = (residual ? z : 0) + SiLU(sums + bias), also written as the next layer's input
//   SWIGLU    SiLU(sums of gate feature n) * sums of up feature n (weight rows n and F + n)
//   ROPE      features n and n + Dh/2 of a head, which are a rotary pair: q -> attention input [B][T][H][Dh], k and v -> cache
//             slot seq_len[b] + node at position seq_len[b] + depth (paper, section 2, "Tree decoding")
// Norm, rotary embedding, activation and bias as kernels of their own: 43 launches per step of the tiny shape, 28 this way.
enum { F32_PLAIN, F32_ADD, F32_BIAS_SILU, F32_SWIGLU, F32_ROPE };
struct F32Rope {
    const float *table; const int32_t *seq_len, *page_table; const TreeDev *tree;
    float *kpages, *vpages, *qbuf; int32_t *flags;
    int max_pages, n_pages, layer, H, Dh, T, max_pos;
};
struct F32Epilogue {
    float *out; int ld;
    const float *gain; float eps;                                      // NORM
    const float *bias; float *z; int residual;                         // BIAS_SILU
    F32Rope rope;                                                      // ROPE
};
template <int MODE, bool NORM, bool VEC>
__global__ __launch_bounds__(256, 2) void gemm_f32_kernel(const float *__restrict__ X, const float *__restrict__ W, int M, int N, int K, F32Epilogue o) {
    constexpr int NB = MODE == F32_SWIGLU || MODE == F32_ROPE ? 2 : 1;              // features per lane
    __shared__ f32x4_t red[NB][4][64];
    __shared__ float red_sq[4][16];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, r = lane & 15, g = lane >> 4;
    const int m0 = blockIdx.y * 16;
    // first feature and the distance of the second one.  ROPE: the 16-feature pieces of the first half of each q, k and v head
    int n0 = blockIdx.x * 16, second = N, part = 0;
    if (MODE == F32_ROPE) {
        const int half = o.rope.Dh >> 1, pieces = half >> 4;
        part = blockIdx.x / pieces;                                    // q heads, then k heads, then v heads
        n0 = part * o.rope.Dh + (blockIdx.x - part * pieces) * 16;
        second = half;
    }
    const float *xr = X + (size_t)min(m0 + r, M - 1) * K + 4 * g, *wr = W + (size_t)min(n0 + r, N - 1) * K + 4 * g;
    const float *gr = NORM ? o.gain + 4 * g : nullptr;
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
    f32x4_t a[4], b[NB][4], gn[4];
    auto fetch = [&](int k0) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            a[u] = four(xr, k0 + 64 * u);
#pragma unroll
            for (int i = 0; i < NB; ++i) b[i][u] = four(wr + (size_t)i * second * K, k0 + 64 * u);
            if (NORM) gn[u] = four(gr, k0 + 64 * u);
        }
    };
    fetch(wave * 16);
    // what the end needs, requested while the operands are under way
    const int m = threadIdx.x >> 4, n = threadIdx.x & 15, row = m0 + m, col = n0 + n;
    const bool live = row < M && col < N;
    float before = 0.f, bias = 0.f;
    if (MODE == F32_ADD && live) before = o.out[(size_t)row * o.ld + col];
    if (MODE == F32_BIAS_SILU && live) {
        bias = o.bias[col];
        if (o.residual) before = o.z[(size_t)row * N + col];
    }
    float cs = 1.f, sn = 0.f;
    size_t at = 0;
    bool fits = false, cached = false;
    if (MODE == F32_ROPE) {
        const F32Rope &p = o.rope;
        const int bb = min(row, M - 1) / p.T, node = min(row, M - 1) - bb * p.T, L = p.seq_len[bb];
        fits = L >= 0 && L + p.T <= p.max_pages * 16 && L + p.tree->max_depth < p.max_pos;
        if (fits) {
            const int j = (n0 % p.Dh) + n, half = p.Dh >> 1, slot = L + node;
            const float *t = p.table + ((size_t)(L + p.tree->depth[node]) * half + j) * 2;
            cs = t[0];
            sn = t[1];
            const int page = p.page_table[(size_t)bb * p.max_pages + (slot >> 4)];
            cached = (unsigned)page < (unsigned)p.n_pages;
            at = kv_block_base(p.layer, p.n_pages, cached ? page : 0, p.H, part % p.H, p.Dh) + (size_t)(slot & 15) * p.Dh + j;
        }
    }
    // A sum per (piece, element), added as a tree: chains of K / 256 products.  Where there are two features two pieces share a sum
    // (with 32 of them per lane only one wave fits a SIMD: 2048 wide, 128 rows, a step 4.5 % slower), and every sweep of 256 is added
    // up by itself, so that a product is rounded no more often on its way than with a sum per piece.  Error of a normed product
    // against 64 bits at K = 256 / 2048 / 4096: 9.1e-8 / 1.09e-7 / 1.21e-7; with the shared sums kept over all of K 9.9e-8 / 1.67e-7 /
    // 2.20e-7; with a sum per piece, behind a norm of its own, 9.5e-8 / 1.36e-7 / 1.70e-7.  It costs no time (20 registers fewer:
    // 1024 wide, 16 rows, a verification 114.5 -> 111.8 us).
    constexpr int NP = 4 / NB;
    f32x4_t part_acc[NB][NP][4], swept[NB];
    auto clear = [&](int i) {
#pragma unroll
        for (int u = 0; u < NP; ++u)
#pragma unroll
            for (int e = 0; e < 4; ++e) part_acc[i][u][e] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    };
    auto sum = [&](int i) {
        f32x4_t by_piece[NP];
#pragma unroll
        for (int u = 0; u < NP; ++u) by_piece[u] = (part_acc[i][u][0] + part_acc[i][u][1]) + (part_acc[i][u][2] + part_acc[i][u][3]);
        f32x4_t all = by_piece[0] + by_piece[1];
        if constexpr (NP == 4) all += by_piece[2] + by_piece[3];
        return all;
    };
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        clear(i);
        swept[i] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    }
    float sq = 0.f;
    for (int k0 = wave * 16; k0 < K; k0 += 256) {
        f32x4_t ca[4], cb[NB][4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            ca[u] = a[u];
#pragma unroll
            for (int i = 0; i < NB; ++i) cb[i][u] = b[i][u];
            if (NORM) ca[u] *= gn[u];
        }
        if (NORM) {                                                    // likewise: a chain of K / 256
            f32x4_t q = a[0] * a[0];
#pragma unroll
            for (int u = 1; u < 4; ++u)
#pragma unroll
                for (int e = 0; e < 4; ++e) q[e] = fmaf(a[u][e], a[u][e], q[e]);
            sq += (q[0] + q[1]) + (q[2] + q[3]);
        }
        if (k0 + 256 < K) fetch(k0 + 256);
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int i = 0; i < NB; ++i) part_acc[i][u % NP][e] = __builtin_amdgcn_mfma_f32_16x16x4f32(ca[u][e], cb[i][u][e], part_acc[i][u % NP][e], 0, 0, 0);
        if constexpr (NB > 1)
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                swept[i] += sum(i);
                clear(i);
            }
    }
#pragma unroll
    for (int i = 0; i < NB; ++i) red[i][wave][lane] = NB > 1 ? swept[i] : sum(i);      // [v]: row 4 g + v, feature r
    if (NORM) {
        sq += __shfl_xor(sq, 16, 64);
        sq += __shfl_xor(sq, 32, 64);
        if (g == 0) red_sq[wave][r] = sq;
    }
    __syncthreads();
    if (row >= M) return;
    const int from = (m >> 2) * 16 + n;
    const float rstd = NORM ? 1.0f / sqrtf(((red_sq[0][m] + red_sq[1][m]) + (red_sq[2][m] + red_sq[3][m])) / (float)K + o.eps) : 1.0f;
    float s[NB];
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        const float p0 = red[i][0][from][m & 3], p1 = red[i][1][from][m & 3], p2 = red[i][2][from][m & 3], p3 = red[i][3][from][m & 3];
        // 1 / rms behind the sum is a rounding of the result that a normed X would not have; one rounding for all of this makes up for it
        s[i] = NORM ? (float)((((double)p0 + p1) + ((double)p2 + p3)) * rstd) : (p0 + p1) + (p2 + p3);
    }
    if (MODE == F32_ROPE) {
        const F32Rope &p = o.rope;
        if (n == 0 && !(fits && cached)) atomicOr(p.flags, fits ? FLAG_BAD_PAGE : FLAG_CAPACITY);      // bad table entry: the row's K/V are not written
        const int sec = part / p.H, half = p.Dh >> 1;
        if (!fits || (sec > 0 && !cached)) return;
        const float y0 = sec < 2 ? s[0] * cs - s[NB - 1] * sn : s[0], y1 = sec < 2 ? s[NB - 1] * cs + s[0] * sn : s[NB - 1];
        float *dst = sec == 0 ? p.qbuf + (size_t)row * p.H * p.Dh + n0 + n : (sec == 1 ? p.kpages : p.vpages) + at;
        dst[0] = y0;
        dst[half] = y1;
        return;
    }
    if (!live) return;
    float y = s[0];
    if (MODE == F32_ADD) y += before;
    if (MODE == F32_BIAS_SILU) {
        y = silu_f(y + bias) + before;
        o.z[(size_t)row * N + col] = y;
    }
    if (MODE == F32_SWIGLU) y = silu_f(y) * s[NB - 1];
    o.out[(size_t)row * o.ld + col] = y;
}

// VEC where K % 4 == 0: X, W and the gains start at 256-byte boundaries of the workspace and the arena, so every row is 16-byte
// aligned.  Only the width of the FFN may be anything; d and the heads' widths are multiples of 64.
template <int MODE, bool NORM>
static int run_f32(hipStream_t s, const float *X, const float *W, int M, int N, int K, int tiles, const F32Epilogue &o) {
    dim3 grid(tiles, ceil_div(M, 16)), block(256);
    if (K % 4 == 0) hipLaunchKernelGGL((gemm_f32_kernel<MODE, NORM, true>), grid, block, 0, s, X, W, M, N, K, o);
    else if constexpr (!NORM) hipLaunchKernelGGL((gemm_f32_kernel<MODE, NORM, false>), grid, block, 0, s, X, W, M, N, K, o);
    else return fail(HYDRA_E_UNSUPPORTED, "fp32 family: d is a multiple of 64");
    HYDRA_LAUNCH_CHECK("gemm_f32_kernel");
    return HYDRA_OK;
}

int launch_gemm_f32(hydra_ctx *c, hipStream_t s, const float *X, const float *W, float *part, int M, int N, int K) {
    (void)c;
    F32Epilogue o{};
    o.out = part; o.ld = N;
    return run_f32<F32_PLAIN, false>(s, X, W, M, N, K, ceil_div(N, 16), o);
}
int launch_f32_norm_gemm(hydra_ctx *c, hipStream_t s, const float *x, const float *gain, const float *W, float *part, int M, int N) {
    F32Epilogue o{};
    o.out = part; o.ld = N; o.gain = gain; o.eps = c->m.rms_eps;
    return run_f32<F32_PLAIN, true>(s, x, W, M, N, c->m.d, ceil_div(N, 16), o);
}
int launch_f32_add(hydra_ctx *c, hipStream_t s, const float *X, const float *W, float *x, int M, int K) {
    F32Epilogue o{};
    o.out = x; o.ld = c->m.d;
    return run_f32<F32_ADD, false>(s, X, W, M, c->m.d, K, ceil_div(c->m.d, 16), o);
}
int launch_f32_bias_silu(hydra_ctx *c, hipStream_t s, const float *X, const float *W, int M, int K, const float *bias, float *z, bool residual, float *out) {
    F32Epilogue o{};
    o.out = out; o.ld = c->m.d; o.bias = bias; o.z = z; o.residual = residual ? 1 : 0;
    return run_f32<F32_BIAS_SILU, false>(s, X, W, M, c->m.d, K, ceil_div(c->m.d, 16), o);
}
int launch_f32_swiglu(hydra_ctx *c, hipStream_t s, const float *x, const float *gain, const float *W, float *act, int M) {
    F32Epilogue o{};
    o.out = act; o.ld = c->m.ffn; o.gain = gain; o.eps = c->m.rms_eps;
    return run_f32<F32_SWIGLU, true>(s, x, W, M, c->m.ffn, c->m.d, ceil_div(c->m.ffn, 16), o);
}
int launch_f32_qkv_rope(hydra_ctx *c, hipStream_t s, const float *x, const float *gain, const float *W, int M, int layer, const int32_t *seq_len,
                        const hydra_kv *kv, float *qbuf, int32_t *flags) {
    F32Epilogue o{};
    o.gain = gain; o.eps = c->m.rms_eps;
    o.rope = F32Rope{rope_dev(c), seq_len, kv->page_table, tree_dev(c), (float *)kv->k_pages, (float *)kv->v_pages, qbuf, flags,
                     kv->max_pages, kv->n_pages, layer, c->m.n_heads, c->m.head_dim, c->tree.T, c->m.max_pos};
    return run_f32<F32_ROPE, true>(s, x, W, M, 3 * c->m.d, c->m.d, 3 * c->m.n_heads * (c->m.head_dim / 32), o);
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
