// fp32 storage family: a plain VALU GEMM and a tree attention.  Used by fp32 models (small, launch-bound), where what a
// kernel costs is its chain of dependent memory round trips and cross-lane steps, not bandwidth.
#include "device_common.h"
#include "internal.h"

namespace hydra {

typedef __attribute__((ext_vector_type(4))) float f32x4_t;
typedef float f32x4_u __attribute__((ext_vector_type(4), aligned(4)));      // the caller's pages: no more than float alignment is known

// Sums v[0..R) over the 64 lanes, R a power of two up to 16: afterwards lane l holds the sum of v[l % R] in v[0].  Each
// step halves the values a lane carries: it keeps those whose index agrees with one bit of its lane number and hands the
// others to its partner, so R sums take R - 1 + log2(64 / R) exchanges instead of 6 R.
template <int R>
__device__ __forceinline__ float lanes_sum(float (&v)[R], int lane) {
#pragma unroll
    for (int half = R / 2; half > 0; half >>= 1) {
        const bool up = (lane & half) != 0;
#pragma unroll
        for (int i = 0; i < half; ++i) {
            const float keep = up ? v[i + half] : v[i], give = up ? v[i] : v[i + half];
            v[i] = keep + __shfl_xor(give, half, 64);
        }
    }
    float s = v[0];
#pragma unroll
    for (int o = R; o < 64; o <<= 1) s += __shfl_xor(s, o, 64);
    return s;
}

// part[m][n] = sum_k X[m][k] W[n][k].  One wave per output feature n and R rows of X; lanes stride over k, four
// consecutive k a lane where K is a multiple of four (rows are then 16-byte aligned), then one reduction over the lanes
// for all R rows together.  Bound by the latency of one or two rounds of loads and of the reduction: with single floats
// and a separate wave reduction per row a launch of the tiny shape (16 rows, K = 256) took 6.2 us, and 8.3 on average
// over a generation; R follows the rows of the call so that a draft phase of a few rows does not load sixteen.
template <int R, bool VEC>
__global__ __launch_bounds__(256) void gemm_f32_kernel(const float *__restrict__ X, const float *__restrict__ W,
                                                        float *__restrict__ part, int M, int N, int K, int ld) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int n = blockIdx.x * 4 + wave;
    const int m0 = blockIdx.y * R;
    if (n >= N) return;                                              // whole waves
    float acc[R];
    const float *xr[R];
#pragma unroll
    for (int i = 0; i < R; ++i) { acc[i] = 0.f; xr[i] = X + (size_t)min(m0 + i, M - 1) * K; }
    const float *wr = W + (size_t)n * K;
    if (VEC) {
        for (int k = lane * 4; k < K; k += 256) {
            const f32x4_t w = *reinterpret_cast<const f32x4_t *>(wr + k);
            f32x4_t x[R];
#pragma unroll
            for (int i = 0; i < R; ++i) x[i] = *reinterpret_cast<const f32x4_t *>(xr[i] + k);
#pragma unroll
            for (int i = 0; i < R; ++i) {
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[i] = fmaf(x[i][e], w[e], acc[i]);
            }
        }
    } else {
        for (int k = lane; k < K; k += 64) {
            const float w = wr[k];
#pragma unroll
            for (int i = 0; i < R; ++i) acc[i] = fmaf(xr[i][k], w, acc[i]);
        }
    }
    const float s = lanes_sum<R>(acc, lane);
    if (lane < R && m0 + lane < M) part[(size_t)(m0 + lane) * ld + n] = s;
}

int launch_gemm_f32(hydra_ctx *c, hipStream_t s, const float *X, const float *W, float *part, int M, int N, int K) {
    (void)c;
    // K % 4 == 0: X and W start at 256-byte boundaries of the workspace and the arena, so every row is 16-byte aligned
    const bool vec = K % 4 == 0;
    const int r = M <= 1 ? 1 : M <= 2 ? 2 : M <= 4 ? 4 : M <= 8 ? 8 : 16;
    dim3 grid(ceil_div(N, 4), ceil_div(M, r)), block(256);
#define GEMM_F32(Rv)                                                                                                  \
    case Rv:                                                                                                          \
        if (vec) hipLaunchKernelGGL((gemm_f32_kernel<Rv, true>), grid, block, 0, s, X, W, part, M, N, K, N);            \
        else     hipLaunchKernelGGL((gemm_f32_kernel<Rv, false>), grid, block, 0, s, X, W, part, M, N, K, N);           \
        break
    switch (r) { GEMM_F32(1); GEMM_F32(2); GEMM_F32(4); GEMM_F32(8); GEMM_F32(16); }
#undef GEMM_F32
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
        if (m_new == -INFINITY) continue;                           // nothing visible yet (wave-uniform)
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
