// Generic kernels of the verify round: one straightforward kernel per step, templated on the
// storage type (float or bf16) of weights / cache (WT) and of activations (AT; float in both paths).
// They serve the fp32 configuration and are the fallback wherever no specialised bf16 kernel
// applies (shapes the matrix-core kernels do not serve).
#include "wisv_internal.h"

namespace wisv {

template <typename T> __device__ __forceinline__ void load8(const T *p, float *out);
template <> __device__ __forceinline__ void load8<float>(const float *p, float *out) {
    float4 a = *reinterpret_cast<const float4 *>(p), b = *reinterpret_cast<const float4 *>(p + 4);
    out[0] = a.x; out[1] = a.y; out[2] = a.z; out[3] = a.w;
    out[4] = b.x; out[5] = b.y; out[6] = b.z; out[7] = b.w;
}
template <> __device__ __forceinline__ void load8<bf16_t>(const bf16_t *p, float *out) {
    uint4 a = *reinterpret_cast<const uint4 *>(p);
    uint32_t w[4] = {a.x, a.y, a.z, a.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        out[2 * i] = __uint_as_float(w[i] << 16);
        out[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
    }
}

// float sum over a block of NT threads (NT multiple of 64); every thread gets the result
template <int NT> __device__ __forceinline__ float block_sum(float v, float *red) {
    v = wave_sum(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    float t = 0.f;
#pragma unroll
    for (int w = 0; w < NT / 64; ++w) t += red[w];
    return t;
}
template <int NT> __device__ __forceinline__ float block_max(float v, float *red) {
    v = wave_max(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    float t = red[0];
#pragma unroll
    for (int w = 1; w < NT / 64; ++w) t = fmaxf(t, red[w]);
    return t;
}

// ------------------------------------------------------------------------------------------ inputs of a host-pointer round
// Reads pinned host memory over the link: a kernel in the stream's own queue instead of one copy command per argument
// (seven of about 10 us each for a small round).  Every load of a thread goes out before its first store.
__global__ __launch_bounds__(256) void k_unpack(const uint4 *__restrict__ host, uint4 *__restrict__ dev, size_t n) {
    const size_t i0 = (size_t)blockIdx.x * 1024 + threadIdx.x;
    uint4 v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = host[min(i0 + 256 * u, n - 1)];
#pragma unroll
    for (int u = 0; u < 4; ++u)
        if (i0 + 256 * u < n) dev[i0 + 256 * u] = v[u];
}

void launch_unpack(Ctx *c, const void *host, void *dev, size_t bytes) {
    const size_t n = bytes / 16;
    if (!n) return;
    hipLaunchKernelGGL(k_unpack, dim3((unsigned)((n + 1023) / 1024)), dim3(256), 0, c->stream, (const uint4 *)host, (uint4 *)dev, n);
}

// ------------------------------------------------------------------------------------------ RMSNorm
// x[m] += y[0][m] + ... + y[n_partial-1][m] (fixed order), then out[m] = x[m] / sqrt(mean(x^2)+eps) * g
// NP: the most slices a launch may hold (the loads of all NP are issued whatever n_partial is); 0: the first launch of a
// forward, where x[m] is the embedding of row m's token and the rows' slots and positions are noted too: row m =
// (stream b = m / k, position j = m % k) sits at L_b + j (one launch instead of three: 96 rows 4.2 + 9.1 + 4.7 us before)
// ss_out != null: the 1 / rms is left to whoever adds up the product's slices (out = x * g, ss_out[m] = sum of x^2)
struct FirstRows {
    const int32_t *tokens, *stream_ids, *kv_len;
    const void *embed;
    int vocab, k, max_batch, max_ctx;
    int32_t *row_slot, *row_pos;
};
template <typename WT> __device__ __forceinline__ float4 load4(const WT *p);
template <> __device__ __forceinline__ float4 load4<float>(const float *p) { return *reinterpret_cast<const float4 *>(p); }
template <> __device__ __forceinline__ float4 load4<bf16_t>(const bf16_t *p) {
    const uint2 v = *reinterpret_cast<const uint2 *>(p);
    return make_float4(__uint_as_float(v.x << 16), __uint_as_float(v.x & 0xffff0000u), __uint_as_float(v.y << 16), __uint_as_float(v.y & 0xffff0000u));
}
template <typename WT, typename AT, int NP>
__global__ __launch_bounds__(1024) void k_rmsnorm(float *x, const float *__restrict__ y, int n_partial, size_t partial_stride,
                          const WT *__restrict__ g, int d, float eps, ActBuf out, float *out_f32, float *ss_out, FirstRows first) {
    __shared__ float red[16];
    const int m = blockIdx.x;
    float *xr = x + (size_t)m * d;
    const WT *er = nullptr;
    if (NP == 0) {
        const int b = m / first.k, s = min(max(first.stream_ids[b], 0), first.max_batch - 1);
        er = (const WT *)first.embed + (size_t)min(max(first.tokens[m], 0), first.vocab - 1) * d;
        if (threadIdx.x == 0) {
            first.row_slot[m] = s;
            first.row_pos[m] = min(max(first.kv_len[s], 0) + m - b * first.k, first.max_ctx - 1);
        }
    }
    float ss = 0.f;
    // 1024 threads, four consecutive elements each per pass.  Every slice is requested before the first is used
    // (no load sits behind a branch: slices past the last re-read it and count as zero) and added in slice order.
    // The first pass's elements stay in registers for the second phase.
    float4 v0 = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int i = threadIdx.x * 4; i < d; i += 4096) {
        float4 v = NP == 0 ? load4<WT>(er + i) : *reinterpret_cast<const float4 *>(xr + i);
        float4 part[NP ? NP : 1];
        const int np = max(n_partial, 1);
#pragma unroll
        for (int p = 0; p < NP; ++p)
            part[p] = *reinterpret_cast<const float4 *>(y + (size_t)min(p, np - 1) * partial_stride + (size_t)m * d + i);
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            const bool on = p < n_partial;   // a select, not a product: the unused re-read may hold anything
            v.x += on ? part[p].x : 0.f; v.y += on ? part[p].y : 0.f; v.z += on ? part[p].z : 0.f; v.w += on ? part[p].w : 0.f;
        }
        if (NP == 0 || n_partial) *reinterpret_cast<float4 *>(xr + i) = v;
        if (i < 4096) v0 = v;
        ss += (v.x * v.x + v.y * v.y) + (v.z * v.z + v.w * v.w);
    }
    if (NP == 0 && !g) return;      // the norm is folded into the product that follows
    ss = block_sum<1024>(ss, red);
    const float inv = ss_out ? 1.0f : 1.0f / sqrtf(ss / (float)d + eps);
    if (ss_out && threadIdx.x == 0) ss_out[m] = ss;
    for (int i = threadIdx.x * 4; i < d; i += 4096) {
        const float4 v = i < 4096 ? v0 : *reinterpret_cast<const float4 *>(xr + i);
        float4 r;
        r.x = v.x * inv * Elem<WT>::load(g + i);
        r.y = v.y * inv * Elem<WT>::load(g + i + 1);
        r.z = v.z * inv * Elem<WT>::load(g + i + 2);
        r.w = v.w * inv * Elem<WT>::load(g + i + 3);
        // a representation whose pointer is null has no reader this round and is not written
        if (out.f) *reinterpret_cast<float4 *>(out.f + (size_t)m * d + i) = r;
        if (out.hi) {
            bf16_t h[4], l[4];
            split2(r.x, h[0], l[0]);
            split2(r.y, h[1], l[1]);
            split2(r.z, h[2], l[2]);
            split2(r.w, h[3], l[3]);
            *reinterpret_cast<uint2 *>(out.hi + (size_t)m * d + i) = make_uint2(h[0] | ((uint32_t)h[1] << 16), h[2] | ((uint32_t)h[3] << 16));
            *reinterpret_cast<uint2 *>(out.lo + (size_t)m * d + i) = make_uint2(l[0] | ((uint32_t)l[1] << 16), l[2] | ((uint32_t)l[3] << 16));
        }
        if (out.h16)
            *reinterpret_cast<uint2 *>(out.h16 + (size_t)m * d + i) = make_uint2(f32_to_f16(r.x) | ((uint32_t)f32_to_f16(r.y) << 16),
                                                                                 f32_to_f16(r.z) | ((uint32_t)f32_to_f16(r.w) << 16));
        if (out_f32) *reinterpret_cast<float4 *>(out_f32 + (size_t)m * d + i) = r;
    }
}

template <int NP>
static void launch_rmsnorm_np(Ctx *c, int rows, int n_partial, const void *g, const ActBuf &out, float *out_f32, int row0, float *ss_out,
                              const FirstRows &first = {}) {
    const int d = c->cfg.d_model;
    const size_t stride = (size_t)c->slice_rows * d;
    float *x = c->x + (size_t)row0 * d, *y = c->y + (size_t)row0 * d;
    if (c->bf16)
        hipLaunchKernelGGL((k_rmsnorm<bf16_t, float, NP>), dim3(rows), dim3(1024), 0, c->stream, x, y, n_partial,
                           stride, (const bf16_t *)g, d, c->cfg.rms_eps, out, out_f32, ss_out, first);
    else
        hipLaunchKernelGGL((k_rmsnorm<float, float, NP>), dim3(rows), dim3(1024), 0, c->stream, x, y, n_partial,
                           stride, (const float *)g, d, c->cfg.rms_eps, out, out_f32, ss_out, first);
}

void launch_rmsnorm(Ctx *c, int rows, int n_partial, const void *g, const ActBuf &out, float *out_f32, int row0, float *ss_out) {
    ProfScope ps(c, KC_NORM);
    static_assert(MAX_SPLITS <= 16, "the widest instantiation below covers every slice count");
    // the kernel requests as many slices as its instantiation holds: the smallest one that covers n_partial
    if (n_partial <= 4) launch_rmsnorm_np<4>(c, rows, n_partial, g, out, out_f32, row0, ss_out);
    else if (n_partial <= 8) launch_rmsnorm_np<8>(c, rows, n_partial, g, out, out_f32, row0, ss_out);
    else launch_rmsnorm_np<16>(c, rows, n_partial, g, out, out_f32, row0, ss_out);
}

void launch_embed(Ctx *c, const Fwd &f, const void *g, const ActBuf &out, float *ss_out) {
    ProfScope ps(c, KC_EMBED);
    launch_rmsnorm_np<0>(c, f.rows, 0, g, out, nullptr, 0, ss_out,
                         FirstRows{f.tokens, f.stream_ids, c->d_kv_len, c->embed, c->cfg.vocab, f.k, c->cfg.max_batch, c->cfg.max_ctx,
                                   c->row_slot, c->row_pos});
}

// ------------------------------------------------------------------------------------------ GEMM (fallback)
// Y[r, o] = sum_i A[r, i] W[o, i]; one wave per output feature, MT rows per pass, kd % 8 == 0
// SWIGLU: W stacks gate over up; the wave of feature o takes both of its rows and H[r, o] = silu(gate) * up
// Bound by latency at the small shapes it serves: every row of a pass is requested before the first is used (rows past the last
// re-read it).  The tiny fp32 target, four rows: 1.5 to 2 us per launch, 1.5 to 2.6 with each row's loads behind a branch, and
// SwiGLU needs no launch of its own (2 us and a gap); the whole call 178 -> 155 us.  With SwiGLU a pass takes four rows whatever
// their count: eight read the weights half as often and leave half as many waves.  fp32, 1024 to 2 x 2816 features, us per launch
// (event pairs), four / eight: 5 rows 11.4 / 13.1, 8 12.2 / 14.0, 16 16.8 / 19.3, 32 26.2 / 27.1, 128 77 / 82, 512 285 / 299.
template <typename WT, typename AT, int MT, bool SWIGLU>
__global__ void k_gemm_ref(const AT *__restrict__ A, const WT *__restrict__ W, float *__restrict__ Y, ActBuf H, int rows, int n, int kd) {
    constexpr int NW = SWIGLU ? 2 : 1;
    const int lane = threadIdx.x & 63, o = blockIdx.x * 4 + (threadIdx.x >> 6), r0 = blockIdx.y * MT;
    if (o >= n) return;
    float acc[NW][MT];
#pragma unroll
    for (int w = 0; w < NW; ++w)
#pragma unroll
        for (int t = 0; t < MT; ++t) acc[w][t] = 0.f;
    const WT *wr = W + (size_t)o * kd;
    for (int i = lane * 8; i < kd; i += 512) {
        float wv[NW][8], av[MT][8];
#pragma unroll
        for (int w = 0; w < NW; ++w) load8<WT>(wr + (size_t)w * n * kd + i, wv[w]);
#pragma unroll
        for (int t = 0; t < MT; ++t) load8<AT>(A + (size_t)min(r0 + t, rows - 1) * kd + i, av[t]);
#pragma unroll
        for (int t = 0; t < MT; ++t)
#pragma unroll
            for (int w = 0; w < NW; ++w)
#pragma unroll
                for (int e = 0; e < 8; ++e) acc[w][t] = fmaf(av[t][e], wv[w][e], acc[w][t]);
    }
#pragma unroll
    for (int t = 0; t < MT; ++t) {
        float s[NW];
#pragma unroll
        for (int w = 0; w < NW; ++w) s[w] = wave_sum(acc[w][t]);
        if (lane != 0 || r0 + t >= rows) continue;
        if (SWIGLU) act_store(H, (size_t)(r0 + t) * n + o, s[0] / (1.0f + expf(-s[0])) * s[NW - 1]);
        else Y[(size_t)(r0 + t) * n + o] = s[0];
    }
}

template <int MT, bool SWIGLU> static void launch_gemm_ref_t(Ctx *c, const float *A, const void *W, float *Y, const ActBuf &H, int rows, int n, int kd) {
    const dim3 grid((n + 3) / 4, (rows + MT - 1) / MT);
    if (c->bf16)
        hipLaunchKernelGGL((k_gemm_ref<bf16_t, float, MT, SWIGLU>), grid, dim3(256), 0, c->stream, A, (const bf16_t *)W, Y, H, rows, n, kd);
    else
        hipLaunchKernelGGL((k_gemm_ref<float, float, MT, SWIGLU>), grid, dim3(256), 0, c->stream, A, (const float *)W, Y, H, rows, n, kd);
}

void launch_gemm_ref(Ctx *c, const float *A, const void *W, float *Y, int rows, int n, int kd, int kclass) {
    ProfScope ps(c, kclass);
    if (rows <= 4) launch_gemm_ref_t<4, false>(c, A, W, Y, ActBuf{}, rows, n, kd);
    else launch_gemm_ref_t<8, false>(c, A, W, Y, ActBuf{}, rows, n, kd);
}

void launch_gemm_ref_swiglu(Ctx *c, const float *A, const void *W, const ActBuf &H, int rows, int features, int kd) {
    ProfScope ps(c, KC_GEMM_GATEUP);
    launch_gemm_ref_t<4, true>(c, A, W, nullptr, H, rows, features, kd);
}

// ------------------------------------------------------------------------------------------ RoPE + KV append
// grid (rows, H + 2G), block hd/2.  q heads: rotate -> q operand; k heads: rotate -> cache; v heads: copy -> cache
template <typename WT, typename AT>
__global__ void k_rope_append(const float *__restrict__ qkv, int n_partial, size_t partial_stride, int H, int G, int hd, const int32_t *__restrict__ row_slot,
                              const int32_t *__restrict__ row_pos, const float *__restrict__ cs,
                              const float *__restrict__ sn, AT *q_out, WT *kv_layer, size_t slot_stride, int ctx_pad,
                              const float *__restrict__ ss, int n_ss, int d_model, float eps) {
    const int m = blockIdx.x, hh = blockIdx.y, i = threadIdx.x, half = hd >> 1;
    const int d_q = H * hd, d_kv = G * hd, pos = row_pos[m];
    const float *src = qkv + (size_t)m * (d_q + 2 * d_kv) + (size_t)hh * hd;
    float a = src[i], b = src[i + half];
    for (int p = 1; p < n_partial; ++p) {   // fixed order: slice 0 + slice 1 + ...
        a += src[p * partial_stride + i];
        b += src[p * partial_stride + i + half];
    }
    if (n_ss > 0) {   // the slices are products of x * gain: the deferred 1 / rms of the folded RMSNorm
        float t = 0.f;
        for (int p = 0; p < n_ss; ++p) t += ss[(size_t)p * gridDim.x + m];
        const float inv = 1.0f / sqrtf(t / (float)d_model + eps);
        a *= inv;
        b *= inv;
    }
    const float co = cs[(size_t)pos * half + i], si = sn[(size_t)pos * half + i];
    if (hh < H) {
        AT *dst = q_out + (size_t)m * d_q + (size_t)hh * hd;
        Elem<AT>::store(dst + i, a * co - b * si);
        Elem<AT>::store(dst + i + half, b * co + a * si);
    } else if (hh < H + G) {
        WT *dst = kv_layer + (size_t)row_slot[m] * slot_stride + ((size_t)(hh - H) * ctx_pad + pos) * hd;
        Elem<WT>::store(dst + i, a * co - b * si);
        Elem<WT>::store(dst + i + half, b * co + a * si);
    } else {
        WT *dst = kv_layer + (size_t)row_slot[m] * slot_stride + (size_t)(hh - H) * ctx_pad * hd;   // V planes follow the G K planes
        Elem<WT>::store(dst + v_plane_index(pos, i, hd), a);
        Elem<WT>::store(dst + v_plane_index(pos, i + half, hd), b);
    }
}

void launch_rope_append(Ctx *c, const Fwd &f, int layer, int n_partial, int n_ss) {
    const size_t pstride = (size_t)c->slice_rows * c->d_qkv;
    ProfScope ps(c, KC_ROPE);
    const wisv_config &g = c->cfg;
    const size_t slot_stride = (size_t)2 * g.n_kv_heads * c->ctx_pad * g.head_dim;
    dim3 grid(f.rows, g.n_heads + 2 * g.n_kv_heads), block(g.head_dim / 2);
    void *kvl = kv_ptr(c, layer, 0, 0);
    if (c->bf16)
        hipLaunchKernelGGL((k_rope_append<bf16_t, float>), grid, block, 0, c->stream, c->qkv, n_partial, pstride, g.n_heads, g.n_kv_heads,
                           g.head_dim, c->row_slot, c->row_pos, c->rope_cos, c->rope_sin, c->q, (bf16_t *)kvl,
                           slot_stride, c->ctx_pad, c->ss, n_ss, g.d_model, g.rms_eps);
    else
        hipLaunchKernelGGL((k_rope_append<float, float>), grid, block, 0, c->stream, c->qkv, n_partial, pstride, g.n_heads, g.n_kv_heads,
                           g.head_dim, c->row_slot, c->row_pos, c->rope_cos, c->rope_sin, c->q, (float *)kvl,
                           slot_stride, c->ctx_pad, c->ss, n_ss, g.d_model, g.rms_eps);
}

// ------------------------------------------------------------------------------------------ attention (fallback)
// one block per (row, query head): scores of the visible keys in LDS, float softmax, then P.V
template <typename WT, typename AT>
__global__ void k_attn_ref(const AT *__restrict__ q, const WT *__restrict__ kv_layer, size_t slot_stride, int H, int G,
                           int hd, int ctx_pad, const int32_t *__restrict__ row_slot,
                           const int32_t *__restrict__ row_pos, ActBuf o) {
    extern __shared__ float smem[];
    float *qs = smem;            // [hd]
    float *red = smem + hd;      // [256 + 4]
    float *sc = red + 260;       // [n_vis]
    const int m = blockIdx.x, h = blockIdx.y, g = h / (H / G), tid = threadIdx.x;
    const int n_vis = row_pos[m] + 1;
    const WT *kc = kv_layer + (size_t)row_slot[m] * slot_stride + (size_t)g * ctx_pad * hd;
    const WT *vc = kc + (size_t)G * ctx_pad * hd;
    if (tid < hd) qs[tid] = Elem<AT>::load(q + (size_t)m * H * hd + (size_t)h * hd + tid);
    __syncthreads();
    const float scale = 1.0f / sqrtf((float)hd);
    float mx = -INFINITY;
    for (int s = tid; s < n_vis; s += 256) {
        float acc = 0.f, kvv[8];
        for (int i = 0; i < hd; i += 8) {
            load8<WT>(kc + (size_t)s * hd + i, kvv);
#pragma unroll
            for (int e = 0; e < 8; ++e) acc = fmaf(qs[i + e], kvv[e], acc);
        }
        acc *= scale;
        sc[s] = acc;
        mx = fmaxf(mx, acc);
    }
    mx = block_max<256>(mx, red + 256);
    float sum = 0.f;
    for (int s = tid; s < n_vis; s += 256) {
        float e = expf(sc[s] - mx);
        sc[s] = e;
        sum += e;
    }
    sum = block_sum<256>(sum, red + 256);   // also makes every sc[] visible
    const int dim = tid % hd, part = tid / hd, nparts = 256 / hd;
    float acc = 0.f;
    for (int s = part; s < n_vis; s += nparts) acc = fmaf(sc[s], Elem<WT>::load(vc + v_plane_index(s, dim, hd)), acc);
    red[tid] = acc;
    __syncthreads();
    if (part == 0) {
        for (int p = 1; p < nparts; ++p) acc += red[p * hd + dim];
        act_store(o, (size_t)m * H * hd + (size_t)h * hd + dim, acc / sum);
    }
}

void launch_attn_ref(Ctx *c, const Fwd &f, int layer) {
    ProfScope ps(c, KC_ATTN);
    const wisv_config &g = c->cfg;
    const size_t slot_stride = (size_t)2 * g.n_kv_heads * c->ctx_pad * g.head_dim;
    // the kernel keeps every visible score in LDS: contexts beyond what a workgroup may hold are not served
    const size_t lds = sizeof(float) * (g.head_dim + 260 + f.max_len_ub);
    static bool allowed_bf16[MAX_DEVICES], allowed_f32[MAX_DEVICES];
    const void *kern = c->bf16 ? reinterpret_cast<const void *>(&k_attn_ref<bf16_t, float>) : reinterpret_cast<const void *>(&k_attn_ref<float, float>);
    if (lds > 150 * 1024 || (lds > 64 * 1024 && !allow_big_lds(c, kern, c->bf16 ? allowed_bf16 : allowed_f32))) {
        c->launch_failed = true;
        c->launch_err = "the generic attention kernel holds one score per visible position in LDS: a context of " +
                        std::to_string(f.max_len_ub) + " positions does not fit (this shape is not served by the MFMA attention kernel)";
        return;
    }
    dim3 grid(f.rows, g.n_heads);
    void *kvl = kv_ptr(c, layer, 0, 0);
    if (c->bf16)
        hipLaunchKernelGGL((k_attn_ref<bf16_t, float>), grid, dim3(256), lds, c->stream, (const float *)c->q,
                           (const bf16_t *)kvl, slot_stride, g.n_heads, g.n_kv_heads, g.head_dim, c->ctx_pad,
                           c->row_slot, c->row_pos, act_planes(c->o, c->o_planes));
    else
        hipLaunchKernelGGL((k_attn_ref<float, float>), grid, dim3(256), lds, c->stream, (const float *)c->q,
                           (const float *)kvl, slot_stride, g.n_heads, g.n_kv_heads, g.head_dim, c->ctx_pad, c->row_slot,
                           c->row_pos, act_planes(c->o, c->o_planes));
}

// ------------------------------------------------------------------------------------------ V plane <-> rows
// rows: [G][len][hd] (what the host hands over); plane: one (layer, slot) V plane [G][ctx_pad / 32][hd][32]
template <typename WT>
__global__ void k_v_reblock(WT *rows, WT *plane, int len, int hd, int ctx_pad, bool to_plane) {
    const int g = blockIdx.y;
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (size_t)len * hd) return;
    const int pos = i / hd, dim = i % hd;
    WT *r = rows + ((size_t)g * len + pos) * hd + dim, *q = plane + (size_t)g * ctx_pad * hd + v_plane_index(pos, dim, hd);
    if (to_plane) *q = *r;
    else *r = *q;
}

void launch_v_reblock(Ctx *c, void *rows, void *plane, int len, bool to_plane) {
    const wisv_config &g = c->cfg;
    dim3 grid((unsigned)(((size_t)len * g.head_dim + 255) / 256), g.n_kv_heads);
    if (c->bf16)
        hipLaunchKernelGGL(k_v_reblock<bf16_t>, grid, dim3(256), 0, c->stream, (bf16_t *)rows, (bf16_t *)plane, len, g.head_dim,
                           c->ctx_pad, to_plane);
    else
        hipLaunchKernelGGL(k_v_reblock<float>, grid, dim3(256), 0, c->stream, (float *)rows, (float *)plane, len, g.head_dim,
                           c->ctx_pad, to_plane);
}

// after a prefill chunk: the slot's length grows by the chunk; after the last one pred_next = the last row's greedy token
__global__ __launch_bounds__(64) void k_set_pred_next(int32_t *kv_len, int32_t *pred_next, const uint2 *best, int slot, int row, int new_len,
                                                      int parts) {
    const int token = row >= 0 ? greedy_token(greedy_part(best, parts, row, threadIdx.x)) : 0;
    if (threadIdx.x) return;
    if (row >= 0) pred_next[slot] = token;
    kv_len[slot] = new_len;
}

void launch_set_pred_next(Ctx *c, int slot, int row, int new_len) {
    const int parts = row >= 0 ? greedy_cut(c->cand).parts : 1;
    hipLaunchKernelGGL(k_set_pred_next, dim3(1), dim3(64), 0, c->stream, c->d_kv_len, c->d_pred_next, c->best, slot, row, new_len, parts);
}

}  // namespace wisv
