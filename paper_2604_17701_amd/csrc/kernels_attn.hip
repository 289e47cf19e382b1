// Grouped-query attention of the drafted block over the KV cache (bf16 cache, head_dim 128):
// the K query rows of a stream x the query heads that share one KV head form one tile of up to 64 rows, so
// every cached key/value byte is read once per (stream, KV head) and meets all of them.
//
// One workgroup = (k-split, KV head, stream); its waves take steps of 32 keys round-robin and never meet before
// the end: nothing is staged in LDS.  K rows go straight from the cache into the A operand of S^T = K Q^T
// (16x16x32 MFMA, two tiles of 16 keys per step, queries as two bf16 terms in the B operand).  The keys of a
// step are dealt to the two tiles so that lane group g ends up holding the scores of the eight consecutive keys
// 8 g .. 8 g + 7 of every query: after the float online softmax these eight probabilities are, as they stand,
// the B operand of O^T += V^T P^T on the 16x16x32 MFMA (two bf16 terms again, so P.V is exact to 2^-17), whose A
// operand - 16 features x 32 keys of V^T - is one 16-byte load per lane from the cache's V plane, which keeps
// 32 positions of a feature contiguous for exactly this reason.  Waves are merged through LDS at the end with
// the usual (max, sum, unnormalised output) rule in wave order; k-splits, when there are several, by a small
// kernel, otherwise the workgroup writes the attention output itself.
#include <algorithm>

#include "wisv_internal.h"

namespace wisv {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

constexpr int HD = 128, STEP = 32;

struct AttnArgs {
    const bf16_t *kv_layer;   // this layer's cache: [slot][K|V][G] planes of ctx_pad * 128
    size_t slot_stride;       // elements per slot
    int H, G, rep, K, max_ctx, ctx_pad, n_splits, rows;
    const int32_t *row_slot, *row_pos;
    float *po, *pm, *pl;      // partials [split][rows][H][128], [split][rows][H]  (n_splits > 1); pm in units of ln 2
    ActBuf o;                 // attention output [rows][H][128]                    (n_splits == 1)
    // the kernel sums the k-split slices of the QKV product itself and rotates q (a round: and k, and appends k and v)
    const float *qkv;         // [n_partial][partial_stride] slices of [rows][H*128 + 2 G*128]
    int n_partial;
    size_t partial_stride;
    const float *cs, *sn;     // rotary tables [max_ctx][64]
    // n_ss > 0: the slices are products of x * gain; row m is scaled by 1 / sqrt(sum_p ss[p][m] / d_model + eps)
    const float *ss;          // [n_ss][rows]
    int n_ss, d_model;
    float eps;
    bf16_t *kv_write;         // == kv_layer
};

// NQ: 16-row query tiles; NW: waves per workgroup.  Every workgroup rotates the queries it needs from the slices of the
// QKV product.  A round (!PROMPT): the workgroup of a (stream, KV head) whose k-split ends the sequence also writes the
// new k, v rows before any of its waves reads them (no other split reads them).  PROMPT: a block of a prompt's chunk, whose
// k, v rows k_kv_append has written (a block reads those of the blocks before it).
// NP: the most slices of the QKV product a launch may hold (all NP are requested whatever n_partial is, slices past
// the last re-read it); NSS: the most partial sums of squares (0: the rows want no 1 / rms of a folded RMSNorm)
//
// PROMPT is bound by the vector and matrix instructions of its waves, about as many cycles of either per step: two waves per
// SIMD overlap them, which takes at most 256 registers and 80 KB of LDS.  Three query tiles meet that (four spill), and the
// waves' outputs are merged in two parts of the features.  us per layer, event pairs (4.5 of bracketing), mean of the two chunks of a
// prompt of 1999 tokens / the one of 512, four query heads per KV head, the queries still rotated by a kernel before this one: four
// tiles, one wave per SIMD 87.5 / 26.7; four capped with spills 77.1 / 33.1; three 67.0 / 23.7; two 92.0 / 30.3.  That
// kernel, which rotated the queries and appended k and v, and this one together: 117.6 / 42.1 with four tiles, 86.1 / 30.3
// with three and the rotation inside.
// Rounds of three and four tiles, one workgroup per CU at most, keep the registers of one wave (143 rows: 42.0 us, capped 42.7).
constexpr int attn_merge_parts(int nq) { return nq > 2 ? 2 : 1; }
template <int NQ, int NW, bool PROMPT, int NP, int NSS>
__global__ __launch_bounds__(64 * NW, PROMPT && NQ < 4 ? 2 : 1) void k_attn_mfma(AttnArgs a) {
    extern __shared__ __align__(16) unsigned char lds[];
    constexpr int PARTS = attn_merge_parts(NQ);
    // (a prompt's last blocks see the most keys: they start first)
    const int split = blockIdx.x, g = blockIdx.y, b = PROMPT ? gridDim.z - 1 - blockIdx.z : blockIdx.z;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, bj = lane & 15, bg = lane >> 4;
    const int m0 = b * a.K;
    const int L = a.row_pos[m0], slot = a.row_slot[m0];
    const int K = min(a.K, a.rows - m0);   // a prompt's last block of rows may be short; a round's blocks never are
    const int n_keys = min(L + K, a.max_ctx), R = a.rep * K;
    const bf16_t *kc = a.kv_layer + (size_t)slot * a.slot_stride + (size_t)g * a.ctx_pad * HD;
    const bf16_t *vc = kc + (size_t)a.G * a.ctx_pad * HD;
    const int n_steps = (n_keys + STEP - 1) / STEP, sps = (n_steps + a.n_splits - 1) / a.n_splits;
    int s_begin = split * sps, s_end = min(n_steps, s_begin + sps);
    // A round with several k-splits: the last split appends the block's k, v rows, so it owns every step from the one
    // that holds position L on (at most two steps more than its share); the others stop there
    const bool appends = !PROMPT && split == a.n_splits - 1;
    if (!PROMPT && a.n_splits > 1) {
        const int tail = L / STEP;
        if (appends) {
            s_begin = min(s_begin, tail);
            s_end = n_steps;
        } else {
            s_end = min(s_end, tail);
            s_begin = min(s_begin, s_end);
        }
    }

    // ---- the first step's loads go out before anything else.  Lane (bj, bg): tile A row bj is key
    //      8 (bj / 4) + bj % 4 of the step, tile B row bj the key four further; V^T row bj of feature tile dt.
    u32x4 ka[4], kb[4], va[8];
    const int krow = 8 * (bj >> 2) + (bj & 3);
#define WISV_ATTN_LOAD_K(s_)                                                                              \
    {                                                                                                     \
        const bf16_t *pa_ = kc + (size_t)min((s_) * STEP + krow, n_keys - 1) * HD + 8 * bg;               \
        const bf16_t *pb_ = kc + (size_t)min((s_) * STEP + krow + 4, n_keys - 1) * HD + 8 * bg;           \
        _Pragma("unroll") for (int t = 0; t < 4; ++t) {                                                   \
            ka[t] = *reinterpret_cast<const u32x4 *>(pa_ + 32 * t);                                       \
            kb[t] = *reinterpret_cast<const u32x4 *>(pb_ + 32 * t);                                       \
        }                                                                                                 \
    }
#define WISV_ATTN_LOAD_V(s_)                                                                              \
    {                                                                                                     \
        const bf16_t *pv_ = vc + ((size_t)(s_) * HD + bj) * STEP + 8 * bg;                                \
        _Pragma("unroll") for (int dt = 0; dt < 8; ++dt) va[dt] = *reinterpret_cast<const u32x4 *>(pv_ + (size_t)dt * 16 * STEP); \
    }
    constexpr int QREG = NQ > 1 ? 1 : NQ;
    u32x4 qhi[QREG][4], qlo[QREG][4];
    u32x4 *qs = reinterpret_cast<u32x4 *>(lds);   // [NQ][4][2][64] query operands; the merge at the end re-uses the space
    int s = s_begin + wave;
    {
        // this wave's first step is requested now; if it holds appended rows it is requested again below
        const int s0 = min(s, n_steps - 1);
        WISV_ATTN_LOAD_K(s0)
        WISV_ATTN_LOAD_V(s0)
    }
    {
        // ---- RoPE + append.  Work item = (row, pair of features i, i + 64): q rows rho < R of this KV head's query
        //      heads go, rotated and split into two bf16 terms, straight into the operand layout in LDS; the K new
        //      rows of k (rotated) and v go to the cache.  Slices are added in slice order.
        const int d_q = a.H * HD, d_kv = a.G * HD, d_all = d_q + 2 * d_kv;
        bf16_t *kw = a.kv_write + (size_t)slot * a.slot_stride + (size_t)g * a.ctx_pad * HD;
        bf16_t *vw = kw + (size_t)a.G * a.ctx_pad * HD;
        bf16_t *q16 = reinterpret_cast<bf16_t *>(qs);
        for (int it = tid; it < (16 * NQ + (appends ? 2 * K : 0)) * 16; it += 64 * NW) {
            const int row = it >> 4, i = (it & 15) * 4;   // features i .. i + 3 and their partners i + 64 .. i + 67
            int j, col;                      // token of the block, first column of the head in a qkv row
            if (row < 16 * NQ) {
                const int rho = min(row, R - 1);
                j = rho / a.rep;
                col = (g * a.rep + rho % a.rep) * HD;
            } else if (row < 16 * NQ + K) {
                j = row - 16 * NQ;
                col = d_q + g * HD;
            } else {
                j = row - 16 * NQ - K;
                col = d_q + d_kv + g * HD;
            }
            const float *src = a.qkv + (size_t)(m0 + j) * d_all + col + i;
            // every slice is requested before the first is used (slices past the last re-read it and count as 0)
            floatx4 xs[NP], ys[NP];
#pragma unroll
            for (int p = 0; p < NP; ++p) {
                const size_t off = (size_t)min(p, a.n_partial - 1) * a.partial_stride;
                xs[p] = *reinterpret_cast<const floatx4 *>(src + off);
                ys[p] = *reinterpret_cast<const floatx4 *>(src + off + 64);
            }
            float ssp[NSS ? NSS : 1];
            if (NSS) {
#pragma unroll
                for (int p = 0; p < NSS; ++p) ssp[p] = a.ss[(size_t)min(p, a.n_ss - 1) * a.rows + m0 + j];
            }
            const int pos = min(L + j, a.max_ctx - 1);
            const floatx4 co = *reinterpret_cast<const floatx4 *>(a.cs + (size_t)pos * 64 + i);
            const floatx4 si = *reinterpret_cast<const floatx4 *>(a.sn + (size_t)pos * 64 + i);
            floatx4 x = xs[0], y = ys[0];
#pragma unroll
            for (int p = 1; p < NP; ++p) {
                const bool on = p < a.n_partial;
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    x[c] += on ? xs[p][c] : 0.f;
                    y[c] += on ? ys[p][c] : 0.f;
                }
            }
            if (NSS) {   // the deferred 1 / rms of the folded RMSNorm (sums of squares in slice order)
                float t = 0.f;
#pragma unroll
                for (int p = 0; p < NSS; ++p) t += p < a.n_ss ? ssp[p] : 0.f;
                const float inv = 1.0f / sqrtf(t / (float)a.d_model + a.eps);
#pragma unroll
                for (int c = 0; c < 4; ++c) { x[c] *= inv; y[c] *= inv; }
            }
            float r0[4], r1[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                r0[c] = x[c] * co[c] - y[c] * si[c];
                r1[c] = y[c] * co[c] + x[c] * si[c];
            }
            if (row < 16 * NQ) {
                // element (rho, dim) of operand (nq, t = dim / 32, plane): lane 16 ((dim % 32) / 8) + rho % 16, slot dim % 8
                const int nq = row >> 4, bjq = row & 15;
                const int e = i & 7, ln = 16 * ((i & 31) >> 3) + bjq, t0 = i >> 5;
                uint2 h0, l0, h1, l1;
                if (row >= R) {
#pragma unroll
                    for (int c = 0; c < 4; ++c) r0[c] = r1[c] = 0.f;
                }
                split2x2(r0[0], r0[1], h0.x, l0.x);
                split2x2(r0[2], r0[3], h0.y, l0.y);
                split2x2(r1[0], r1[1], h1.x, l1.x);
                split2x2(r1[2], r1[3], h1.y, l1.y);
                *reinterpret_cast<uint2 *>(q16 + ((((nq * 4 + t0) * 2 + 0) * 64 + ln) << 3) + e) = h0;
                *reinterpret_cast<uint2 *>(q16 + ((((nq * 4 + t0) * 2 + 1) * 64 + ln) << 3) + e) = l0;
                *reinterpret_cast<uint2 *>(q16 + ((((nq * 4 + t0 + 2) * 2 + 0) * 64 + ln) << 3) + e) = h1;
                *reinterpret_cast<uint2 *>(q16 + ((((nq * 4 + t0 + 2) * 2 + 1) * 64 + ln) << 3) + e) = l1;
            } else if (row < 16 * NQ + K) {
                bf16_t k0[4], k1[4];
#pragma unroll
                for (int c = 0; c < 4; ++c) { k0[c] = f32_to_bf16(r0[c]); k1[c] = f32_to_bf16(r1[c]); }
                *reinterpret_cast<uint2 *>(kw + (size_t)pos * HD + i) = make_uint2(k0[0] | ((unsigned)k0[1] << 16), k0[2] | ((unsigned)k0[3] << 16));
                *reinterpret_cast<uint2 *>(kw + (size_t)pos * HD + i + 64) = make_uint2(k1[0] | ((unsigned)k1[1] << 16), k1[2] | ((unsigned)k1[3] << 16));
            } else {
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    vw[v_plane_index(pos, i + c, HD)] = f32_to_bf16(x[c]);
                    vw[v_plane_index(pos, i + c + 64, HD)] = f32_to_bf16(y[c]);
                }
            }
        }
        __syncthreads();   // the appended rows and the query operands are visible to the whole workgroup
    }
    // (no load below is conditional - a branch around a load makes the compiler wait for it on the spot: a wave
    // without a further step re-reads a step that exists and ignores it)
    if (!PROMPT) {
        const int s0 = min(s, n_steps - 1);
        if ((s0 + 1) * STEP > L) {
            WISV_ATTN_LOAD_K(s0)
            WISV_ATTN_LOAD_V(s0)
        }
    }

    // ---- queries as MFMA B operands (two bf16 terms): lane (bj, bg) holds Q[rho = 16 nq + bj][32 t + 8 bg ..].
    //      One query tile lives in registers; more would crowd out the accumulators and are re-read from LDS at each use.
    if (NQ == 1) {
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            qhi[0][t] = qs[(t * 2 + 0) * 64 + lane];
            qlo[0][t] = qs[(t * 2 + 1) * 64 + lane];
        }
    }

    float m_run[NQ], l_run[NQ];
    floatx4 oacc[NQ][8];
#pragma unroll
    for (int nq = 0; nq < NQ; ++nq) {
        m_run[nq] = -INFINITY;
        l_run[nq] = 0.f;
#pragma unroll
        for (int dt = 0; dt < 8; ++dt) oacc[nq][dt] = floatx4{0.f, 0.f, 0.f, 0.f};
    }

    const float scale = 0.08838834764831845f * 1.4426950408889634f;   // log2(e) / sqrt(128): scores in units of ln 2
    for (; s < s_end; s += NW) {
        const int kbase = s * STEP + 8 * bg;     // this lane's eight keys: kbase .. kbase + 7
        const int s_next = min(s + NW, n_steps - 1);
        u32x4 phi[NQ], plo[NQ];
#pragma unroll
        for (int nq = 0; nq < NQ; ++nq) {
            floatx4 sa = {0.f, 0.f, 0.f, 0.f}, sb = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                u32x4 qh, ql;
                if (NQ > 1) {
                    qh = qs[((nq * 4 + t) * 2 + 0) * 64 + lane];
                    ql = qs[((nq * 4 + t) * 2 + 1) * 64 + lane];
                } else {
                    qh = qhi[nq][t];
                    ql = qlo[nq][t];
                }
                sa = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*reinterpret_cast<bf16x8 *>(&ka[t]), *reinterpret_cast<bf16x8 *>(&qh), sa, 0, 0, 0);
                sb = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*reinterpret_cast<bf16x8 *>(&kb[t]), *reinterpret_cast<bf16x8 *>(&qh), sb, 0, 0, 0);
                sa = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*reinterpret_cast<bf16x8 *>(&ka[t]), *reinterpret_cast<bf16x8 *>(&ql), sa, 0, 0, 0);
                sb = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*reinterpret_cast<bf16x8 *>(&kb[t]), *reinterpret_cast<bf16x8 *>(&ql), sb, 0, 0, 0);
            }
            // lane holds keys kbase + e (e = 0..3 from tile A, 4..7 from tile B) of query rho = 16 nq + bj
            const int rho = nq * 16 + bj;
            const int qpos = L + rho / a.rep;
            float sv[8], mx = -INFINITY;
            if (s * STEP + STEP - 1 <= L) {
                // every query of the block sees every key of this step (wave-uniform): no mask.  Rows past R hold
                // zero queries; their scores are finite and never stored.
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    sv[e] = (e < 4 ? sa[e] : sb[e - 4]) * scale;
                    mx = fmaxf(mx, sv[e]);
                }
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const int kp = kbase + e;
                    const float x = e < 4 ? sa[e] : sb[e - 4];
                    sv[e] = (rho < R && kp <= qpos && kp < n_keys) ? x * scale : -INFINITY;
                    mx = fmaxf(mx, sv[e]);
                }
            }
            mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
            mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
            // Scores are in units of ln 2, so the exponentials are single v_exp_f32 instructions; exp2(-inf) = 0 covers
            // masked keys and a row's first step, and a row that has seen no key at all subtracts 0 instead of -inf.
            const float m_new = fmaxf(m_run[nq], mx);
            const float m_sub = m_new == -INFINITY ? 0.f : m_new;
            const float alpha = __builtin_amdgcn_exp2f(m_run[nq] - m_sub);
            float p[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) p[e] = __builtin_amdgcn_exp2f(sv[e] - m_sub);
            l_run[nq] = l_run[nq] * alpha + (((p[0] + p[1]) + (p[2] + p[3])) + ((p[4] + p[5]) + (p[6] + p[7])));
            m_run[nq] = m_new;
            // the running maximum rarely moves after a row's first steps: scaling by exactly 1 is skipped (wave-uniform)
            if (__any(alpha != 1.f)) {
#pragma unroll
                for (int dt = 0; dt < 8; ++dt) oacc[nq][dt] *= alpha;
            }
            uint32_t h[4], l[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) split2x2(p[2 * e], p[2 * e + 1], h[e], l[e]);
            phi[nq] = u32x4{h[0], h[1], h[2], h[3]};
            plo[nq] = u32x4{l[0], l[1], l[2], l[3]};
            __builtin_amdgcn_sched_barrier(0);   // one query tile at a time: their temporaries must not pile up
        }
        // the K registers are free: request the next step's keys
        WISV_ATTN_LOAD_K(s_next)
        // positions past the end of the sequence may hold anything (0 x NaN would poison the sum): clear them
        if (s * STEP + STEP > n_keys) {
#pragma unroll
            for (int dt = 0; dt < 8; ++dt)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const uint32_t keep = (kbase + 2 * e < n_keys ? 0xffffu : 0u) | (kbase + 2 * e + 1 < n_keys ? 0xffff0000u : 0u);
                    va[dt][e] &= keep;
                }
        }
        // O^T tiles: rows = 16 features (A operand = V^T), columns = 16 queries, k = this lane group's 8 keys
#pragma unroll
        for (int dt = 0; dt < 8; ++dt) {
#pragma unroll
            for (int nq = 0; nq < NQ; ++nq) {
                oacc[nq][dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*reinterpret_cast<bf16x8 *>(&va[dt]),
                                                                      *reinterpret_cast<bf16x8 *>(&phi[nq]), oacc[nq][dt], 0, 0, 0);
                oacc[nq][dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*reinterpret_cast<bf16x8 *>(&va[dt]),
                                                                      *reinterpret_cast<bf16x8 *>(&plo[nq]), oacc[nq][dt], 0, 0, 0);
            }
        }
        WISV_ATTN_LOAD_V(s_next)
    }
#undef WISV_ATTN_LOAD_K
#undef WISV_ATTN_LOAD_V

    // ---- sums over the four lane groups (each held eight keys of every step), fixed order
#pragma unroll
    for (int nq = 0; nq < NQ; ++nq) {
        const float l1 = l_run[nq] + __shfl_xor(l_run[nq], 16, 64);
        l_run[nq] = l1 + __shfl_xor(l1, 32, 64);
    }

    // ---- merge the waves.  Every wave publishes (m, l) of its queries, rescales its output to the common
    //      maximum and publishes that too; wave w then adds up feature tiles w, w + NW, .. of all waves in
    //      wave order.  LDS: sm, sl [NW][NQ][16] floats, then so [NW][NQ][8][64] floatx4.
    float *sm = reinterpret_cast<float *>(lds), *sl = sm + NW * NQ * 16;
    floatx4 *so = reinterpret_cast<floatx4 *>(sl + NW * NQ * 16);
    __syncthreads();   // every wave is done with the query operands that live in the same LDS
    if (bg == 0) {
#pragma unroll
        for (int nq = 0; nq < NQ; ++nq) {
            sm[(wave * NQ + nq) * 16 + bj] = m_run[nq];
            sl[(wave * NQ + nq) * 16 + bj] = l_run[nq];
        }
    }
    __syncthreads();
    float m_all[NQ], l_all[NQ];
#pragma unroll
    for (int nq = 0; nq < NQ; ++nq) {
        float mx = -INFINITY;
        for (int w = 0; w < NW; ++w) mx = fmaxf(mx, sm[(w * NQ + nq) * 16 + bj]);
        float ls = 0.f;
        for (int w = 0; w < NW; ++w) {
            const float mw = sm[(w * NQ + nq) * 16 + bj];
            if (mw != -INFINITY) ls += sl[(w * NQ + nq) * 16 + bj] * exp2f(mw - mx);
        }
        m_all[nq] = mx;
        l_all[nq] = ls;
        m_run[nq] = m_run[nq] == -INFINITY ? 0.f : exp2f(m_run[nq] - mx);   // from here on: the weight of this wave's output
    }
    // (Written out as a loop: with the parts as calls of a lambda the compiler gives the loop over the keys eleven registers fewer and
    // four waits more at one query tile.  us per layer, event pairs: 4 rows over 512 tokens 13.4 -> 12.8, over 4096 15.1 -> 14.4, 12 rows
    // 14.2 -> 13.3, 32 rows 15.7 -> 15.0; two to four tiles and prompts the same.)
    constexpr int DP = 8 / PARTS;   // feature tiles merged at a time
#pragma unroll
    for (int part = 0; part < PARTS; ++part) {
        if (part) __syncthreads();   // the part before has been read
#pragma unroll
        for (int nq = 0; nq < NQ; ++nq)
#pragma unroll
            for (int dt = 0; dt < DP; ++dt) so[((wave * NQ + nq) * DP + dt) * 64 + lane] = oacc[nq][part * DP + dt] * m_run[nq];
        __syncthreads();
        for (int dl = wave; dl < DP; dl += NW) {
            const int dt = part * DP + dl;
#pragma unroll
            for (int nq = 0; nq < NQ; ++nq) {
                const int rho = nq * 16 + bj;
                floatx4 acc = so[((0 * NQ + nq) * DP + dl) * 64 + lane];
                for (int w = 1; w < NW; ++w) acc += so[((w * NQ + nq) * DP + dl) * 64 + lane];
                if (rho >= R) continue;
                // lane holds features 16 dt + 4 bg + r of query rho
                const int m = m0 + rho / a.rep, h = g * a.rep + rho % a.rep;
                if (a.n_splits == 1) {
                    const float inv = 1.0f / l_all[nq];
                    act_store4(a.o, ((size_t)m * a.H + h) * HD + 16 * dt + 4 * bg, acc[0] * inv, acc[1] * inv, acc[2] * inv, acc[3] * inv);
                } else {
                    const size_t row = ((size_t)split * a.rows + m) * a.H + h;
                    *reinterpret_cast<floatx4 *>(a.po + row * HD + 16 * dt + 4 * bg) = acc;
                    if (dt == 0 && bg == 0) {
                        a.pm[row] = m_all[nq];
                        a.pl[row] = l_all[nq];
                    }
                }
            }
        }
    }
}

// ------------------------------------------------------------------------------------------ a prompt's keys and values
// The chunk's rows lie at consecutive positions of one slot.  One workgroup = one block of 32 positions of the cache x one KV
// head, k (blockIdx.z 0: rotated, 16-byte stores) or v (1: turned over in LDS, since the V plane keeps 32 positions of a feature
// together).  Slices are added in slice order; n_ss as in AttnArgs (at most 1).  Event pairs, chunks of 1000 / 512 rows of the 8B
// shape: 10.6 / 6.6 us; a workgroup per row and head, which rotated the queries too, 27.5 / 14.4.
struct AppendArgs {
    const float *qkv;
    int n_partial;
    size_t partial_stride;
    int rows, d_q, G, ctx_pad, d_model, n_ss;
    const int32_t *row_slot, *row_pos;
    const float *cs, *sn, *ss;
    float eps;
    bf16_t *kv_layer;
    size_t slot_stride;
};
__global__ __launch_bounds__(256) void k_kv_append(AppendArgs a) {
    __shared__ float vt[HD][STEP + 1];
    const int g = blockIdx.y, tid = threadIdx.x, r = tid >> 3, c0 = (tid & 7) * 8;   // row of the block; features c0 .. + 7 and c0 + 64 ..
    const int pos0 = a.row_pos[0], slot = a.row_slot[0], pb = pos0 / STEP + blockIdx.x;
    const int m = pb * STEP - pos0 + r, mc = min(max(m, 0), a.rows - 1), pos = pos0 + mc;   // rows outside the chunk re-read one inside
    const bool is_v = blockIdx.z != 0;
    const float *src = a.qkv + (size_t)mc * (a.d_q + 2 * a.G * HD) + a.d_q + (is_v ? a.G * HD : 0) + g * HD + c0;
    floatx4 x[4];   // features c0, c0 + 4, c0 + 64, c0 + 68
#pragma unroll
    for (int i = 0; i < 4; ++i) x[i] = *reinterpret_cast<const floatx4 *>(src + (i >> 1) * 64 + (i & 1) * 4);
    const float ssm = a.ss[mc];
    for (int p = 1; p < a.n_partial; ++p)
#pragma unroll
        for (int i = 0; i < 4; ++i) x[i] += *reinterpret_cast<const floatx4 *>(src + p * a.partial_stride + (i >> 1) * 64 + (i & 1) * 4);
    if (a.n_ss) {
        const float inv = 1.0f / sqrtf(ssm / (float)a.d_model + a.eps);
#pragma unroll
        for (int i = 0; i < 4; ++i) x[i] *= inv;
    }
    const bool live = m >= 0 && m < a.rows;
    bf16_t *kc = a.kv_layer + (size_t)slot * a.slot_stride + (size_t)g * a.ctx_pad * HD;
    if (!is_v) {
        uint32_t lo[4], hi[4];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const floatx4 co = *reinterpret_cast<const floatx4 *>(a.cs + (size_t)pos * 64 + c0 + 4 * i);
            const floatx4 si = *reinterpret_cast<const floatx4 *>(a.sn + (size_t)pos * 64 + c0 + 4 * i);
            float f0[4], f1[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                f0[e] = x[i][e] * co[e] - x[2 + i][e] * si[e];
                f1[e] = x[2 + i][e] * co[e] + x[i][e] * si[e];
            }
            lo[2 * i] = f32x2_to_bf16x2(f0[0], f0[1]); lo[2 * i + 1] = f32x2_to_bf16x2(f0[2], f0[3]);
            hi[2 * i] = f32x2_to_bf16x2(f1[0], f1[1]); hi[2 * i + 1] = f32x2_to_bf16x2(f1[2], f1[3]);
        }
        if (live) {
            *reinterpret_cast<uint4 *>(kc + (size_t)pos * HD + c0) = make_uint4(lo[0], lo[1], lo[2], lo[3]);
            *reinterpret_cast<uint4 *>(kc + (size_t)pos * HD + c0 + 64) = make_uint4(hi[0], hi[1], hi[2], hi[3]);
        }
        return;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) vt[c0 + (i >> 1) * 64 + (i & 1) * 4 + e][r] = x[i][e];
    __syncthreads();
    // thread: sixteen positions of one feature
    const int dim = tid >> 1, p0 = (tid & 1) * 16, m_first = pb * STEP - pos0 + p0;
    bf16_t *vp = kc + (size_t)a.G * a.ctx_pad * HD + ((size_t)pb * HD + dim) * STEP + p0;
    uint32_t w[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) w[i] = f32x2_to_bf16x2(vt[dim][p0 + 2 * i], vt[dim][p0 + 2 * i + 1]);
    if (m_first >= 0 && m_first + 16 <= a.rows) {
        *reinterpret_cast<uint4 *>(vp) = make_uint4(w[0], w[1], w[2], w[3]);
        *reinterpret_cast<uint4 *>(vp + 8) = make_uint4(w[4], w[5], w[6], w[7]);
    } else {   // the chunk begins or ends inside: the other positions keep what they hold
#pragma unroll
        for (int i = 0; i < 16; ++i)
            if (m_first + i >= 0 && m_first + i < a.rows) vp[i] = (bf16_t)(w[i >> 1] >> (16 * (i & 1)));
    }
}
static void launch_kv_append(Ctx *c, const Fwd &f, int layer, int n_partial, int n_ss) {
    const wisv_config &g = c->cfg;
    ProfScope ps(c, KC_ROPE);
    const AppendArgs a{c->qkv, n_partial, (size_t)c->slice_rows * c->d_qkv, f.rows, c->d_q, g.n_kv_heads, c->ctx_pad, g.d_model, n_ss,
                       c->row_slot, c->row_pos, c->rope_cos, c->rope_sin, c->ss, g.rms_eps, (bf16_t *)kv_ptr(c, layer, 0, 0),
                       (size_t)2 * g.n_kv_heads * c->ctx_pad * g.head_dim};
    // the first row may lie anywhere in its block of positions
    hipLaunchKernelGGL(k_kv_append, dim3((f.rows + STEP - 2) / STEP + 1, g.n_kv_heads, 2), dim3(256), 0, c->stream, a);
}

// o[m][h][:] = sum_s 2^(m_s - m*) O_s / sum_s 2^(m_s - m*) l_s (the maxima are kept in units of ln 2), splits in index
// order; one block per (row, head).
// Splits are taken BATCH at a time, all loads of a batch issued before the first is used (slots past the last
// split re-read it and weigh zero), batches chained with the same rescaling rule.
template <int BATCH>
__global__ void k_attn_combine(const float *__restrict__ po, const float *__restrict__ pm, const float *__restrict__ pl,
                               int n_splits, int rows, int H, ActBuf o) {
    const int m = blockIdx.x, h = blockIdx.y, d = threadIdx.x;
    float mx = -INFINITY, num = 0.f, den = 0.f;
    for (int s0 = 0; s0 < n_splits; s0 += BATCH) {
        float ms[BATCH], ls[BATCH], os[BATCH];
#pragma unroll
        for (int i = 0; i < BATCH; ++i) {
            const size_t row = ((size_t)min(s0 + i, n_splits - 1) * rows + m) * H + h;
            ms[i] = pm[row];
            ls[i] = pl[row];
            os[i] = po[row * HD + d];
        }
        float bmx = mx;
#pragma unroll
        for (int i = 0; i < BATCH; ++i) bmx = fmaxf(bmx, s0 + i < n_splits ? ms[i] : -INFINITY);
        if (bmx == -INFINITY) continue;
        const float keep = mx == -INFINITY ? 0.f : exp2f(mx - bmx);
        num *= keep;
        den *= keep;
#pragma unroll
        for (int i = 0; i < BATCH; ++i) {
            const bool on = s0 + i < n_splits && ms[i] != -INFINITY;
            const float w = on ? exp2f(ms[i] - bmx) : 0.f;
            den = fmaf(w, on ? ls[i] : 0.f, den);
            num = fmaf(w, on ? os[i] : 0.f, num);
        }
        mx = bmx;
    }
    act_store(o, ((size_t)m * H + h) * HD + d, num / den);
}

template <int NQ, int NW, bool PROMPT, int NP, int NSS> static bool launch_nq_t(Ctx *c, const AttnArgs &a, dim3 grid) {
    // the merge area at the end of the kernel, which also holds the parked query operands before that
    const size_t lds = std::max((size_t)NW * NQ * (2 * 16 * 4 + 8 / attn_merge_parts(NQ) * 64 * 16), (size_t)NQ * 8 * 1024);
    static bool allowed[MAX_DEVICES];
    if (lds > 64 * 1024 && !allow_big_lds(c, reinterpret_cast<const void *>(&k_attn_mfma<NQ, NW, PROMPT, NP, NSS>), allowed)) return false;
    hipLaunchKernelGGL((k_attn_mfma<NQ, NW, PROMPT, NP, NSS>), grid, dim3(64 * NW), lds, c->stream, a);
    return true;
}
// The prologue requests as many slices as its instantiation holds, 32 bytes of each per item: the smallest one that
// covers the count (rounds of more than 16 rows leave 2 to 10, a prompt's chunk 1 to 4, or more when it is short)
template <int NQ, int NW> static bool launch_nq(Ctx *c, const AttnArgs &a, dim3 grid) {
    if (a.n_ss > 0) return launch_nq_t<NQ, NW, false, MAX_SPLITS, MAX_SPLITS>(c, a, grid);
    if (a.n_partial <= 2) return launch_nq_t<NQ, NW, false, 2, 0>(c, a, grid);
    if (a.n_partial <= 5) return launch_nq_t<NQ, NW, false, 5, 0>(c, a, grid);
    return launch_nq_t<NQ, NW, false, MAX_SPLITS, 0>(c, a, grid);
}
template <int NQ, int NW> static bool launch_prompt_nq(Ctx *c, const AttnArgs &a, dim3 grid) {
    if (a.n_partial <= 2) return a.n_ss ? launch_nq_t<NQ, NW, true, 2, 1>(c, a, grid) : launch_nq_t<NQ, NW, true, 2, 0>(c, a, grid);
    if (a.n_partial <= 4) return a.n_ss ? launch_nq_t<NQ, NW, true, 4, 1>(c, a, grid) : launch_nq_t<NQ, NW, true, 4, 0>(c, a, grid);
    return a.n_ss ? launch_nq_t<NQ, NW, true, MAX_SPLITS, 1>(c, a, grid) : launch_nq_t<NQ, NW, true, MAX_SPLITS, 0>(c, a, grid);
}

// One workgroup per (stream, KV head) when that fills the chip (then the workgroup writes the output itself);
// otherwise k-splits of at least one 32-key step per wave, never more workgroups than CUs (a second round of
// workgroups costs more than the splits gain: 12 streams x 8 KV heads over 2048 cached tokens, 3 splits = 288
// workgroups 44.7 us, 2 splits 29.1 us; 24 streams over 4096: 2 splits 112.8 us, 1 split 98.7 us) and 16 in all
// (one stream over 512: the round takes 3.51 ms with 3 splits and their combine kernel, 3.55 ms with one).
// 0: the shape is not served.
//
// A prompt's chunk has more rows than the 64 query rows one workgroup meets: it is cut into blocks of about 48 query rows,
// each treated as a stream of its own whose cached length is its first row's position (k_kv_append has written the
// whole chunk's k, v rows before, and a block's causal limit is its own last position).  Blocks of 64 / rep tokens take 1.07 to 1.76
// times as long with 4 to 20 query heads per KV head, 1 to 8 KV heads, 128 to 1000 tokens behind nothing or 1000; the same with 128 / 8
// heads over 128 tokens and, being the same two tokens, with 22 to 24 heads per KV head.  With 25 to 32 query heads per KV head
// that is one token, and blocks of two (four query tiles, one workgroup per CU) read the keys half as often: they are taken where
// they fill seven eighths of their last round of 256 workgroups.  us per layer, event pairs, blocks of one / two, tokens behind
// nothing and behind 1000: 1000 tokens, 28 / 1 heads (500 workgroups of two) 61.5 / 53.7 and 103.8 / 99.5, 64 / 2 heads (1000)
// 117.9 / 108.5 and 202 / 195, 112 / 4 heads (2000) 218 / 189 and 387 / 362; 512 tokens, 28 / 1 heads (256) 29.6 / 28.9 and 50.7 /
// 53.0.  Below that line: 256 tokens, 28 / 1 heads (128) 16.2 / 21.5 and 28.5 / 44.8; 640 tokens (320) 41.1 / 37.6 and 71.5 / 83.5.
static int attn_block(const Ctx *c, const Fwd &f) {
    const wisv_config &g = c->cfg;
    const int rep = g.n_heads / g.n_kv_heads;
    if (!c->bf16 || g.head_dim != HD || rep > 64 || f.rows != f.batch * f.k) return 0;
    if (rep * f.k <= 64) return f.k;
    if (!f.prefill) return 0;   // a round's larger block goes to the generic kernel
    const int wgs = (f.rows + 1) / 2 * g.n_kv_heads, rounds = (wgs + 255) / 256;
    if (rep > 24 && rep <= 32 && 8 * wgs >= 7 * 256 * rounds) return 2;
    return std::max(1, 48 / rep);
}
static int attn_splits(const Ctx *c, const Fwd &f) {
    const wisv_config &g = c->cfg;
    const int block = attn_block(c, f);
    if (!block) return 0;
    const int nw = g.n_heads / g.n_kv_heads * block <= 32 ? 8 : 4;
    const int n_steps = (f.max_len_ub + STEP - 1) / STEP, wgs = (f.rows + block - 1) / block * g.n_kv_heads;
    const int want = std::max(1, std::min(256 / wgs, (n_steps + nw - 1) / nw));
    // 16: one batch of the combine kernel; a round smaller than the ctx's largest finds room for more splits than that one
    return std::max(1, std::min(std::min(want, 16), (int)std::min<size_t>(64, c->att_cap / f.rows)));
}

// With several k-splits every split repeats the query part of the prologue (it sums the QKV slices of its queries
// and rotates them; the split that ends the sequence also appends).  That always beat or equalled a kernel of its own
// for RoPE and the append: 8 rows over 4096 cached tokens 4.04 -> 3.92 ms per round; 96 rows, 2 splits 6.34 -> 6.15;
// 72 rows, 3 splits 6.25 -> 6.09; 32 rows over 4096 tokens, 8 splits 4.98 -> 4.86; 24 rows over 8192 tokens, 16
// splits 4.88 -> 4.89.  k_rope_append serves the shapes this kernel does not take.
bool attn_one_block(const Ctx *c, const Fwd &f) { return attn_block(c, f) == f.k; }

// c->o from the k-split partials in c->att_o / att_m / att_l
void launch_attn_combine(Ctx *c, const Fwd &f, int n_splits) {
    const wisv_config &g = c->cfg;
    ProfScope ps(c, KC_ATTN_COMBINE);
    if (n_splits <= 4)
        hipLaunchKernelGGL(k_attn_combine<4>, dim3(f.rows, g.n_heads), dim3(HD), 0, c->stream, c->att_o, c->att_m, c->att_l,
                           n_splits, f.rows, g.n_heads, act_planes(c->o, c->o_planes));
    else
        hipLaunchKernelGGL(k_attn_combine<16>, dim3(f.rows, g.n_heads), dim3(HD), 0, c->stream, c->att_o, c->att_m, c->att_l,
                           n_splits, f.rows, g.n_heads, act_planes(c->o, c->o_planes));
}

// c->qkv holds the n_partial k-split slices of the QKV product
bool launch_attn_mfma(Ctx *c, const Fwd &f, int layer, int n_partial, bool with_combine, int *n_splits, int n_ss) {
    const wisv_config &g = c->cfg;
    const int block = attn_block(c, f), rep = g.n_heads / g.n_kv_heads, R = rep * block;
    const bool prompt = block != f.k;
    AttnArgs a;
    a.n_splits = attn_splits(c, f);
    if (!a.n_splits || (prompt && n_ss > 1)) return false;
    a.kv_layer = (const bf16_t *)kv_ptr(c, layer, 0, 0);
    a.kv_write = (bf16_t *)kv_ptr(c, layer, 0, 0);
    a.slot_stride = (size_t)2 * g.n_kv_heads * c->ctx_pad * g.head_dim;
    a.H = g.n_heads; a.G = g.n_kv_heads; a.rep = rep; a.K = block; a.max_ctx = g.max_ctx; a.ctx_pad = c->ctx_pad; a.rows = f.rows;
    a.row_slot = c->row_slot; a.row_pos = c->row_pos;
    a.po = c->att_o; a.pm = c->att_m; a.pl = c->att_l;
    a.o = act_planes(c->o, c->o_planes);
    a.qkv = c->qkv; a.n_partial = n_partial; a.partial_stride = (size_t)c->slice_rows * c->d_qkv;
    a.cs = c->rope_cos; a.sn = c->rope_sin;
    a.ss = c->ss; a.n_ss = n_ss; a.d_model = g.d_model; a.eps = g.rms_eps;
    if (prompt) launch_kv_append(c, f, layer, n_partial, n_ss);
    dim3 grid(a.n_splits, g.n_kv_heads, (f.rows + block - 1) / block);
    {
        ProfScope ps(c, KC_ATTN);
        bool ok;
        switch ((R + 15) / 16) {
            case 1: ok = launch_nq<1, 8>(c, a, grid); break;   // (a prompt's blocks have at least 25 query rows)
            case 2: ok = prompt ? launch_prompt_nq<2, 8>(c, a, grid) : launch_nq<2, 8>(c, a, grid); break;
            case 3: ok = prompt ? launch_prompt_nq<3, 4>(c, a, grid) : launch_nq<3, 4>(c, a, grid); break;
            default: ok = prompt ? launch_prompt_nq<4, 4>(c, a, grid) : launch_nq<4, 4>(c, a, grid); break;
        }
        if (!ok) return false;
    }
    if (n_splits) *n_splits = a.n_splits;
    if (a.n_splits > 1 && with_combine) launch_attn_combine(c, f, a.n_splits);
    return true;
}

}  // namespace wisv
