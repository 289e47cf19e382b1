// Decision head, mismatch localisation and the first-reject scan (Sec. V-A eqs. feature_concat /
// head_forward / mlp_form; eq. threshold; Alg. 1 last block).
//
//   1. head     one launch for two things that do not need each other: the head's first layer over [h^D ; h^T ; c] for every
//               position with an uploaded h^D row, and the search for every row's greedy token among the LM head's candidates
//   2. decide   per stream: the parts of that search merged, localisation, second layer and accept probabilities of the scored
//               positions (FH: positions with an h^D row; SH: mismatch positions with one), mismatch mask, earliest rejected
//               position, accepted length, correction token, and the commit of the stream state
#include <algorithm>

#include "wisv_internal.h"

namespace wisv {

// dst[r][0..cols_pad) = src[r][0..cols) followed by zeros
template <typename WT>
__global__ void k_pad_cols(const WT *__restrict__ src, WT *__restrict__ dst, int cols, int cols_pad) {
    const int r = blockIdx.x;
    for (int i = threadIdx.x; i < cols_pad; i += blockDim.x)
        dst[(size_t)r * cols_pad + i] = i < cols ? src[(size_t)r * cols + i] : (WT)0;
}

void launch_pad_cols(Ctx *c, const void *src, void *dst, int rows, int cols, int cols_pad) {
    if (c->bf16)
        hipLaunchKernelGGL(k_pad_cols<bf16_t>, dim3(rows), dim3(256), 0, c->stream, (const bf16_t *)src, (bf16_t *)dst, cols, cols_pad);
    else
        hipLaunchKernelGGL(k_pad_cols<float>, dim3(rows), dim3(256), 0, c->stream, (const float *)src, (float *)dst, cols, cols_pad);
}

// ------------------------------------------------------------------------------------------ greedy tokens
// Bound by latency: a round trip of eight loads per thread and the merge.  Candidates lie [slot][row] (see store_tile), so lanes
// run along the rows of a line first and along the slots after that; with a workgroup for each row, which uses 8 bytes of a line,
// and one part the search took, us per launch of its own at 128256 tokens over 4 / 15 / 96 / 143 / 512 rows, 7.5 / 12.5 / 9.4 / 9.3
// / 13.7, now 2.1 / 2.7 / 1.9 / 2.3 / 3.0 (event pairs less the 4.5 of an empty one).
template <int NTH> __device__ __forceinline__ void search_candidates(const Candidates &cd, const GreedyCut &cut, int wg, uint2 *best) {
    __shared__ float bv[NTH / 64][16];
    __shared__ int bi[NTH / 64][16];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, width = 1 << cut.shift, step = NTH >> cut.shift;
    const int part = wg % cut.parts, r = tid & (width - 1), m = (wg / cut.parts << cut.shift) + r, mc = min(m, cd.rows - 1);
    const int end = min(cd.n, (part + 1) * cut.per);
    float v = -INFINITY;
    int idx = 0x7fffffff;
    for (int i0 = part * cut.per + (tid >> cut.shift); i0 < end; i0 += 8 * step) {
        uint2 p[8];   // candidates past the end re-read the last one: same value, same index
        if (cd.pairs) {
#pragma unroll
            for (int u = 0; u < 8; ++u) p[u] = cd.pairs[(size_t)min(i0 + step * u, end - 1) * cd.rows + mc];
        } else {
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int i = min(i0 + step * u, end - 1);
                p[u] = make_uint2(__float_as_uint(cd.logits[(size_t)mc * cd.n + i]), i);
            }
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) keep_better(v, idx, __uint_as_float(p[u].x), (int)p[u].y);
    }
    for (int o = 32; o >= width; o >>= 1) keep_better(v, idx, __shfl_xor(v, o, 64), __shfl_xor(idx, o, 64));
    if (lane < width) { bv[wave][lane] = v; bi[wave][lane] = idx; }
    __syncthreads();
    if (tid >= width || m >= cd.rows) return;
    for (int w = 1; w < NTH / 64; ++w) keep_better(v, idx, bv[w][tid], bi[w][tid]);
    best[(size_t)m * GREEDY_PARTS + part] = make_uint2(__float_as_uint(v), (uint32_t)idx);
}

__global__ __launch_bounds__(512) void k_argmax(Candidates cd, GreedyCut cut, uint2 *best) { search_candidates<512>(cd, cut, blockIdx.x, best); }

void launch_argmax(Ctx *c) {
    ProfScope ps(c, KC_ARGMAX);
    const GreedyCut cut = greedy_cut(c->cand);
    hipLaunchKernelGGL(k_argmax, dim3(cut.wgs), dim3(512), 0, c->stream, c->cand, cut, c->best);
}

// ------------------------------------------------------------------------------------------ the head's first layer
// u = W1 [h^D ; h^T ; c] for every position with an uploaded row, without ever writing the concatenated vector: the three
// column slices of W1 meet h^D (read through hd_row from what the device uploaded), h^T (the target's final hidden state)
// and c (the stream's CSI vector) where they lie.  Which of these positions count is localisation's business and is left
// to k_decide, so that nothing here waits for the greedy tokens.
//
// bf16 weights: W1 is held re-tiled for the 16x16x32 MFMA (kernels_gemm.hip).  One workgroup = RB row-blocks of 16 hidden
// units x NT tiles of 16 positions x one split of the columns; its WK waves split those columns again and each wave builds
// its own B operands (16 positions x 32 columns, two bf16 terms) straight from global memory - no two waves of a workgroup
// need the same columns, so nothing is staged in LDS.  The waves' accumulators are added through LDS in wave order into
// one partial sum per (split, position, hidden unit), which k_decide adds up in split order.  Positions without an
// uploaded row are never loaded; a tile without one exits.
//
// Bound by what a workgroup reads, at some 50 GB/s per CU, behind two dependent loads (row map, operands): a row-block of W1
// is 200 KB at the 8B shape, h^D and h^T of a tile 330 KB.
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

struct HeadArgs {
    const u32x4 *w1t;          // re-tiled W1 [nrb][nkt][64] (bf16 path)
    const void *w1;            // W1 [dJ][din] row-major (generic path)
    int nkt, nrb, dJ, dD, dT, dC, din;
    const void *hd;            // uploaded drafter hidden states [n_hd][dD], weight dtype
    const int32_t *hd_row;     // [rows] or null (identity)
    int n_hd;
    const float *h_t, *csi;    // [rows][dT], [batch][dC]
    int k, rows, act;
    const void *b1, *w2;
    float *u;                  // bf16 path: first-layer partial sums [split][rows][16 nrb]; generic: second-layer sums [rows]
    int gx, tiles, kt_per_split;   // bf16 path: workgroups along the hidden units and the positions; columns of a split
    // workgroups from search0 on look for greedy tokens instead
    Candidates cand;
    GreedyCut cut;
    int search0;
    uint2 *best;
};

// the uploaded row of position m, or -1
__device__ __forceinline__ int head_row(const int32_t *hd_row, int n_hd, int m) {
    const int hr = hd_row ? hd_row[m] : m;
    return hr >= 0 && hr < n_hd ? hr : -1;
}

// element c < din of z = [h^D ; h^T ; c] of position m
template <typename WT> __device__ __forceinline__ float head_z(const HeadArgs &a, int m, int hr, int c) {
    // all three sources at clamped places (no load behind a branch), the right one selected
    const float d = Elem<WT>::load((const WT *)a.hd + (size_t)hr * a.dD + min(c, a.dD - 1));
    const float t = a.h_t[(size_t)m * a.dT + min(max(c - a.dD, 0), a.dT - 1)];
    const float v = a.csi[(size_t)(m / a.k) * a.dC + min(max(c - a.dD - a.dT, 0), a.dC - 1)];
    return c < a.dD ? d : c < a.dD + a.dT ? t : v;
}

__device__ __forceinline__ float head_act(int act, float v) { return act == WISV_ACT_RELU ? fmaxf(v, 0.f) : v / (1.0f + expf(-v)); }

// WK waves split the columns of the split; a wave multiplies RB row-blocks of hidden units with NT tiles of 16 positions (every
// A operand meets NT B operands and every B operand RB A operands) and requests TB k-tiles at a time
template <int WK, int RB, int NT, int TB>
__global__ __launch_bounds__(64 * WK) void k_head_fused(HeadArgs a) {
    if ((int)blockIdx.x >= a.search0) {
        search_candidates<64 * WK>(a.cand, a.cut, blockIdx.x - a.search0, a.best);
        return;
    }
    const int wg = blockIdx.x, rb0 = wg % a.gx * RB, tile0 = wg / a.gx % a.tiles * NT, split = wg / (a.gx * a.tiles);
    const int tid = threadIdx.x, lane = tid & 63, wk = tid >> 6, bj = lane & 15, bg = lane >> 4;
    int m[NT], hr[NT];
    bool sc[NT], any = false;
    const bf16_t *hd_row[NT];
    const float *ht_row[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        m[t] = (tile0 + t) * 16 + bj;
        hr[t] = head_row(a.hd_row, a.n_hd, min(m[t], a.rows - 1));
        sc[t] = m[t] < a.rows && hr[t] >= 0;
        any = any || sc[t];
        hd_row[t] = (const bf16_t *)a.hd + (size_t)max(hr[t], 0) * a.dD;
        ht_row[t] = a.h_t + (size_t)min(m[t], a.rows - 1) * a.dT;
    }
    if (!__any(any)) return;         // every wave sees the same positions: the whole workgroup leaves together

    const int kt0 = split * a.kt_per_split, kt1 = min(a.nkt, kt0 + a.kt_per_split), sub = (kt1 - kt0 + WK - 1) / WK;
    const int k_begin = min(kt1, kt0 + wk * sub), k_end = min(kt1, k_begin + sub);
    floatx4 acc[RB][NT];
#pragma unroll
    for (int r = 0; r < RB; ++r)
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[r][t] = floatx4{0.f, 0.f, 0.f, 0.f};
    // one B operand (two bf16 terms) of position tile t against the RB A operands
    auto mma = [&](const u32x4 (&av)[RB], int t, u32x4 bh, u32x4 bl, bool two) {
        if (!sc[t]) { bh = u32x4{0u, 0u, 0u, 0u}; bl = bh; }
#pragma unroll
        for (int r = 0; r < RB; ++r) {
            u32x4 a_ = av[r];
            acc[r][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*reinterpret_cast<bf16x8 *>(&a_), *reinterpret_cast<bf16x8 *>(&bh), acc[r][t], 0, 0, 0);
            if (two) acc[r][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*reinterpret_cast<bf16x8 *>(&a_), *reinterpret_cast<bf16x8 *>(&bl), acc[r][t], 0, 0, 0);
        }
    };
    auto split8 = [&](const float (&z)[8], u32x4 &bh, u32x4 &bl) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            bf16_t h0, l0, h1, l1;
            split2(z[2 * e], h0, l0);
            split2(z[2 * e + 1], h1, l1);
            bh[e] = h0 | ((uint32_t)h1 << 16);
            bl[e] = l0 | ((uint32_t)l1 << 16);
        }
    };
    // A wave's k-tiles fall into three runs (uniform per wave): tiles inside h^D, tiles inside h^T, and the rest (a tile
    // that straddles two sources, the CSI features, the padding).  Each run is a loop without branches around its
    // loads: TB tiles are requested at once (tiles past the run re-read its last one and are not used).  The launcher
    // sends only widths that are multiples of 8 here, so a lane's eight columns never straddle two sources inside a run.
    const int d_end = a.dD / 32, t_begin = (a.dD + 31) / 32, t_end = (a.dD + a.dT) / 32;   // [0, d_end) in h^D; [t_begin, t_end) in h^T
    const u32x4 *wt[RB];   // row-blocks past the last re-read it; their results are not written
#pragma unroll
    for (int r = 0; r < RB; ++r) wt[r] = a.w1t + (size_t)min(rb0 + r, a.nrb - 1) * a.nkt * 64 + lane;
    {   // ---- h^D: bf16 values are their own high term, there is no low term
        const int r0 = k_begin, r1 = min(k_end, d_end);
        for (int k0 = r0; k0 < r1; k0 += TB) {
            u32x4 av[TB][RB], hv[TB][NT];
#pragma unroll
            for (int u = 0; u < TB; ++u) {
                const int kt = min(k0 + u, r1 - 1);
#pragma unroll
                for (int r = 0; r < RB; ++r) av[u][r] = wt[r][(size_t)kt * 64];
#pragma unroll
                for (int t = 0; t < NT; ++t) hv[u][t] = *reinterpret_cast<const u32x4 *>(hd_row[t] + kt * 32 + bg * 8);
            }
#pragma unroll
            for (int u = 0; u < TB; ++u)
                if (k0 + u < r1) {
#pragma unroll
                    for (int t = 0; t < NT; ++t) mma(av[u], t, hv[u][t], u32x4{0u, 0u, 0u, 0u}, false);
                }
        }
    }
    {   // ---- h^T: float, split into two bf16 terms
        const int r0 = max(k_begin, t_begin), r1 = min(k_end, t_end);
        for (int k0 = r0; k0 < r1; k0 += TB) {
            u32x4 av[TB][RB];
            floatx4 f0[TB][NT], f1[TB][NT];
#pragma unroll
            for (int u = 0; u < TB; ++u) {
                const int kt = min(k0 + u, r1 - 1);
#pragma unroll
                for (int r = 0; r < RB; ++r) av[u][r] = wt[r][(size_t)kt * 64];
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                    f0[u][t] = *reinterpret_cast<const floatx4 *>(ht_row[t] + kt * 32 + bg * 8 - a.dD);
                    f1[u][t] = *reinterpret_cast<const floatx4 *>(ht_row[t] + kt * 32 + bg * 8 - a.dD + 4);
                }
            }
#pragma unroll
            for (int u = 0; u < TB; ++u)
                if (k0 + u < r1) {
#pragma unroll
                    for (int t = 0; t < NT; ++t) {
                        const float z[8] = {f0[u][t][0], f0[u][t][1], f0[u][t][2], f0[u][t][3], f1[u][t][0], f1[u][t][1], f1[u][t][2], f1[u][t][3]};
                        u32x4 bh, bl;
                        split8(z, bh, bl);
                        mma(av[u], t, bh, bl, true);
                    }
                }
        }
    }
    for (int kt = k_begin; kt < k_end; ++kt) {   // ---- the rest, element by element (a handful of tiles)
        if (kt < d_end || (kt >= t_begin && kt < t_end)) continue;
        u32x4 av[RB];
#pragma unroll
        for (int r = 0; r < RB; ++r) av[r] = wt[r][(size_t)kt * 64];
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            // the three sources are read at clamped places and the right one is selected: one latency for the tile instead
            // of one per element (positions that are not scored are zeroed by mma)
            float z[8], zd[8], zt[8], zc[8];
            const float *csi = a.csi + (size_t)(min(m[t], a.rows - 1) / a.k) * a.dC;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int col = kt * 32 + bg * 8 + e;
                zd[e] = bf16_to_f32(hd_row[t][min(col, a.dD - 1)]);
                zt[e] = ht_row[t][min(max(col - a.dD, 0), a.dT - 1)];
                zc[e] = csi[min(max(col - a.dD - a.dT, 0), a.dC - 1)];
            }
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int col = kt * 32 + bg * 8 + e;
                z[e] = col < a.dD ? zd[e] : col < a.dD + a.dT ? zt[e] : col < a.din ? zc[e] : 0.f;
            }
            u32x4 bh, bl;
            split8(z, bh, bl);
            mma(av, t, bh, bl, true);
        }
    }
    // ---- the waves' column slices, added in wave order, an operand tile by one wave
    constexpr int OPS = RB * NT, PART = OPS < 4 ? OPS : 4;   // operand tiles added at a time
    static_assert(OPS % PART == 0, "");
    __shared__ floatx4 red[WK][PART][64];
    const int dJp = 16 * a.nrb;
#pragma unroll
    for (int i0 = 0; i0 < OPS; i0 += PART) {
        if (i0) __syncthreads();
#pragma unroll
        for (int i = 0; i < PART; ++i) red[wk][i][lane] = acc[(i0 + i) / NT][(i0 + i) % NT];
        __syncthreads();
        if (wk >= PART) continue;
        const int r = (i0 + wk) / NT, t = (i0 + wk) % NT;
        floatx4 u = red[0][wk][lane];
        for (int w = 1; w < WK; ++w) u += red[w][wk][lane];
        bool on = false;
#pragma unroll
        for (int q = 0; q < NT; ++q) on = q == t ? sc[q] : on;
        // lane (bj, bg) holds u[hidden 16 (rb0 + r) + 4 bg + e][position bj of tile t]
        if (on && rb0 + r < a.nrb)
            *reinterpret_cast<floatx4 *>(a.u + ((size_t)split * a.rows + (tile0 + t) * 16 + bj) * dJp + (rb0 + r) * 16 + bg * 4) = u;
    }
}

// Generic form (float weights, or shapes the re-tiled form does not serve): one workgroup of 16 waves per position, both
// layers at once.  Bound by latency (4 rows of the tiny fp32 target: 18 us when four waves took one hidden unit
// after the other, 5 us now): a wave works on UJ hidden units at once, all loads of a step of columns before the first use.  The
// units' products are then added by four threads, unit j by thread j % 4 in rising order, and the four sums in pairs.
template <typename WT>
__global__ __launch_bounds__(1024) void k_head_ref(HeadArgs a) {
    constexpr int UJ = 4, GROUP = 16 * UJ * 4;            // hidden units per wave at once; per pass over val
    __shared__ float val[GROUP], red[4];
    if ((int)blockIdx.x >= a.search0) {
        search_candidates<1024>(a.cand, a.cut, blockIdx.x - a.search0, a.best);
        return;
    }
    const int m = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int hr = head_row(a.hd_row, a.n_hd, m);
    if (hr < 0) return;
    float t = 0.f;
    for (int g0 = 0; g0 < a.dJ; g0 += GROUP) {
        for (int j0 = g0 + wave * UJ; j0 < min(g0 + GROUP, a.dJ); j0 += 16 * UJ) {
            float dot[UJ], bias[UJ];
            const WT *wr[UJ];
#pragma unroll
            for (int i = 0; i < UJ; ++i) {                // units past the last re-read it
                dot[i] = 0.f;
                wr[i] = (const WT *)a.w1 + (size_t)min(j0 + i, a.dJ - 1) * a.din;
                bias[i] = Elem<WT>::load((const WT *)a.b1 + min(j0 + i, a.dJ - 1));
            }
            for (int c = lane; c < a.din; c += 64) {
                const float z = head_z<WT>(a, m, hr, c);
#pragma unroll
                for (int i = 0; i < UJ; ++i) dot[i] = fmaf(Elem<WT>::load(wr[i] + c), z, dot[i]);
            }
#pragma unroll
            for (int i = 0; i < UJ; ++i) {
                dot[i] = wave_sum(dot[i]);
                if (lane == 0 && j0 + i < a.dJ) val[j0 + i - g0] = head_act(a.act, dot[i] + bias[i]);
            }
        }
        __syncthreads();
        if (tid < 4)
            for (int j = g0 + tid; j < min(g0 + GROUP, a.dJ); j += 4) t = fmaf(Elem<WT>::load((const WT *)a.w2 + j), val[j - g0], t);
        __syncthreads();
    }
    if (tid < 4) red[tid] = t;
    __syncthreads();
    if (tid == 0) a.u[m] = (red[0] + red[1]) + (red[2] + red[3]);
}

// One workgroup per stream, one wave per position: is it a mismatch (Alg. 1's localisation against the target's greedy token)
// and does the upload protocol have it scored (Sec. III-B: full-hidden streams everywhere, selective-hidden ones at
// mismatches); the second layer from the first layer's partial sums (lanes take four hidden units at a time, then a fixed
// shuffle tree); threshold.  Then the first wave finds the earliest rejected position, and the commit.
struct DecideArgs {
    int batch, k, rows, max_batch, gate_all, commit, act;
    const int32_t *stream_ids, *tokens, *proto, *hd_row;
    const uint2 *best;         // the rows' greedy tokens, in parts
    int parts, n_hd;
    const float *tau;
    const float *u;            // first-layer partial sums [splits][rows][16 nrb], or (splits == 0) second-layer sums [rows]
    int splits, dJ, nrb;
    const void *b1, *w2, *b2;
    int bf16;
    int32_t *kv_len, *pred_next;
    float *p_acc;
    int32_t *alen, *ytok, *targ;
    uint32_t *mask_out, *status_out;
};
constexpr int HEAD_MAX_SPLITS = 8;
__global__ __launch_bounds__(64 * WISV_MAX_K) void k_decide(DecideArgs a) {
    __shared__ int flags[WISV_MAX_K];   // 1: mismatch, 2: rejected, 4: wanted for the decision but not uploaded
    __shared__ int greedy[WISV_MAX_K];
    const int b = blockIdx.x, lane = threadIdx.x & 63, j = threadIdx.x >> 6, m = b * a.k + j;
    const int slot = min(max(a.stream_ids[b], 0), a.max_batch - 1);
    const int token = a.tokens[m], proto = a.proto[b];
    const int hr = head_row(a.hd_row, a.n_hd, m);
    const float tau = a.tau[b];
    const int pn = a.pred_next[slot];
    const uint2 part = greedy_part(a.best, a.parts, lane & 16 ? max(m - 1, 0) : m, lane);
    // second layer; a position that is not scored reads sums that nobody wrote (inside the buffer) and drops the result
    float s2 = 0.f;
    if (a.splits) {
        const int dJp = 16 * a.nrb;
        for (int j0 = lane * 4; j0 < dJp; j0 += 256) {
            float4 part[HEAD_MAX_SPLITS];
#pragma unroll
            for (int p = 0; p < HEAD_MAX_SPLITS; ++p)   // splits past the last re-read it and are not added
                part[p] = *reinterpret_cast<const float4 *>(a.u + ((size_t)min(p, a.splits - 1) * a.rows + m) * dJp + j0);
            float b1[4], w2[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                b1[e] = bf16_to_f32(((const bf16_t *)a.b1)[min(j0 + e, a.dJ - 1)]);
                w2[e] = bf16_to_f32(((const bf16_t *)a.w2)[min(j0 + e, a.dJ - 1)]);
            }
            float u[4] = {part[0].x, part[0].y, part[0].z, part[0].w};
#pragma unroll
            for (int p = 1; p < HEAD_MAX_SPLITS; ++p) {
                const bool on = p < a.splits;
                u[0] += on ? part[p].x : 0.f; u[1] += on ? part[p].y : 0.f; u[2] += on ? part[p].z : 0.f; u[3] += on ? part[p].w : 0.f;
            }
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (j0 + e < a.dJ) s2 = fmaf(w2[e], head_act(a.act, u[e] + b1[e]), s2);
        }
        s2 = wave_sum(s2);
    } else {
        s2 = a.u[m];
    }
    const int merged = greedy_token(part), own = __builtin_amdgcn_readlane(merged, 0), before = __builtin_amdgcn_readlane(merged, 16);
    const bool mismatch = token != (j == 0 ? pn : before);
    const bool sc = (a.gate_all || proto == WISV_PROTO_FH || mismatch) && hr >= 0;
    const float bias = a.bf16 ? bf16_to_f32(*(const bf16_t *)a.b2) : *(const float *)a.b2;
    if (lane == 0) {
        greedy[j] = own;
        const float p = sc ? 1.0f / (1.0f + expf(s2 + bias)) : 1.0f;   // p_accept = 1 - sigmoid(s); 1 where not evaluated
        a.p_acc[m] = p;
        const bool decides = a.gate_all || mismatch, missing = decides && !sc;
        flags[j] = (mismatch ? 1 : 0) | (missing || (decides && !(p >= tau)) ? 2 : 0) | (missing ? 4 : 0);
        if (a.targ) {
            a.targ[b * (a.k + 1) + j + 1] = own;
            if (j == 0) a.targ[b * (a.k + 1)] = pn;
        }
    }
    __syncthreads();
    if (j != 0) return;
    const int fl = flags[min(lane, a.k - 1)];
    const bool live = lane < a.k;
    const uint64_t mask = __ballot(live && (fl & 1)), rejected = __ballot(live && (fl & 2)), missing = __ballot(live && (fl & 4));
    if (lane != 0) return;
    const int first = rejected ? __ffsll((unsigned long long)rejected) - 1 : a.k;
    const int y = first == 0 ? pn : greedy[first - 1];
    a.alen[b] = first;
    a.ytok[b] = y;
    if (a.mask_out) a.mask_out[b] = (uint32_t)mask;
    if (a.status_out) a.status_out[b] = missing ? WISV_STATUS_MISSING_HIDDEN : 0;
    if (a.commit) {
        a.kv_len[slot] += first;
        a.pred_next[slot] = y;
    }
}

// How the first layer is cut: two or four row-blocks x one or two tiles of 16 positions, and as many splits of the columns (of at
// least eight k-tiles) as make one round of 256 workgroups; of the two the one whose workgroups read less (a row-block of W1
// costs a KiB per k-tile, 16 positions two KiB).  The search's workgroups (4 to 256 of them) come last in the grid and share CUs
// with these: first in it 96 rows take 14.6 us instead of 12.2; counted as part of the round 143 rows 24.2 instead of 16.2
// and 256 rows 26.3 instead of 20.6, 512 rows the same (128256 tokens, event pairs).
struct HeadCut { int rb, nt, gx, tiles, splits, kt_per_split; };
static HeadCut head_cut(int rows, int nrb, int nkt) {
    const int pos = (rows + 15) / 16;
    HeadCut best{};
    double least = 0;
    for (int rb : {2, 4}) {
        HeadCut h;
        h.rb = rb;
        h.nt = pos == 1 ? 1 : 2;
        if (h.nt == 1 && rb == 4) break;
        h.gx = (nrb + h.rb - 1) / h.rb;
        h.tiles = (pos + h.nt - 1) / h.nt;
        const int s = std::max(1, std::min(std::min(HEAD_MAX_SPLITS, 256 / (h.gx * h.tiles)), nkt / 8));
        h.kt_per_split = (nkt + s - 1) / s;
        h.splits = (nkt + h.kt_per_split - 1) / h.kt_per_split;
        const double reads = (double)(h.rb + 2 * h.nt) * h.kt_per_split * ((h.gx * h.tiles * h.splits + 255) / 256);
        if (!best.rb || reads < least) best = h, least = reads;
    }
    return best;
}
static bool head_tiled(const Ctx *c) { return c->head_w1_t && c->cfg.d_draft % 8 == 0; }
size_t head_scratch_floats(const Ctx *c, int rows) {
    const int nrb = (c->cfg.d_head_hidden + 15) / 16;
    size_t most = rows;
    for (int r = 16;; r += 16) {      // the cut depends on the number of tiles of 16 positions
        const int n = std::min(r, rows);
        most = std::max(most, (size_t)head_cut(n, nrb, c->din_pad / 32).splits * n * 16 * nrb);
        if (n == rows) return most;
    }
}

void launch_head_decide(Ctx *c, const Fwd &f, const wisv_round_in &in, const wisv_round_out &out, bool find_tokens) {
    const wisv_config &g = c->cfg;
    HeadArgs a{};
    a.w1t = (const u32x4 *)c->head_w1_t; a.w1 = c->head_w1;
    a.dJ = g.d_head_hidden; a.dD = g.d_draft; a.dT = g.d_model; a.dC = g.d_csi; a.din = g.d_draft + g.d_model + g.d_csi;
    a.nkt = c->din_pad / 32; a.nrb = (g.d_head_hidden + 15) / 16;
    a.hd = in.hd; a.hd_row = in.hd_row; a.n_hd = in.n_hd;
    a.h_t = c->h_t; a.csi = in.csi;
    a.k = f.k; a.rows = f.rows; a.act = g.head_act;
    a.b1 = c->head_b1; a.w2 = c->head_w2;
    a.u = c->hu;
    a.cand = c->cand; a.best = c->best;
    a.cut = greedy_cut(c->cand);
    const int search = find_tokens ? a.cut.wgs : 0;
    int splits = 0;
    if (in.n_hd == 0) {          // nothing was uploaded: localisation only
        if (find_tokens) launch_argmax(c);
    } else {
        ProfScope ps(c, KC_HEAD);
        if (head_tiled(c)) {
            const HeadCut h = head_cut(f.rows, a.nrb, a.nkt);
            a.gx = h.gx; a.tiles = h.tiles; a.kt_per_split = h.kt_per_split;
            splits = h.splits;
            a.search0 = h.gx * h.tiles * h.splits;
            const dim3 grid(a.search0 + search);
            if (h.nt == 1) hipLaunchKernelGGL((k_head_fused<8, 2, 1, 6>), grid, dim3(512), 0, c->stream, a);
            else if (h.rb == 2) hipLaunchKernelGGL((k_head_fused<8, 2, 2, 4>), grid, dim3(512), 0, c->stream, a);
            else hipLaunchKernelGGL((k_head_fused<8, 4, 2, 3>), grid, dim3(512), 0, c->stream, a);
        } else {
            a.search0 = f.rows;
            const dim3 grid(a.search0 + search);
            if (c->bf16) hipLaunchKernelGGL(k_head_ref<bf16_t>, grid, dim3(1024), 0, c->stream, a);
            else hipLaunchKernelGGL(k_head_ref<float>, grid, dim3(1024), 0, c->stream, a);
        }
    }
    DecideArgs d{};
    d.batch = f.batch; d.k = f.k; d.rows = f.rows; d.max_batch = g.max_batch; d.act = g.head_act;
    d.gate_all = (in.flags & WISV_FLAG_GATE_ALL) ? 1 : 0; d.commit = (in.flags & WISV_FLAG_NO_COMMIT) ? 0 : 1;
    d.stream_ids = in.stream_ids; d.tokens = in.draft_tokens; d.proto = in.proto; d.best = c->best; d.parts = a.cut.parts;
    d.hd_row = in.hd_row; d.n_hd = in.n_hd; d.tau = in.tau;
    d.u = c->hu; d.splits = splits; d.dJ = g.d_head_hidden; d.nrb = a.nrb;
    d.b1 = c->head_b1; d.w2 = c->head_w2; d.b2 = c->head_b2; d.bf16 = c->bf16 ? 1 : 0;
    d.kv_len = c->d_kv_len; d.pred_next = c->d_pred_next;
    d.p_acc = out.p_accept; d.alen = out.accepted_len; d.ytok = out.correction_token; d.targ = out.target_argmax;
    d.mask_out = out.mismatch_mask; d.status_out = out.status;
    ProfScope ps(c, KC_DECIDE);
    hipLaunchKernelGGL(k_decide, dim3(f.batch), dim3(64 * f.k), 0, c->stream, d);
}

}  // namespace wisv
