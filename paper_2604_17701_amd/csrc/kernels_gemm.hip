// Weight-streaming bf16 GEMM for a small number of activation rows (the memory-bound regime of the
// verify round: every weight byte is read once per round and meets at most a few hundred rows).
//
// Y[m, n] = sum_k X[m, k] W[n, k] is computed "swapped": the 16x16x32 MFMA takes a 16-row block of W as
// its A operand and 16 activation rows as its B operand, so the output-feature dimension fills the
// matrix core however few rows there are.  W is stored re-tiled: tile (rb, kt) holds W[16rb..+16][32kt..+32]
// as 64 lanes x 8 bf16 in exactly the order the MFMA wants, so that one wave-wide 16-byte load fetches a
// contiguous KiB and a wave walking along k reads one contiguous stream.  Activations arrive as two bf16
// planes (x = hi + lo, written by whichever kernel produced them), one MFMA each: the products are then
// exact to about 2^-17 while the weights stay bf16; the second MFMA costs issue slots this memory-bound
// kernel has to spare.
//
// A workgroup is WR x WK waves: WR groups of RB row-blocks share the activation chunk in LDS, and WK slices
// of the workgroup's k-range whose accumulators are added through LDS in slice order.  The grid's y
// dimension splits k into partial outputs, its z dimension walks tiles of 16 NT rows.
// The weight stream is software-pipelined through a ring of U register slots: the steady-state loop has no
// branches, and every slot is refilled right after the MFMAs that read it (scheduling barriers keep that
// order), so that the compiler's wait counts let U loads stay in flight.
#include <algorithm>

#include "wisv_internal.h"

namespace wisv {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// ------------------------------------------------------------------------------------------ re-tiling
// out[((rb * nkt + kt) * 64 + lane) * 8 + e] = W[row(rb, lane % 16)][32 kt + 8 (lane / 16) + e]
// pair_rows > 0: W stacks two matrices of pair_rows rows each (gate over up); row-block rb then holds
// gate rows 8rb..8rb+7 in its rows 0..7 and up rows 8rb..8rb+7 in its rows 8..15, so that one MFMA tile
// carries both halves of SwiGLU for 8 features.
// overflow != null: every element is converted to an IEEE half (nearest-even; magnitudes below 2^-14 keep what a
// subnormal half holds, an absolute error of at most 2^-25); *overflow is set when one does not fit the half range
__global__ void k_retile(const bf16_t *__restrict__ W, int n_rows, int kd, int nrb, int nkt, int pair_rows,
                         uint4 *__restrict__ out, int32_t *overflow) {
    const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (size_t)nrb * nkt * 64) return;
    const int lane = idx & 63;
    const size_t tile = idx >> 6;
    const int kt = tile % nkt, rb = tile / nkt, i = lane & 15;
    int row;
    bool valid;
    if (pair_rows > 0) {
        const int f = rb * 8 + (i & 7);
        row = (i >> 3) * pair_rows + f;
        valid = f < pair_rows;
    } else {
        row = rb * 16 + i;
        valid = row < n_rows;
    }
    uint4 v = make_uint4(0, 0, 0, 0);
    if (valid) v = *reinterpret_cast<const uint4 *>(W + (size_t)row * kd + 32 * kt + 8 * (lane >> 4));
    if (overflow) {
        uint32_t w[4] = {v.x, v.y, v.z, v.w};
        bool bad = false;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float a = __uint_as_float(w[e] << 16), b = __uint_as_float(w[e] & 0xffff0000u);
            bad = bad || !(fabsf(a) <= 65504.0f) || !(fabsf(b) <= 65504.0f);
            w[e] = (uint32_t)__builtin_bit_cast(uint16_t, (_Float16)a) | ((uint32_t)__builtin_bit_cast(uint16_t, (_Float16)b) << 16);
        }
        if (bad) atomicOr(overflow, 1);
        v = make_uint4(w[0], w[1], w[2], w[3]);
    }
    out[idx] = v;
}

void launch_retile(Ctx *c, const void *W, int n_rows, int kd, int pair_rows, void *out, int nrb, int32_t *overflow) {
    const int nkt = kd / 32;
    const size_t total = (size_t)nrb * nkt * 64;
    hipLaunchKernelGGL(k_retile, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, c->stream, (const bf16_t *)W,
                       n_rows, kd, nrb, nkt, pair_rows, (uint4 *)out, overflow);
}

// row-blocks are padded to a multiple of 16 so that a workgroup may own up to 16 of them
int ws_padded_row_blocks(int n_rows) { return ((n_rows + 15) / 16 + 15) / 16 * 16; }
// gate/up pairs: 8 features per row-block
int ws_padded_pair_blocks(int features) { return ((features + 7) / 8 + 15) / 16 * 16; }

// ------------------------------------------------------------------------------------------ the GEMM
enum { EPI_PARTIAL = 0, EPI_SWIGLU = 1, EPI_ARGMAX = 2, EPI_RESID = 3 };

struct GemmArgs {
    const u32x4 *Wt;           // re-tiled weights [nrb][nkt][64]
    const bf16_t *Xhi, *Xlo;   // activation planes [M][kd]
    const uint16_t *X16;       // the activations as one half each (k_gemm_mm with ONE term; Wt then holds halves too)
    int M, N, kd, nrb, nkt, kt_per_split;
    int kcw;                   // k-tiles per wave staged in LDS at a time (a multiple of the prefetch depth)
    float *Yp;                 // EPI_PARTIAL: [S][split_stride];  EPI_ARGMAX with logits != null: [M][N]
    size_t split_stride;
    ActBuf H;                  // EPI_SWIGLU: [M][N] float + planes (N = features)
    uint2 *cand;               // EPI_ARGMAX: (value, index) [slot][M]
    int gx, gz, gs;            // k_gemm_mm, k_gemm_pipe: row-block groups, row tiles and k-splits the 1-D grid decodes into
    int per;                   // k_gemm_pipe: consecutive k-splits a workgroup takes one after the other
    // PRO: the activations are the attention output, still in k-split partials (up to WS_PRO_SPLITS of them):
    // o [split][rows][heads][128], running maximum m (in units of ln 2) and sum l [split][rows][heads]
    const float *att_o, *att_m, *att_l;
    int att_splits, att_rows, att_H;
    // PRO_NORM: the activations are the residual stream, still to be updated: v = xin + the n_partial slices of the
    // previous product (ys), a = v * gain (the RMSNorm gain; its 1 / rms factor is applied by whoever sums this
    // product's slices).  Workgroups with blockIdx.x == 0 also write v to xout and the sum of v^2 over their k-range
    // to ss_out[split][row].
    const float *xin, *ys;
    float *xout, *ss_out;
    const bf16_t *gain;
    int n_partial;
    size_t ys_stride;
    // EPI_RESID (a product whose k-split stays inside the workgroup: complete sums): v = xin + Y is written to xout,
    // v * gain to H (float and two-term planes: the next block's RMSNorm without its 1 / rms), and the sum of v^2 over
    // the workgroup's 16 RB features of every row to ss_out[row-block group][row]; xin may be xout.
    // EPI_SWIGLU with ss_in: the activations came that way; both halves are scaled by
    // 1 / sqrt(sum of the n_ss_in partial sums of the row / kd + rms_eps) before the SiLU.
    const float *ss_in;
    int n_ss_in;
    float rms_eps;
};
enum { PRO_NONE = 0, PRO_ATTN = 1, PRO_NORM = 2 };

// ------------------------------------------------------------------------------------------ epilogues
// acc[r][t][e] = Y[m = m_base + 16 t + lane % 16][row 4 (lane / 16) + e of row-block rb0 + r]; `split` is the
// partial-output slice, `slot` the wave's candidate slot (one per group of RB row-blocks)
template <int NT, int RB, int EPI>
__device__ __forceinline__ void ws_epilogue(const GemmArgs &g, floatx4 (&acc)[RB][NT], int m_base, int rb0, int split,
                                            int slot, int lane, const float *s_inv, const floatx4 (&res_x)[RB][NT],
                                            const uint2 (&res_g)[RB]) {
    const int bj = lane & 15, bg = lane >> 4;
    if (EPI == EPI_PARTIAL) {
        float *out = g.Yp + (size_t)split * g.split_stride;
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const int m = m_base + t * 16 + bj;
            if (m >= g.M) continue;
#pragma unroll
            for (int r = 0; r < RB; ++r) {
                const int n = (rb0 + r) * 16 + bg * 4;
                if (n + 3 < g.N && (g.N & 3) == 0) *reinterpret_cast<floatx4 *>(out + (size_t)m * g.N + n) = acc[r][t];
                else
                    for (int e = 0; e < 4; ++e)
                        if (n + e < g.N) out[(size_t)m * g.N + n + e] = acc[r][t][e];
            }
        }
    } else if (EPI == EPI_SWIGLU) {
        // rows 0..7 of a block are gate, rows 8..15 up, of features 8 (rb0 + r) ..: lanes 32..63 hold the up
        // values that lanes 0..31 need
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const int m = m_base + t * 16 + bj;
            if (g.ss_in) {   // the deferred 1 / rms of a folded RMSNorm, computed by the kernel's prologue
                const float inv = s_inv[min(t * 16 + bj, 16 * NT - 1)];
#pragma unroll
                for (int r = 0; r < RB; ++r)
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[r][t][e] *= inv;
            }
#pragma unroll
            for (int r = 0; r < RB; ++r) {
                floatx4 up;
#pragma unroll
                for (int e = 0; e < 4; ++e) up[e] = __shfl_xor(acc[r][t][e], 32, 64);
                if (bg < 2 && m < g.M) {
                    const int f = (rb0 + r) * 8 + bg * 4;
                    float hv[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float gt = acc[r][t][e];
                        hv[e] = gt / (1.0f + expf(-gt)) * up[e];
                    }
                    if (f + 3 < g.N && (g.N & 3) == 0) act_store4(g.H, (size_t)m * g.N + f, hv[0], hv[1], hv[2], hv[3]);
                    else
                        for (int e = 0; e < 4; ++e)
                            if (f + e < g.N) act_store(g.H, (size_t)m * g.N + f + e, hv[e]);
                }
            }
        }
    } else if (EPI == EPI_RESID) {
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const int m = m_base + t * 16 + bj;
            float q2 = 0.f;
#pragma unroll
            for (int r = 0; r < RB; ++r) {
                const int n = (rb0 + r) * 16 + bg * 4;     // N is a multiple of 16 here (checked by the launcher)
                if ((rb0 + r) * 16 >= g.N) continue;       // a padding row-block (uniform over the wave)
                const floatx4 xv = res_x[r][t];            // requested when the kernel started
                const uint2 gw = res_g[r];
                const floatx4 v = {xv[0] + acc[r][t][0], xv[1] + acc[r][t][1], xv[2] + acc[r][t][2], xv[3] + acc[r][t][3]};
                if (m < g.M) {
                    *reinterpret_cast<floatx4 *>(g.xout + (size_t)m * g.N + n) = v;
                    act_store4(g.H, (size_t)m * g.N + n, v[0] * __uint_as_float(gw.x << 16), v[1] * __uint_as_float(gw.x & 0xffff0000u),
                               v[2] * __uint_as_float(gw.y << 16), v[3] * __uint_as_float(gw.y & 0xffff0000u));
                }
                q2 += (v[0] * v[0] + v[1] * v[1]) + (v[2] * v[2] + v[3] * v[3]);
            }
            q2 += __shfl_xor(q2, 16, 64);
            q2 += __shfl_xor(q2, 32, 64);
            if (bg == 0 && m < g.M && rb0 * 16 < g.N) g.ss_out[(size_t)slot * g.M + m] = q2;
        }
    } else {   // EPI_ARGMAX: best (value, lowest index) of this wave's 16*RB features for every row
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const int m = m_base + t * 16 + bj;
            float best = -INFINITY;
            int idx = 0x7fffffff;
#pragma unroll
            for (int r = 0; r < RB; ++r)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int n = (rb0 + r) * 16 + bg * 4 + e;
                    const float v = acc[r][t][e];
                    if (n < g.N) {
                        if (g.Yp && m < g.M) g.Yp[(size_t)m * g.N + n] = v;
                        if (v > best || (v == best && n < idx)) { best = v; idx = n; }
                    }
                }
#pragma unroll
            for (int o = 16; o < 64; o <<= 1) {
                const float ov = __shfl_xor(best, o, 64);
                const int oi = __shfl_xor(idx, o, 64);
                if (ov > best || (ov == best && oi < idx)) { best = ov; idx = oi; }
            }
            if (bg == 0 && m < g.M) g.cand[(size_t)slot * g.M + m] = make_uint2(__float_as_uint(best), (uint32_t)idx);
        }
    }
}

// NT: 16-row activation tiles per wave; RB: row-blocks per wave; WR x WK waves per workgroup; U: prefetch depth;
// PRO_ATTN: the activations are combined from the attention kernel's k-split partials while they are staged (the rule
// of k_attn_combine: weights e^(m_s - max m), splits in index order), so that no kernel of its own has to do it.
// PRO_NORM: the activations are the residual stream plus the previous product's slices, times the norm gain (see
// GemmArgs); WK == 1 and a single activation chunk
// WHOLE: every wave has a whole number of ring turns (the launcher checks), so no load and no product is guarded: the guarded
// last turn waits for each of its loads in turn.  us per launch over 4 / 15 rows: gate/up 38.6 / 41.9 -> 37.9 / 40.5, down
// 18.8 / 19.9 -> 18.1 / 19.1, O with the residual inside (eight k-tiles per wave, all requested at once) 12.1 -> 11.7.
template <int NT, int RB, int WR, int WK, int U, int PRO, int EPI, bool WHOLE>
__global__ __launch_bounds__(64 * WR * WK, PRO == PRO_NORM ? 6 : 1) void k_gemm_ws(GemmArgs g) {
    extern __shared__ __align__(16) unsigned char lds[];
    constexpr int NTH = 64 * WR * WK;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, wr = wave / WK, wk = wave % WK;
    const int kt0 = blockIdx.y * g.kt_per_split;
    const int ntile = min(g.kt_per_split, g.nkt - kt0);
    const int sub = (ntile + WK - 1) / WK;                         // k-tiles per wave
    const int my0 = wk * sub, myn = max(0, min(sub, ntile - my0));
    const int rb0 = (blockIdx.x * WR + wr) * RB;
    const bool active = rb0 < g.nrb;                               // RB * WR divides nrb (padded)
    const int m_base = blockIdx.z * (16 * NT), Mt = min(16 * NT, g.M - m_base);   // this workgroup's rows

    // ---- start the weight stream before anything else: it does not depend on the activations
    const u32x4 *wp[RB];
    u32x4 abuf[U][RB];
#pragma unroll
    for (int r = 0; r < RB; ++r) wp[r] = g.Wt + ((size_t)(active ? rb0 + r : 0) * g.nkt + kt0 + my0) * 64 + lane;
    if (active) {
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int r = 0; r < RB; ++r)
                if (WHOLE || u < myn) abuf[u][r] = __builtin_nontemporal_load(wp[r] + (size_t)u * 64);
    }

    floatx4 acc[RB][NT];
#pragma unroll
    for (int r = 0; r < RB; ++r)
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[r][t] = floatx4{0.f, 0.f, 0.f, 0.f};

    // EPI_RESID: the residual stream and the gain of this wave's outputs are requested now, by the waves that will
    // run the epilogue (lane (bj, bg): row m_base + 16 t + bj, features 16 (rb0 + r) + 4 bg ..)
    floatx4 res_x[RB][NT];
    uint2 res_g[RB];
    if (EPI == EPI_RESID && wk == 0) {
#pragma unroll
        for (int r = 0; r < RB; ++r) {
            const int n = min((rb0 + r) * 16, g.N - 16) + (lane >> 4) * 4;
            res_g[r] = *reinterpret_cast<const uint2 *>(g.gain + n);
#pragma unroll
            for (int t = 0; t < NT; ++t)
                res_x[r][t] = *reinterpret_cast<const floatx4 *>(g.xin + (size_t)min(m_base + t * 16 + (lane & 15), g.M - 1) * g.N + n);
        }
    }

    // ---- activations: chunk ch holds, for every k-slice w, its tiles [ch kcw, (ch+1) kcw) as
    //      lds[ch & 1][plane][w][m][kcw * 64 + 16 bytes]; the 16 spreads rows over the banks
    const int kcw = g.kcw, pitch = kcw * 64 + 16, wk_bytes = Mt * pitch, plane_bytes = WK * wk_bytes,
              buf_bytes = 2 * plane_bytes;
    const int nchunk = (sub + kcw - 1) / kcw;
    auto stage = [&](int ch) {
        unsigned char *dst = lds + (size_t)(ch & 1) * buf_bytes;
        const int vec_per_row = kcw * 4, per_wk = Mt * vec_per_row;
        if (PRO == PRO_NORM) {
            // An item is four consecutive features of one row; the four lane groups of a wave share 16 items and take
            // four slices each (every load is unconditional: slices past the last re-read it and count as zero), then
            // add their sums in a fixed order: ((x + s0..s3) + (s4..s7)) + ((s8..s11) + (s12..s15)).
            float *ssq = reinterpret_cast<float *>(lds + 2 * buf_bytes);   // per item: sum of v^2
            const int grp = lane >> 4, np = max(g.n_partial, 1);
            const int item_per_row = kcw * 8, n_item = Mt * item_per_row;
            for (int base = wave * 16; base < n_item; base += (NTH / 64) * 16) {
                const int raw = base + (lane & 15), it = min(raw, n_item - 1);
                const int m = it / item_per_row, v = it - m * item_per_row, lt = v >> 3;
                const bool live = raw < n_item && lt < sub && lt < ntile;
                const int col = (kt0 + min(lt, ntile - 1)) * 32 + (v & 7) * 4;
                const size_t off = (size_t)(m_base + m) * g.kd + col;
                const floatx4 xa = *reinterpret_cast<const floatx4 *>(g.xin + off);
                floatx4 sa[4];
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    sa[q] = *reinterpret_cast<const floatx4 *>(g.ys + (size_t)min(grp * 4 + q, np - 1) * g.ys_stride + off);
                const uint2 gw = *reinterpret_cast<const uint2 *>(g.gain + col);
                floatx4 t = grp == 0 ? xa : floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const bool on = grp * 4 + q < g.n_partial;   // a select: the unused re-read may hold anything
#pragma unroll
                    for (int e = 0; e < 4; ++e) t[e] += on ? sa[q][e] : 0.f;
                }
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    t[e] += __shfl_xor(t[e], 16, 64);
                    t[e] += __shfl_xor(t[e], 32, 64);
                }
                bf16_t h[4], l[4];
                split2(t[0] * __uint_as_float(gw.x << 16), h[0], l[0]);
                split2(t[1] * __uint_as_float(gw.x & 0xffff0000u), h[1], l[1]);
                split2(t[2] * __uint_as_float(gw.y << 16), h[2], l[2]);
                split2(t[3] * __uint_as_float(gw.y & 0xffff0000u), h[3], l[3]);
                if (live) {
                    unsigned char *d = dst + (size_t)m * pitch + v * 8;
                    if (grp == 0) *reinterpret_cast<uint2 *>(d) = make_uint2(h[0] | ((uint32_t)h[1] << 16), h[2] | ((uint32_t)h[3] << 16));
                    if (grp == 1) *reinterpret_cast<uint2 *>(d + plane_bytes) = make_uint2(l[0] | ((uint32_t)l[1] << 16), l[2] | ((uint32_t)l[3] << 16));
                    if (grp == 2 && blockIdx.x == 0) *reinterpret_cast<floatx4 *>(g.xout + off) = t;
                }
                if (grp == 3 && raw < n_item) ssq[raw] = live ? (t[0] * t[0] + t[1] * t[1]) + (t[2] * t[2] + t[3] * t[3]) : 0.f;
            }
            return;
        }
        for (int i = tid; i < WK * per_wk; i += NTH) {
            const int w = i / per_wk, rem = i - w * per_wk, m = rem / vec_per_row, v = rem - m * vec_per_row;
            const int lt = ch * kcw + (v >> 2), kt = w * sub + lt;          // tile within the slice / the workgroup range
            if (lt < sub && kt < ntile) {
                unsigned char *d = dst + (size_t)w * wk_bytes + (size_t)m * pitch + v * 16;
                if (PRO == PRO_ATTN) {
                    // eight consecutive features of one head (head_dim 128) of row m_base + m
                    const int col = (kt0 + kt) * 32 + (v & 3) * 8, head = col >> 7, dd = col & 127;
                    float ms[WS_PRO_SPLITS], ls[WS_PRO_SPLITS];
                    floatx4 oa[WS_PRO_SPLITS], ob[WS_PRO_SPLITS];
#pragma unroll
                    for (int sp = 0; sp < WS_PRO_SPLITS; ++sp) {   // splits past the last re-read it and weigh zero
                        const size_t row = ((size_t)min(sp, g.att_splits - 1) * g.att_rows + m_base + m) * g.att_H + head;
                        ms[sp] = g.att_m[row];
                        ls[sp] = g.att_l[row];
                        oa[sp] = *reinterpret_cast<const floatx4 *>(g.att_o + row * 128 + dd);
                        ob[sp] = *reinterpret_cast<const floatx4 *>(g.att_o + row * 128 + dd + 4);
                    }
                    float mx = -INFINITY;
#pragma unroll
                    for (int sp = 0; sp < WS_PRO_SPLITS; ++sp) mx = fmaxf(mx, sp < g.att_splits ? ms[sp] : -INFINITY);
                    float den = 0.f, num[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int sp = 0; sp < WS_PRO_SPLITS; ++sp) {
                        const bool on = sp < g.att_splits && ms[sp] != -INFINITY;
                        const float wgt = on ? exp2f(ms[sp] - mx) : 0.f;   // the maxima are in units of ln 2
                        den = fmaf(wgt, on ? ls[sp] : 0.f, den);
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            num[e] = fmaf(wgt, on ? oa[sp][e] : 0.f, num[e]);
                            num[4 + e] = fmaf(wgt, on ? ob[sp][e] : 0.f, num[4 + e]);
                        }
                    }
                    uint32_t hw[4], lw[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        bf16_t h0, l0, h1, l1;
                        split2(num[2 * e] / den, h0, l0);
                        split2(num[2 * e + 1] / den, h1, l1);
                        hw[e] = h0 | ((uint32_t)h1 << 16);
                        lw[e] = l0 | ((uint32_t)l1 << 16);
                    }
                    *reinterpret_cast<uint4 *>(d) = make_uint4(hw[0], hw[1], hw[2], hw[3]);
                    *reinterpret_cast<uint4 *>(d + plane_bytes) = make_uint4(lw[0], lw[1], lw[2], lw[3]);
                } else {
                    const size_t off = (size_t)(m_base + m) * g.kd + (size_t)(kt0 + kt) * 32 + (v & 3) * 8;
                    *reinterpret_cast<uint4 *>(d) = *reinterpret_cast<const uint4 *>(g.Xhi + off);
                    *reinterpret_cast<uint4 *>(d + plane_bytes) = *reinterpret_cast<const uint4 *>(g.Xlo + off);
                }
            }
        }
    };
    const int bj = lane & 15, bg = lane >> 4;
    // B operands of one k-tile: lanes whose row does not exist read row Mt - 1 and are zeroed (no branch)
    auto mfma_tile = [&](const unsigned char *buf, int lt, const u32x4 *a) {
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const int m = t * 16 + bj;
            const unsigned char *p = buf + (size_t)min(m, Mt - 1) * pitch + (lt * 32 + bg * 8) * 2;
            uint4 bh = *reinterpret_cast<const uint4 *>(p);
            uint4 bl = *reinterpret_cast<const uint4 *>(p + plane_bytes);
            if (m >= Mt) { bh = make_uint4(0, 0, 0, 0); bl = bh; }
#pragma unroll
            for (int r = 0; r < RB; ++r) {
                u32x4 av = a[r];
                acc[r][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*reinterpret_cast<bf16x8 *>(&av),
                                                                   *reinterpret_cast<bf16x8 *>(&bh), acc[r][t], 0, 0, 0);
                acc[r][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*reinterpret_cast<bf16x8 *>(&av),
                                                                   *reinterpret_cast<bf16x8 *>(&bl), acc[r][t], 0, 0, 0);
            }
        }
    };
    // EPI_SWIGLU after a folded RMSNorm: 1 / rms of every row from the partial sums of squares the producer left.
    // Wave w takes rows w, w + waves, ..; its loads go out before the staging loads and are reduced after them
    // (lane-strided sums in index order, then a fixed shuffle tree).
    __shared__ float s_inv[16 * NT];
    float ssv[4] = {0.f, 0.f, 0.f, 0.f};
    const bool scale_rows = EPI == EPI_SWIGLU && g.ss_in != nullptr;
    if (scale_rows && wave < Mt) {
#pragma unroll
        for (int q = 0; q < 4; ++q) ssv[q] = g.ss_in[(size_t)min(lane + 64 * q, g.n_ss_in - 1) * g.M + m_base + wave];
    }
    stage(0);
    if (scale_rows) {
        for (int r = wave; r < Mt; r += NTH / 64) {
            float v = 0.f;
            if (r == wave) {   // the first row's partial sums are already here
#pragma unroll
                for (int q = 0; q < 4; ++q) v += lane + 64 * q < g.n_ss_in ? ssv[q] : 0.f;
                for (int p = lane + 256; p < g.n_ss_in; p += 64) v += g.ss_in[(size_t)p * g.M + m_base + r];
            } else {
                for (int p = lane; p < g.n_ss_in; p += 64) v += g.ss_in[(size_t)p * g.M + m_base + r];
            }
            v = wave_sum(v);
            if (lane == 0) s_inv[r] = 1.0f / sqrtf(v / (float)g.kd + g.rms_eps);
        }
    }
    for (int ch = 0; ch < nchunk; ++ch) {
        __syncthreads();   // chunk ch is staged; everyone is done with the buffer chunk ch + 1 goes to
        if (PRO == PRO_NORM && blockIdx.x == 0 && wave == 0) {
            // sum of v^2 of every row over this k-range: the items of a row in index order, lanes then a fixed tree
            const float *ssq = reinterpret_cast<const float *>(lds + 2 * buf_bytes);
            const int item_per_row = kcw * 8;
            for (int m = 0; m < Mt; ++m) {
                float q2 = 0.f;
                for (int i = lane; i < item_per_row; i += 64) q2 += ssq[m * item_per_row + i];
                q2 = wave_sum(q2);
                if (lane == 0) g.ss_out[(size_t)blockIdx.y * g.M + m_base + m] = q2;
            }
        }
        if (ch + 1 < nchunk) stage(ch + 1);
        if (!active) continue;
        const unsigned char *buf = lds + (size_t)(ch & 1) * buf_bytes + (size_t)wk * wk_bytes;
        const int kend = min(myn, (ch + 1) * kcw);
        int kt = ch * kcw;
        // steady state: U tiles consumed and U refills issued per pass, no conditionals in between
        for (; kt + U <= kend && kt + 2 * U <= myn; kt += U) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                mfma_tile(buf, kt + u - ch * kcw, abuf[u]);
                // the slot is free once its MFMAs have issued: refill it, and keep this order
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int r = 0; r < RB; ++r) abuf[u][r] = __builtin_nontemporal_load(wp[r] + (size_t)(kt + u + U) * 64);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if (WHOLE) {   // the last turn
            if (kt < kend)
#pragma unroll
                for (int u = 0; u < U; ++u) mfma_tile(buf, kt + u - ch * kcw, abuf[u]);
            continue;
        }
        // the last tiles of the slice (and slices shorter than 2 U): guarded
        for (; kt < kend; kt += U) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (kt + u < kend) {
                    u32x4 a[RB];
#pragma unroll
                    for (int r = 0; r < RB; ++r) {
                        a[r] = abuf[u][r];
                        if (kt + u + U < myn) abuf[u][r] = __builtin_nontemporal_load(wp[r] + (size_t)(kt + u + U) * 64);
                    }
                    mfma_tile(buf, kt + u - ch * kcw, a);
                }
            }
        }
    }

    // ---- add the WK k-slices of each row-block group through LDS, in slice order
    if (WK > 1) {
        __syncthreads();
        floatx4 *red = reinterpret_cast<floatx4 *>(lds);
        if (wk > 0 && active) {
#pragma unroll
            for (int r = 0; r < RB; ++r)
#pragma unroll
                for (int t = 0; t < NT; ++t)
                    red[(((size_t)(wr * (WK - 1) + wk - 1) * RB + r) * NT + t) * 64 + lane] = acc[r][t];
        }
        __syncthreads();
        if (wk > 0 || !active) return;
        for (int s = 1; s < WK; ++s)
#pragma unroll
            for (int r = 0; r < RB; ++r)
#pragma unroll
                for (int t = 0; t < NT; ++t) acc[r][t] += red[(((size_t)(wr * (WK - 1) + s - 1) * RB + r) * NT + t) * 64 + lane];
    } else if (!active) {
        return;
    }

    ws_epilogue<NT, RB, EPI>(g, acc, m_base, rb0, blockIdx.y, blockIdx.x * WR + wr, lane, s_inv, res_x, res_g);
}

// ------------------------------------------------------------------------------------------ many rows
// The compute-bound regime (hundreds of rows) uses the 32x32x16 MFMA, which sustains about 1.5 times
// the rate of the 16x16x32 one and needs half the B-operand bytes per flop.  Its A operand wants lane l to
// hold row l % 32 and the 8 k-values of slot l / 32.  Two vertically adjacent re-tiled row-blocks (lane l:
// row l % 16, k-group l / 16 of a 32-wide k-tile) hold two such operands - 32 weight rows with k-groups (0, 2)
// and (1, 3) - each lane of which is a 16-byte piece of one of the two tiles, so they are loaded directly in
// that order.  The activations are staged in LDS already split the same way: operand `op` of k-tile kt and
// 32-row tile t holds, at lane l, X[32 t + l % 32][32 kt + 8 op + 16 (l / 32) ..+8] - a wave stores and later
// reads a contiguous KiB.
//
// More than 160 rows.  Eight waves, two per SIMD (a lone wave issues in order and leaves the matrix pipe idle while it
// issues anything else): WN x WM of them, a wave owns RP pairs of row-blocks of W, streamed straight into a ring of U
// register slots as above, and meets 32 NT rows of the workgroup's row tile.  Staging is double-buffered in chunks of KC k-tiles: the loads of chunk ch + 1 are
// issued before the MFMAs of chunk ch and written to LDS after them.  The 1-D grid is decoded so that the row
// tiles sharing a slice of W run on the same XCD at the same time (workgroup ids are dealt round-robin to the
// 8 XCDs): W then comes from HBM once and from that L2 afterwards.
typedef float floatx16 __attribute__((ext_vector_type(16)));
// Plain results: a lane's four consecutive floats stored as they stand would put 16 bytes into each of 32 rows twice per store,
// and the four stores of a tile a quarter each into the same lines.  So a tile is turned over in 4 KiB of LDS that belong to
// the wave (the 16-byte pieces of a row permuted, so that neither side meets a bank twice) and leaves as 128-byte runs of eight
// rows per store.  us per launch, before and after: down over 512 rows 66.1 -> 62.0, over 143 rows 34.5 -> 33.4; QKV over 1000
// rows 108.5 -> 104.5; O over 143 rows 16.7 -> 16.0; 32 and 96 rows the same.  What an epilogue still costs is its bytes: 143 rows
// leave 18 MB of QKV slices, 4 us.  SwiGLU's 2-byte results gain nothing this way (512 rows 115.2 -> 116, 1000 rows 225 -> 228).
// Candidates for the greedy token lie [slot][row]: a wave's 32 rows fill whole lines, where [row][slot] put 4 bytes of every
// XCD into each (LM head of 32000 tokens over 143 rows 60.8 -> 57.8 us, of 128256 tokens over 96 rows 213 -> 190, over 143 rows
// 245 -> 222; the search that reads them is search_candidates, 7.0 us over either before and 6.4 and 6.8 now).
// one 32 x 32 tile of plain results to rows m0 .., columns n0 ..
__device__ __forceinline__ void store_tile(const GemmArgs &g, float *out, floatx4 *turn, const floatx16 &a, int m0, int n0, int lane) {
    const int mj = lane & 31, h = lane >> 5;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // the wave's LDS accesses stay in this order
#pragma unroll
    for (int v = 0; v < 4; ++v) turn[mj * 8 + ((2 * v + h) ^ ((mj >> 1) & 7))] = floatx4{a[4 * v], a[4 * v + 1], a[4 * v + 2], a[4 * v + 3]};
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    floatx4 o[4];   // row 8 i + lane / 8, columns 4 (lane % 8) .. + 3
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int r = 8 * i + (lane >> 3);
        o[i] = turn[r * 8 + ((lane & 7) ^ ((r >> 1) & 7))];
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int m = m0 + 8 * i + (lane >> 3), n = n0 + 4 * (lane & 7);
        if (m >= g.M) continue;
        if (n + 3 < g.N && (g.N & 3) == 0) *reinterpret_cast<floatx4 *>(out + (size_t)m * g.N + n) = o[i];
        else
            for (int e = 0; e < 4; ++e)
                if (n + e < g.N) out[(size_t)m * g.N + n + e] = o[i][e];
    }
}
// acc[p][t][e] = Y[m = m_base + 32 t + lane % 32][row 8 (e / 4) + 4 (lane / 32) + e % 4 of the 32 rows that
// row-blocks rb0 + 2 p and rb0 + 2 p + 1 make]
// rb_end: row-blocks from here on belong to another workgroup (SwiGLU only)
// turn: 4 KiB of the wave's own
template <int NT, int RP, int EPI>
__device__ __forceinline__ void mm_epilogue(const GemmArgs &g, floatx16 (&acc)[RP][NT], int m_base, int rb0, int split,
                                            int slot, int lane, floatx4 *turn, int rb_end = 0x7fffffff) {
    const int mj = lane & 31, h = lane >> 5;
    if (EPI == EPI_PARTIAL) {
        float *out = g.Yp + (size_t)split * g.split_stride;
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int p = 0; p < RP; ++p) store_tile(g, out, turn, acc[p][t], m_base + 32 * t, (rb0 + 2 * p) * 16, lane);
    } else if (EPI == EPI_SWIGLU) {
        // a row-block holds 8 gate rows over 8 up rows of the same features: this lane's registers 8 b + c and
        // 8 b + 4 + c are gate and up of feature 8 (rb0 + 2 p + b) + 4 h + c
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const int m = m_base + 32 * t + mj;
            if (m >= g.M) continue;
#pragma unroll
            for (int p = 0; p < RP; ++p)
#pragma unroll
                for (int b = 0; b < 2; ++b) {
                    if (rb0 + 2 * p + b >= rb_end) continue;
                    const int f = (rb0 + 2 * p + b) * 8 + 4 * h;
                    float hv[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float gt = acc[p][t][8 * b + e], up = acc[p][t][8 * b + 4 + e];
                        hv[e] = gt / (1.0f + expf(-gt)) * up;
                    }
                    if (f + 3 < g.N && (g.N & 3) == 0) act_store4(g.H, (size_t)m * g.N + f, hv[0], hv[1], hv[2], hv[3]);
                    else
                        for (int e = 0; e < 4; ++e)
                            if (f + e < g.N) act_store(g.H, (size_t)m * g.N + f + e, hv[e]);
                }
        }
    } else {   // EPI_ARGMAX: best (value, lowest index) of this wave's 32 RP features for every row
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const int m = m_base + 32 * t + mj;
            float best = -INFINITY;
            int idx = 0x7fffffff;
#pragma unroll
            for (int p = 0; p < RP; ++p) {
                if (g.Yp) store_tile(g, g.Yp, turn, acc[p][t], m_base + 32 * t, (rb0 + 2 * p) * 16, lane);
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const int n = (rb0 + 2 * p) * 16 + 8 * (e / 4) + 4 * h + (e % 4);
                    const float v = acc[p][t][e];
                    if (n < g.N && (v > best || (v == best && n < idx))) { best = v; idx = n; }
                }
            }
            const float ov = __shfl_xor(best, 32, 64);
            const int oi = __shfl_xor(idx, 32, 64);
            if (ov > best || (ov == best && oi < idx)) { best = ov; idx = oi; }
            if (h == 0 && m < g.M) g.cand[(size_t)slot * g.M + m] = make_uint2(__float_as_uint(best), (uint32_t)idx);
        }
    }
}

// NT: 32-row tiles per wave; NW waves: WM along the rows, NW / WM along the row-blocks; RP: pairs of row-blocks per
// wave; KC: k-tiles per LDS chunk; U: register slots of a wave's weight stream
// NPL: 2 = activations as two bf16 terms (planes hi and lo, two MFMAs per operand pair); 1 = one half-precision term
// (plane X16 against half-precision weight tiles, one MFMA per pair: half the matrix-core work and half the staging)
// SHORT: an accumulator holds one chunk's products only (2 KC NPL of them); finished chunks are added up in a second set of
// registers.  Every addition to a float sum rounds at the size of the whole sum, so one chain over k rounds 2 NPL times per
// k-tile at full size, short chains mostly at a fraction of it.  Prompts take this form for their two-term products over k:
// a bf16 key that lands on the wrong side of a rounding boundary moves every later score of its stream (512 tokens, first
// layer of the 8B shape: 1 of 2600 cached entries with one chain, 1 of 6200 so, 1 of 6000 and 1 of 5400 with chains of 2 and 4
// chunks; passes of four rows, whose k is split into 16 slices, 1 of 5500).  The additions hide behind the matrix
// instructions of the other wave (512 rows: QKV 66.6 -> 69.4 us, down 120.7 -> 123.9).  gate/up keeps one chain: the cache's
// error does not see it (5.63e-4 either way), and 512 rows would take 253 us in this shape against 197 in the wide one.
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
template <int NPL> __device__ __forceinline__ floatx16 mm_mfma(const u32x4 &a, const u32x4 &b, const floatx16 &c) {
    if (NPL == 2) return __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<const bf16x8 *>(&a), *reinterpret_cast<const bf16x8 *>(&b), c, 0, 0, 0);
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(*reinterpret_cast<const f16x8 *>(&a), *reinterpret_cast<const f16x8 *>(&b), c, 0, 0, 0);
}
template <int NT, int WM, int NW, int RP, int KC, int U, int EPI, int NPL, bool DEEP = false, bool WEAVE = false, bool SHORT = false>
__global__ __launch_bounds__(64 * NW) void k_gemm_mm(GemmArgs g) {
    extern __shared__ __align__(16) unsigned char lds[];
    static_assert(U % KC == 0, "a turn of the ring is a whole number of chunks");
    constexpr int WN = NW / WM, RB = 2 * RP;
    constexpr int NTW = NT * WM;                          // 32-row tiles of the workgroup
    constexpr int OPS = KC * NTW * 2;                     // B operands of one plane in a chunk
    constexpr int PER_WAVE = (NPL * OPS + NW - 1) / NW;   // operand loads a wave issues per chunk (all planes)
    constexpr int BUF = NPL * OPS * 1024;                 // bytes of one chunk buffer
    constexpr int G = 2 * NPL;                            // operand groups (op, plane) of a k-tile
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, wn = wave / WM, wm = wave % WM;
    // ---- which (row-block group bx, k-split by, row tile z)
    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
    const int z = slot % g.gz, q = (slot / g.gz) * 8 + xcd;
    if (q >= g.gx * g.gs) return;                         // the whole workgroup leaves: no barrier is reached
    const int bx = q % g.gx, by = q / g.gx;
    const int kt0 = by * g.kt_per_split;
    const int ntile = min(g.kt_per_split, g.nkt - kt0);
    const int rb0 = (bx * WN + wn) * RB;
    const bool active = rb0 < g.nrb;                      // RB divides the padded number of row-blocks
    const int m_base = z * (32 * NTW);

    // A operands straight from the re-tiled W: lane l of operand `op` of pair p wants row l % 32 of the pair and
    // k-group 2 (l / 32) + op, which row-block rb0 + 2 p + (l % 32) / 16 keeps at lane 16 (2 (l / 32) + op) + l % 16.
    // A wave-wide load then reads four contiguous 256-byte runs, and the two operands of a pair together read
    // both of its tiles exactly once.  Waves that differ only in wm stream the same row-blocks: the second one
    // finds them in the vector L1.
    const u32x4 *wp = g.Wt + ((size_t)((active ? rb0 : 0) + ((lane & 31) >> 4)) * g.nkt + kt0) * 64 + 32 * (lane >> 5) + (lane & 15);
    const size_t wstep = (size_t)2 * g.nkt * 64;          // from one pair of row-blocks to the next
    u32x4 abuf[U][RP][2];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
        for (int p = 0; p < RP; ++p)
#pragma unroll
            for (int op = 0; op < 2; ++op)   // a slot past the last k-tile re-reads that tile and is never used
                abuf[u][p][op] = wp[p * wstep + (size_t)min(u, ntile - 1) * 64 + 16 * op];

    floatx16 acc[RP][NT];
#pragma unroll
    for (int p = 0; p < RP; ++p)
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[p][t][e] = 0.f;
    floatx16 sum[SHORT ? RP : 1][SHORT ? NT : 1];         // SHORT: the finished chains
    const floatx16 zero = {};
    if (SHORT) {
#pragma unroll
        for (int p = 0; p < RP; ++p)
#pragma unroll
            for (int t = 0; t < NT; ++t) sum[p][t] = zero;
    }

    // ---- staging: operand id i in [0, 2 OPS): plane i / OPS, then (k-tile, row tile, op) = ((i % OPS) / (2 NTW),
    //      ((i % OPS) / 2) % NTW, i % 2); wave w takes ids w, w + NW, ...  No load is conditional (a branch would
    //      make the compiler wait for each one at once): rows past M re-read row M - 1, k-tiles past the end
    //      re-read the last one; neither is ever used.
    static_assert((NPL * OPS) % NW == 0, "every wave stages the same number of operands");
    const int srow = m_base + (lane & 31);
    const int scol = (lane >> 5) * 16;
    constexpr int TURN = U / KC;   // chunks per turn of the ring
    constexpr int SD = DEEP ? TURN : 1;   // chunks of activations in flight
    u32x4 sreg[SD][PER_WAVE];
#define WISV_MM_STAGE_LOAD(ch, S)                                                                                   \
    _Pragma("unroll") for (int j = 0; j < PER_WAVE; ++j) {                                                         \
        const int i = wave + NW * j, pl = i / OPS, rem = i % OPS, lt = rem / (2 * NTW), t = (rem / 2) % NTW, op = rem & 1; \
        const int kt = min((ch) * KC + lt, ntile - 1);                                                             \
        const int row = min(srow + 32 * t, g.M - 1);                                                               \
        sreg[S][j] = *reinterpret_cast<const u32x4 *>((NPL == 1 ? g.X16 : pl ? g.Xlo : g.Xhi) + (size_t)row * g.kd +  \
                                                   (size_t)(kt0 + kt) * 32 + 8 * op + scol);                       \
    }
#define WISV_MM_STAGE_STORE(ch, S)                                                                                  \
    _Pragma("unroll") for (int j = 0; j < PER_WAVE; ++j)                                                           \
        *reinterpret_cast<u32x4 *>(lds + (size_t)((ch) & 1) * BUF + (size_t)(wave + NW * j) * 1024 + lane * 16) = sreg[S][j];
    // A k-tile is G groups (op, plane) of NT B operands, each feeding NT RP independent MFMAs.  The B
    // operands of group gi + 1 are read from LDS before the MFMAs of group gi issue (scheduling barriers keep
    // that order): the LDS latency hides behind matrix work, the other wave of the SIMD fills what is left.
    // WEAVE asks the scheduler to place those reads between the MFMAs instead (one read after every RP of them),
    // and reads the first group of the chunk's next k-tile the same way: the matrix pipe does not drain while
    // eight reads issue.  Measured gain only for the widest products without k-splits (512 rows: gate/up
    // 142 -> 135 us; the down projection loses 3 %).
    // group og of k-tile lt: plane og % NPL, operand og / NPL
#define WISV_MM_READ_B(lt, og, DST)                                                                                \
    _Pragma("unroll") for (int t = 0; t < NT; ++t)                                                                 \
        DST[t] = *reinterpret_cast<const u32x4 *>(buf + ((((og) % NPL) * OPS) + (((lt) * NTW + t) * 2 + (og) / NPL)) * 1024);
// (SHORT: the first group of a chunk starts new chains and adds up the old ones, finished a barrier ago)
#define WISV_MM_GROUP(lt, og, A, SRC)                                                                              \
    _Pragma("unroll") for (int t = 0; t < NT; ++t) _Pragma("unroll") for (int p = 0; p < RP; ++p) {                \
        if (SHORT && (lt) == 0 && (og) == 0) {                                                                     \
            sum[p][t] += acc[p][t];                                                                                \
            acc[p][t] = mm_mfma<NPL>(A[p][0], SRC[t], zero);                                                       \
        } else acc[p][t] = mm_mfma<NPL>(A[p][(og) / NPL], SRC[t], acc[p][t]);                                      \
    }
    u32x4 bv[2][NT];

    // One chunk: CC (a compile-time number) places it in a turn of the weight ring, which spans U / KC chunks.
    // The next chunk's activations are requested before this chunk's MFMAs and written to LDS after them; the
    // write must wait for exactly these loads while the weight refills issued after them stay in flight, and
    // the compiler can count those only if every path through the chunk issues the same number of loads.
    // Loads complete in order, so that wait also ends every weight refill issued before them, which caps the ring
    // at about one chunk whatever U is.  DEEP keeps as many chunks of activations in flight as the ring has
    // (requested right after the previous occupant of their registers went to LDS, a whole turn before they are
    // written): the wait then ends only refills that are due in the same chunk anyway.
#define WISV_MM_CHUNK(ch, CC)                                                                                      \
    {                                                                                                              \
        __syncthreads(); /* chunk ch is in LDS; nobody still reads the buffer chunk ch + 1 goes to */             \
        /* this wave's row tiles start at tile wm NT of the workgroup's */                                        \
        const unsigned char *buf = lds + (size_t)((ch) & 1) * BUF + (size_t)(wm * NT) * 2048 + lane * 16;          \
        const int kbase = (ch) * KC;                                                                               \
        if (!DEEP) { WISV_MM_STAGE_LOAD((ch) + 1, 0) }                                                             \
        _Pragma("unroll") for (int lt = 0; lt < KC; ++lt) {                                                        \
            if (kbase + lt < ntile) { /* uniform per wave; no load inside, so the load counts hold on every path */ \
                if (!WEAVE || lt == 0) {                                                                           \
                    WISV_MM_READ_B(lt, 0, bv[0])                                                                   \
                    if (WEAVE) __builtin_amdgcn_sched_barrier(0);                                                  \
                }                                                                                                  \
                _Pragma("unroll") for (int og = 0; og < G; ++og) {                                                 \
                    if (og < G - 1) { WISV_MM_READ_B(lt, og + 1, bv[(og + 1) & 1]) }                               \
                    else if (WEAVE && lt + 1 < KC) { WISV_MM_READ_B(lt + 1, 0, bv[0]) }                            \
                    if (!WEAVE) __builtin_amdgcn_sched_barrier(0);                                                 \
                    WISV_MM_GROUP(lt, og, abuf[(CC) * KC + lt], bv[og & 1])                                        \
                    if (WEAVE && (og < G - 1 || lt + 1 < KC)) {                                                    \
                        /* one LDS read of the next group after every RP matrix instructions of this one */       \
                        _Pragma("unroll") for (int t = 0; t < NT; ++t) {                                           \
                            __builtin_amdgcn_sched_group_barrier(0x008, RP, 0);                                    \
                            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);                                     \
                        }                                                                                          \
                    }                                                                                              \
                    __builtin_amdgcn_sched_barrier(0);                                                             \
                }                                                                                                  \
            }                                                                                                      \
            /* refill the slot right after its use; past the end the last tile is re-read into a slot nobody uses */ \
            _Pragma("unroll") for (int p = 0; p < RP; ++p) _Pragma("unroll") for (int op = 0; op < 2; ++op)        \
                abuf[(CC) * KC + lt][p][op] = wp[p * wstep + (size_t)min(kbase + lt + TURN * KC, ntile - 1) * 64 + 16 * op]; \
            __builtin_amdgcn_sched_barrier(0);                                                                     \
        }                                                                                                          \
        WISV_MM_STAGE_STORE((ch) + 1, DEEP ? ((CC) + 1) % TURN : 0)                                                \
        if (DEEP) { WISV_MM_STAGE_LOAD((ch) + 1 + TURN, ((CC) + 1) % TURN) }                                       \
    }

    const int nchunk = (ntile + KC - 1) / KC;
    if (DEEP) {
#pragma unroll
        for (int cc = 0; cc < TURN; ++cc) { WISV_MM_STAGE_LOAD(cc, cc) }
        WISV_MM_STAGE_STORE(0, 0)
        WISV_MM_STAGE_LOAD(TURN, 0)
    } else {
        WISV_MM_STAGE_LOAD(0, 0)
        WISV_MM_STAGE_STORE(0, 0)
    }
    int ch = 0;
    for (; ch + TURN <= nchunk; ch += TURN) {   // whole turns: no branch around any load
#pragma unroll
        for (int cc = 0; cc < TURN; ++cc) WISV_MM_CHUNK(ch + cc, cc)
    }
#pragma unroll
    for (int cc = 0; cc < TURN - 1; ++cc)       // the last, partial turn
        if (ch + cc < nchunk) WISV_MM_CHUNK(ch + cc, cc)
#undef WISV_MM_CHUNK
#undef WISV_MM_STAGE_LOAD
#undef WISV_MM_STAGE_STORE
#undef WISV_MM_READ_B
#undef WISV_MM_GROUP
    __syncthreads();   // every wave is done with the staged operands: the epilogue turns its tiles over there
    if (!active) return;
    static_assert(2 * BUF >= NW * 4096, "4 KiB of LDS per wave");
    if (SHORT) {
#pragma unroll
        for (int p = 0; p < RP; ++p)
#pragma unroll
            for (int t = 0; t < NT; ++t) acc[p][t] = sum[p][t] + acc[p][t];
    }
    mm_epilogue<NT, RP, EPI>(g, acc, m_base + wm * (32 * NT), rb0, by, bx * WN + wn, lane, reinterpret_cast<floatx4 *>(lds) + wave * 256);
}

// ------------------------------------------------------------------------------------------ tens of rows
// One row tile (17 to 160 rows) against the whole weight stream.  Weights and activations both go to LDS by direct loads
// (global_load_lds, 1 KiB per wave instruction, no registers) through a ring of NS stages of KC k-tiles.  A stage is
// waited for by count (loads complete in order) by the waves that loaded it, and one barrier per stage makes it visible
// and frees the buffer of the stage before.  The loads are inline assembly without outputs: the compiler orders every
// LDS read after every such load it knows of, which would drain the ring at each stage; the waits below are the only
// ones.
//
// Four of the eight waves multiply, the other four only issue loads, two of them the weights and two the activations:
// issuing one takes tens of cycles, which a multiplying wave loses on the matrix pipe.
//
// Without SHORT the order of the sums is that of k_gemm_mm and of the k-slice workgroups this kernel replaced, bit for bit (a token
// of a near-tie, once turned, stays turned).  CH == 1: every output is one chain of products over the workgroup's
// k-tiles (SHORT, as in k_gemm_mm: one per stage), a wave multiplies 32 weight rows by every row tile.  CH == 4 (at most 64 rows): four chains, k-tile i in
// chain i % 4, added as ((0 + 1) + 2) + 3; the waves are 2 x 2, 64 weight rows (wn) and one k-tile of every stage (wk)
// each, a wave's stages alternate between its two chains, and at the end it hands one of its two row-block pairs to its
// partner and finishes the other.
//
// What bounds it: bytes into a CU.  Weights and activations together arrive at about 41 GB/s per CU whatever the depth
// of the ring (3, 4 and 5 stages the same +- 1 %, 2 stages 30 % slower) and whether or not anything is multiplied (in
// a first form, 143 rows, gate/up of the 8B shape: 56 us, 54 without the matrix instructions, 47 with the weights
// alone), so beyond 32 rows, where weights alone (6.2 TB/s over 256 CUs) stop being the limit, time grows with the
// activations every workgroup re-reads from L2.  Against the workgroups it replaced, us per launch at the 8B shape, 32 /
// 96 / 143 rows: gate/up 49.0 / 61.8 / 76.3 -> 38.0 / 42.8 / 49.2, down 23.6 / 33.3 / 40.9 -> 19.6 / 24.6 / 34.6,
// QKV (two terms) 14.1 / 20.4 / 27.3 -> 10.3 / 18.4 / 23.1, O (two terms) 10.9 / 14.8 / 20.4 -> 8.3 / 12.4 / 16.8, LM head of
// 32000 tokens 53.3 / 70.0 / 82.8 -> 45.4 / 49.4 / 55.1, of 128256 tokens over 28 rows 207 -> 188 (results still leaving in
// 16-byte pieces; what whole lines took off stands at store_tile).

// a wave-uniform pointer, in scalar registers
__device__ __forceinline__ const unsigned char *scalar_ptr(const void *p) {
    const uint64_t v = (uint64_t)p;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return (const unsigned char *)(((uint64_t)hi << 32) | lo);
}
// lane l: 16 bytes from base + voff to lds_addr + 16 l
__device__ __forceinline__ void lds_load_1k(uint32_t lds_addr, uint32_t voff, const void *base) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds_addr), "v"(voff), "s"(base) : "memory", "m0");
}
__device__ __forceinline__ void lds_load_1k_nt(uint32_t lds_addr, uint32_t voff, const void *base) {   // read once: streamed
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt" ::"s"(lds_addr), "v"(voff), "s"(base) : "memory", "m0");
}
// at most `left` stages of N loads each may still be on their way; then meet the other waves
template <int N, int NS> __device__ __forceinline__ void pipe_wait(int left) {
    static_assert(NS == 3 || NS == 4, "one branch per count of stages left");
    static_assert(N * (NS - 2) <= 63, "vmcnt holds six bits");
    if (left >= NS - 2) asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(N * (NS - 2)) : "memory");
    else if (NS == 4 && left == 1) asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(N) : "memory");
    else asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
}

// RBW: row-blocks of weights per workgroup, 8 or 7 (with 7 the last pair's second half is another workgroup's: its
// products are of whatever the ring holds there and are not written)
template <int NT, int KC, int NS, int RBW, int CH, int EPI, int NPL, bool SHORT = false>
__global__ __launch_bounds__(512) void k_gemm_pipe(GemmArgs g) {
    extern __shared__ __align__(16) unsigned char lds[];
    static_assert(CH == 1 || (CH == 4 && KC == 2 && NT <= 2), "four chains: a k-tile per wave half and stage");
    static_assert(!SHORT || CH == 1, "a stage's products are one chain");
    constexpr int WB = RBW * KC, AB = NPL * KC * NT * 2;  // 1 KiB loads of weights / activations in a stage
    constexpr int NW = WB / 2, NA = AB / 2;               // per loading wave
    static_assert(WB % 2 == 0 && AB % 2 == 0, "the two waves of a kind issue the same number of loads");
    constexpr int WSLOT = 8 * KC, STAGE = (WSLOT + AB) * 1024;
    const int tid = threadIdx.x, lane = tid & 63, wave8 = __builtin_amdgcn_readfirstlane(tid >> 6), wave = wave8 & 3;
    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
    // (quotients come out of vector registers: made scalar here, so that every address below is)
    const int q = slot * 8 + xcd, groups = (g.gs + g.per - 1) / g.per;
    if (q >= g.gx * groups) return;                       // the whole workgroup leaves: no barrier is reached
    const int by = __builtin_amdgcn_readfirstlane(q / g.gx), bx = q - by * g.gx;
    // k-tiles of the first split and of the workgroup's last one; their stages run through the ring without a break
    const int split0 = by * g.per, n_split = min(g.per, g.gs - split0);
    const int kt0 = split0 * g.kt_per_split, whole = g.kt_per_split;
    const int tail = min(whole, g.nkt - kt0 - (n_split - 1) * whole), ntile = n_split == 1 ? tail : whole;
    const int per_split = (whole + KC - 1) / KC;
    const int nst = (n_split - 1) * per_split + (tail + KC - 1) / KC;   // every wave passes nst barriers (CH == 4: and two more)

    if (wave8 >= 4) {
        const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)lds;
        const int half = wave & 1;
        if (wave < 2) {
            // ---- weights: NW tiles of a stage (tile i = half NW + j: row-block i / KC, k-tile i % KC)
            const unsigned char *base = scalar_ptr(g.Wt + ((size_t)bx * RBW * g.nkt + kt0) * 64);
            const int rb_last = g.nrb - 1 - bx * RBW;         // row-blocks past the last re-read it (RBW == 7)
            int first = 0, at = 0;                            // of the next stage to load: its split's first k-tile, its place there
            auto issue = [&](int st) {
                const uint32_t buf = lds0 + (uint32_t)(st % NS) * STAGE;
                const int kt_last = min(whole, g.nkt - kt0 - first) - 1;
#pragma unroll
                for (int j = 0; j < NW; ++j) {
                    const int i = half * NW + j, rb = min(i / KC, rb_last), kt = first + min(at * KC + i % KC, kt_last);
                    lds_load_1k_nt(buf + i * 1024, lane * 16 + (uint32_t)(rb * g.nkt + kt) * 1024u, base);
                }
                if (++at == per_split) at = 0, first += whole;
            };
            for (int st = 0; st < min(NS - 1, nst); ++st) issue(st);
            for (int st = 0; st < nst; ++st) {
                pipe_wait<NW, NS>(min(NS - 2, nst - 1 - st));
                if (st + NS - 1 < nst) issue(st + NS - 1);    // into the buffer of stage st - 1, which nobody reads any more
            }
        } else {
            // ---- activations: NA KiB of a stage (two planes: one wave each), 8 rows x 64 columns or 16 rows x 32 per load,
            //      so that a row contributes whole 128- or 64-byte runs.  LDS keeps rows of KC * 64 bytes whose 16-byte
            //      pieces are permuted (piece c of row r sits at c ^ swz(r)): the operand reads then spread over the banks.
            constexpr int PCS = KC * 4, RPL = 64 / PCS;       // pieces per row, rows per load
            const unsigned char *base = scalar_ptr((const unsigned char *)(NPL == 1 ? g.X16 : half ? g.Xlo : g.Xhi) + (size_t)kt0 * 64);
            const int piece = (lane % PCS) ^ (KC == 2 ? lane / 8 : (lane / 16) & 3);
            const uint32_t last_odd = piece >= 4 ? 64u : 0u;  // of a last stage with one k-tile: the missing tile re-reads the present one
            uint32_t avo[NA];
#pragma unroll
            for (int j = 0; j < NA; ++j) {
                const int r = (half * NA + j) % (NT * 32 / RPL) * RPL + lane / PCS;
                // rows past M re-read row M - 1; their results are not written
                avo[j] = (uint32_t)min(r, g.M - 1) * (uint32_t)g.kd * 2u + (uint32_t)(piece * 16);
            }
            int first = 0, at = 0;
            auto issue = [&](int st) {
                const uint32_t buf = lds0 + (uint32_t)(st % NS) * STAGE + (WSLOT + half * NA) * 1024, k = (uint32_t)(first + at * KC) * 64u;
                const bool alone = KC == 2 && at * 2 + 1 >= min(whole, g.nkt - kt0 - first);
#pragma unroll
                for (int j = 0; j < NA; ++j) lds_load_1k(buf + j * 1024, avo[j] + (alone ? k - last_odd : k), base);
                if (++at == per_split) at = 0, first += whole;
            };
            for (int st = 0; st < min(NS - 1, nst); ++st) issue(st);
            for (int st = 0; st < nst; ++st) {
                pipe_wait<NA, NS>(min(NS - 2, nst - 1 - st));
                if (st + NS - 1 < nst) issue(st + NS - 1);
            }
        }
        if (CH == 4) asm volatile("s_barrier\n\ts_barrier" ::: "memory");   // the two of the chains' sum below
        return;
    }

    // ---- the multiplying waves
    constexpr int P = CH == 4 ? 2 : 1, SETS = CH == 4 ? 2 : 1, UN = CH == 4 ? 2 : 2 * KC;   // pairs, chains, operands of a stage
    const int wn = CH == 4 ? wave >> 1 : wave, wk = CH == 4 ? wave & 1 : 0;
    floatx16 acc[SETS][P][NT];
#pragma unroll
    for (int c = 0; c < SETS; ++c)
#pragma unroll
        for (int p = 0; p < P; ++p)
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[c][p][t][e] = 0.f;
    // operand `op` of pair p: lane l wants row l % 32 of the pair and k-group 2 (l / 32) + op (as in k_gemm_mm)
    const unsigned char *ap = lds + (wn * 2 * P + ((lane & 31) >> 4)) * KC * 1024 + (32 * (lane >> 5) + (lane & 15)) * 16;
    const unsigned char *bp = lds + WSLOT * 1024 + (lane & 31) * (KC * 64);
    const int swz = KC == 2 ? lane & 7 : (lane >> 2) & 3;
    struct Ops { u32x4 a[UN][P], b[UN][NPL][NT]; };
    // Where the registers allow it (AHEAD) a stage's operands are read while the products of the stage before run; else
    // those products must not sink below the reads
    constexpr bool AHEAD = 16 * SETS * P * NT + 8 * UN * (P + NPL * NT) <= 200;
    auto fetch = [&](int st, Ops &o) {
        if (!AHEAD) __builtin_amdgcn_sched_barrier(0);
        // this wave's reads of the stage before are done (its buffer is overwritten after the barrier); stage st is there
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        const unsigned char *as = ap + (size_t)(st % NS) * STAGE, *bs = bp + (size_t)(st % NS) * STAGE;
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            const int kt = CH == 4 ? wk : u >> 1, op = u & 1;
#pragma unroll
            for (int p = 0; p < P; ++p) o.a[u][p] = *reinterpret_cast<const u32x4 *>(as + (p * 2 * KC + kt) * 1024 + op * 256);
#pragma unroll
            for (int pl = 0; pl < NPL; ++pl)
#pragma unroll
                for (int t = 0; t < NT; ++t)
                    o.b[u][pl][t] = *reinterpret_cast<const u32x4 *>(bs + (pl * NT + t) * (KC * 2048) + ((kt * 4 + op + 2 * (lane >> 5)) ^ swz) * 16);
        }
    };
    auto multiply = [&](const Ops &o, floatx16 (&ac)[P][NT], int u0, int u1) {   // compile-time numbers once inlined
        if constexpr (SHORT) {
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                floatx16 chain = {};
#pragma unroll
                for (int u = u0; u < u1; ++u)
#pragma unroll
                    for (int pl = 0; pl < NPL; ++pl) chain = mm_mfma<NPL>(o.a[u][0], o.b[u][pl][t], chain);
                ac[0][t] += chain;
            }
            return;
        }
#pragma unroll
        for (int u = u0; u < u1; ++u)
#pragma unroll
            for (int pl = 0; pl < NPL; ++pl)
#pragma unroll
                for (int t = 0; t < NT; ++t)
#pragma unroll
                    for (int p = 0; p < P; ++p) ac[p][t] = mm_mfma<NPL>(o.a[u][p], o.b[u][pl][t], ac[p][t]);
    };
    // No branch around the products in the loops: a merge would move every accumulator between register files.
    auto last = [&](const Ops &o, floatx16 (&ac)[P][NT], int nt) {   // of a split of nt k-tiles: with KC == 2 its last stage may hold one
        const bool odd = KC == 2 && (nt & 1);
        if (CH == 4) {
            if (!odd || wk == 0) multiply(o, ac, 0, UN);
        } else {
            multiply(o, ac, 0, 2);
            if (KC == 2 && !odd) multiply(o, ac, 2, UN);
        }
    };
    const int rb0 = bx * RBW + wn * 2 * P + wk * 2, rb_end = min(g.nrb, (bx + 1) * RBW);
    floatx4 *turn = reinterpret_cast<floatx4 *>(lds + (size_t)NS * STAGE) + wave * 256;   // (the ring may still be filling for the next split)
    Ops o0, o1;
    int st = 0;
    static_assert(NT < 5 || !AHEAD, "several splits per workgroup: the plain loop only");
    if constexpr (AHEAD) {
        fetch(0, o0);
        for (; st + 2 < nst; st += 2) {
            fetch(st + 1, o1);
            multiply(o0, acc[0], 0, UN);
            fetch(st + 2, o0);
            multiply(o1, acc[SETS - 1], 0, UN);
        }
        if (st + 1 < nst) {
            fetch(st + 1, o1);
            multiply(o0, acc[0], 0, UN);
            last(o1, acc[SETS - 1], ntile);
        } else {
            last(o0, acc[0], ntile);
        }
    } else if constexpr (CH == 1) {
        // (the only form that takes several splits: see the launcher)
        for (int sp = 0; sp + 1 < n_split; ++sp) {
            for (const int end = st + per_split - 1; st < end; ++st) {
                fetch(st, o0);
                multiply(o0, acc[0], 0, UN);
            }
            fetch(st++, o0);
            last(o0, acc[0], whole);
            if (rb0 < rb_end) mm_epilogue<NT, 1, EPI>(g, acc[0], 0, rb0, split0 + sp, rb0 >> 1, lane, turn, rb_end);
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[0][0][t][e] = 0.f;
        }
        for (; st + 1 < nst; ++st) {
            fetch(st, o0);
            multiply(o0, acc[0], 0, UN);
        }
        fetch(st, o0);
        last(o0, acc[0], tail);
    } else {
        for (; st + 2 < nst; st += 2) {
            fetch(st, o0);
            multiply(o0, acc[0], 0, UN);
            fetch(st + 1, o0);
            multiply(o0, acc[SETS - 1], 0, UN);
        }
        fetch(st, o0);
        if (st + 1 < nst) {
            multiply(o0, acc[0], 0, UN);
            fetch(st + 1, o0);
            last(o0, acc[SETS - 1], ntile);
        } else {
            last(o0, acc[0], ntile);
        }
    }

    const int split = split0 + n_split - 1;
    if constexpr (CH == 4) {
        // wave (wn, wk) holds chains wk and 2 + wk; it hands pair 1 - wk to its partner and finishes pair wk
        floatx4 *red = reinterpret_cast<floatx4 *>(lds);   // [wave][chain][NT][4][64]
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");   // every read of the last stages is done
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    floatx4 v;
#pragma unroll
                    for (int i = 0; i < 4; ++i) v[i] = wk ? acc[c][0][t][4 * e + i] : acc[c][1][t][4 * e + i];
                    red[(((wave * 2 + c) * NT + t) * 4 + e) * 64 + lane] = v;
                }
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        floatx16 out[1][NT];
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const floatx4 p0 = red[((((wave ^ 1) * 2 + 0) * NT + t) * 4 + e) * 64 + lane];
                const floatx4 p1 = red[((((wave ^ 1) * 2 + 1) * NT + t) * 4 + e) * 64 + lane];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float m0 = wk ? acc[0][1][t][4 * e + i] : acc[0][0][t][4 * e + i];
                    const float m1 = wk ? acc[1][1][t][4 * e + i] : acc[1][0][t][4 * e + i];
                    out[0][t][4 * e + i] = wk ? ((p0[i] + m0) + p1[i]) + m1 : ((m0 + p0[i]) + m1) + p1[i];
                }
            }
        if (rb0 < rb_end) mm_epilogue<NT, 1, EPI>(g, out, 0, rb0, split, rb0 >> 1, lane, turn, rb_end);
    } else {
        if (rb0 < rb_end) mm_epilogue<NT, 1, EPI>(g, acc[0], 0, rb0, split, rb0 >> 1, lane, turn, rb_end);
    }
}

// ------------------------------------------------------------------------------------------ launch
// LDS bytes: activation chunk (two planes, WK slices; two buffers when a slice needs several chunks),
// or the slice-reduction scratch if that is larger
static size_t ws_lds(int Mt, int kcw, int sub, int NT, int RB, int WR, int WK) {
    const size_t x = (size_t)(sub > kcw ? 2 : 1) * 2 * WK * Mt * (kcw * 64 + 16);
    const size_t red = (size_t)WR * (WK - 1) * RB * NT * 1024;
    return std::max(x, red);
}

template <int NT, int RB, int WR, int WK, int U, int EPI, int PRO, bool WHOLE>
static bool launch_ws_u(Ctx *c, GemmArgs &g, int splits, size_t soft_budget) {
    const int sub = (g.kt_per_split + WK - 1) / WK, Mt = std::min(g.M, 16 * NT);
    // largest chunk (a multiple of U) within the soft budget, else within what a CU has
    int kcw = (sub + U - 1) / U * U;
    for (size_t budget : {soft_budget, (size_t)150 * 1024}) {
        kcw = (sub + U - 1) / U * U;
        while (kcw > U && ws_lds(Mt, kcw, sub, NT, RB, WR, WK) > budget) kcw = (kcw / 2 + U - 1) / U * U;
        if (ws_lds(Mt, kcw, sub, NT, RB, WR, WK) <= budget) break;
    }
    size_t lds = ws_lds(Mt, kcw, sub, NT, RB, WR, WK);
    if (PRO == PRO_NORM) {
        // one chunk only (the row sums of squares are taken once), and room for one float per staged item behind
        // the two chunk buffers
        if (sub > kcw || WK != 1) return false;
        lds = (size_t)2 * 2 * Mt * (kcw * 64 + 16) + (size_t)Mt * kcw * 8 * 4;
    }
    if (lds > 150 * 1024) return false;
    g.kcw = kcw;
    static bool allowed[MAX_DEVICES];     // per instantiation
    if (lds > 64 * 1024 && !allow_big_lds(c, reinterpret_cast<const void *>(&k_gemm_ws<NT, RB, WR, WK, U, PRO, EPI, WHOLE>), allowed))
        return false;
    dim3 grid((g.nrb / RB + WR - 1) / WR, splits, (g.M + 16 * NT - 1) / (16 * NT));
    hipLaunchKernelGGL((k_gemm_ws<NT, RB, WR, WK, U, PRO, EPI, WHOLE>), grid, dim3(64 * WR * WK), lds, c->stream, g);
    return true;
}
// U: ring slots of the guarded form; UW: of the form for slices of whole turns, taken where the shape has them (every matrix of
// the 8B shape does)
template <int NT, int RB, int WR, int WK, int U, int UW, int EPI, int PRO = PRO_NONE>
static bool launch_ws_t(Ctx *c, GemmArgs &g, int splits, size_t soft_budget) {
    const bool whole = g.nkt == splits * g.kt_per_split && g.kt_per_split % (WK * UW) == 0 && g.nrb % (RB * WR) == 0;
    if (whole) return launch_ws_u<NT, RB, WR, WK, UW, EPI, PRO, true>(c, g, splits, soft_budget);
    return launch_ws_u<NT, RB, WR, WK, U, EPI, PRO, false>(c, g, splits, soft_budget);
}

constexpr int MM_RP = 2;            // pairs of row-blocks per wave of k_gemm_mm
constexpr int MM_RB = 2 * MM_RP;

template <int NT, int WM, int NW, int KC, int U, int EPI, int NPL, bool DEEP = false, bool WEAVE = false, bool SHORT = false>
static bool launch_mm_t(Ctx *c, GemmArgs &g, int splits) {
    constexpr int WN = NW / WM, NTW = NT * WM;
    g.gx = (g.nrb + WN * MM_RB - 1) / (WN * MM_RB);
    g.gz = (g.M + 32 * NTW - 1) / (32 * NTW);
    g.gs = splits;
    const size_t lds = (size_t)2 * NPL * KC * NTW * 2 * 1024;   // two buffers, NPL planes, 2 operands per (k-tile, row tile)
    static bool allowed[MAX_DEVICES];     // per instantiation
    if (lds > 64 * 1024 &&
        !allow_big_lds(c, reinterpret_cast<const void *>(&k_gemm_mm<NT, WM, NW, MM_RP, KC, U, EPI, NPL, DEEP, WEAVE, SHORT>), allowed))
        return false;
    const unsigned grid = (unsigned)((g.gx * g.gs + 7) / 8 * 8 * g.gz);
    hipLaunchKernelGGL((k_gemm_mm<NT, WM, NW, MM_RP, KC, U, EPI, NPL, DEEP, WEAVE, SHORT>), dim3(grid), dim3(64 * NW), lds, c->stream, g);
    return true;
}

// ---- k_gemm_pipe: 128 (or 112) weight rows x one row tile per workgroup
constexpr int PIPE_RB = 8, PIPE_MAX_ROWS = 160;
template <int NT, int KC, int RBW, int CH, int EPI, int NPL, bool SHORT = false> static bool launch_pipe_t(Ctx *c, GemmArgs &g, int splits) {
    constexpr int NS = KC == 2 ? 3 : 4;                        // see the kernel: deeper rings measure the same
    constexpr int STAGE = KC * (8 + NPL * NT * 2);             // KiB
    constexpr size_t lds = (size_t)(NS * STAGE + 16) * 1024;   // the ring, and 4 KiB per multiplying wave for the epilogue
    static_assert(lds <= 150 * 1024, "what allow_big_lds asks for");
    static_assert(CH != 4 || NS * STAGE >= 32 * NT, "the four chains are added up in the ring");
    g.gx = (g.nrb + RBW - 1) / RBW;
    g.gz = 1;
    g.gs = splits;
    // More splits than fill the chip once (129 to 160 rows keep the counts that tiles of 512 weight rows asked for: 16 for the
    // down projection at the 8B shape, 512 workgroups): a workgroup takes several in one pass of the ring.  143 rows: 45 us
    // as 512 workgroups, 41 in k_gemm_mm, 34.6 as 256 of two splits.
    g.per = NT == 5 ? std::max(1, std::min(splits, (g.gx * splits + 255) / 256)) : 1;
    static bool allowed[MAX_DEVICES];     // per instantiation
    if (lds > 64 * 1024 && !allow_big_lds(c, reinterpret_cast<const void *>(&k_gemm_pipe<NT, KC, NS, RBW, CH, EPI, NPL, SHORT>), allowed)) return false;
    const unsigned grid = (unsigned)((g.gx * ((splits + g.per - 1) / g.per) + 7) / 8 * 8);
    hipLaunchKernelGGL((k_gemm_pipe<NT, KC, NS, RBW, CH, EPI, NPL, SHORT>), dim3(grid), dim3(512), lds, c->stream, g);
    return true;
}
template <int NT, int CH, int EPI, int NPL> static bool launch_pipe_nt(Ctx *c, GemmArgs &g, int splits) {
    if constexpr (NPL == 1 && EPI == EPI_SWIGLU) {
        // no k-split here: seven row-blocks per workgroup when that fills whole rounds of 256 CUs better (14336 features:
        // 256 workgroups instead of 224: 32 / 96 / 143 rows 39.0 / 46.5 / 55.9 -> 36.6 / 44.6 / 52.8 us in an earlier form)
        auto fill = [&](int rbw) { const int wgs = (g.nrb + rbw - 1) / rbw; return (double)wgs / ((wgs + 255) / 256 * 256); };
        if (fill(7) > fill(8)) return launch_pipe_t<NT, 2, 7, CH, EPI, NPL>(c, g, splits);
    }
    return launch_pipe_t<NT, NPL == 1 || CH == 4 ? 2 : 1, 8, CH, EPI, NPL>(c, g, splits);
}
template <int EPI, int NPL> static bool launch_pipe(Ctx *c, GemmArgs &g, int splits) {
    // Four chains up to 64 rows, except for a product without k-splits over so many weight rows (>= 200 groups of 512: a
    // vocabulary of 100 thousand) that one chain per output always filled the chip
    if constexpr (EPI != EPI_PARTIAL)
        if (g.M <= 64 && (g.nrb + 31) / 32 >= 200)
            return g.M <= 32 ? launch_pipe_nt<1, 1, EPI, NPL>(c, g, splits) : launch_pipe_nt<2, 1, EPI, NPL>(c, g, splits);
    switch ((g.M + 31) / 32) {
        case 1: return launch_pipe_nt<1, 4, EPI, NPL>(c, g, splits);
        case 2: return launch_pipe_nt<2, 4, EPI, NPL>(c, g, splits);
        case 3: return launch_pipe_nt<3, 1, EPI, NPL>(c, g, splits);
        case 4: return launch_pipe_nt<4, 1, EPI, NPL>(c, g, splits);
        default: return launch_pipe_nt<5, 1, EPI, NPL>(c, g, splits);
    }
}

// Workgroup shapes of k_gemm_mm (more than 160 rows), tiles of 128 rows: met by 4 x 2 waves (256 weight rows per
// workgroup, every weight tile loaded by two waves), or - "wide" - by 8 x 1 waves with four row tiles each (512 weight
// rows, half the L2 traffic per flop, but half as many workgroups), or - "narrow" - by 2 x 2 waves (128 weight rows; two
// workgroups share a CU).  With k-splits wide pays when it still fills the chip (>= 200 workgroups) and a split keeps
// >= 24 k-tiles; without them the shape with the fewest rounds of workgroups, weighted by what a round of that shape
// costs, is taken.
enum { MM_NARROW = 0, MM_NORMAL = 1, MM_WIDE = 2 };   // 2 x 2, 4 x 2, 8 x 1 waves
static int mm_layout(int rows, int nrb, int nkt, bool can_split, int max_splits) {
    const int tiles = (rows + 127) / 128;
    const int base8 = ((nrb + 8 * MM_RB - 1) / (8 * MM_RB)) * tiles, base4 = ((nrb + 4 * MM_RB - 1) / (4 * MM_RB)) * tiles;
    if (!can_split) {
        // A workgroup takes about the same time however many of them run, so the cost is rounds of 256 workgroups
        // times the time of one round, measured on gate/up of 4096 x 5504 over 256 rows, one round in every shape: wide
        // 108.6 us, 4 x 2 waves 81.6, narrow 62.6 (over 512 rows narrow needs two rounds: 106.4, 83.0 and 112.8).
        // 14336 features over 384 rows: 336 workgroups of 4 x 2 waves 163.6 us, 168 wide ones 119.2.
        const int base2 = ((nrb + 2 * MM_RB - 1) / (2 * MM_RB)) * tiles;
        const double c8 = (base8 + 255) / 256 * 1.34, c4 = (base4 + 255) / 256 * 1.0, c2 = (base2 + 255) / 256 * 0.76;
        return c8 <= c4 && c8 <= c2 ? MM_WIDE : c4 <= c2 ? MM_NORMAL : MM_NARROW;
    }
    const int s = std::max(1, std::min(256 / std::max(1, base8), max_splits));
    return base8 * s >= 200 && nkt / s >= 24 ? MM_WIDE : MM_NORMAL;
}

// returns the number of row tiles and of row-blocks a workgroup covers
static int mm_shape(int rows, int layout, int *rb_per_wg) {
    *rb_per_wg = (layout == MM_WIDE ? 8 : layout == MM_NORMAL ? 4 : 2) * MM_RB;
    return (rows + 127) / 128;
}

// More than 160 rows: k_gemm_mm
template <int EPI, int NPL> static bool launch_ws_many_t(Ctx *c, GemmArgs &g, int splits, int layout) {
    if (layout == MM_WIDE) {
        if (EPI != EPI_PARTIAL) return launch_mm_t<4, 1, 8, 2, 2, EPI, NPL, false, true>(c, g, splits);
        return launch_mm_t<4, 1, 8, 2, 2, EPI, NPL>(c, g, splits);
    }
    if constexpr (EPI != EPI_PARTIAL) {   // products with k-splits never take it
        if (layout == MM_NARROW) {
            // gate/up: a ring of two chunks with the activations staged as deep (5504 features over 176 / 256 rows 58.5 / 63.0
            // -> 53.9 / 62.1 us; the LM head of 16000 tokens 64.2 / 69.3 without it, 60.3 / 68.3 if it took it)
            if (EPI == EPI_SWIGLU) return launch_mm_t<2, 2, 4, 2, 4, EPI, NPL, true>(c, g, splits);
            return launch_mm_t<2, 2, 4, 2, 2, EPI, NPL>(c, g, splits);
        }
    }
    return launch_mm_t<2, 2, 8, 2, 2, EPI, NPL>(c, g, splits);
}
// Two-term products of a prompt: the same kernels with short chains (see k_gemm_mm), no wide form (its accumulators leave no
// registers for a second set)
template <int EPI> static bool launch_short(Ctx *c, GemmArgs &g, int splits) {
    switch ((g.M + 31) / 32) {
        case 1: return launch_pipe_t<1, 2, 8, 1, EPI, 2, true>(c, g, splits);
        case 2: return launch_pipe_t<2, 2, 8, 1, EPI, 2, true>(c, g, splits);
        case 3: return launch_pipe_t<3, 1, 8, 1, EPI, 2, true>(c, g, splits);
        case 4: return launch_pipe_t<4, 1, 8, 1, EPI, 2, true>(c, g, splits);
        case 5: return launch_pipe_t<5, 1, 8, 1, EPI, 2, true>(c, g, splits);
        default: return launch_mm_t<2, 2, 8, 2, 2, EPI, 2, false, false, true>(c, g, splits);
    }
}
// Wh: the half-precision tiles, or null for the two-term product on the bf16 tiles already in g.Wt
template <int EPI> static bool launch_ws_many(Ctx *c, GemmArgs &g, int splits, int layout, const void *Wh, bool short_chains = false) {
    // Up to 160 rows (five 32-row tiles: the accumulators of a sixth do not fit a wave's registers) one pass over the
    // weights in k_gemm_pipe; see there for both sides.
    const bool pipe = g.M <= PIPE_MAX_ROWS;
    if (Wh && g.X16) {
        g.Wt = (const u32x4 *)Wh;
        if (pipe) return launch_pipe<EPI, 1>(c, g, splits);
        return launch_ws_many_t<EPI, 1>(c, g, splits, layout);
    }
    if constexpr (EPI == EPI_PARTIAL)
        if (short_chains) return launch_short<EPI>(c, g, splits);
    if (pipe) return launch_pipe<EPI, 2>(c, g, splits);
    return launch_ws_many_t<EPI, 2>(c, g, splits, layout);
}

bool ws_supported(const Ctx *c, int rows, int kd) {
    return c->bf16 && kd % 32 == 0 && rows >= 1;
}

static void fill_args(GemmArgs &g, const void *Wt, const ActBuf &X, int rows, int n, int kd) {
    g.Wt = (const u32x4 *)Wt;
    g.Xhi = X.hi; g.Xlo = X.lo; g.X16 = X.h16;
    g.M = rows; g.N = n; g.kd = kd;
    g.nrb = ws_padded_row_blocks(n); g.nkt = kd / 32;
}

// Slices of 8 k-tiles (QKV and O at the 8B shape) stay at a ring of four (of eight: QKV 9.4 -> 9.9 us, O 6.3 -> 6.8), slices of
// 28 (down) take four turns of seven (18.8 -> 18.1).  So do all lengths that seven divides, whether four does or not: down from as
// many features as make slices of 14 / 21 / 28 / 35 / 42 / 56 k-tiles, 4 rows, event pairs, with the ring of four 14.8 / 19.7 / 23.0
// / 31.3 / 33.3 / 41.7 us, of seven 13.5 / 18.0 / 22.5 / 28.1 / 31.2 / 40.5; 15 rows alike.
static bool launch_ws_partial_t(Ctx *c, GemmArgs &g, int splits) {
    if (g.kt_per_split % 7) return launch_ws_t<1, 1, 8, 1, 4, 4, EPI_PARTIAL>(c, g, splits, 40 * 1024);
    return launch_ws_t<1, 1, 8, 1, 4, 7, EPI_PARTIAL>(c, g, splits, 40 * 1024);
}

// Y partial slices: returns the number of slices written to `Yp` ([S][split_stride]), 0 if the shape cannot
// be served (nothing was launched)
int launch_gemm_ws_partial(Ctx *c, const void *Wt, const ActBuf &X, float *Yp, size_t split_stride, int max_splits,
                           int rows, int n, int kd, int kclass, const AttnPartials *ap, const void *Wh, bool prompt) {
    ProfScope ps(c, kclass);
    GemmArgs g{};
    fill_args(g, Wt, X, rows, n, kd);
    g.Yp = Yp; g.split_stride = split_stride;
    int s;
    int layout = MM_NORMAL;
    const bool short_chains = prompt && !(Wh && X.h16);
    if (rows <= 16) {
        // one row-block per wave: split k until about 6144 waves stream (three workgroups per CU), a wave keeps
        // at least 8 k-tiles
        s = (6144 + g.nrb - 1) / g.nrb;
        s = std::max(1, std::min(s, std::min(max_splits, std::max(1, g.nkt / 8))));
    } else {
        // about one workgroup per CU over (row-block groups) x (row tiles) x splits; a split keeps >= 8 k-tiles
        const int max_s = std::min(max_splits, std::max(1, g.nkt / 8));
        int rb_per_wg = PIPE_RB, tiles = 1;
        if (rows > 128) {   // (k_gemm_pipe up to 160 rows keeps the split counts of the tiles of 128 rows)
            layout = short_chains ? MM_NORMAL : mm_layout(rows, g.nrb, g.nkt, true, max_s);
            tiles = mm_shape(rows, layout, &rb_per_wg);
        }
        const int base = ((g.nrb + rb_per_wg - 1) / rb_per_wg) * tiles;
        s = std::max(1, std::min(256 / std::max(1, base), max_s));
        if (short_chains) {
            // up to four splits where they come to fewer rounds of 256 workgroups a split: slices are shorter sums (QKV at
            // the 8B shape over 768 rows, 144 workgroups a split: 1 split 113 us, 2 splits 124, 3 splits 95; over 1000 rows, 192
            // a split: 115, 127 and 138, 4 splits 117)
            auto rounds = [&](int t) { return (base * t + 255) / 256; };
            for (int t = s + 1; t <= std::min(4, max_s); ++t)
                if (rounds(t) * s < rounds(s) * t + (rows <= PIPE_MAX_ROWS)) s = t;   // (few rows: slices cost little, a tie goes to more)
        }
    }
    g.kt_per_split = (g.nkt + s - 1) / s;
    const int splits = (g.nkt + g.kt_per_split - 1) / g.kt_per_split;
    if (ap) {   // the activations are the attention output, still in k-split partials
        if (rows > 16 || ap->splits < 1 || ap->splits > WS_PRO_SPLITS || kd != ap->heads * 128) return 0;
        g.att_o = ap->o; g.att_m = ap->m; g.att_l = ap->l;
        g.att_splits = ap->splits; g.att_rows = ap->rows; g.att_H = ap->heads;
        return launch_ws_t<1, 1, 8, 1, 4, 4, EPI_PARTIAL, PRO_ATTN>(c, g, splits, 40 * 1024) ? splits : 0;
    }
    const bool ok = rows <= 16 ? launch_ws_partial_t(c, g, splits)
                               : launch_ws_many<EPI_PARTIAL>(c, g, splits, layout, Wh, short_chains);
    return ok ? splits : 0;
}

// The product that opens a block, with the block's RMSNorm folded in (at most 16 rows): the kernel adds the previous
// product's n_partial slices (c->y) to the residual stream x_in while it stages it, writes the sum to x_out, feeds
// x * gain to the matrix cores and leaves the sum of squares of every row in ss[split][row]; whoever adds this
// product's slices multiplies by 1 / sqrt(sum ss / kd + eps).  Returns the number of slices, 0 if the shape is not
// served (nothing was launched).
int launch_gemm_ws_normfold(Ctx *c, const void *Wt, const float *x_in, float *x_out, int n_partial, const void *gain,
                            float *Yp, size_t split_stride, int max_splits, int rows, int n, int kd, float *ss, int kclass) {
    if (rows > 16 || n_partial > MAX_SPLITS) return 0;
    ProfScope ps(c, kclass);
    GemmArgs g{};
    fill_args(g, Wt, ActBuf{}, rows, n, kd);
    g.Yp = Yp; g.split_stride = split_stride;
    int s = (6144 + g.nrb - 1) / g.nrb;
    s = std::max(1, std::min(s, std::min(max_splits, std::max(1, g.nkt / 8))));
    g.kt_per_split = (g.nkt + s - 1) / s;
    const int splits = (g.nkt + g.kt_per_split - 1) / g.kt_per_split;
    g.xin = x_in; g.xout = x_out; g.ys = c->y; g.ys_stride = (size_t)c->slice_rows * kd; g.n_partial = n_partial;
    g.gain = (const bf16_t *)gain; g.ss_out = ss;
    return launch_ws_t<1, 1, 8, 1, 4, 4, EPI_PARTIAL, PRO_NORM>(c, g, splits, 40 * 1024) ? splits : 0;
}

// A product that closes a residual branch, complete inside one kernel (at most 16 rows): one row-block per
// workgroup, 16 waves split k among them and add their results through LDS, and the epilogue adds the residual
// stream, writes it back, writes x * gain as the next block's activations and the rows' partial sums of squares to
// ss[row-block][row] (see EPI_RESID).  `ap`: the activations are still the attention kernel's k-split partials.
// Returns the number of partial sums per row, 0 if the shape is not served (nothing was launched).
int launch_gemm_ws_resid(Ctx *c, const void *Wt, const ActBuf &X, const AttnPartials *ap, float *x, const void *gain,
                         const ActBuf &A_out, float *ss, int rows, int n, int kd, int kclass) {
    if (rows > 16 || n % 16 || (ap && (ap->splits < 1 || ap->splits > WS_PRO_SPLITS || kd != ap->heads * 128))) return 0;
    ProfScope ps(c, kclass);
    GemmArgs g{};
    fill_args(g, Wt, X, rows, n, kd);
    g.kt_per_split = g.nkt;
    g.xin = x; g.xout = x; g.gain = (const bf16_t *)gain; g.H = A_out; g.ss_out = ss;
    if (ap) {
        g.att_o = ap->o; g.att_m = ap->m; g.att_l = ap->l;
        g.att_splits = ap->splits; g.att_rows = ap->rows; g.att_H = ap->heads;
        return launch_ws_t<1, 1, 1, 16, 4, 8, EPI_RESID, PRO_ATTN>(c, g, 1, 150 * 1024) ? n / 16 : 0;
    }
    return launch_ws_t<1, 1, 1, 16, 4, 8, EPI_RESID>(c, g, 1, 150 * 1024) ? n / 16 : 0;
}

// gate/up with the SwiGLU fused (single split): H[rows][F] = silu(gate) * up.  Every row-block of the
// re-tiled matrix holds 8 gate and 8 up rows.
bool launch_gemm_ws_swiglu(Ctx *c, const void *Wt, const ActBuf &X, const ActBuf &H, int rows, int features, int kd,
                           int kclass, const void *Wh, const float *ss, int n_ss, int planes) {
    ProfScope ps(c, kclass);
    GemmArgs g{};
    fill_args(g, Wt, X, rows, features, kd);
    g.nrb = ws_padded_pair_blocks(features);
    g.kt_per_split = g.nkt;
    g.H = H;
    if (n_ss > 0) {   // X holds x * gain: the kernel scales by 1 / rms itself (the streaming kernel only)
        if (rows > 16) return false;
        g.ss_in = ss; g.n_ss_in = n_ss; g.rms_eps = c->cfg.rms_eps;
    }
    if (rows <= 16) {
        // no k-split here, so the workgroup count is fixed by the shape: seven waves per workgroup when that fills
        // whole rounds of 256 CUs better than eight (14336 features: 256 workgroups instead of 224)
        auto fill = [&](int wr) { const int wgs = (g.nrb + wr - 1) / wr; return (double)wgs / ((wgs + 255) / 256 * 256); };
        if (fill(7) > fill(8)) return launch_ws_t<1, 1, 7, 1, 16, 16, EPI_SWIGLU>(c, g, 1, 36 * 1024);
        return launch_ws_t<1, 1, 8, 1, 16, 16, EPI_SWIGLU>(c, g, 1, 36 * 1024);
    }
    // more than 16 rows: H has one consumer, the down projection, and `planes` names the representation it reads;
    // the others (at 512 rows 59 of 73 MB) are not written
    g.H = act_planes(g.H, planes);
    return launch_ws_many<EPI_SWIGLU>(c, g, 1, mm_layout(rows, g.nrb, g.nkt, false, 1), Wh);
}

// LM head with the argmax fused: the candidates of every row's greedy token in c->cand; logits kept only on request
bool launch_gemm_ws_argmax(Ctx *c, const void *Wt, const ActBuf &X, float *logits, int rows, int n, int kd, int kclass,
                           const void *Wh) {
    GemmArgs g{};
    fill_args(g, Wt, X, rows, n, kd);
    g.kt_per_split = g.nkt;
    g.Yp = logits;
    g.cand = c->cand_pairs;               // at most one slot per row-block
    const int slots = rows <= 16 ? g.nrb : rows <= PIPE_MAX_ROWS ? g.nrb / 2 : (g.nrb + MM_RB - 1) / MM_RB;
    c->cand = Candidates{c->cand_pairs, nullptr, slots, rows};
    ProfScope ps(c, kclass);
    return rows <= 16 ? launch_ws_t<1, 1, 8, 1, 16, 16, EPI_ARGMAX>(c, g, 1, 70 * 1024)
                      : launch_ws_many<EPI_ARGMAX>(c, g, 1, mm_layout(rows, g.nrb, g.nkt, false, 1), Wh);
}

}  // namespace wisv
