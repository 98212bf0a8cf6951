// Dirty-row transform (the Compute step of Sec. 3.3 in re-apply form): for every
// vertex v of A_l gather the layer's input row
//     GraphConv  x            GraphSAGE  [h_self | x]        GIN  (1+eps) h_self + x
// (x = X^l[v], divided by the in-degree for mean), multiply by the weight
// matrix on the matrix cores, add the bias, apply the activation, and emit
//     D^l[v] = h_new - H^l[v],   H^l[v] = h_new
// so that the next hop can forward the delta (Sec. 3.3.3).
//
// Tiling: a workgroup of four wavefronts computes a tile of rows x columns, each
// wavefront accumulators of 32 x 32 (k_transform_split, k_transform_bf16; few rows:
// wave_gemm). K is consumed in slices of 32 staged through LDS. Later slices are
// already on their way from memory into registers while the matrix cores work on
// the current one: the weights (an L2 hit) one step ahead, the gathered rows (HBM
// latency) STAGES steps ahead. The fetch is branch-free (addresses are clamped, the row
// mode is a template parameter) and touches no loaded value, so nothing waits on
// memory until the registers are written to LDS; scaling, the SAGE/GIN combination
// and zero padding are applied at that point.
//
// Layers whose output is much narrower than their input (the classifier layer) are
// handled "project first": aggregation and the linear map commute, so the deltas are
// multiplied by the neighbour weights before they are scattered, the cached aggregate
// holds sum_u H[u] W_neigh (d_out wide), and the row transform only adds it
// (scaled for mean) to h_self W_self + b in the epilogue.
#include "common.h"
#include "kernels.h"
#include <algorithm>

#include "rows.h"
#include "push.h"

// Bias, (projected aggregate,) activation, delta against the stored row, store. Everything that
// is read (old rows, aggregate rows) is read in batches of TN*16 loads before anything is written:
// a load may not move above an earlier store to the same array, so interleaving them would pay one
// memory round trip per element.
template <int TM, int TN>
__device__ __forceinline__ void epilogue(const TArgs &a, floatx16 (&acc)[TM][TN], const uint32_t *s_vtx,
                                         const float *s_scale, uint32_t row0, uint32_t count, uint32_t n0, int wm, int wn,
                                         int lane) {
#pragma unroll
    for (int sm = 0; sm < TM; ++sm) {
        float old[TN][16], add[TN][16];
#pragma unroll
        for (int sn = 0; sn < TN; ++sn) {
            const uint32_t col = n0 + (wn * TN + sn) * 32 + (lane & 31);
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int lr = (wm * TM + sm) * 32 + (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3);
                float o = 0.0f, ad = 0.0f;
                if (col < a.N && row0 + lr < count) {
                    const size_t hidx = (size_t)s_vtx[lr] * a.N + col;
                    if (a.out_mode == 1)
                        o = a.store ? __bfloat162float(((const __hip_bfloat16 *)a.Hout)[hidx]) : ((const float *)a.Hout)[hidx];
                    if (a.addend) ad = a.addend[hidx] * (a.addend_scaled ? s_scale[lr] : 1.0f);
                }
                old[sn][r] = o;
                add[sn][r] = ad;
            }
        }
#pragma unroll
        for (int sn = 0; sn < TN; ++sn) {
            const uint32_t col = n0 + (wn * TN + sn) * 32 + (lane & 31);
            if (col >= a.N) continue;
            const float bias = a.bias[col];
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int lr = (wm * TM + sm) * 32 + (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3);
                const uint32_t slot = row0 + lr;
                if (slot >= count) continue;
                float z = acc[sm][sn][r] + bias + add[sn][r];
                if (a.act == RIPPLE_ACT_RELU) z = z > 0.0f ? z : 0.0f;
                if (a.out_mode == 0) {
                    a.tmp_out[(size_t)slot * a.tmp_out_ld + col] = z;
                } else if (a.out_mode == 2) {
                    a.tmp_out[(size_t)s_vtx[lr] * a.tmp_out_ld + col] = z;
                } else {
                    const size_t hidx = (size_t)s_vtx[lr] * a.N + col;
                    if (a.store) {
                        const __hip_bfloat16 zr = __float2bfloat16(z);
                        z = __bfloat162float(zr);
                        ((__hip_bfloat16 *)a.Hout)[hidx] = zr;
                    } else {
                        ((float *)a.Hout)[hidx] = z;
                    }
                    if (a.D) a.D[hidx] = a.d_old ? old[sn][r] : z - old[sn][r];
                }
            }
        }
    }
}

// 16-byte (bf16: 8-byte) accesses of the epilogues. full = false: a row's last group when the width is not a multiple of
// four; a load takes the whole group all the same (see floatx4u), a store the valid numbers.
__device__ __forceinline__ floatx4 ld4(const float *p) { return *(const floatx4u *)p; }
__device__ __forceinline__ void st4(float *p, floatx4 v, bool full, uint32_t n_valid) {
    if (full) {
        *(floatx4u *)p = v;
        return;
    }
    if (n_valid > 0) p[0] = v.x;
    if (n_valid > 1) p[1] = v.y;
    if (n_valid > 2) p[2] = v.z;
    if (n_valid > 3) p[3] = v.w;
}
__device__ __forceinline__ floatx4 ld4_bf16(const __hip_bfloat16 *p) {
    floatx4 r;
    const uintx2u w = *(const uintx2u *)p;
    r.x = bf_lo(w.x);
    r.y = bf_hi(w.x);
    r.z = bf_lo(w.y);
    r.w = bf_hi(w.y);
    return r;
}

// One round of the staged epilogue: U groups of four consecutive columns per thread. What the round
// reads and writes is fixed at compile time, so that its loads form one branch-free batch (a branch
// between two loads makes the second wait for the first):
//   EPI 0: act(z) goes to tmp_out (by slot or by vertex); nothing is read
//   EPI 1: H is updated;  EPI 2: H is updated and the delta row written
//   VEC: every group is whole (row widths that are multiples of four); BF: bf16 embeddings
template <int BN, int U, bool VEC, int EPI, bool BF>
struct EpiRound {
    floatx4 old[U], add[U];
    uint32_t nv[U];                                        // valid columns of the group (0: nothing to do)

    // request the old row and the addend of round it0 (no stores in here, no branches between the loads). Groups that
    // will not be stored read a valid address all the same (the row of vertex 0 for slots past the end, the
    // row's last four columns for padded columns), and a missing addend reads the bias instead.
    __device__ __forceinline__ void load(const TArgs &a, const uint32_t *s_vtx, const float *s_scale, uint32_t row0,
                                         uint32_t count, uint32_t n0, int tid, int it0) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int idx = tid + (it0 + u) * 256;
            const int r = idx / (BN / 4), c4 = (idx % (BN / 4)) * 4;
            const uint32_t col = n0 + c4;
            const uint32_t lim = (a.split_col && col < a.split_col) ? a.N1 : a.N;   // end of the block of columns `col` lies in
            nv[u] = (row0 + r < count && col < lim) ? min(4u, lim - col) : 0u;
            old[u] = (floatx4)(0.0f);
            add[u] = (floatx4)(0.0f);
            if (EPI == 0) continue;
            const uint32_t lcol = min(col, last_group(a.N));
            const size_t hidx = (size_t)s_vtx[r] * a.N + lcol;
            old[u] = BF ? ld4_bf16((const __hip_bfloat16 *)a.Hout + hidx) : ld4((const float *)a.Hout + hidx);
            const floatx4 t = ld4(a.addend ? a.addend + hidx : a.bias + lcol);
            const float sc = a.addend ? (a.addend_scaled ? s_scale[r] : 1.0f) : 0.0f;
            add[u] = a.addend ? t * sc : (floatx4)(0.0f);
        }
    }

    // bias, addend, activation, delta, stores
    __device__ __forceinline__ void finish(const TArgs &a, const float *Cs, const uint32_t *s_vtx, uint32_t row0,
                                           uint32_t n0, int tid, int it0) const {
        constexpr int C_LD = BN + 4;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (!nv[u]) continue;
            const int idx = tid + (it0 + u) * 256;
            const int r = idx / (BN / 4), c4 = (idx % (BN / 4)) * 4;
            const uint32_t col = n0 + c4, slot = row0 + r;
            const bool full = VEC || nv[u] == 4u;
            floatx4 v = *(const floatx4 *)&Cs[r * C_LD + c4] + *(const floatx4 *)(a.bias + col) + add[u];   // bias is padded
            if (a.act == RIPPLE_ACT_RELU) {
                v.x = v.x > 0.0f ? v.x : 0.0f;
                v.y = v.y > 0.0f ? v.y : 0.0f;
                v.z = v.z > 0.0f ? v.z : 0.0f;
                v.w = v.w > 0.0f ? v.w : 0.0f;
            }
            if (EPI == 0) {
                const size_t orow = (a.out_mode == 0) ? slot : s_vtx[r];
                if (a.split_col && col >= a.split_col) st4(a.tmp_out2 + orow * a.tmp_out2_ld + (col - a.split_col), v, full, nv[u]);
                else st4(a.tmp_out + orow * a.tmp_out_ld + col, v, full, nv[u]);
                continue;
            }
            const size_t hidx = (size_t)s_vtx[r] * a.N + col;
            if (BF) {
                uint2 w;
                w.x = pack_bf16x2(v.x, v.y);
                w.y = pack_bf16x2(v.z, v.w);
                unsigned short *hp = (unsigned short *)a.Hout + hidx;
                if (full) {
                    uintx2u wu;
                    wu.x = w.x;
                    wu.y = w.y;
                    *(uintx2u *)hp = wu;
                } else {
                    if (nv[u] > 0) hp[0] = (unsigned short)(w.x & 0xFFFFu);
                    if (nv[u] > 1) hp[1] = (unsigned short)(w.x >> 16);
                    if (nv[u] > 2) hp[2] = (unsigned short)(w.y & 0xFFFFu);
                    if (nv[u] > 3) hp[3] = (unsigned short)(w.y >> 16);
                }
                v.x = bf_lo(w.x);
                v.y = bf_hi(w.x);
                v.z = bf_lo(w.y);
                v.w = bf_hi(w.y);
            } else {
                st4((float *)a.Hout + hidx, v, full, nv[u]);
            }
            if (EPI == 2) st4(a.D + hidx, a.d_old ? old[u] : v - old[u], full, nv[u]);
        }
    }
};

// The global reads (old row, addend) run one round ahead of the stores: the first round is requested
// while the accumulators settle in LDS, each later one before the previous round is finished, so that
// only one memory round trip per tile is exposed.
template <int BN, int ITER, int U, bool VEC, int EPI, bool BF>
__device__ __forceinline__ void epilogue_rounds(const TArgs &a, const float *Cs, const uint32_t *s_vtx, const float *s_scale,
                                                uint32_t row0, uint32_t count, uint32_t n0, int tid) {
    EpiRound<BN, U, VEC, EPI, BF> ra, rb;
    ra.load(a, s_vtx, s_scale, row0, count, n0, tid, 0);
    __syncthreads();                                       // the tile is in LDS
#pragma unroll 1
    for (int it0 = 0; it0 < ITER; it0 += 2 * U) {
        rb.load(a, s_vtx, s_scale, row0, count, n0, tid, it0 + U);
        ra.finish(a, Cs, s_vtx, row0, n0, tid, it0);
        if (it0 + 2 * U < ITER) ra.load(a, s_vtx, s_scale, row0, count, n0, tid, it0 + 2 * U);
        rb.finish(a, Cs, s_vtx, row0, n0, tid, it0 + U);
    }
}

template <int BN, int ITER, int U, bool VEC, bool BF>
__device__ __forceinline__ void epilogue_pick(const TArgs &a, const float *Cs, const uint32_t *s_vtx, const float *s_scale,
                                              uint32_t row0, uint32_t count, uint32_t n0, int tid) {
    if (a.out_mode != 1) epilogue_rounds<BN, ITER, U, VEC, 0, BF>(a, Cs, s_vtx, s_scale, row0, count, n0, tid);
    else if (a.D) epilogue_rounds<BN, ITER, U, VEC, 2, BF>(a, Cs, s_vtx, s_scale, row0, count, n0, tid);
    else epilogue_rounds<BN, ITER, U, VEC, 1, BF>(a, Cs, s_vtx, s_scale, row0, count, n0, tid);
}

// Epilogue of the pipelined kernels: the accumulators are laid out row-major in LDS (over the A/B
// staging area, which is free by then), so that every thread handles four consecutive columns of a
// row. An addend is only read when H is updated (out_mode 1).
template <int TM, int TN, int BM, int BN, bool BF>
__device__ __forceinline__ void epilogue_staged(const TArgs &a, floatx16 (&acc)[TM][TN], float *Cs, const uint32_t *s_vtx,
                                                const float *s_scale, uint32_t row0, uint32_t count, uint32_t n0, int wm,
                                                int wn, int tid) {
    constexpr int C_LD = BN + 4;
    constexpr int ITER = BM * BN / 4 / 256, U = (ITER % 8 == 0) ? 4 : (ITER % 6 == 0) ? 3 : ITER / 2;
    static_assert(U >= 1 && ITER % (2 * U) == 0, "tile size");
    const int lane = tid & 63;
    const bool vec = (a.N & 3u) == 0 && (a.out_mode == 1 || (a.tmp_out_ld & 3u) == 0) &&
                     (a.split_col == 0 || ((a.N1 & 3u) == 0 && (a.tmp_out2_ld & 3u) == 0));
    __syncthreads();                                       // every wavefront is done with the A/B slices
#pragma unroll
    for (int sm = 0; sm < TM; ++sm)
#pragma unroll
        for (int sn = 0; sn < TN; ++sn)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int lr = (wm * TM + sm) * 32 + (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3);
                Cs[lr * C_LD + (wn * TN + sn) * 32 + (lane & 31)] = acc[sm][sn][r];
            }
    if (vec) epilogue_pick<BN, ITER, U, true, BF>(a, Cs, s_vtx, s_scale, row0, count, n0, tid);
    else epilogue_pick<BN, ITER, U, false, BF>(a, Cs, s_vtx, s_scale, row0, count, n0, tid);
}

static TArgs base_args(ripple_ctx *c, uint32_t l, const uint32_t *list, const uint32_t *count_d) {
    const LayerDev &ly = c->layers[l - 1];
    TArgs a;
    a.list = list;
    a.count_ptr = count_d;
    a.Hprev = c->H[l - 1];
    a.X = c->X[l];
    a.in_meta = c->in_meta;
    a.mean = (ly.agg == RIPPLE_AGG_MEAN) ? 1 : 0;
    a.one_plus_eps = 1.0f + ly.eps;
    a.d_in = ly.d_in;
    a.tmp_in = nullptr;
    a.tmp_ld = 0;
    a.store = c->store;
    a.Hout = c->H[l];
    a.D = nullptr;
    a.d_old = 0;
    a.tmp_out = nullptr;
    a.tmp_out_ld = 0;
    a.split_col = 0;
    a.N1 = ly.d_out;
    a.tmp_out2 = nullptr;
    a.tmp_out2_ld = 0;
    a.addend = nullptr;
    a.addend_scaled = 1;
    a.addend2 = nullptr;
    a.den = nullptr;
    a.range_rows = &c->ctr->range_rows;
    a.a_mode = 0;
    a.out_mode = 1;
    a.act = 0;
    a.W = ly.W0;
    a.Wq = ly.W0q;
    a.Wt = (c->store && c->opt_bf16_mfma) ? ly.W0h : nullptr;   // bf16 storage: bf16 matrix cores
    a.wt_ld = ly.K0pad;
    a.Wp = ly.W0p;
    a.wp_k = rp_round_up(ly.K, 128);
    a.wp_lift = ly.lift0;
    a.bias = ly.b0;
    a.K = ly.K;
    a.Kpad = ly.K0pad;
    a.N = ly.d_out;
    a.Npad = ly.N0pad;
    return a;
}

// Project-first layers have no matrix product left per row: h = act(Y[v] * scale + PS[v] + b), with
// Y the projected aggregate and PS the cached self term (absent for GraphConv).
template <bool BF>
__device__ __forceinline__ void addend_only_rows(const TArgs &a, uint32_t gw, uint32_t nw) {
    constexpr int R = 8;                                   // rows per wavefront and round: their loads overlap
    const uint32_t count = *a.count_ptr;
    const int lane = threadIdx.x & 63;
    for (uint32_t s0 = gw * R; s0 < count; s0 += nw * R) {
        uint32_t v[R];
        float sc[R];
#pragma unroll
        for (int u = 0; u < R; ++u) v[u] = a.list[min(s0 + u, count - 1u)];
#pragma unroll
        for (int u = 0; u < R; ++u) {
            const uint32_t deg = a.in_meta[v[u]].y;        // read in any case: no branch between the loads
            sc[u] = a.mean ? 1.0f / (float)(deg > 1u ? deg : 1u) : 1.0f;
        }
        bool bad[R];
#pragma unroll
        for (int u = 0; u < R; ++u) bad[u] = false;
        if (a.den) {                                       // attention: numerator / denominator, 0 without in-neighbours
#pragma unroll
            for (int u = 0; u < R; ++u) {
                const float dn = a.den[v[u]];
                bad[u] = !isfinite(dn) && s0 + u < count;
                sc[u] = (a.in_meta[v[u]].y > 0u && dn > 0.0f) ? 1.0f / dn : 0.0f;
            }
        }
        const float *p2 = a.addend2 ? a.addend2 : a.addend;
        const float w2 = a.addend2 ? 1.0f : 0.0f;
        for (uint32_t col = lane; col < a.N; col += 64) {
            float y[R], p[R], old[R];
#pragma unroll
            for (int u = 0; u < R; ++u) {                  // rows past the end repeat the last one and are not stored
                const size_t hidx = (size_t)v[u] * a.N + col;
                y[u] = a.addend[hidx];
                p[u] = p2[hidx];                           // unconditional: a branch here would serialise the loads
                old[u] = BF ? __bfloat162float(((const __hip_bfloat16 *)a.Hout)[hidx]) : ((const float *)a.Hout)[hidx];
            }
            const float b = a.bias[col];
#pragma unroll
            for (int u = 0; u < R; ++u) {
                if (s0 + u >= count) continue;
                const size_t hidx = (size_t)v[u] * a.N + col;
                float z = y[u] * sc[u] + b + (w2 != 0.0f ? p[u] : 0.0f);
                if (a.den && !isfinite(z)) bad[u] = true;      // an overflowed exponential: inf / inf, or inf itself
                if (a.act == RIPPLE_ACT_RELU) z = z > 0.0f ? z : 0.0f;
                if (BF) {
                    const __hip_bfloat16 zr = __float2bfloat16(z);
                    z = __bfloat162float(zr);
                    ((__hip_bfloat16 *)a.Hout)[hidx] = zr;
                } else {
                    ((float *)a.Hout)[hidx] = z;
                }
                if (a.D) a.D[hidx] = a.d_old ? old[u] : z - old[u];
            }
        }
        if (a.den) {
            uint32_t n_bad = 0;
#pragma unroll
            for (int u = 0; u < R; ++u) n_bad += __ballot(bad[u]) != 0ull ? 1u : 0u;
            if (n_bad && lane == 0) atomicAdd(a.range_rows, n_bad);
        }
    }
}

// The same for many rows, four columns per thread over the flattened (slot, group) space: rows of a narrow layer
// (47 columns) leave a quarter of a wavefront idle when a lane is a column, and consecutive slots are mostly consecutive vertices, so
// consecutive lanes read consecutive addresses across row ends. OLD: the stored row is read (a delta row is written); KIND 1: there is a
// cached self term, 2: attention (denominators; a row that is not finite is counted by the thread with its first such column).
// Bound by memory; with a number per thread it was bound by the two divisions and the three index reads of
// each: 2.4 M rows of 47 with a self term 411 -> 298 us (1.4 GB: 4.6 TB/s), 1 M of them scattered over the graph 203 -> 186, 2.4 M bf16
// rows 196 -> 178. (Four groups per round: 305, 186 and 186.) Attention, 300 updates on 31 M edges: rows of 47 columns 119 -> 64 us, of 256
// with rows of changes 119 -> 105; below three million numbers the row-by-row kernel takes 11 us and this one no less.
template <bool BF, bool OLD, int KIND>
__global__ __launch_bounds__(256) void k_transform_addend_flat(TArgs a) {
    constexpr int U = 2;                                   // groups per thread and round: their loads overlap
    const uint32_t count = *a.count_ptr, groups = (a.N + 3u) / 4u;
    const uint32_t total = count * groups;                 // < 2^32 (checked by the launch)
    const uint32_t stride = gridDim.x * blockDim.x, t0 = blockIdx.x * blockDim.x + threadIdx.x;
    if (t0 >= total) return;
    const uint32_t d_slot = stride / groups, d_g = stride - d_slot * groups;   // one division per thread: what a stride adds to slot and group
    uint32_t slot = t0 / groups, g = t0 - slot * groups;
    for (uint64_t e0 = t0; e0 < total; e0 += (uint64_t)stride * U) {
        uint32_t col[U], sl[U];
        size_t hidx[U];
        float sc[U], dn[U];
        floatx4 y[U], p[U], old[U];
        bool ok[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            ok[u] = e0 + (uint64_t)u * stride < total;
            sl[u] = ok[u] ? slot : count - 1u;             // past the end: the last row again, not stored
            col[u] = 4u * g;
            slot += d_slot;
            g += d_g;
            if (g >= groups) {
                g -= groups;
                ++slot;
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t v = a.list[sl[u]];
            hidx[u] = (size_t)v * a.N + col[u];
            if (KIND == 2) {                               // numerator / denominator, 0 without in-neighbours
                dn[u] = a.den[v];
                sc[u] = (a.in_meta[v].y > 0u && dn[u] > 0.0f) ? 1.0f / dn[u] : 0.0f;
            } else {
                const uint32_t deg = a.mean ? a.in_meta[v].y : 1u;
                sc[u] = 1.0f / (float)(deg > 1u ? deg : 1u);
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {                      // (up to three numbers past a row: the arrays have room behind them)
            y[u] = *(const floatx4u *)(a.addend + hidx[u]);
            p[u] = old[u] = (floatx4)(0.0f);
            if (KIND == 1) p[u] = *(const floatx4u *)(a.addend2 + hidx[u]);
            if (OLD && BF) {
                const uintx2u w = *(const uintx2u *)((const __hip_bfloat16 *)a.Hout + hidx[u]);
                old[u].x = __uint_as_float(w.x << 16);
                old[u].y = __uint_as_float(w.x & 0xFFFF0000u);
                old[u].z = __uint_as_float(w.y << 16);
                old[u].w = __uint_as_float(w.y & 0xFFFF0000u);
            } else if (OLD) {
                old[u] = *(const floatx4u *)((const float *)a.Hout + hidx[u]);
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (!ok[u]) continue;
            const uint32_t n = min(4u, a.N - col[u]);
            floatx4 z, dl;
            __hip_bfloat16 zr[4];
            bool bad = KIND == 2 && !isfinite(dn[u]);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const float b = a.bias[min(col[u] + (uint32_t)k, a.N - 1u)];
                float t = y[u][k] * sc[u] + b + p[u][k];
                if (KIND == 2) bad |= (uint32_t)k < n && !isfinite(t);
                if (a.act == RIPPLE_ACT_RELU) t = t > 0.0f ? t : 0.0f;
                if (BF) {
                    zr[k] = __float2bfloat16(t);
                    t = __bfloat162float(zr[k]);
                }
                z[k] = t;
                dl[k] = a.d_old ? old[u][k] : t - old[u][k];
            }
            if (KIND == 2 && __builtin_expect(bad, 0)) {
                bool first = col[u] == 0u || isfinite(dn[u]);
                const float *row = a.addend + (hidx[u] - col[u]);
                for (uint32_t k = 0; k < col[u] && first; ++k) first = isfinite(row[k] * sc[u] + a.bias[k]);
                if (first) atomicAdd(a.range_rows, 1u);
            }
            if (n == 4u) {
                if (BF) {
                    uintx2u w;
                    w.x = __float_as_uint(z.x) >> 16 | (__float_as_uint(z.y) & 0xFFFF0000u);
                    w.y = __float_as_uint(z.z) >> 16 | (__float_as_uint(z.w) & 0xFFFF0000u);
                    *(uintx2u *)((__hip_bfloat16 *)a.Hout + hidx[u]) = w;
                } else {
                    *(floatx4u *)((float *)a.Hout + hidx[u]) = z;
                }
                if (OLD) *(floatx4u *)(a.D + hidx[u]) = dl;
            } else {
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    if ((uint32_t)k >= n) continue;
                    if (BF) ((__hip_bfloat16 *)a.Hout)[hidx[u] + k] = zr[k];
                    else ((float *)a.Hout)[hidx[u] + k] = z[k];
                    if (OLD) a.D[hidx[u] + k] = dl[k];
                }
            }
        }
    }
}

// Small hops of a project-first layer: the row update, and (the workgroups from nb on) T brought up to date with the messages
// that push_edges<.., 2> has sent: T += m, element by element as rp_message made it.
__global__ __launch_bounds__(256) void k_small_addend(TArgs a, uint32_t nb, const uint32_t *src_list, const uint32_t *src_count,
                                                      const float *PD, uint32_t ldd, float *T, uint32_t ldt, int packed) {
    if (blockIdx.x < nb) {
        if (a.store) addend_only_rows<true>(a, blockIdx.x * 4u + (threadIdx.x >> 6), nb * 4u);
        else addend_only_rows<false>(a, blockIdx.x * 4u + (threadIdx.x >> 6), nb * 4u);
        return;
    }
    const uint32_t count = *src_count, lane = threadIdx.x & 63u, nw = (gridDim.x - nb) * 4u;
    for (uint32_t i = (blockIdx.x - nb) * 4u + (threadIdx.x >> 6); i < count; i += nw) {
        const uint32_t u = src_list[i];
        for (uint32_t c0 = 0; c0 < a.N; c0 += 64u) {
            const uint32_t col = c0 + lane;
            const float p = col < a.N ? PD[(size_t)u * ldd + col] : 0.0f, t = col < a.N ? T[(size_t)u * ldt + col] : 0.0f;
            const float m = rp_message(p - t, packed != 0);
            if (col < a.N) T[(size_t)u * ldt + col] = packed ? t + m : p;
        }
    }
}

void rp_launch_small_addend(ripple_ctx *c, uint32_t l, bool emit_delta) {
    const LayerDev &ly = c->layers[l - 1];
    TArgs a = base_args(c, l, c->list[l], &c->ctr->set[l].a);
    a.D = emit_delta ? c->D[l & 1] : nullptr;
    a.d_old = rp_layer_mono(c, l + 1) ? 1 : 0;
    a.addend = c->X[l];
    a.act = (int)ly.act_out;
    a.addend2 = ly.selfc ? ly.PS : nullptr;
    const uint32_t nb = std::min(rp_div_up(c->last_a[l] + c->last_a[l] / 2u + 32u, 32), c->n_cu * 8);
    const uint32_t nt = std::min(rp_div_up(c->last_a[l - 1] + c->last_a[l - 1] / 2u + 4u, 4), c->n_cu * 4);
    hipLaunchKernelGGL(k_small_addend, dim3(nb + nt), dim3(256), 0, c->stream, a, nb, c->list[l - 1], &c->ctr->set[l - 1].a, c->PD, c->pd_ld,
                       ly.T, ly.ldt, (int)ly.packed);
}

// Many rows: every lane busy, whatever the row width. (Fewer: the launch is what counts.)
static bool launch_addend_flat(ripple_ctx *c, const TArgs &a, uint32_t rows_hint) {
    if ((uint64_t)c->n_cap * a.N >= (1ull << 32) || (rows_hint < 65536u && (uint64_t)rows_hint * a.N < (3u << 20))) return false;
    const dim3 grid(c->n_cu * 16), block(256);
#define RP_FLAT(BF, OLD)                                                                                            \
    do {                                                                                                            \
        if (a.den) hipLaunchKernelGGL((k_transform_addend_flat<BF, OLD, 2>), grid, block, 0, c->stream, a);         \
        else if (a.addend2) hipLaunchKernelGGL((k_transform_addend_flat<BF, OLD, 1>), grid, block, 0, c->stream, a);\
        else hipLaunchKernelGGL((k_transform_addend_flat<BF, OLD, 0>), grid, block, 0, c->stream, a);               \
    } while (0)
    if (a.store && a.D) RP_FLAT(true, true);
    else if (a.store) RP_FLAT(true, false);
    else if (a.D) RP_FLAT(false, true);
    else RP_FLAT(false, false);
#undef RP_FLAT
    return true;
}

__global__ __launch_bounds__(256) void k_transform_addend_only(TArgs a) {
    const uint32_t gw = (blockIdx.x * blockDim.x + threadIdx.x) >> 6, nw = (gridDim.x * blockDim.x) >> 6;
    if (a.store) addend_only_rows<true>(a, gw, nw);
    else addend_only_rows<false>(a, gw, nw);
}

// [h_self | x] rows whose halves are not multiples of four columns wide (a group of four would straddle them; only layers
// that concatenate and do not cache their self term get here): same tiling, scalar gathers, no prefetch.
__device__ __forceinline__ float load_a1(const TArgs &a, uint32_t v, float scale, uint32_t k) {
    if (k >= a.K) return 0.0f;
    return (k < a.d_in) ? rp_load_h(a.Hprev, a.store, (size_t)v * a.d_in + k) : a.X[(size_t)v * a.d_in + (k - a.d_in)] * scale;
}

template <int WAVES_M, int WAVES_N>
__global__ __launch_bounds__(256) void k_transform_generic(TArgs a) {
    constexpr int TM = 2, TN = 2;
    constexpr int BM = WAVES_M * 64, BN = WAVES_N * 64;
    __shared__ float As[BM][T_BK + 1];
    __shared__ float Bs[T_BK][BN];
    __shared__ uint32_t s_vtx[BM];
    __shared__ float s_scale[BM];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave / WAVES_N, wn = wave % WAVES_N;
    const uint32_t count = *a.count_ptr;
    const uint32_t n_tiles = (count + BM - 1) / BM;
    const uint32_t n0 = blockIdx.y * BN;
    for (uint32_t tile = blockIdx.x; tile < n_tiles; tile += gridDim.x) {
        const uint32_t row0 = tile * BM;
        __syncthreads();
        for (int r = tid; r < BM; r += 256) {
            uint32_t slot = row0 + r;
            uint32_t v = 0;
            float sc = 1.0f;
            if (slot < count) {
                v = a.list[slot];
                if (a.mean) {
                    uint32_t deg = a.in_meta[v].y;
                    sc = 1.0f / (float)(deg > 1u ? deg : 1u);
                }
            }
            s_vtx[r] = v;
            s_scale[r] = sc;
        }
        __syncthreads();
        floatx16 acc[TM][TN];
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;
        for (uint32_t k0 = 0; k0 < a.Kpad; k0 += T_BK) {
            for (int idx = tid; idx < BM * T_BK; idx += 256) {
                const int r = idx / T_BK, k = idx % T_BK;
                const uint32_t slot = row0 + r;
                As[r][k] = (slot < count) ? load_a1(a, s_vtx[r], s_scale[r], k0 + k) : 0.0f;
            }
            for (int idx = tid; idx < T_BK * (BN / 4); idx += 256) {
                const int kr = idx / (BN / 4), c4 = (idx % (BN / 4)) * 4;
                *(float4 *)&Bs[kr][c4] = *(const float4 *)(a.W + (size_t)(k0 + kr) * a.Npad + n0 + c4);
            }
            __syncthreads();
#pragma unroll
            for (int kk = 0; kk < T_BK; kk += 2) {
                const int kq = kk + (lane >> 5);
                float av[TM], bv[TN];
#pragma unroll
                for (int i = 0; i < TM; ++i) av[i] = As[(wm * TM + i) * 32 + (lane & 31)][kq];
#pragma unroll
                for (int j = 0; j < TN; ++j) bv[j] = Bs[kq][(wn * TN + j) * 32 + (lane & 31)];
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[i], bv[j], acc[i][j], 0, 0, 0);
            }
            __syncthreads();
        }
        epilogue<TM, TN>(a, acc, s_vtx, s_scale, row0, count, n0, wm, wn, lane);
    }
}

// ---------------------------------------------------------------------------------
// bf16 matrix-core variant (embeddings stored in bfloat16): MFMA 32x32x16 bf16 with fp32
// accumulation. Same tiling, prefetch and epilogue; the gathered rows are rounded to bf16 when
// they are written to LDS, the weights come from a transposed bf16 copy so that the eight
// consecutive k a lane feeds into one MFMA are one 16-byte LDS read for both operands.
// ---------------------------------------------------------------------------------
#define TB_LD 40                                            // LDS row stride in bf16 (80 bytes)

template <int WAVES_M, int WAVES_N, int TM, int TN, int STAGES, int MODE>
__global__ __launch_bounds__(256, 2) void k_transform_bf16(TArgs a) {
    constexpr int STORE = 1;
    constexpr int BM = WAVES_M * TM * 32, BN = WAVES_N * TN * 32;
    constexpr int NA = BM / 32, NB = BN / 64;              // per thread per slice: float4 of A, 16-byte chunks of B
    constexpr bool TWO = (MODE == 2) || (MODE == 1);
    constexpr int A_BYTES = BM * TB_LD * 2, B_BYTES = BN * TB_LD * 2, C_BYTES = BM * (BN + 4) * 4;
    constexpr int S_BYTES = (A_BYTES + B_BYTES > C_BYTES) ? A_BYTES + B_BYTES : C_BYTES;
    static_assert(A_BYTES % 16 == 0, "alignment of the weight slice");
    __shared__ __attribute__((aligned(16))) char smem[S_BYTES];   // A and B slices; reused by the staged epilogue
    unsigned short (*As)[TB_LD] = (unsigned short (*)[TB_LD]) smem;
    unsigned short (*Bs)[TB_LD] = (unsigned short (*)[TB_LD])(smem + A_BYTES);
    __shared__ uint32_t s_vtx[BM];
    __shared__ float s_scale[BM];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave / WAVES_N, wn = wave % WAVES_N;
    const uint32_t count = *a.count_ptr;
    const uint32_t n_tiles = (count + BM - 1) / BM;
    const uint32_t n0 = blockIdx.y * BN;

    for (uint32_t tile = blockIdx.x; tile < n_tiles; tile += gridDim.x) {
        const uint32_t row0 = tile * BM;
        __syncthreads();
        for (int r = tid; r < BM; r += 256) {
            uint32_t slot = row0 + r;
            uint32_t v = 0;
            float sc = 1.0f;
            if (slot < count) {
                v = a.list[slot];
                if (a.mean) {
                    uint32_t deg = a.in_meta[v].y;
                    sc = 1.0f / (float)(deg > 1u ? deg : 1u);
                }
            }
            s_vtx[r] = v;
            s_scale[r] = sc;
        }
        __syncthreads();

        floatx16 acc[TM][TN];
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

        uint32_t my_v[NA], my_slot[NA];
#pragma unroll
        for (int i = 0; i < NA; ++i) {
            const int r = (tid + i * 256) / (T_BK / 4);
            my_v[i] = s_vtx[r];
            my_slot[i] = min(row0 + r, count - 1u);
        }
        const uint32_t c4a = (tid % (T_BK / 4)) * 4;

        floatx4 ra[STAGES][NA], rq[TWO ? STAGES : 1][TWO ? NA : 1];
        uintx4 rb[NB];
#pragma unroll
        for (int i = 0; i < NB; ++i) {                     // weights first, as in every step of the loop
            const int idx = tid + i * 256;
            const int n = idx / 4, kc = (idx % 4) * 8;
            rb[i] = *(const uintx4 *)(a.Wt + (size_t)(n0 + n) * a.wt_ld + kc);
        }
#pragma unroll
        for (int st = 0; st < STAGES; ++st)
#pragma unroll
            for (int i = 0; i < NA; ++i) {
                floatx4 q = (floatx4)(0.0f);
                fetch_raw<MODE, STORE>(a, my_v[i], my_slot[i], (uint32_t)st * T_BK + c4a, ra[st][i], q);
                if constexpr (TWO) rq[st][i] = q;
            }
        __builtin_amdgcn_sched_barrier(0);

        for (uint32_t kbase = 0; kbase < a.Kpad; kbase += STAGES * T_BK) {    // staging registers rotate by unrolling
#pragma unroll
          for (int s = 0; s < STAGES; ++s) {
            const uint32_t k0 = kbase + s * T_BK;
            if (k0 >= a.Kpad) break;
            __syncthreads();
#pragma unroll
            for (int i = 0; i < NA; ++i) {
                const int r = (tid + i * 256) / (T_BK / 4);
                floatx4 q = (floatx4)(0.0f);
                if constexpr (TWO) q = rq[s][i];
                const floatx4 val = finish_raw<MODE, STORE>(a, ra[s][i], q, k0 + c4a, s_scale[r]);
                uint2 pk;
                pk.x = pack_bf16x2(val.x, val.y);
                pk.y = pack_bf16x2(val.z, val.w);
                *(uint2 *)&As[r][c4a] = pk;
            }
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                const int idx = tid + i * 256;
                const int n = idx / 4, kc = (idx % 4) * 8;
                *(uintx4 *)&Bs[n][kc] = rb[i];
            }
            __syncthreads();
            {
                const uint32_t kb = min(k0 + T_BK, a.Kpad - T_BK);
#pragma unroll
                for (int i = 0; i < NB; ++i) {
                    const int idx = tid + i * 256;
                    const int n = idx / 4, kc = (idx % 4) * 8;
                    rb[i] = *(const uintx4 *)(a.Wt + (size_t)(n0 + n) * a.wt_ld + kb + kc);
                }
            }
            {
                const uint32_t kn = k0 + STAGES * T_BK + c4a;
#pragma unroll
                for (int i = 0; i < NA; ++i) {
                    floatx4 q = (floatx4)(0.0f);
                    fetch_raw<MODE, STORE>(a, my_v[i], my_slot[i], kn, ra[s][i], q);
                    if constexpr (TWO) rq[s][i] = q;
                }
            }
            __builtin_amdgcn_sched_barrier(0);             // requests stay above the matrix-core work
#pragma unroll
            for (int kh = 0; kh < 2; ++kh) {
                const int ko = kh * 16 + (lane >> 5) * 8;
                bf16x8 av[TM], bv[TN];
#pragma unroll
                for (int i = 0; i < TM; ++i)
                    av[i] = __builtin_bit_cast(bf16x8, *(const uintx4 *)&As[(wm * TM + i) * 32 + (lane & 31)][ko]);
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    bv[j] = __builtin_bit_cast(bf16x8, *(const uintx4 *)&Bs[(wn * TN + j) * 32 + (lane & 31)][ko]);
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[i], bv[j], acc[i][j], 0, 0, 0);
            }
          }
        }
        epilogue_staged<TM, TN, BM, BN, true>(a, acc, (float *)smem, s_vtx, s_scale, row0, count, n0, wm, wn, tid);
    }
}

// The grid holds about one workgroup per expected tile (a grid-stride loop covers any excess):
// workgroups that start at different times do not all sit in their memory phase at once, which a
// grid of resident, persistent workgroups does.
static uint32_t tile_grid(const ripple_ctx *c, uint32_t rows_hint, uint32_t bm, uint32_t floor_wg) {
    const uint64_t want = ((uint64_t)rows_hint + rows_hint / 4) / bm + 1;
    const uint64_t cap = (uint64_t)c->n_cap / bm + 1;
    return (uint32_t)std::max<uint64_t>(floor_wg, std::min(want, cap));
}

// tiles of 64 x 256 (128 x 128) where there are enough for every compute unit to have several, small ones below
template <int MODE>
static void launch_bf16(ripple_ctx *c, const TArgs &a, uint32_t rows_hint) {
    const bool many = rows_hint >= 64u * 4u * c->n_cu;
    if (a.Npad >= 256 && many) {
        hipLaunchKernelGGL((k_transform_bf16<1, 4, 2, 2, 3, MODE>), dim3(tile_grid(c, rows_hint, 64, c->n_cu * 2), a.Npad / 256),
                           dim3(256), 0, c->stream, a);
    } else if (a.Npad == 128 && many) {
        hipLaunchKernelGGL((k_transform_bf16<2, 2, 2, 2, 3, MODE>), dim3(tile_grid(c, rows_hint, 128, c->n_cu * 2), 1), dim3(256), 0,
                           c->stream, a);
    } else if (a.Npad % 128 == 0) {
        hipLaunchKernelGGL((k_transform_bf16<1, 4, 1, 1, 3, MODE>), dim3(tile_grid(c, rows_hint, 32, c->n_cu * 2), a.Npad / 128), dim3(256), 0,
                           c->stream, a);
    } else {
        hipLaunchKernelGGL((k_transform_bf16<2, 2, 1, 1, 3, MODE>), dim3(tile_grid(c, rows_hint, 64, c->n_cu * 2), a.Npad / 64), dim3(256), 0,
                           c->stream, a);
    }
}

// Some thousand rows: fp32 numbers as three bf16 parts on the bf16 matrix cores (see k_split_stream: six products, the small terms summed
// apart, closer to 64-bit sums than fp32 products; sums that are not finite are made again from fp32 products). Tiles of 32 x 128, or
// 64 x 64 where the matrix is 64 columns wide, a wavefront 32 x 32 of them; the rows pass through LDS, split as they are written there, the
// weights come from the L2 in the order in which the matrix cores take them. What bounds it is the chain of slices (LDS, barrier,
// products) and the workgroups that share a compute unit's matrix cores: six bf16 products take 3/8 of the fp32 products' time.
// 256 -> 256 against the same tiles of fp32 products (launch included): 10 K rows with a cached row 20.6 -> 15.8 us, 35 K rows 40 -> 31 (23 for
// the bytes alone), without it 18.4 -> 12.7 and 22 -> 16.8; both products of an MLP on 10 K rows 37 -> 31 and 26 -> 18.
// Three workgroups per compute unit where a row number comes from one place; those that add two up hold both for four slices, and with the
// registers of a third workgroup 15 of them were spilled: two workgroups.
template <int WAVES_M, int WAVES_N, int STAGES, int MODE, int STORE>
__global__ __launch_bounds__(256, (WAVES_N == 4 && MODE != 2 && !(MODE == 1 && STORE) ? 3 : 2)) void k_transform_split(TArgs a) {
    constexpr int BM = WAVES_M * 32, BN = WAVES_N * 32;
    constexpr int NA = BM / 32;                            // groups of four numbers per thread and slice
    constexpr bool TWO = (MODE == 2) || (MODE == 1 && STORE == 1);
    constexpr int PL = STORE && MODE == 4 ? 1 : 3;         // parts of a row number (bf16 rows are exact as they are)
    constexpr int A_BYTES = 2 * PL * BM * TB_LD * 2, C_BYTES = BM * (BN + 4) * 4;
    __shared__ __attribute__((aligned(16))) char smem[A_BYTES > C_BYTES ? A_BYTES : C_BYTES];   // two slices of rows; reused by the staged epilogue
    typedef unsigned short (*slice_t)[BM][TB_LD];
    slice_t As[2] = {(slice_t)smem, (slice_t)(smem + A_BYTES / 2)};
    __shared__ uint32_t s_vtx[BM];
    __shared__ float s_scale[BM];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave / WAVES_N, wn = wave % WAVES_N;
    const uint32_t count = *a.count_ptr;
    const uint32_t n_tiles = (count + BM - 1) / BM;
    const uint32_t n0 = blockIdx.y * BN, col = n0 + wn * 32 + (lane & 31);
    const uintx4 *Wp = (const uintx4 *)a.Wp + (size_t)(lane >> 5) * a.Npad + col;    // eight k of the lane's column
    const size_t part = (size_t)(a.wp_k / 8u) * a.Npad, step = 2u * a.Npad;
    const float down = 1.0f / ((PL == 3 ? PARTS_LIFT : 1.0f) * a.wp_lift);   // (see PARTS_LIFT)

    for (uint32_t tile = blockIdx.x; tile < n_tiles; tile += gridDim.x) {
        const uint32_t row0 = tile * BM;
        __syncthreads();                                   // previous tile's epilogue has read s_vtx
        for (int r = tid; r < BM; r += 256) {
            const uint32_t v = a.list[min(row0 + r, count - 1u)];   // rows past the end repeat the last one and are never stored
            float sc = 1.0f;
            if (a.mean) {
                const uint32_t deg = a.in_meta[v].y;
                sc = 1.0f / (float)(deg > 1u ? deg : 1u);
            }
            s_vtx[r] = v;
            s_scale[r] = sc;
        }
        __syncthreads();
        uint32_t my_v[NA], my_slot[NA];
#pragma unroll
        for (int i = 0; i < NA; ++i) {
            const int r = (tid + i * 256) / (T_BK / 4);
            my_v[i] = s_vtx[r];
            my_slot[i] = min(row0 + r, count - 1u);
        }
        const uint32_t c4a = (tid % (T_BK / 4)) * 4;
        floatx4 ra[STAGES][NA], rq[TWO ? STAGES : 1][TWO ? NA : 1];
        uintx4 bq[2][3];                                   // weights of step g (16 k) in bq[g & 1]
        auto load_w = [&](uint32_t g) {
            const uint32_t at = min(g, a.Kpad / 16u - 1u); // past the end: the last step once more, not used
#pragma unroll
            for (int p = 0; p < 3; ++p) bq[g & 1][p] = Wp[p * part + at * step];
        };
        load_w(0);
        load_w(1);
#pragma unroll
        for (int st = 0; st < STAGES; ++st)
#pragma unroll
            for (int i = 0; i < NA; ++i) {
                floatx4 q = (floatx4)(0.0f);
                fetch_raw<MODE, STORE>(a, my_v[i], my_slot[i], (uint32_t)st * T_BK + c4a, ra[st][i], q);
                if constexpr (TWO) rq[st][i] = q;
            }
        __builtin_amdgcn_sched_barrier(0);
        floatx16 acc[1][1], cor;
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[0][0][r] = cor[r] = 0.0f;
        for (uint32_t kbase = 0; kbase < a.Kpad; kbase += STAGES * T_BK) {    // staging registers rotate by unrolling
#pragma unroll
          for (int s = 0; s < STAGES; ++s) {
            const uint32_t k0 = kbase + s * T_BK;
            if (k0 >= a.Kpad) break;
            static_assert(STAGES % 2 == 0, "the LDS buffers alternate");
#pragma unroll
            for (int i = 0; i < NA; ++i) {
                const int r = (tid + i * 256) / (T_BK / 4);
                floatx4 q = (floatx4)(0.0f);
                if constexpr (TWO) q = rq[s][i];
                uintx2 parts[PL];
                const floatx4 x = finish_raw<MODE, STORE>(a, ra[s][i], q, k0 + c4a, s_scale[r]);
                split_parts<PL>(PL == 3 ? x * PARTS_LIFT : x, parts);
#pragma unroll
                for (int p = 0; p < PL; ++p) *(uintx2 *)&As[s & 1][p][r][c4a] = parts[p];
            }
            __syncthreads();                               // (one per slice: the other buffer was read before the last one)
#pragma unroll
            for (int i = 0; i < NA; ++i) {                 // rows of the slice STAGES steps ahead (clamped: harmless past the end)
                floatx4 q = (floatx4)(0.0f);
                fetch_raw<MODE, STORE>(a, my_v[i], my_slot[i], k0 + STAGES * T_BK + c4a, ra[s][i], q);
                if constexpr (TWO) rq[s][i] = q;
            }
            __builtin_amdgcn_sched_barrier(0);             // requests stay above the matrix-core work
            bf16x8 av[2][PL];
#pragma unroll
            for (int kk = 0; kk < 2; ++kk)
#pragma unroll
                for (int p = 0; p < PL; ++p) av[kk][p] = __builtin_bit_cast(bf16x8, *(const uintx4 *)&As[s & 1][p][wm * 32 + (lane & 31)][kk * 16 + (lane >> 5) * 8]);
#pragma unroll
            for (int kk = 0; kk < 2; ++kk) {
#define TERM(dst, x, w) dst = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[kk][x], __builtin_bit_cast(bf16x8, bq[kk][w]), dst, 0, 0, 0)
                TERM(cor, 0, 2);
                TERM(acc[0][0], 0, 0);
                if constexpr (PL == 3) {
                    TERM(cor, 2, 0);
                    TERM(cor, 1, 1);
                    TERM(cor, 1, 0);
                }
                TERM(cor, 0, 1);
#undef TERM
                load_w(k0 / 16u + kk + 2u);
            }
          }
        }
        bool bad = false;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            acc[0][0][r] = (acc[0][0][r] + cor[r]) * down;
            bad |= !__builtin_isfinite(acc[0][0][r]);
        }
        if (__builtin_expect(__any(bad && col < a.N), 0)) {
            const uint32_t lr = wm * 32 + (lane & 31);
            const floatx16 sum = fp32_block<MODE, STORE>(a, min(row0 + lr, count - 1u), s_vtx[lr], s_scale[lr], col, lane);
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[0][0][r] = __builtin_isfinite(acc[0][0][r]) ? acc[0][0][r] : sum[r];
        }
        epilogue_staged<1, 1, BM, BN, STORE != 0>(a, acc, (float *)smem, s_vtx, s_scale, row0, count, n0, wm, wn, tid);
    }
}

template <int MODE, int STORE>
__global__ __launch_bounds__(256) void k_transform_wave(TArgs a) {
    wave_gemm<MODE, STORE>(a, (blockIdx.x * 256u + threadIdx.x) >> 6, gridDim.x * 4u);
}

// Few rows: a product per wavefront (wave_gemm); more: tiles. Every matrix has its parts (wp_k >= Kpad: no read leaves them).
template <int MODE, int STORE>
static void launch_fast(ripple_ctx *c, const TArgs &a, uint32_t rows_hint) {
    if constexpr (MODE != 2) {                             // (never pays)
        if (!c->opt_split && wave_gemm_pays(a, rows_hint)) {
            // wavefronts for half as many rows again as expected; a set that turns out larger still finds every SIMD busy
            const uint32_t waves = std::max(wave_gemm_waves(a, rows_hint + rows_hint / 2u), c->n_cu * 4);
            hipLaunchKernelGGL((k_transform_wave<MODE, STORE>), dim3(rp_div_up(waves, 4)), dim3(256), 0, c->stream, a);
            return;
        }
    }
    if (a.Npad % 128 == 0) {
        hipLaunchKernelGGL((k_transform_split<1, 4, 4, MODE, STORE>), dim3(tile_grid(c, rows_hint, 32, c->n_cu * 2), a.Npad / 128), dim3(256), 0, c->stream, a);
    } else {
        hipLaunchKernelGGL((k_transform_split<2, 2, 4, MODE, STORE>), dim3(tile_grid(c, rows_hint, 64, c->n_cu * 2), a.Npad / 64), dim3(256), 0, c->stream, a);
    }
}

static void launch_t(ripple_ctx *c, const TArgs &a, uint32_t rows_hint) {
    if (rp_launch_stream(c, a, rows_hint)) return;
    const uint32_t gx = c->n_cu * 2;
    if (a.a_mode == 1 && (a.d_in & 3u)) {
        if (a.Npad >= 256) hipLaunchKernelGGL((k_transform_generic<1, 4>), dim3(gx, a.Npad / 256), dim3(256), 0, c->stream, a);
        else if (a.Npad == 128) hipLaunchKernelGGL((k_transform_generic<2, 2>), dim3(gx, 1), dim3(256), 0, c->stream, a);
        else hipLaunchKernelGGL((k_transform_generic<4, 1>), dim3(gx, 1), dim3(256), 0, c->stream, a);
        return;
    }
#define T_CASE(M)                                            \
    case M:                                                  \
        if (a.store && a.Wt) launch_bf16<M>(c, a, rows_hint);           \
        else if (a.store) launch_fast<M, 1>(c, a, rows_hint);   \
        else launch_fast<M, 0>(c, a, rows_hint);                \
        break;
    switch (a.a_mode) {
        T_CASE(0)
        T_CASE(1)
        T_CASE(2)
        T_CASE(4)
    default:
        if (a.store) launch_fast<3, 1>(c, a, rows_hint);   // compact fp32 rows; the storage type only shapes the epilogue
        else launch_fast<3, 0>(c, a, rows_hint);
        break;
    }
#undef T_CASE
}

// Project-first layers: P[v] = H^{l-1}[v] W_neigh for the listed vertices, no bias, no activation.
//   bootstrap: into the layer's T (what every vertex has sent: the aggregates are then summed from it)
//   otherwise: into c->PD, from where rp_launch_messages turns the rows into this hop's messages
TArgs rp_project_args(ripple_ctx *c, uint32_t l, const uint32_t *list, const uint32_t *count_d, bool bootstrap) {
    const LayerDev &ly = c->layers[l - 1];
    TArgs a = base_args(c, l, list, count_d);
    a.mean = 0;
    a.W = ly.Wn;
    a.Wq = ly.Wnq;
    a.Wt = nullptr;                                // messages are differences of such products: fp32 weights (in parts) also for bf16 rows
    a.Wp = ly.Wnp;
    a.wp_k = rp_round_up(ly.d_in, 128);
    a.bias = ly.bzero;
    a.K = ly.d_in;
    a.Kpad = rp_round_up(ly.d_in, 32);
    a.act = RIPPLE_ACT_NONE;
    a.tmp_out = bootstrap ? ly.T : c->PD;
    a.tmp_out_ld = bootstrap ? ly.ldt : c->pd_ld;
    a.Hout = nullptr;
    a.out_mode = 2;
    a.a_mode = 4;
    return a;
}

void rp_launch_project(ripple_ctx *c, uint32_t l, const uint32_t *list, const uint32_t *count_d, bool bootstrap) {
    launch_t(c, rp_project_args(c, l, list, count_d, bootstrap), bootstrap ? c->n_cap : rp_rows_guess(c, l - 1));
}

// Layers handled project-first that also cache their self term: both products of H^{l-1}[v], with W_self (into PS)
// and with W_neigh (into T at the bootstrap, else into c->PD), from one pass over the rows, against the
// layer's combined weight matrix [W_self | W_neigh] (second block from column 64 on).
bool rp_has_project_both(const ripple_ctx *c, uint32_t l) { return c->layers[l - 1].Wc != nullptr; }

TArgs rp_project_both_args(ripple_ctx *c, uint32_t l, const uint32_t *list, const uint32_t *count_d, bool bootstrap) {
    const LayerDev &ly = c->layers[l - 1];
    TArgs a = base_args(c, l, list, count_d);
    a.mean = 0;
    a.W = ly.Wc;
    a.Wq = ly.Wcq;
    a.Wt = nullptr;
    a.Wp = ly.Wcp;
    a.wp_k = rp_round_up(ly.d_in, 128);
    a.bias = ly.bzero_c;
    a.K = ly.d_in;
    a.Kpad = rp_round_up(ly.d_in, 32);
    a.N = 64 + ly.d_out;
    a.Npad = 128;
    a.act = RIPPLE_ACT_NONE;
    a.a_mode = 4;
    a.out_mode = 2;
    a.Hout = nullptr;
    a.tmp_out = ly.PS;
    a.tmp_out_ld = ly.d_out;
    a.split_col = 64;
    a.N1 = ly.d_out;
    a.tmp_out2 = bootstrap ? ly.T : c->PD;
    a.tmp_out2_ld = bootstrap ? ly.ldt : c->pd_ld;
    return a;
}

void rp_launch_project_both(ripple_ctx *c, uint32_t l, const uint32_t *list, const uint32_t *count_d, bool bootstrap) {
    TArgs a = rp_project_both_args(c, l, list, count_d, bootstrap);
    launch_t(c, a, bootstrap ? c->n_cap : rp_rows_guess(c, l - 1));
}

// Attention layer l: P[v] = H^{l-1}[v] W0 for the listed vertices (fp32, no bias, no activation).
void rp_launch_gat_project(ripple_ctx *c, uint32_t l, const uint32_t *list, const uint32_t *count_d) {
    const LayerDev &ly = c->layers[l - 1];
    TArgs a = base_args(c, l, list, count_d);
    a.mean = 0;
    a.Wt = nullptr;
    a.bias = ly.bzero;
    a.act = RIPPLE_ACT_NONE;
    a.a_mode = 4;
    a.out_mode = 2;
    a.tmp_out = ly.P;
    a.tmp_out_ld = ly.ldp;
    a.Hout = nullptr;
    launch_t(c, a, (list == c->all_list) ? c->n_cap : rp_rows_guess(c, l - 1));
}

// Cached self term of layer l: PS[v] = H^{l-1}[v] W_self for the listed vertices (fp32, no bias).
TArgs rp_self_project_args(ripple_ctx *c, uint32_t l, const uint32_t *list, const uint32_t *count_d) {
    const LayerDev &ly = c->layers[l - 1];
    TArgs a = base_args(c, l, list, count_d);
    a.mean = 0;
    a.W = ly.W0;                                   // W_self: the first d_in rows (the kernel zeroes k >= K)
    a.Wq = ly.W0q;
    a.Wt = nullptr;
    a.bias = ly.bzero;
    a.K = ly.d_in;
    a.Kpad = rp_round_up(ly.d_in, 32);
    a.act = RIPPLE_ACT_NONE;
    a.a_mode = 4;
    a.out_mode = 2;
    a.tmp_out = ly.PS;
    a.tmp_out_ld = ly.d_out;
    a.Hout = nullptr;
    return a;
}

void rp_launch_self_project(ripple_ctx *c, uint32_t l, const uint32_t *list, const uint32_t *count_d) {
    launch_t(c, rp_self_project_args(c, l, list, count_d), (list == c->all_list) ? c->n_cap : rp_rows_guess(c, l - 1));
}

// Re-apply layer l (1-based) to the vertices in `list` (count on the device).
// emit_delta: write D^l (into the ping-pong buffer of parity l) for the next hop.
void rp_launch_transform(ripple_ctx *c, uint32_t l, const uint32_t *list, const uint32_t *count_d, bool emit_delta) {
    const LayerDev &ly = c->layers[l - 1];
    TArgs a = base_args(c, l, list, count_d);
    a.D = emit_delta ? c->D[l & 1] : nullptr;
    a.d_old = rp_layer_mono(c, l + 1) ? 1 : 0;
    a.a_mode = (ly.self_mode == RIPPLE_SELF_NONE) ? 0 : (ly.self_mode == RIPPLE_SELF_CONCAT ? 1 : 2);
    // expected row count: the previous batch's (bootstrap passes the list of all live vertices)
    const uint32_t hint = (list == c->all_list) ? c->n_cap : rp_rows_guess(c, l);
    if (ly.agg == RIPPLE_AGG_ATTN) {             // h = act(numerator / denominator + b): no product left per row
        a.addend = c->X[l];
        a.den = ly.den;
        a.act = (int)ly.act_out;
        if (!launch_addend_flat(c, a, hint)) hipLaunchKernelGGL(k_transform_addend_only, dim3(c->n_cu * 8), dim3(256), 0, c->stream, a);
        return;
    }
    if (ly.proj) {                               // aggregate already multiplied by W_neigh: add it in the epilogue
        a.addend = c->X[l];
        a.act = (int)ly.act_out;
        if (ly.self_mode == RIPPLE_SELF_NONE || ly.selfc) {
            a.addend2 = ly.selfc ? ly.PS : nullptr;
            if (!launch_addend_flat(c, a, hint)) hipLaunchKernelGGL(k_transform_addend_only, dim3(c->n_cu * 8), dim3(256), 0, c->stream, a);
            return;
        }
        a.a_mode = 4;                            // h_self * W_self: the first d_in rows of W0
        a.K = ly.d_in;
        a.Kpad = rp_round_up(ly.d_in, 32);
        launch_t(c, a, hint);
        return;
    }
    if (ly.selfc) {                              // act((x * scale) W_neigh + PS[v] + b)
        a.a_mode = 0;
        a.W = ly.Wn;
        a.Wq = ly.Wnq;
        a.Wt = nullptr;
        a.Wp = ly.Wnp;
        a.wp_k = rp_round_up(ly.d_in, 128);
        a.K = ly.d_in;
        a.Kpad = rp_round_up(ly.d_in, 32);
        a.addend = ly.PS;
        a.addend_scaled = 0;
        a.act = (int)ly.act_out;
        launch_t(c, a, hint);
        return;
    }
    if (ly.d_hidden == 0) {
        a.act = (int)ly.act_out;
        launch_t(c, a, hint);
        return;
    }
    // two-stage update: hidden = act_inner(row W0 + b0) -> tmp, then h = act_out(hidden W1 + b1)
    TArgs s1 = a;
    s1.N = ly.d_hidden;
    s1.act = (int)ly.act_inner;
    s1.out_mode = 0;
    s1.tmp_out = c->tmp;
    s1.tmp_out_ld = ly.d_hidden;
    s1.Hout = nullptr;
    s1.D = nullptr;
    launch_t(c, s1, hint);
    TArgs s2 = a;
    s2.a_mode = 3;
    s2.tmp_in = c->tmp;
    s2.tmp_ld = ly.d_hidden;
    s2.mean = 0;
    s2.W = ly.W1;
    s2.Wq = ly.W1q;
    s2.Wt = nullptr;
    s2.Wp = ly.W1p;
    s2.wp_k = rp_round_up(ly.d_hidden, 128);
    s2.wp_lift = ly.lift1;
    s2.bias = ly.b1;
    s2.K = ly.d_hidden;
    s2.Kpad = ly.K1pad;
    s2.N = ly.d_out;
    s2.Npad = ly.N1pad;
    s2.act = (int)ly.act_out;
    s2.out_mode = 1;
    launch_t(c, s2, hint);
}
