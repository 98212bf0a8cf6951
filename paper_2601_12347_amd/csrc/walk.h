// The out-edge walk from a hop's set, shared by the frontier kernels and the fused kernels of small hops.
#pragma once
#include "common.h"

#define MARK_CHUNK 256

// mark the out-neighbours of every vertex of A_{l-1}. Every wavefront walks a contiguous run of
// 256-edge chunks of the flattened out-edge space, so only its first chunk needs a search over the
// whole list; the 64 rows after the chunk's first one are described in registers (one per lane:
// where the row's edges start in the pool, and the first edge of the next row) and an edge finds its
// row with shuffles. Nothing to do on a discovering hop (the in-row scan finds A_l).
// Small frontiers (SparseArgs given): a marked vertex is entered into the hop's bitmap at once and the
// first wavefront to do so appends it to the hop's list, so no scan of the whole bitmap is needed
// afterwards; the list is then in no particular order.
struct SparseArgs {
    uint32_t *bm;                  // the hop's bitmap (zero on entry)
    const uint32_t *alive;
    uint32_t *list, *count;        // the hop's list and its length (zero on entry)
    // with eoff (all entered vertices are appended then, long_dup): the degree prefix over the list is written along with it. `count` is a DevCtr::Set: one 64-bit addition
    // reserves list positions and the stretch of the out-edge space that goes with them, so the prefix is in list order
    uint32_t *eoff;
    const uint2 *out_meta;
    uint32_t *isum;                // += in-degrees of the entries (statistics), with eoff
    uint32_t *touched;             // += vertices first entered by an out-edge (statistics)
    // roots merged in by the same kernel: sinks of changed edges, created vertices, the previous hop's set (self term)
    const uint32_t *st_dst, *n_struct;
    uint32_t struct_cap;
    const uint32_t *list0, *count0, *bm_vadd;
    int self_term;
    // optional second list: vertices with more than long_min in-neighbours are appended there instead
    const uint2 *in_meta;
    uint32_t long_min;
    uint32_t *long_list, *long_count;
    int long_dup;                  // those vertices are appended to the hop's list as well
};

// T vertices per lane (0xFFFFFFFF: none): the T marks go out together and one reservation covers all of
// them (two round trips instead of 2 T). To be called by all 64 lanes together.
template <int T>
__device__ __forceinline__ void sparse_enter_many(const SparseArgs &s, const uint32_t *v, bool from_edge) {
    bool live[T], fresh[T], lng[T];
    uint32_t d_out[T], d_in[T];                             // requested beside the live bits, whether or not the vertex turns out to be new
#pragma unroll
    for (int t = 0; t < T; ++t) {
        const bool some = v[t] != 0xFFFFFFFFu;
        live[t] = some && rp_bit(s.alive, v[t]);
        d_out[t] = (some && s.eoff) ? s.out_meta[v[t]].y : 0u;
        d_in[t] = (some && (s.eoff || s.long_list)) ? s.in_meta[v[t]].y : 0u;
    }
#pragma unroll
    for (int t = 0; t < T; ++t) {
        fresh[t] = false;
        if (live[t]) {
            const uint32_t m = 1u << (v[t] & 31);
            fresh[t] = !(atomicOr(&s.bm[v[t] >> 5], m) & m);
        }
    }
#pragma unroll
    for (int t = 0; t < T; ++t) lng[t] = fresh[t] && s.long_list && d_in[t] > s.long_min;
    unsigned long long mask[T], lmask[T];
    uint32_t total = 0, ltotal = 0;
#pragma unroll
    for (int t = 0; t < T; ++t) {
        mask[t] = __ballot(fresh[t] && (!lng[t] || s.long_dup));
        lmask[t] = __ballot(lng[t]);
        total += (uint32_t)__popcll(mask[t]);
        ltotal += (uint32_t)__popcll(lmask[t]);
    }
    if (!(total + ltotal)) return;
    const int lane = rp_lane();
    uint32_t base = 0, lbase = 0;
    if (s.eoff) {
        uint32_t off[T], run = 0, din = 0;
#pragma unroll
        for (int t = 0; t < T; ++t) {
            off[t] = fresh[t] ? d_out[t] : 0u;
            din += fresh[t] ? d_in[t] : 0u;
        }
#pragma unroll
        for (int t = 0; t < T; ++t) {
            const uint32_t dg = off[t], x = rp_wave_scan(dg);
            off[t] = run + x - dg;
            run += (uint32_t)__builtin_amdgcn_readlane((int)x, 63);
        }
        din = (uint32_t)__builtin_amdgcn_readlane((int)rp_wave_scan(din), 63);
        unsigned long long at = 0;
        if (lane == 0) {
            at = atomicAdd((unsigned long long *)s.count, ((unsigned long long)run << 32) | total);
            if (ltotal) lbase = atomicAdd(s.long_count, ltotal);
            if (from_edge && s.touched) atomicAdd(s.touched, total);
            atomicAdd(s.isum, din);
        }
        base = __shfl((uint32_t)at, 0);
        lbase = __shfl(lbase, 0);
        const uint32_t e = __shfl((uint32_t)(at >> 32), 0);
        const unsigned long long below = (1ull << lane) - 1ull;
#pragma unroll
        for (int t = 0; t < T; ++t) {
            if (fresh[t]) {
                const uint32_t p = base + (uint32_t)__popcll(mask[t] & below);
                s.list[p] = v[t];
                s.eoff[p] = e + off[t];
            }
            if (lng[t]) s.long_list[lbase + (uint32_t)__popcll(lmask[t] & below)] = v[t];
            base += (uint32_t)__popcll(mask[t]);
            lbase += (uint32_t)__popcll(lmask[t]);
        }
        return;
    }
    if (lane == 0) {
        if (total) base = atomicAdd(s.count, total);
        if (ltotal) lbase = atomicAdd(s.long_count, ltotal);
        if (from_edge && s.touched) atomicAdd(s.touched, total + ltotal);
    }
    base = __shfl(base, 0);
    lbase = __shfl(lbase, 0);
    const unsigned long long below = (1ull << lane) - 1ull;
#pragma unroll
    for (int t = 0; t < T; ++t) {
        if (fresh[t] && (!lng[t] || s.long_dup)) s.list[base + (uint32_t)__popcll(mask[t] & below)] = v[t];
        if (lng[t]) s.long_list[lbase + (uint32_t)__popcll(lmask[t] & below)] = v[t];
        base += (uint32_t)__popcll(mask[t]);
        lbase += (uint32_t)__popcll(lmask[t]);
    }
}

// one vertex per valid lane; to be called by all 64 lanes together
__device__ __forceinline__ void sparse_enter(const SparseArgs &s, uint32_t v, bool valid, bool from_edge) {
    const uint32_t one[1] = {valid ? v : 0xFFFFFFFFu};
    sparse_enter_many<1>(s, one, from_edge);
}

template <bool SPARSE>
__device__ __forceinline__ void frontier_walk(const uint32_t *list, const uint32_t *count_ptr, const uint32_t *eoff,
                                              const uint2 *out_meta, const uint32_t *out_pool, uint8_t *mk,
                                              const SparseArgs &sp, uint32_t gw, uint32_t nw) {
    const uint32_t count = *count_ptr;
    if (count == 0) return;
    constexpr int T = MARK_CHUNK / 64;
    const int lane = rp_lane();
    const uint32_t M = count_ptr[1];
    // few out-edges: 64-edge chunks (only the first of a lane's T slots is used) so that more wavefronts share them
    const uint32_t chunk = (SPARSE && M <= 16384u) ? 64u : (uint32_t)MARK_CHUNK;
    const uint32_t n_chunks = (M + chunk - 1) / chunk;
    const uint32_t per = (n_chunks + nw - 1) / nw;
    const uint32_t c_begin = min(n_chunks, gw * per), c_end = min(n_chunks, c_begin + per);
    if (c_begin >= c_end) return;
    const uint32_t last = count - 1;
    uint32_t i_lo = rp_seg_search_wave(eoff, 0, last, c_begin * chunk);
    uint32_t rbase, bnd;                                    // lane j: row i_lo + j
    {
        const uint32_t ri = min(last, i_lo + lane);
        rbase = out_meta[list[ri]].x - eoff[ri];                // pool position of edge e: rbase + e (mod 2^32)
        bnd = rp_row_end(eoff, count, M, i_lo + lane);
    }
    for (uint32_t c = c_begin; c < c_end; ++c) {
        const uint32_t e0 = c * chunk, e1 = min(M, e0 + chunk);
        const bool fits = __shfl(bnd, 63) > e1 - 1;         // every row of the chunk is among the 64 held
        uint32_t v[T];
        uint32_t i_nx;
        if (fits) {
#pragma unroll
            for (int t = 0; t < T; ++t) {
                const uint32_t e = e0 + lane + 64 * t;
                const int r = (int)min(63u, rp_count_le(bnd, e));
                const uint32_t base = __shfl(rbase, r);
                v[t] = (e < e1) ? out_pool[base + e] : 0xFFFFFFFFu;
            }
            i_nx = min(last, i_lo + rp_count_le(bnd, e1));
        } else {
            const uint32_t i_hi = rp_seg_forward(eoff, i_lo, last, e1 - 1);
#pragma unroll
            for (int t = 0; t < T; ++t) {
                const uint32_t e = e0 + lane + 64 * t;
                v[t] = 0xFFFFFFFFu;
                if (e < e1) {
                    const uint32_t i = rp_seg_search(eoff, i_lo, i_hi, e);
                    const uint32_t u = list[i];
                    v[t] = out_pool[out_meta[u].x + (e - eoff[i])];
                }
            }
            i_nx = rp_seg_forward(eoff, i_hi, last, e1);
        }
        uint32_t rbase_n, bnd_n;                            // next chunk's rows, requested before the marks
        {
            const uint32_t ri = min(last, i_nx + lane);
            rbase_n = out_meta[list[ri]].x - eoff[ri];
            bnd_n = rp_row_end(eoff, count, M, i_nx + lane);
        }
        if (SPARSE) {
            sparse_enter_many<T>(sp, v, true);
        } else {
#pragma unroll
            for (int t = 0; t < T; ++t)
                if (v[t] != 0xFFFFFFFFu) mk[v[t]] = 1;       // plain byte stores: idempotent, no atomics
        }
        i_lo = i_nx;
        rbase = rbase_n;
        bnd = bnd_n;
    }
}

// Edges c0 * MARK_CHUNK .. (c0 + C) * MARK_CHUNK - 1 of the flattened out-edge space, four per lane and chunk: destination v (0xFFFFFFFF past
// the end) and source u, and (WT) the edge's weight w. By all 64 lanes; rows are found as in frontier_walk.
template <int C, int WT>
__device__ __forceinline__ void walk_collect(const uint32_t *list, uint32_t count, uint32_t M, const uint32_t *eoff, const uint2 *out_meta,
                                             const uint32_t *out_pool, const float *out_w, uint32_t c0, uint32_t (&v)[4 * C], uint32_t (&u)[4 * C],
                                             float (&w)[WT ? 4 * C : 1]) {
    const int lane = rp_lane();
    const uint32_t last = count - 1;
    uint32_t i_lo = c0 * MARK_CHUNK < M ? rp_seg_search_wave(eoff, 0, last, c0 * MARK_CHUNK) : 0u;
#pragma unroll
    for (int k = 0; k < C; ++k) {
        const uint32_t e0 = (c0 + k) * MARK_CHUNK, e1 = min(M, e0 + MARK_CHUNK);
#pragma unroll
        for (int t = 0; t < 4; ++t) v[4 * k + t] = 0xFFFFFFFFu;
        if (e0 >= M) continue;                              // (the same for all lanes)
        const uint32_t ri = min(last, i_lo + lane), rsrc = list[ri], rbase = out_meta[rsrc].x - eoff[ri], bnd = rp_row_end(eoff, count, M, i_lo + lane);
        uint32_t i_hi = i_lo;
        const bool fits = __shfl(bnd, 63) > e1 - 1;
        if (!fits) i_hi = rp_seg_forward(eoff, i_lo, last, e1 - 1);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const uint32_t e = e0 + lane + 64 * t;
            const int r = (int)min(63u, rp_count_le(bnd, e));
            uint32_t src = __shfl(rsrc, r), at = __shfl(rbase, r) + e;
            if (!fits && e < e1) {
                const uint32_t i = rp_seg_search(eoff, i_lo, i_hi, e);
                src = list[i];
                at = out_meta[src].x + (e - eoff[i]);
            }
            u[4 * k + t] = src;
            if (e < e1) v[4 * k + t] = out_pool[at];
            if (WT) w[WT ? 4 * k + t : 0] = e < e1 ? out_w[at] : 0.0f;
        }
        i_lo = fits ? min(last, i_lo + rp_count_le(bnd, e1)) : rp_seg_forward(eoff, i_hi, last, e1);
    }
}

// roots of a hop, one vertex per lane and round: sinks of changed edges, created vertices, the previous hop's set (self term)
__device__ __forceinline__ void enter_roots(const uint32_t *list, const uint32_t *count_ptr, const SparseArgs &sp, uint32_t gw, uint32_t nw) {
    const int lane = rp_lane();
    const uint32_t n_s = min(*sp.n_struct, sp.struct_cap), n_0 = *sp.count0, n_p = sp.self_term ? *count_ptr : 0u;
    const uint32_t total = n_s + n_0 + n_p;
    for (uint32_t base = gw * 64; base < total; base += nw * 64) {
        const uint32_t i = base + lane;
        uint32_t v = 0;
        bool valid = i < total;
        if (valid) {
            if (i < n_s) v = sp.st_dst[i];
            else if (i < n_s + n_0) {
                v = sp.list0[i - n_s];
                valid = rp_bit(sp.bm_vadd, v);
            } else v = list[i - n_s - n_0];
        }
        sparse_enter(sp, v, valid, false);
    }
}

SparseArgs rp_sparse_args(ripple_ctx *c, uint32_t l, uint32_t *list, uint32_t *count, bool self_term);   // frontier.hip
