// The walk along a list's in-edges that the pull kernels share: scatter.hip (hops and bootstrap), attention.hip.
#pragma once
#include "common.h"
#include <algorithm>

#define PULL_CHUNK 256
#define PULL_RUN 8                      // chunks a wavefront takes at a time on a large hop
// How the flattened in-edge space of a list, `total` entries, is cut for nw wavefronts: chunks of `chunk` edges (64 edges a wavefront step, PULL_CHUNK at
// most), `per` chunks to a run. A chunk is one chain of dependent reads (descriptors, ids, marks, rows), so hops of few in-edges are cut into halves or
// quarters of a chunk as long as every wavefront still gets at most one: up to 64 nw in-edges (0.5 M on 8,192 wavefronts) chunks of 64, up to 128 nw (1.05 M) chunks of
// 128. A hop of 470 K in-edges is 7,300 chains of a quarter of the length and not 1,800.
//   In-edges, rows, 256 / 64 or 128 edges a chunk: 278 K, a thousand messages of 128 columns 18.8 / 11.0 us; 482 K, 9 K of 256 46.6 / 21.5; 468 K rows of 256
//   all gathered 86.9 / 70.8 (the first three with what the flush of k_scatter_pull gained).
// Not further: above that, from 1.05 M to 2.1 M in-edges, up to half of the wavefronts have no chunk of 256, but with more chunks than wavefronts
// every wavefront asks the counter for another run, one after the other. Two-layer batches and bootstraps, limits as they are / twice as high, us:
// 1.1 M in-edges, sums of 128 columns 316 / 385, of 60 222 / 304, attention's bootstrap 272 / 416, deterministic (no counter) 372 / 383; 2.05 M 402 / 511,
// 276 / 418, 354 / 607, 459 / 484.
struct RunCut {
    uint32_t chunk, n_chunks, per, n_runs;
    __host__ __device__ __forceinline__ uint32_t span() const { return chunk * per; }
};
__host__ __device__ __forceinline__ RunCut rp_run_cut(uint32_t total, uint32_t nw) {
    RunCut c;
    c.chunk = (total - 1u) / 64u < nw ? 64u : ((total - 1u) / 128u < nw ? 128u : (uint32_t)PULL_CHUNK);
    c.n_chunks = (uint32_t)(((unsigned long long)total + c.chunk - 1u) / c.chunk);
    const uint32_t p = c.n_chunks / (2u * nw);
    c.per = p < 1u ? 1u : (p > PULL_RUN ? PULL_RUN : p);
    c.n_runs = (c.n_chunks + c.per - 1u) / c.per;
    return c;
}
// ... and the most runs that in-rows of up to `entries` entries can give: nw while chunks are small, 4 nw + 1 while runs are shorter than PULL_RUN chunks
static inline size_t rp_max_runs(uint64_t entries, uint32_t nw) {
    return (size_t)std::min<uint64_t>(entries / 64u + 2, std::max<uint64_t>(4ull * nw + 1, entries / (PULL_CHUNK * PULL_RUN) + 2));
}

// the next run's number, fetched by lane 0 for the wavefront
__device__ __forceinline__ uint32_t rp_next_run(uint32_t *counter, int lane) {
    uint32_t r = 0;
    if (lane == 0) r = atomicAdd(counter, 1u);
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)r);
}

struct PullArgs {
    const uint32_t *list;          // destinations, ascending
    const uint32_t *count_ptr;
    const uint32_t *ioff;          // in-degree prefix over the list
    const uint2 *in_meta;
    const uint32_t *in_pool;
    const float *in_w;             // edge weights parallel to in_pool (weighted-sum layers), or null
    const uint32_t *bm_prev;       // A_{l-1} as bitmap
    uint32_t *bm_cur;              // bitmap of A_l: receivers are marked here when discovering
    const float *D;                // delta rows, indexed by vertex
    uint32_t ldd;                  // their row stride
    uint32_t msg_bytes;            // packed message rows (k_scatter_pull4): size of the table in bytes, below 4 GB
    uint32_t d;
    float *X;
    DevCtr *ctr;
    uint32_t l;
    int mode, ratio, allow_disc;
    // the hop's messages may have been listed and sorted instead (rp_hop_listed): then the pull leaves the hop alone
    const uint32_t *m_count;       // |A_{l-1}| and, in the next word, the number of messages
    uint32_t sorted_cap;           // entries the host sorted (0: no list was made)
    int sorted_force;
    // the same hop pushed (DISC = 0), or its set marked (DISC = 1), by the same launch where the hop turns out not to be this kernel's
    int others;
    const uint32_t *out_list, *out_eoff;   // A_{l-1} and its out-degree prefix
    const uint2 *out_meta;
    const uint32_t *out_pool;
    const float *out_w;
    uint8_t *mk;
    // deterministic variants only
    const uint32_t *bm_rec;        // destinations that are recomputed from all their in-neighbours (bootstrap inference), or null
    const void *Hprev;             // what a recomputed row sums: rows of H^{l-1} (storage format `store`) ...
    const float *R;                // ... or, for a project-first layer, of T (what every vertex has sent so far)
    uint32_t ldr;                  // its row stride (H: d)
    int store;
    uint32_t side_runs;            // runs the side entries have room for (two entries per run)
    uint32_t *side_v;              // per run: the destinations of its first and last in-edge, if it has sums for them
    float *side_acc;               // ... and those sums, d floats per entry
};

// The part both pull kernels share: which in-edges a chunk holds. Lane j describes row i_lo + j of the
// list: destination rv, pool position of edge e is rbase + e (mod 2^32), and bnd = first edge of row
// i_lo + j + 1 (the total beyond the list's end). ALL: every in-edge counts, no source is tested.
template <int T, int WT, int ALL = 0>
struct PullScan {
    uint32_t i_lo, rv, rbase, bnd;
    uint32_t i_nx, rv_n, rbase_n, bnd_n;

    __device__ __forceinline__ void begin(const PullArgs &a, uint32_t count, uint32_t e_begin, int lane) {
        const uint32_t last = count - 1;
        i_lo = rp_seg_search_wave(a.ioff, 0, last, e_begin);
        const uint32_t ri = min(last, i_lo + lane);
        rv = a.list[ri];
        rbase = a.in_meta[rv].x - a.ioff[ri];
        bnd = a.ioff[min(count, i_lo + 1 + lane)];
    }
    // edge e0 + 64 t + lane of the chunk [e0, e1): its destination, source, weight and whether the source is in
    // A_{l-1}; then requests the rows of the next chunk, which are in flight while this chunk's messages are gathered
    __device__ __forceinline__ void chunk(const PullArgs &a, uint32_t count, uint32_t e0, uint32_t e1, int lane,
                                          uint32_t (&my_v)[T], uint32_t (&my_u)[T], float (&my_w)[WT ? T : 1], bool (&dirty)[T]) {
        const uint32_t last = count - 1;
        const bool fits = __shfl(bnd, 63) > e1 - 1;         // every row of the chunk is among the 64 held
        if (fits) {
#pragma unroll
            for (int t = 0; t < T; ++t) {
                const uint32_t e = e0 + 64 * t + lane;
                const int r = (int)min(63u, rp_count_le(bnd, e));
                my_v[t] = __shfl(rv, r);
                const uint32_t base = __shfl(rbase, r);
                my_u[t] = 0;
                dirty[t] = false;
                if (WT) my_w[t] = 0.0f;
                if (e < e1) {
                    my_u[t] = a.in_pool[base + e];
                    if (WT) my_w[t] = a.in_w[base + e];
                    dirty[t] = ALL || ((a.bm_prev[my_u[t] >> 5] >> (my_u[t] & 31)) & 1u);
                }
            }
            i_nx = min(last, i_lo + rp_count_le(bnd, e1));
        } else {
            // Short rows (a stretch of vertices with fewer than four in-neighbours on average, e.g. vertices created
            // by earlier batches, which sit together at the end of the id range): the chunk is taken in pieces of
            // 64 rows, each like a chunk that fits. (A search per edge instead made such chunks several times as
            // slow as the others, and since a wavefront's chunks are neighbours, the wavefronts at the end of the
            // id range then held up the whole hop: 2.1 -> 3.8 ms after 400 batches that each create 100 vertices.)
#pragma unroll
            for (int t = 0; t < T; ++t) {
                my_v[t] = 0;
                my_u[t] = 0;
                if (WT) my_w[t] = 0.0f;
                dirty[t] = false;
            }
            uint32_t il = i_lo, rv_p = rv, rb_p = rbase, bn_p = bnd, es = e0;
            for (;;) {
                const uint32_t top = min(e1, (uint32_t)__shfl(bn_p, 63));   // edges [es, top) lie in the 64 rows held
#pragma unroll
                for (int t = 0; t < T; ++t) {
                    const uint32_t e = e0 + 64 * t + lane;
                    const int r = (int)min(63u, rp_count_le(bn_p, e));
                    const uint32_t v = __shfl(rv_p, r);
                    const uint32_t base = __shfl(rb_p, r);
                    if (e >= es && e < top) {
                        my_v[t] = v;
                        my_u[t] = a.in_pool[base + e];
                        if (WT) my_w[t] = a.in_w[base + e];
                        dirty[t] = ALL || ((a.bm_prev[my_u[t] >> 5] >> (my_u[t] & 31)) & 1u);
                    }
                }
                if (top >= e1) break;
                es = top;
                il = min(last, il + 64u);
                const uint32_t rp = min(last, il + lane);
                rv_p = a.list[rp];
                rb_p = a.in_meta[rv_p].x - a.ioff[rp];
                bn_p = a.ioff[min(count, il + 1 + lane)];
            }
            i_nx = min(last, il + rp_count_le(bn_p, e1));
        }
        const uint32_t ri = min(last, i_nx + lane);
        rv_n = a.list[ri];
        rbase_n = a.in_meta[rv_n].x - a.ioff[ri];
        bnd_n = a.ioff[min(count, i_nx + 1 + lane)];
    }
    __device__ __forceinline__ void advance() {
        i_lo = i_nx;
        rv = rv_n;
        rbase = rbase_n;
        bnd = bnd_n;
    }
};

#ifdef __HIPCC__
// Two rows of 16 lanes (or the two halves) trade places and are added, without LDS: odd rows (the upper half) of the first operand against even rows (the
// lower half) of the second.
__device__ __forceinline__ float swap_add16(float x, float y) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);   // rows 0 and 2: x over the two rows, rows 1 and 3: y
}
__device__ __forceinline__ float swap_add32(float x, float y) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);   // lower half: x over both halves, upper half: y
}
// A destination whose in-edges lie in several runs is summed in run order: every run leaves its share in one of its two rows of
// `part` (the first for a destination that began in an earlier run, the second for one that begins here and goes on), and says in
// `cut` which destination goes on and up to which run; a wavefront per run then adds the parts up. Atomics in their place would make
// the sum depend on which run came first, from one bootstrap to the next.
struct CutRows {
    uint2 *cut;                    // per run: the destination (or 0xFFFFFFFF), the run of its last in-edge
    float *part;                   // per run: two rows
};
// in an array of 2 runs (1 + row) numbers
static inline CutRows rp_cut_rows(float *p, size_t runs) { return {(uint2 *)p, p + 2 * runs}; }
// Row 2 r + 1 of `part` plus rows 2 (r + 1), ... 2 r_last, for PARTS_B blocks of 64 columns from `col` on (the caller's lane): eight
// rows of all blocks are on their way at a time.
#define PARTS_B 4
__device__ __forceinline__ void rp_sum_parts(const float *part, uint32_t ld, uint32_t r, uint32_t r_last, uint32_t col, float (&t)[PARTS_B]) {
    constexpr int G = 8;
#pragma unroll
    for (int b = 0; b < PARTS_B; ++b) t[b] = part[(size_t)(2u * r + 1u) * ld + min(col + 64u * b, ld - 1u)];
    for (uint32_t f = r + 1u; f <= r_last; f += G) {
        float p[G][PARTS_B];
#pragma unroll
        for (int g = 0; g < G; ++g)
            if (f + (uint32_t)g <= r_last)
#pragma unroll
                for (int b = 0; b < PARTS_B; ++b) p[g][b] = part[(size_t)(2u * (f + (uint32_t)g)) * ld + min(col + 64u * b, ld - 1u)];
#pragma unroll
        for (int g = 0; g < G; ++g)
            if (f + (uint32_t)g <= r_last)
#pragma unroll
                for (int b = 0; b < PARTS_B; ++b) t[b] += p[g][b];
    }
}
#endif
