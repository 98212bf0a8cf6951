// Frontier construction (the per-hop slice of the propagation tree, Sec. 3.3):
//   A_l = (S  u  Out(A_{l-1})  u  [A_{l-1} if the layer reads the vertex's own
//          embedding]  u  V_added)  n  Alive
// as a bitmap and as an ascending list, plus the exclusive scan of out-degrees
// over that list, which lets the next hop's edge walk be split evenly over
// wavefronts regardless of degree skew.
#include "common.h"
#include "kernels.h"
#include "walk.h"
#include <cstring>

#define RP_STATIC_BLOCKS 16384u                  // entries of the static array (see below): blocks a compaction may have

// The walk that also lists the hop's messages: (destination, source) pairs in buckets by destination, each with room of its own, for
// k_scatter_list. A workgroup holds 16 K edges in registers, counts its share of every bucket in LDS, takes that much room at once and writes.
// `cap`: the messages the host expects at most; a hop with more is marked only.
// In place of a list in edge order and a radix sort of it (4.6 M pairs: 0.09 ms for the walk, 0.24 for the sort and its launches; here 0.117
// for the walk and 0.036 for k_list_order).
#define LIST_C 4
// up to here a tile is a quarter of that: most compute units would have none (220 K walked edges of an attention hop 64 us / 21, 140 K of a sum 30 / 13; 2 M 38 / 38)
#define LIST_SMALL (1u << 20)
struct ListWalk {
    uint2 *pairs;
    const float *out_w;            // weighted sums: weights beside the out-rows, and where they go beside the pairs
    float *pair_w;
    uint32_t *cnt;
    ListCut cut;
    uint32_t cap;
    // attention hops: messages to vertices that are recomputed anyway are not listed
    int attn, force;
    const uint32_t *bm_prev, *bm_sink, *bm_vadd;
    const uint2 *in_meta;
    uint32_t long_min;
};
// the tiles of a list walk, C chunks of 256 edges to a wavefront
template <int C, int WT>
__device__ __forceinline__ void list_tiles(const uint32_t *list, uint32_t count, uint32_t M, const uint32_t *eoff, const uint2 *out_meta,
                                           const uint32_t *out_pool, uint8_t *mk, DevCtr *ctr, uint32_t l, const ListWalk &w, uint32_t *s_at) {
    constexpr uint32_t NONE = 0xFFFFFFFFu, FULL = 0xFF000000u;
    constexpr uint32_t TILE = 16u * C;                      // chunks of a workgroup
    const uint32_t wave = threadIdx.x >> 6;
    const uint32_t n_tiles = (M + TILE * MARK_CHUNK - 1) / (TILE * MARK_CHUNK);
    for (uint32_t tile = blockIdx.x; tile < n_tiles; tile += gridDim.x) {
        for (uint32_t b = threadIdx.x; b < w.cut.n; b += 1024u) s_at[b] = 0;
        uint32_t v[4 * C], u[4 * C];
        float wt[WT ? 4 * C : 1];
        walk_collect<C, WT>(list, count, M, eoff, out_meta, out_pool, w.out_w, tile * TILE + wave * C, v, u, wt);
        if (w.attn) {
            uint32_t is[4 * C], sink[4 * C];                // all of them on their way together
#pragma unroll
            for (int t = 0; t < 4 * C; ++t) {
                const uint32_t at = v[t] == NONE ? 0u : v[t] >> 5;
                is[t] = w.bm_prev[at] | w.bm_vadd[at];
                sink[t] = w.bm_sink[at];
            }
#pragma unroll
            for (int t = 0; t < 4 * C; ++t) {
                const uint32_t x = v[t], b = x & 31u;
                if (x == NONE) continue;
                mk[x] = 1;
                if (((is[t] >> b) & 1u) || (((sink[t] >> b) & 1u) && w.in_meta[x].y <= w.long_min)) v[t] = NONE;
            }
        }
        __syncthreads();
#pragma unroll
        for (int t = 0; t < 4 * C; ++t)
            if (v[t] != NONE) {
                mk[v[t]] = 1;
                atomicAdd(&s_at[v[t] >> w.cut.shift], 1u);
            }
        __syncthreads();
        for (uint32_t b = threadIdx.x; b < w.cut.n; b += 1024u) {
            const uint32_t n = s_at[b];
            if (!n) continue;
            const uint32_t at = atomicAdd(&w.cnt[b], n);
            const bool fits = at + n <= w.cut.room;
            if (!fits) ctr->pair_over[l] = 1;               // the hop is pushed or pulled
            s_at[b] = fits ? b * w.cut.room + at : FULL;
        }
        __syncthreads();
#pragma unroll
        for (int t = 0; t < 4 * C; ++t)
            if (v[t] != NONE) {
                const uint32_t at = atomicAdd(&s_at[v[t] >> w.cut.shift], 1u);
                if (at < FULL) {
                    w.pairs[at] = make_uint2(v[t], u[t]);
                    if (WT) w.pair_w[at] = wt[WT ? t : 0];
                }
            }
        __syncthreads();
    }
}

template <int WT>
__global__ __launch_bounds__(1024) void k_frontier_list(const uint32_t *list, const uint32_t *count_ptr, const uint32_t *eoff, const uint2 *out_meta,
                                                        const uint32_t *out_pool, uint8_t *mk, DevCtr *ctr, uint32_t l, uint32_t d, int mode, int ratio,
                                                        int allow_disc, ListWalk w) {
    if (allow_disc && rp_hop_mode(ctr, l, d, mode, ratio, allow_disc) == RP_HOP_DISCOVER) return;
    __shared__ uint32_t s_at[RP_LIST_BUCKETS];              // per bucket: this tile's pairs, then where the next one goes
    const uint32_t count = *count_ptr, wave = threadIdx.x >> 6;
    const uint32_t M = count ? count_ptr[1] : 0u;
    if (w.attn ? !rp_gat_list_made(ctr, M, w.cap, w.force) : (M == 0 || M > w.cap)) {
        frontier_walk<false>(list, count_ptr, eoff, out_meta, out_pool, mk, SparseArgs(), blockIdx.x * 16u + wave, gridDim.x * 16u);
        return;
    }
    if (M <= LIST_SMALL) list_tiles<1, WT>(list, count, M, eoff, out_meta, out_pool, mk, ctr, l, w, s_at);
    else list_tiles<LIST_C, WT>(list, count, M, eoff, out_meta, out_pool, mk, ctr, l, w, s_at);
}

__global__ __launch_bounds__(256) void k_frontier_mark(const uint32_t *list, const uint32_t *count_ptr, const uint32_t *eoff, const uint2 *out_meta,
                                                       const uint32_t *out_pool, uint8_t *mk) {
    frontier_walk<false>(list, count_ptr, eoff, out_meta, out_pool, mk, SparseArgs(), (blockIdx.x * blockDim.x + threadIdx.x) >> 6,
                         (gridDim.x * blockDim.x) >> 6);
}

// the out-edge walk and the roots in one kernel, straight into the hop's bitmap and (unordered) list
__global__ __launch_bounds__(256) void k_frontier_sparse(const uint32_t *list, const uint32_t *count_ptr,
                                                         const uint32_t *eoff, const uint2 *out_meta,
                                                         const uint32_t *out_pool, SparseArgs sp) {
    const uint32_t gw = (blockIdx.x * blockDim.x + threadIdx.x) >> 6, nw = (gridDim.x * blockDim.x) >> 6;
    frontier_walk<true>(list, count_ptr, eoff, out_meta, out_pool, nullptr, sp, gw, nw);
    enter_roots(list, count_ptr, sp, gw, nw);
}

struct CompactArgs {
    uint32_t *bm;                  // the layer's bitmap: marks in (a discovering hop sets them here), final set out
    uint8_t *mk;                   // more marks, one byte per vertex (set by the out-edge walk, cleared here), or null
    const uint32_t *bm_prev;       // previous hop's set (layers with a self term) or null
    const uint32_t *bm_sink;       // S or null
    const uint32_t *bm_vadd;       // V_added (read only when bm_sink is set)
    const uint32_t *alive;
    uint32_t n_words;
    const uint2 *out_meta, *in_meta;
    int want_out, want_in;         // emit out-degree / in-degree prefixes over the list
    uint32_t *part_cnt, *part_out, *part_in, *part_tch, *part_rec;    // (part_tch: with touched_out only, part_rec: with gat)
    uint32_t *rep;                 // reporting union or null
    uint32_t *touched_out;         // += vertices that received a message, or null
    uint32_t *list, *eoff, *ioff;  // outputs
    uint32_t *count_out, *msgs_out, *isum_out;
    uint32_t list_cap;             // entries the list has room for (positions beyond are counted, not written)
    HostFlag done;                 // k_bitmap_ids only
    // Attention hops whose messages are listed (rp_gat_listed): the vertices that are recomputed and have in-edges get a list of their own, and the
    // in-degree prefix is over that one. (With the prefix over the whole list, zero for the others, the wavefront whose edges lay on both sides of
    // 400 K vertices that are not recomputed went over those alone: a batch of 0.23 ms took 9.8.)
    const DevCtr *gat;             // null: any other compaction
    uint32_t gat_l, gat_cap, gat_long;
    int gat_force;
    uint32_t *rec_list, *rec_count;
};

// Compaction of a bitmap into its ascending list. A wavefront takes two bitmap words at a time, a lane being a vertex:
// marks, degrees and list entries are then read and written with consecutive addresses (a lane per word read the degrees
// of 32 consecutive vertices each, 64 cache lines per instruction: 15 + 48 us for both passes on 2.45 M vertices;
// reading the degrees takes about 10). S steps of two words per wavefront, four wavefronts per
// workgroup; the vertex's membership and degrees stay in registers between the sums and the list entries.
template <int S>
struct WordRange {
    bool on[S];                    // this lane's vertex of step s is in the set
    uint32_t o[S], i[S];           // its degrees (0 where not wanted or not in the set)
    uint32_t cnt, tch, dout, din;  // the wavefront's totals
    bool some;                     // a listed attention hop: i[s] is zero but for vertices that are recomputed
    uint32_t nrec;                 // ... and how many those are

    static __device__ __forceinline__ uint32_t word(uint32_t w0, int s, int lane) { return w0 + 2u * s + ((uint32_t)lane >> 5); }

    // the final set of words w0 .. w0 + 2 S - 1: marks, bitmap and roots merged and restricted to live vertices
    __device__ __forceinline__ void merge(const CompactArgs &a, uint32_t w0, int lane) {
        uint32_t w[S], live[S], root[S];
        uint8_t m[S];
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const uint32_t idx = word(w0, s, lane), ic = min(idx, a.n_words - 1u);
            live[s] = idx < a.n_words ? a.alive[ic] : 0u;
            w[s] = a.bm[ic];
            m[s] = (a.mk && idx < a.n_words) ? a.mk[(size_t)ic * 32u + ((uint32_t)lane & 31u)] : (uint8_t)0;
            root[s] = 0u;
            if (a.bm_sink) root[s] |= a.bm_sink[ic] | a.bm_vadd[ic];
            if (a.bm_prev) root[s] |= a.bm_prev[ic];
        }
        cnt = tch = 0;
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const uint32_t idx = word(w0, s, lane), b = (uint32_t)lane & 31u;
            const bool lv = (live[s] >> b) & 1u;
            const bool hit = lv && (m[s] != 0 || ((w[s] >> b) & 1u));
            if (m[s]) a.mk[(size_t)idx * 32u + b] = 0;
            on[s] = hit || (lv && ((root[s] >> b) & 1u));
            const unsigned long long mask = __ballot(on[s]);
            tch += (uint32_t)__popcll(__ballot(hit));              // vertices that received at least one message
            cnt += (uint32_t)__popcll(mask);
            if (b == 0 && idx < a.n_words) {
                const uint32_t f = (lane == 0) ? (uint32_t)mask : (uint32_t)(mask >> 32);
                if (f != w[s]) a.bm[idx] = f;
                if (a.rep && f) a.rep[idx] |= f;
            }
        }
    }
    // the set as merge() left it in memory
    __device__ __forceinline__ void read(const CompactArgs &a, uint32_t w0, int lane) {
        uint32_t w[S];
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const uint32_t idx = word(w0, s, lane);
            w[s] = idx < a.n_words ? a.bm[idx] & a.alive[idx] : 0u;
        }
        cnt = tch = 0;
#pragma unroll
        for (int s = 0; s < S; ++s) {
            on[s] = (w[s] >> ((uint32_t)lane & 31u)) & 1u;
            cnt += (uint32_t)__popcll(__ballot(on[s]));
        }
    }
    __device__ __forceinline__ void degrees(const CompactArgs &a, uint32_t w0, int lane) {
        dout = din = nrec = 0;
        some = false;
        if (!(a.want_out | a.want_in)) {
#pragma unroll
            for (int s = 0; s < S; ++s) o[s] = i[s] = 0u;
            return;
        }
        some = a.gat && rp_gat_listed(a.gat, a.gat_l, a.gat_cap, a.gat_force);
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const uint32_t v = (w0 + 2u * s) * 32u + (uint32_t)lane;
            o[s] = (a.want_out && on[s]) ? a.out_meta[v].y : 0u;
            i[s] = (a.want_in && on[s]) ? a.in_meta[v].y : 0u;
        }
        if (some) {
#pragma unroll
            for (int s = 0; s < S; ++s) {
                const uint32_t v = (w0 + 2u * s) * 32u + (uint32_t)lane;
                if (on[s] && !rp_gat_recomputes(a.bm_prev, a.bm_sink, a.bm_vadd, a.in_meta, a.gat_long, v)) i[s] = 0u;
                nrec += (uint32_t)__popcll(__ballot(i[s] != 0u));
            }
        }
#pragma unroll
        for (int s = 0; s < S; ++s) {
            dout += o[s];
            din += i[s];
        }
        dout = (uint32_t)__builtin_amdgcn_readlane((int)rp_wave_scan(dout), 63);
        din = (uint32_t)__builtin_amdgcn_readlane((int)rp_wave_scan(din), 63);
    }
    // list entries and prefixes, from position oc and running sums oo, oi on (some: the list of recomputed vertices from position orec on)
    __device__ __forceinline__ void emit(const CompactArgs &a, uint32_t w0, int lane, uint32_t oc, uint32_t oo, uint32_t oi, uint32_t orec) const {
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const unsigned long long mask = __ballot(on[s]);
            if (!mask) continue;
            const uint32_t pos = oc + __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
            const bool put = on[s] && pos < a.list_cap;
            if (put) a.list[pos] = (w0 + 2u * s) * 32u + (uint32_t)lane;
            oc += (uint32_t)__popcll(mask);
            if (a.want_out) {
                const uint32_t x = rp_wave_scan(o[s]);
                if (put) a.eoff[pos] = oo + x - o[s];
                oo += (uint32_t)__builtin_amdgcn_readlane((int)x, 63);
            }
            if (a.want_in) {
                const uint32_t x = rp_wave_scan(i[s]);
                if (some) {
                    const unsigned long long mr = __ballot(i[s] != 0u);
                    const uint32_t at = orec + __builtin_amdgcn_mbcnt_hi((uint32_t)(mr >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mr, 0u));
                    if (i[s]) {
                        a.rec_list[at] = (w0 + 2u * s) * 32u + (uint32_t)lane;
                        a.ioff[at] = oi + x - i[s];
                    }
                    orec += (uint32_t)__popcll(mr);
                } else if (put) {
                    a.ioff[pos] = oi + x - i[s];
                }
                oi += (uint32_t)__builtin_amdgcn_readlane((int)x, 63);
            }
        }
    }
};

__device__ __forceinline__ void compact_totals(const CompactArgs &a, uint32_t oc, uint32_t oo, uint32_t oi, bool some, uint32_t orec) {
    *a.count_out = oc;
    if (some) *a.rec_count = orec;
    if (a.want_out) {
        a.eoff[oc] = oo;
        if (a.msgs_out) *a.msgs_out = oo;
    }
    if (a.want_in) {
        a.ioff[some ? orec : oc] = oi;
        if (a.isum_out) *a.isum_out = oi;
    }
}

// pass 1: merge the root sets (S, V_added, and the previous hop's set when the layer has a
// self term) into the layer's bitmap, restrict to live vertices, count vertices and
// (optionally) their degrees per block of 8 S words
template <int S>
__global__ __launch_bounds__(256) void k_frontier_count(CompactArgs a) {
    __shared__ uint32_t sh[20];
    const int lane = rp_lane(), wave = threadIdx.x >> 6;
    const uint32_t w0 = (blockIdx.x * 4u + wave) * 2u * S;
    WordRange<S> r;
    r.merge(a, w0, lane);
    r.degrees(a, w0, lane);
    if (lane == 0) {
        sh[wave] = r.cnt;
        sh[4 + wave] = r.dout;
        sh[8 + wave] = r.din;
        sh[12 + wave] = r.tch;
        sh[16 + wave] = r.nrec;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        a.part_cnt[blockIdx.x] = sh[0] + sh[1] + sh[2] + sh[3];
        a.part_out[blockIdx.x] = sh[4] + sh[5] + sh[6] + sh[7];
        a.part_in[blockIdx.x] = sh[8] + sh[9] + sh[10] + sh[11];
        // (added to one counter, 1,196 blocks waited for one another: 22 us for 2.45 M vertices, now 12)
        if (a.touched_out) a.part_tch[blockIdx.x] = sh[12] + sh[13] + sh[14] + sh[15];
        if (r.some) a.part_rec[blockIdx.x] = sh[16] + sh[17] + sh[18] + sh[19];
    }
}

// pass 2: write the ascending list and the degree prefixes
template <int S>
__global__ __launch_bounds__(256) void k_frontier_emit(CompactArgs a) {
    __shared__ uint32_t sh[20], wt[16];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint32_t w0 = (blockIdx.x * 4u + wave) * 2u * S;
    WordRange<S> r;
    r.read(a, w0, lane);                                   // on its way while the blocks before this one are summed
    const bool last = blockIdx.x == gridDim.x - 1;
    uint32_t pc = 0, po = 0, pi = 0, pt = 0, pr = 0;
    for (uint32_t b = tid; b < blockIdx.x; b += 256) {
        pc += a.part_cnt[b];
        po += a.part_out[b];
        pi += a.part_in[b];
    }
    for (uint32_t b = tid; last && a.touched_out && b < gridDim.x; b += 256) pt += a.part_tch[b];
    r.degrees(a, w0, lane);
    for (uint32_t b = tid; r.some && b < blockIdx.x; b += 256) pr += a.part_rec[b];
    pc = rp_wave_scan(pc);
    po = rp_wave_scan(po);
    pi = rp_wave_scan(pi);
    pt = rp_wave_scan(pt);
    if (r.some) pr = rp_wave_scan(pr);
    if (lane == 63) {
        sh[wave] = pc;
        sh[4 + wave] = po;
        sh[8 + wave] = pi;
        sh[12 + wave] = pt;
        sh[16 + wave] = pr;
        wt[wave] = r.cnt;
        wt[4 + wave] = r.dout;
        wt[8 + wave] = r.din;
        wt[12 + wave] = r.nrec;
    }
    __syncthreads();
    uint32_t oc = sh[0] + sh[1] + sh[2] + sh[3], oo = sh[4] + sh[5] + sh[6] + sh[7], oi = sh[8] + sh[9] + sh[10] + sh[11], orec = sh[16] + sh[17] + sh[18] + sh[19];
    for (int k = 0; k < wave; ++k) {
        oc += wt[k];
        oo += wt[4 + k];
        oi += wt[8 + k];
        orec += wt[12 + k];
    }
    r.emit(a, w0, lane, oc, oo, oi, orec);
    if (last && tid == 255) {
        compact_totals(a, oc + r.cnt, oo + r.dout, oi + r.din, r.some, orec + r.nrec);
        if (a.touched_out) *a.touched_out += sh[12] + sh[13] + sh[14] + sh[15];
    }
}

// Both passes in one workgroup, for bitmaps of at most ONE_WORDS words (8,192 vertices): one launch instead of two.
#define ONE_STEPS 8
#define ONE_WORDS (16u * 2u * ONE_STEPS)
__global__ __launch_bounds__(1024) void k_frontier_compact_one(CompactArgs a) {
    __shared__ uint32_t wt[16 * 5];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint32_t w0 = (uint32_t)wave * 2u * ONE_STEPS;
    WordRange<ONE_STEPS> r;
    r.merge(a, w0, lane);
    r.degrees(a, w0, lane);
    if (lane == 0) {
        wt[wave] = r.cnt;
        wt[16 + wave] = r.dout;
        wt[32 + wave] = r.din;
        wt[48 + wave] = r.tch;
        wt[64 + wave] = r.nrec;
    }
    __syncthreads();
    uint32_t oc = 0, oo = 0, oi = 0, orec = 0;
    for (int k = 0; k < wave; ++k) {
        oc += wt[k];
        oo += wt[16 + k];
        oi += wt[32 + k];
        orec += wt[64 + k];
    }
    r.emit(a, w0, lane, oc, oo, oi, orec);
    if (tid == 1023) {
        compact_totals(a, oc + r.cnt, oo + r.dout, oi + r.din, r.some, orec + r.nrec);
        uint32_t t = 0;
        for (int k = 0; k < 16; ++k) t += wt[48 + k];
        if (a.touched_out && t) atomicAdd(a.touched_out, t);
    }
}

// bitmap & alive -> ascending ids and their number, nothing else: every block adds up the words before its own by itself (at
// most RANK_WORDS of them, from the L2), so one launch does it and no scratch is needed.
#define RANK_WORDS 32768u
__global__ __launch_bounds__(256) void k_bitmap_ids(CompactArgs a) {
    constexpr int S = 4;
    __shared__ uint32_t sh[4], wt[4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint32_t w0 = (blockIdx.x * 4u + wave) * 2u * S;
    WordRange<S> r;
    r.read(a, w0, lane);
    uint32_t pc = 0;
    typedef uint32_t uintx4u __attribute__((ext_vector_type(4), aligned(4)));
    const uintx4u *bm4 = (const uintx4u *)a.bm, *al4 = (const uintx4u *)a.alive;   // 8 S words per block: whole groups of four
    for (uint32_t k = tid; k < blockIdx.x * (2u * S); k += 256u) {
        const uintx4u x = bm4[k], y = al4[k];
        pc += __popc(x.x & y.x) + __popc(x.y & y.y) + __popc(x.z & y.z) + __popc(x.w & y.w);
    }
    pc = rp_wave_scan(pc);
    if (lane == 63) {
        sh[wave] = pc;
        wt[wave] = r.cnt;
    }
    __syncthreads();
    uint32_t oc = sh[0] + sh[1] + sh[2] + sh[3];
    for (int k = 0; k < wave; ++k) oc += wt[k];
#pragma unroll
    for (int s = 0; s < S; ++s) r.o[s] = r.i[s] = 0u;
    r.some = false;
    r.emit(a, w0, lane, oc, 0u, 0u, 0u);
    if (blockIdx.x == gridDim.x - 1 && tid == 255) *a.count_out = oc + r.cnt;
    report_done(a.done, gridDim.x);
}

// Words per block: 32 up to half a million vertices (several blocks per compute unit where the graph allows it), 64 above,
// and 256 where 64 would need more blocks than the static array has entries.
static void launch_compact(ripple_ctx *c, const CompactArgs &a) {
    if (a.n_words <= ONE_WORDS) {
        hipLaunchKernelGGL(k_frontier_compact_one, dim3(1), dim3(1024), 0, c->stream, a);
        return;
    }
#define RP_COMPACT(S)                                                                                            \
    do {                                                                                                         \
        const dim3 nb(rp_div_up(a.n_words, 8 * (S)));                                                            \
        hipLaunchKernelGGL((k_frontier_count<S>), nb, dim3(256), 0, c->stream, a);                               \
        hipLaunchKernelGGL((k_frontier_emit<S>), nb, dim3(256), 0, c->stream, a);                                \
    } while (0)
    if (a.n_words <= 16384u) RP_COMPACT(4);
    else if (a.n_words <= 64u * RP_STATIC_BLOCKS) RP_COMPACT(8);
    else RP_COMPACT(32);
#undef RP_COMPACT
}

// degree prefixes over an arbitrary (unsorted) list, one workgroup: out-degrees into eoff (hop 0, and the
// lists of small frontiers) and, with in_meta and ioff given, in-degrees into ioff in the same sweep.
// Every thread takes four consecutive entries per round, so that a list that turns out long (the
// small-frontier path is chosen on the previous batch's sizes) costs a quarter of the round trips.
#define EOFF_PER 4
__global__ __launch_bounds__(1024) void k_list_eoff(const uint32_t *list, const uint32_t *count_ptr,
                                                    const uint2 *out_meta, uint32_t *eoff, uint32_t *msgs_out,
                                                    const uint2 *in_meta, uint32_t *ioff, uint32_t *isum_out) {
    __shared__ uint32_t wo[16], wi[16];
    __shared__ uint32_t carry_o, carry_i;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint32_t count = *count_ptr;
    const bool want_o = eoff != nullptr, want_i = in_meta != nullptr && ioff != nullptr;   // kernel arguments: uniform
    if (tid == 0) {
        carry_o = 0;
        carry_i = 0;
    }
    __syncthreads();
    for (uint32_t base = 0; base < count; base += 1024 * EOFF_PER) {
        const uint32_t i0 = base + tid * EOFF_PER;
        uint32_t v[EOFF_PER], dgo[EOFF_PER], dgi[EOFF_PER];
#pragma unroll
        for (int k = 0; k < EOFF_PER; ++k) v[k] = (i0 + k < count) ? list[i0 + k] : 0u;
        uint32_t so = 0, si = 0;
#pragma unroll
        for (int k = 0; k < EOFF_PER; ++k) {
            const bool on = i0 + k < count;
            dgo[k] = (on && want_o) ? out_meta[v[k]].y : 0u;
            dgi[k] = (on && want_i) ? in_meta[v[k]].y : 0u;
            so += dgo[k];
            si += dgi[k];
        }
        uint32_t inc_o = so, inc_i = si;
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t to = __shfl_up(inc_o, o), ti = __shfl_up(inc_i, o);
            if (lane >= o) {
                inc_o += to;
                inc_i += ti;
            }
        }
        if (lane == 63) {
            wo[wave] = inc_o;
            wi[wave] = inc_i;
        }
        __syncthreads();
        uint32_t off_o = carry_o, off_i = carry_i;
        for (int k = 0; k < wave; ++k) {
            off_o += wo[k];
            off_i += wi[k];
        }
        uint32_t run_o = off_o + inc_o - so, run_i = off_i + inc_i - si;
#pragma unroll
        for (int k = 0; k < EOFF_PER; ++k) {
            if (i0 + k < count) {
                if (want_o) eoff[i0 + k] = run_o;
                if (want_i) ioff[i0 + k] = run_i;
            }
            run_o += dgo[k];
            run_i += dgi[k];
        }
        __syncthreads();
        if (tid == 1023) {
            carry_o = off_o + inc_o;
            carry_i = off_i + inc_i;
        }
        __syncthreads();
    }
    if (tid == 0) {
        if (want_o) {
            eoff[count] = carry_o;
            if (msgs_out) *msgs_out = carry_o;
        }
        if (want_i) {
            ioff[count] = carry_i;
            if (isum_out) *isum_out = carry_i;
        }
    }
}

// allow_disc: the hop may discover its set (pair_cap > 0 then: without a list the launch that discovers marks)
void rp_launch_frontier_mark(ripple_ctx *c, uint32_t l, bool allow_disc, uint32_t pair_cap) {
    if (pair_cap) {
        const ListWalk w = {c->pairs, c->out_w, c->pair_w, c->pair_cnt, rp_list_cut(c, c->last_m[l] ? c->last_m[l] : pair_cap), pair_cap,
                            rp_layer_attn(c, l) ? 1 : 0, c->opt_sorted == 2, c->bm[l - 1], c->bm_sink, c->bm_vadd, c->in_meta, rp_gat_long_min(c)};
        const auto kernel = c->layers[l - 1].agg == RIPPLE_AGG_WSUM ? k_frontier_list<1> : k_frontier_list<0>;
        hipLaunchKernelGGL(kernel, dim3(c->n_cu * 2), dim3(1024), 0, c->stream, c->list[l - 1], &c->ctr->set[l - 1].a, c->eoff[l - 1],
                           c->out_meta, c->out_pool, c->mk, c->ctr, l, c->xw[l], c->opt_scatter, c->opt_pull_ratio, allow_disc ? 1 : 0, w);
        return;
    }
    hipLaunchKernelGGL(k_frontier_mark, dim3(c->n_cu * 8), dim3(256), 0, c->stream, c->list[l - 1], &c->ctr->set[l - 1].a, c->eoff[l - 1],
                       c->out_meta, c->out_pool, c->mk);
}

// all live vertices, ascending, in c->all_list (count in ctr->n_all) with the exclusive scan of
// their in-degrees in c->ioff_all: the work list of a discovering hop
void rp_launch_alive_list(ripple_ctx *c) {
    CompactArgs a;
    memset(&a, 0, sizeof(a));
    a.list_cap = 0xFFFFFFFFu;
    a.bm = c->alive;                               // rewritten with the same bits
    a.alive = c->alive;
    a.n_words = c->n_words;
    a.out_meta = c->out_meta;
    a.in_meta = c->in_meta;
    a.want_in = 1;
    a.part_cnt = c->part_cnt;
    a.part_out = c->part_deg;
    a.part_in = c->part_ideg;
    a.part_tch = c->part_tch;
    a.list = c->all_list;
    a.ioff = c->ioff_all;
    a.count_out = &c->ctr->n_all;
    launch_compact(c, a);
}

// bitmap of layer l, merged with S, V_added (and A_{l-1} when self_term) -> list[l], ctr->set[l].a;
// want_out: eoff[l] and ctr->set[l].m (the next hop's edge walk); want_in: ioff[l], ctr->isum[l]
// pruned: bm[l] already is the hop's final set (max / min layers: candidates whose aggregate did not
// change have been taken out again), so neither marks nor S are merged into it
void rp_launch_frontier_compact(ripple_ctx *c, uint32_t l, bool self_term, bool want_out, bool want_in,
                                bool accumulate_rep, bool pruned, uint32_t gat_cap) {
    CompactArgs a;
    a.gat = gat_cap ? c->ctr : nullptr;
    a.gat_l = l;
    a.gat_cap = gat_cap;
    a.gat_long = rp_gat_long_min(c);
    a.gat_force = c->opt_sorted == 2;
    a.rec_list = c->ioff_all;                      // (the live vertices' prefix is made anew behind an attention hop)
    a.rec_count = &c->ctr->n_rec;
    a.bm = c->bm[l];
    a.mk = pruned ? nullptr : c->mk;
    a.bm_prev = self_term ? c->bm[l - 1] : nullptr;
    a.bm_sink = pruned ? nullptr : c->bm_sink;
    a.bm_vadd = c->bm_vadd;
    a.alive = c->alive;
    a.n_words = c->n_words;
    a.out_meta = c->out_meta;
    a.in_meta = c->in_meta;
    a.want_out = want_out ? 1 : 0;
    a.want_in = want_in ? 1 : 0;
    a.part_cnt = c->part_cnt;
    a.part_out = c->part_deg;
    a.part_in = c->part_ideg;
    a.part_tch = c->part_tch;
    a.part_rec = c->part_rec;
    a.done.flag = nullptr;
    a.rep = accumulate_rep ? c->rep[l] : nullptr;
    a.touched_out = pruned ? nullptr : &c->ctr->touched[l];
    a.list = c->list[l];
    a.eoff = c->eoff[l];
    a.ioff = c->ioff[l];
    a.count_out = &c->ctr->set[l].a;
    a.msgs_out = &c->ctr->set[l].m;
    a.isum_out = &c->ctr->isum[l];
    a.list_cap = 0xFFFFFFFFu;
    launch_compact(c, a);
}

// Candidates of a max / min hop: the vertices marked by the out-edge walk from A_{l-1}, S and V_added,
// into bm[l] and, ascending, into c->all_list (count in ctr->n_all). The aggregation kernel then
// clears the bits of those whose aggregate stays as it is.
void rp_launch_candidates(ripple_ctx *c, uint32_t l) {
    CompactArgs a;
    memset(&a, 0, sizeof(a));
    a.list_cap = 0xFFFFFFFFu;
    a.bm = c->bm[l];
    a.mk = c->mk;
    a.bm_sink = c->bm_sink;
    a.bm_vadd = c->bm_vadd;
    a.alive = c->alive;
    a.n_words = c->n_words;
    a.out_meta = c->out_meta;
    a.in_meta = c->in_meta;
    a.part_cnt = c->part_cnt;
    a.part_out = c->part_deg;
    a.part_in = c->part_ideg;
    a.part_tch = c->part_tch;
    a.touched_out = &c->ctr->touched[l];
    a.want_in = 1;                                 // for the hops that recompute every candidate, and for the choice of the next batch
    a.list = c->all_list;
    a.ioff = c->ioff_all;
    a.isum_out = &c->ctr->isum[l];
    a.count_out = &c->ctr->n_all;
    launch_compact(c, a);
}

static void bitmap_ids(ripple_ctx *c, CompactArgs &a, bool report) {
    a.done.flag = nullptr;
    const uint32_t nb = rp_div_up(a.n_words, 32);
    if (a.n_words <= RANK_WORDS) {
        if (report && nb <= REPORT_WGS) a.done = rp_host_flag(c);
        hipLaunchKernelGGL(k_bitmap_ids, dim3(nb), dim3(256), 0, c->stream, a);
    } else {
        launch_compact(c, a);
    }
    if (report && !a.done.flag) rp_launch_report(c);
}

// any bitmap & alive -> ascending list in `out_list` (room for cap), count in *count_d (both device memory, or pinned host memory)
void rp_launch_bitmap_to_list(ripple_ctx *c, uint32_t *bitmap, uint32_t *out_list, uint32_t cap, uint32_t *count_d, bool report) {
    CompactArgs a;
    memset(&a, 0, sizeof(a));
    a.list_cap = cap;
    a.bm = bitmap;
    a.alive = c->alive;
    a.n_words = c->n_words;
    a.out_meta = c->out_meta;
    a.in_meta = c->in_meta;
    a.part_cnt = c->part_cnt;
    a.part_out = c->part_deg;
    a.part_in = c->part_ideg;
    a.part_tch = c->part_tch;
    a.list = out_list;
    a.count_out = count_d;
    bitmap_ids(c, a, report);
}

// ---------------------------------------------------------------------------------
// the same compaction without any allocation: block sums in a static device array
// ---------------------------------------------------------------------------------
// Per-block partial sums of the two-pass compaction (three arrays of RP_STATIC_BLOCKS entries: vertex
// counts, and the out- and in-degree sums the first pass writes alongside). One copy per GPU, shared by
// every context on that GPU and kept until the process ends; every launch writes the entries it reads,
// so nothing has to be cleared between calls, and calls that overlap on one GPU race on it.
static __device__ __align__(256) uint32_t scratch[3 * RP_STATIC_BLOCKS];
#define RP_MAX_DEVICES 64
static uint32_t *g_scratch_ptr[RP_MAX_DEVICES] = {nullptr};    // the array's address on each GPU

uint32_t rp_static_max_vertices() { return RP_STATIC_BLOCKS * 256u * 32u; }

// Called by init_graph with the context's device current: looks the array's address up once per GPU.
ripple_status rp_static_scratch_init(ripple_ctx *c) {
    if (c->device < 0 || c->device >= RP_MAX_DEVICES) return RIPPLE_OK;      // such a GPU has no no-allocation path
    if (g_scratch_ptr[c->device]) return RIPPLE_OK;
    uint32_t *ptr = nullptr;
    RP_HIP(c, hipGetSymbolAddress((void **)&ptr, HIP_SYMBOL(scratch)));
    g_scratch_ptr[c->device] = ptr;
    return RIPPLE_OK;
}

// bitmap & alive -> ascending ids in ids_out (device, room for cap), set size in *n_out (device). Allocates nothing.
ripple_status rp_launch_affected_static(ripple_ctx *c, uint32_t *bitmap, uint32_t *ids_out, uint32_t cap,
                                        uint32_t *n_out) {
    uint32_t *ptr = (c->device >= 0 && c->device < RP_MAX_DEVICES) ? g_scratch_ptr[c->device] : nullptr;
    if (!ptr) {
        c->err = "the static scratch array was not set up for this GPU";
        return RIPPLE_ESTATE;
    }
    if (rp_div_up(c->n_words, 256) > RP_STATIC_BLOCKS) {
        c->err = "vertex capacity " + std::to_string(c->n_cap) + " exceeds what the no-allocation call supports (" +
                 std::to_string(rp_static_max_vertices()) + ")";
        return RIPPLE_EINVAL;
    }
    CompactArgs a;
    memset(&a, 0, sizeof(a));
    a.bm = bitmap;
    a.alive = c->alive;
    a.n_words = c->n_words;
    a.out_meta = c->out_meta;
    a.in_meta = c->in_meta;
    a.part_cnt = ptr;
    a.part_out = ptr + RP_STATIC_BLOCKS;
    a.part_in = ptr + 2 * RP_STATIC_BLOCKS;
    a.list = ids_out;
    a.list_cap = cap;
    a.count_out = n_out;
    bitmap_ids(c, a, false);
    RP_HIP(c, hipGetLastError());
    // The call's contract is a synchronised stream. The wait for an event behind the last launch gives it and costs 5 us more than a
    // word in pinned memory would; hipStreamSynchronize goes over every launch since the last one and costs 16 more.
    RP_HIP(c, hipEventRecord(c->idle, c->stream));
    RP_HIP(c, hipEventSynchronize(c->idle));
    return RIPPLE_OK;
}

SparseArgs rp_sparse_args(ripple_ctx *c, uint32_t l, uint32_t *list, uint32_t *count, bool self_term) {
    SparseArgs sp;
    sp.bm = c->bm[l];
    sp.alive = c->alive;
    sp.list = list;
    sp.count = count;
    sp.touched = &c->ctr->touched[l];
    sp.st_dst = c->st_dst;
    sp.n_struct = &c->ctr->n_struct;
    sp.struct_cap = c->struct_cap;
    sp.list0 = c->list[0];
    sp.count0 = &c->ctr->set[0].a;
    sp.bm_vadd = c->bm_vadd;
    sp.self_term = self_term ? 1 : 0;
    sp.in_meta = c->in_meta;
    sp.long_min = 0;
    sp.long_list = nullptr;
    sp.long_count = nullptr;
    sp.long_dup = 0;
    sp.eoff = nullptr;
    sp.out_meta = c->out_meta;
    sp.isum = &c->ctr->isum[l];
    return sp;
}

// Candidates of a small max / min hop, listed while they are marked: the set of rp_launch_candidates
// (with A_{l-1} when the layer has a self term) in bm[l] and, unordered, in c->all_list, count in
// ctr->cand[l] (zero since the batch began).
void rp_launch_candidates_sparse(ripple_ctx *c, uint32_t l, bool self_term, uint32_t long_min) {
    SparseArgs sp = rp_sparse_args(c, l, c->all_list, &c->ctr->cand[l], self_term);
    sp.long_min = long_min;                              // candidates with longer in-rows: straight into the queue of the
    sp.long_list = c->eoff[l];                           // workgroup role (free until the hop's set is final), count in
    sp.long_count = &c->ctr->n_long[l];                  // ctr->n_long[l] (zero since the batch began)
    hipLaunchKernelGGL(k_frontier_sparse, dim3(c->n_cu), dim3(256), 0, c->stream, c->list[l - 1], &c->ctr->set[l - 1].a,
                       c->eoff[l - 1], c->out_meta, c->out_pool, sp);
}

// Hop l for a small frontier: out-edge walk from A_{l-1} and the roots (S, V_added, A_{l-1} when self_term)
// straight into bm[l] and list[l] (unordered), then the degree prefixes over that list. Two launches
// instead of the walk plus a scan of the whole bitmap.
// long_min > 0 (attention hops): vertices with more in-neighbours than that are also queued in c->all_list
// (count in ctr->n_long[l], zero since the batch began) for the workgroup role of the aggregation kernel. Nothing reads an in-degree prefix there, and the
// out-degrees' is written along with the list: no second launch (9 us for 1,400 vertices, 20 for 4,300).
void rp_launch_frontier_sparse(ripple_ctx *c, uint32_t l, bool self_term, bool want_out, uint32_t long_min) {
    SparseArgs sp = rp_sparse_args(c, l, c->list[l], &c->ctr->set[l].a, self_term);
    if (long_min) {
        sp.long_min = long_min;
        sp.long_list = c->all_list;
        sp.long_count = &c->ctr->n_long[l];
        sp.long_dup = 1;
        if (want_out) sp.eoff = c->eoff[l];
    }
    hipLaunchKernelGGL(k_frontier_sparse, dim3(c->n_cu), dim3(256), 0, c->stream, c->list[l - 1], &c->ctr->set[l - 1].a,
                       c->eoff[l - 1], c->out_meta, c->out_pool, sp);
    if (!long_min) rp_launch_list_offsets(c, l, want_out);
}

// degree prefixes over the (unordered) list of hop l
void rp_launch_list_offsets(ripple_ctx *c, uint32_t l, bool want_out) {
    hipLaunchKernelGGL(k_list_eoff, dim3(1), dim3(1024), 0, c->stream, c->list[l], &c->ctr->set[l].a, c->out_meta,
                       want_out ? c->eoff[l] : (uint32_t *)nullptr,
                       want_out ? &c->ctr->set[l].m : (uint32_t *)nullptr, c->in_meta, c->ioff[l],
                       &c->ctr->isum[l]);
}
