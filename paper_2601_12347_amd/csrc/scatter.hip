// Delta aggregation (the Send / Aggregate steps of Sec. 3.3): every vertex u of
// A_{l-1} sends m = h_u(new) - h_u(old) (Sec. 3.3.3, sum) along its out-edges
// of the updated graph and the messages arriving at v are added into the cached
// un-normalised sum X^l[v] (the vertex's hop-l inbox, Sec. 3.3.2). Mean needs
// no separate message: X stays a plain sum and the in-degree divides it when
// the row is transformed.
//
// Push kernel: the flattened (source, out-edge) space is cut into equal chunks
// via the out-degree prefix, one wavefront walks a chunk, holds the source's
// delta row in registers across that source's edges and adds it to the
// destination rows with hardware float atomics (order-free, Sec. 3.3.3).
//
// Bootstrap kernel: X^l[v] = sum over v's in-row of H^{l-1}, cut over edges like the pull.
#include "common.h"
#include "kernels.h"
#include "pull_scan.h"
#include "push.h"
#include "walk.h"



typedef uint32_t uintx2 __attribute__((ext_vector_type(2)));

template <int NJ, int PK, int WT>
__global__ __launch_bounds__(256) void k_scatter_push(const uint32_t *list, const uint32_t *count_ptr,
                                                      const uint32_t *eoff, const float *D, uint32_t ldd, uint32_t d,
                                                      const uint2 *out_meta, const uint32_t *out_pool, const float *out_w, float *X,
                                                      DevCtr *ctr, uint32_t l, int mode, int ratio, uint32_t list_cap, int list_force) {
    if (list_cap) {
        const int hm = rp_hop_mode(ctr, l, d, mode, ratio, 0);
        const uint32_t cp = *count_ptr;
        if (rp_hop_listed(ctr, l, d, cp ? count_ptr[1] : 0u, list_cap, list_force, hm)) return;
    }
    if (*count_ptr && blockIdx.x == 0 && threadIdx.x == 0) ctr->hop_mode[l] = 1u + RP_HOP_PUSH;
    push_edges<NJ, PK, WT>(list, count_ptr, eoff, D, nullptr, 0u, ldd, d, out_meta, out_pool, out_w, X, (blockIdx.x * blockDim.x + threadIdx.x) >> 6,
                       (gridDim.x * blockDim.x) >> 6);
}

// (hops that may be pulled: rp_launch_scatter_pull)
void rp_launch_scatter_push(ripple_ctx *c, uint32_t l, uint32_t pair_cap) {
    const bool proj = c->layers[l - 1].proj != 0;           // project-first: messages are already d_out wide
    const uint32_t d = c->xw[l];
    const bool packed = proj && c->layers[l - 1].packed;
    const float *D = packed ? (const float *)c->MSG : (proj ? c->PD : c->D[(l - 1) & 1]);
    const uint32_t ldd = proj ? c->pd_ld : d;
    dim3 grid(c->n_cu * 8), block(256);
    const bool wt = c->layers[l - 1].agg == RIPPLE_AGG_WSUM;
#define PUSH_CASE_WT(NJ, PK, WT)                                                                                   \
    hipLaunchKernelGGL((k_scatter_push<NJ, PK, WT>), grid, block, 0, c->stream, c->list[l - 1], &c->ctr->set[l - 1].a,     \
                       c->eoff[l - 1], D, ldd, d, c->out_meta, c->out_pool, c->out_w, c->X[l], c->ctr, l,  \
                       c->opt_scatter, c->opt_pull_ratio, pair_cap, c->opt_sorted == 2 ? 1 : 0)
#define PUSH_CASE_PK(NJ, PK)                     \
    do {                                         \
        if (wt) PUSH_CASE_WT(NJ, PK, 1);         \
        else PUSH_CASE_WT(NJ, PK, 0);            \
    } while (0)
#define PUSH_CASE(NJ) PUSH_CASE_PK(NJ, 0)
    if (packed) PUSH_CASE_PK(1, 1);
    else if (d <= 64) PUSH_CASE(1);
    else if (d <= 128) PUSH_CASE(2);
    else if (d <= 256) PUSH_CASE(4);
    else if (d <= 512) PUSH_CASE(8);
    else PUSH_CASE(16);
#undef PUSH_CASE
#undef PUSH_CASE_PK
#undef PUSH_CASE_WT
}

// ---------------------------------------------------------------------------------
// pull: segmented reduction over in-rows, keeping only the sources that are in A_{l-1}
// ---------------------------------------------------------------------------------
// The flattened in-edge space of the listed destinations is cut into chunks of up to 256 edges (rp_run_cut) and every
// wavefront takes a contiguous run of chunks, so the row of a chunk's first edge follows from the
// previous chunk instead of a search over the whole list. The 64 rows after that one (vertex, pool
// position, first edge) sit in registers, one per lane; an edge finds its row with shuffles. The next
// chunk's rows are requested before the gathers of the current one.
// DISC = 0: destinations are A_l. DISC = 1 (discovering hop): destinations are all live vertices and
// those that receive a message are marked in the hop's bitmap.
// DET = 1, the deterministic mode's form of both pull kernels. Float addition does not commute bit for bit, so
// every sum has to be taken in an order that is a function of the graph and the batches alone:
//   * the graph store keeps the order of an in-row such a function (rows built in the order the edges were given,
//     appended entries put in id order, holes filled by a fixed rule), the list of destinations is ascending, and
//     the cut of the in-edge space into chunks and of the chunks into runs (every nw-th run is one wavefront's)
//     depends on their number and the grid only;
//   * within a run a wavefront carries a destination's partial sum from chunk to chunk, so a run finishes every
//     destination once. Only the destinations of a run's first and last in-edge can have in-edges in another run;
//     their sums go to two side entries per run instead of memory, and k_pull_fixup adds the entries of one
//     destination in run order. All other rows are written with plain loads and stores by their only writer.
// The changed edges' structural terms have been added before the first hop, in that order too (k_det_terms).
// Bootstrap inference runs the same kernels with every destination marked as recomputed: every in-edge of such a
// row contributes, with the source's current row (of H^{l-1}, or of T for a project-first layer) in place of a
// message, and the sum replaces the row. The hop is always pulled.
//
// WT = 1: every message is multiplied by its edge's weight (weighted sum, m = alpha (h - h_old), Sec. 3.3.3)
__device__ __forceinline__ bool pull_is_listed(const PullArgs &a, int hop_mode) {
    if (!a.sorted_cap) return false;
    const uint32_t cp = *a.m_count;
    return rp_hop_listed(a.ctr, a.l, a.d, cp ? a.m_count[1] : 0u, a.sorted_cap, a.sorted_force, hop_mode);
}
// Whether the hop is pulled (DISC = 0) or discovered by the launch that asks. If not, and nothing else has been launched for it, the launch pushes the
// hop's messages (rows of NJ times 64 columns, PK: packed), or marks its set: a launch of its own that turns out to have nothing to do takes 7 us.
template <int NJ, int PK, int DISC, int WT>
__device__ __forceinline__ bool pull_or_others(const PullArgs &a) {
    const int hm = rp_hop_mode(a.ctr, a.l, a.d, a.mode, a.ratio, a.allow_disc);
    const uint32_t gw = (blockIdx.x * blockDim.x + threadIdx.x) >> 6, nw = (gridDim.x * blockDim.x) >> 6;
    if (DISC) {
        if (hm == RP_HOP_DISCOVER) return true;
        if (a.others) frontier_walk<false>(a.out_list, a.m_count, a.out_eoff, a.out_meta, a.out_pool, a.mk, SparseArgs(), gw, nw);
        return false;
    }
    if (hm == RP_HOP_DISCOVER || pull_is_listed(a, hm)) return false;
    if (hm == RP_HOP_PULL) return true;
    if (a.others) {
        if (*a.m_count && blockIdx.x == 0 && threadIdx.x == 0) a.ctr->hop_mode[a.l] = 1u + RP_HOP_PUSH;
        push_edges<NJ, PK, WT>(a.out_list, a.m_count, a.out_eoff, a.D, nullptr, 0u, a.ldd, a.d, a.out_meta, a.out_pool, a.out_w, a.X, gw, nw);
    }
    return false;
}

template <int NJ, int DISC, int WT, int DET>
__global__ __launch_bounds__(256) void k_scatter_pull(PullArgs a) {
    static_assert(!DET || (!DISC && !WT), "the deterministic form pulls into A_l, unweighted");
    if constexpr (!DET)
        if (!pull_or_others<NJ, 0, DISC, WT>(a)) return;
    const uint32_t count = *a.count_ptr;
    if (count == 0) return;
    if (blockIdx.x == 0 && threadIdx.x == 0) a.ctr->hop_mode[a.l] = 1u + (DISC ? RP_HOP_DISCOVER : RP_HOP_PULL);
    constexpr int G = (NJ >= 8) ? 2 : 16 / NJ;              // rows gathered per round trip
    constexpr int T = PULL_CHUNK / 64;                      // in-edges examined per lane and chunk
    __shared__ uint2 s_e[4][PULL_CHUNK];                    // the chunk's messages: source, destination
    __shared__ float s_w[WT ? 4 : 1][WT ? PULL_CHUNK : 1];
    const int lane = rp_lane(), wave = threadIdx.x >> 6;
    const uint32_t d = a.d;
    const uint32_t total = a.ioff[count];
    const uint32_t gw = (blockIdx.x * blockDim.x + threadIdx.x) >> 6, nw = (gridDim.x * blockDim.x) >> 6;
    const RunCut cut = rp_run_cut(total, nw);
    const uint32_t n_chunks = cut.n_chunks;
    // The chunks are handed out in runs (PULL_RUN chunks on large hops, one chunk when there are fewer chunks than
    // wavefronts would need). A wavefront starts with the run of its own number; after that it fetches runs from a
    // counter until none is left, or, in the deterministic mode, takes every nw-th run (a cut that depends on the
    // number of chunks and the grid alone). One long contiguous run per wavefront is what the first version had:
    // chunks differ in cost (a stretch of short in-rows ends a sum every few edges), stretches of such chunks exist
    // (the vertices that earlier batches created sit together at the end of the id range), and the few wavefronts
    // that owned such a stretch held up the hop (3.4 instead of 2.1 ms after 400 batches that each create 100
    // vertices; in the deterministic mode 7.4 instead of 2.5 ms at hop 2).
    const uint32_t per = cut.per, n_runs = cut.n_runs;
    uint32_t run = gw;                                      // the first run needs no counter
    if (DET && n_runs > a.side_runs) {                      // cannot happen: the side entries are sized for the in-row pool
        if (gw == 0 && lane == 0) a.ctr->error = 9;
        return;
    }
    if (run >= n_runs) {
        if (DET && lane == 0)
            for (; run < a.side_runs; run += nw) a.side_v[2 * run] = a.side_v[2 * run + 1] = 0xFFFFFFFFu;
        return;
    }
    uint32_t c_begin = run * per;
    uint32_t c_end = min(n_chunks, c_begin + per);
    PullScan<T, WT> scan;
    scan.begin(a, count, c_begin * cut.chunk, lane);
    constexpr uint32_t NONE = 0xFFFFFFFFu;
    uint32_t cur = NONE;                                    // destination whose partial sum is held
    const bool rec = DET && a.bm_rec != nullptr;            // every destination is recomputed from all its in-neighbours (bootstrap), or none
    float acc[NJ], xo[NJ];                                  // ... and its old row, where nobody else writes it
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[j] = xo[j] = 0.0f;
    // the destinations of the run's first and last in-edge may have in-edges in other runs: atomics, or (DET) side entries; whether a sum was left for them
    uint32_t v_head = (uint32_t)__shfl((int)scan.rv, 0), v_tail = a.list[rp_seg_search_wave(a.ioff, 0, count - 1, min(total, c_end * cut.chunk) - 1u)];
    bool wrote_head = false, wrote_tail = false;
    // All others have one writer: the old row is read beside the destination's first message and stored with the sum. (Atomics take 3.2 ps a number
    // wherever they go, 30 K rows of 256 numbers alone 24 us: 62 K messages to them 38 us, so 29. The old row read when the sum is complete, as the
    // deterministic mode did, is a stall per destination: 40 K messages to 21 K rows of 256 73 us, with atomics 35, so 25.)
    auto flush = [&]() {
        float *xr = a.X + (size_t)cur * d;
        const bool shared = cur == v_head || cur == v_tail;
        if (DET && shared) {
            xr = a.side_acc + (size_t)(2 * run + (cur == v_head ? 0u : 1u)) * d;
            if (cur == v_head) wrote_head = true;
            else wrote_tail = true;
        }
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            const uint32_t col = lane + 64 * j;
            if (col < d) {
                if (DET && (shared || rec)) xr[col] = acc[j];
                else if (!shared) xr[col] = xo[j] + acc[j];
                else if (acc[j] != 0.0f) unsafeAtomicAdd(&xr[col], acc[j]);
            }
            acc[j] = 0.0f;
        }
        if (DISC && lane == 0) atomicOr(&a.bm_cur[cur >> 5], 1u << (cur & 31));   // once per receiver and wavefront
    };
    for (;;) {
    for (uint32_t c = c_begin; c < c_end; ++c) {
        const uint32_t e0 = c * cut.chunk, e1 = min(total, e0 + cut.chunk);
        uint32_t my_v[T], my_u[T];
        float my_w[WT ? T : 1];
        bool dirty[T];
        scan.chunk(a, count, e0, e1, lane, my_v, my_u, my_w, dirty);
        // the chunk's messages, in edge order
        uint32_t n = 0;
#pragma unroll
        for (int t = 0; t < T; ++t) {
            const bool on = dirty[t] || (rec && e0 + 64u * t + lane < e1);
            const unsigned long long mask = __ballot(on);
            const uint32_t pos = n + __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
            if (on) {
                s_e[wave][pos] = make_uint2(my_u[t], my_v[t]);
                if (WT) s_w[wave][pos] = my_w[t];
            }
            n += (uint32_t)__popcll(mask);
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");   // (LDS accesses of one wavefront are executed in order)
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        for (uint32_t k0 = 0; k0 < n; k0 += G) {
            uint32_t v[G];
            float r[G][NJ], x[G][NJ], w[WT ? G : 1];
            uint32_t before = cur;
            auto rows = [&](auto read) {                     // (past the list's end: its last row again, not added)
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    const uint32_t idx = min(k0 + (uint32_t)g, n - 1u);
                    const uint2 e = s_e[wave][idx];
                    const uint32_t u = (uint32_t)__builtin_amdgcn_readfirstlane((int)e.x);
                    v[g] = (uint32_t)__builtin_amdgcn_readfirstlane((int)e.y);
                    if (WT) w[WT ? g : 0] = s_w[wave][idx];
#pragma unroll
                    for (int j = 0; j < NJ; ++j) r[g][j] = read(u, min((uint32_t)lane + 64u * j, d - 1u));
                    const bool own = v[g] != before && v[g] != v_head && v[g] != v_tail && !rec;   // the first message of an unshared destination
                    before = v[g];
#pragma unroll
                    for (int j = 0; j < NJ; ++j) x[g][j] = own ? a.X[(size_t)v[g] * d + min((uint32_t)lane + 64u * j, d - 1u)] : 0.0f;
                }
            };
            if (!rec) rows([&](uint32_t u, uint32_t col) { return a.D[(size_t)u * a.ldd + col]; });
            else if (a.R) rows([&](uint32_t u, uint32_t col) { return a.R[(size_t)u * a.ldr + col]; });
            else rows([&](uint32_t u, uint32_t col) { return rp_load_h(a.Hprev, a.store, (size_t)u * d + col); });
#pragma unroll
            for (int g = 0; g < G; ++g) {
                if (k0 + (uint32_t)g >= n) continue;
                if (v[g] != cur) {                           // the destination changes: flush its partial sum
                    if (cur != NONE) flush();
                    cur = v[g];
#pragma unroll
                    for (int j = 0; j < NJ; ++j) xo[j] = x[g][j];
                }
#pragma unroll
                for (int j = 0; j < NJ; ++j) acc[j] = WT ? __builtin_fmaf(r[g][j], w[WT ? g : 0], acc[j]) : acc[j] + r[g][j];
            }
        }
        __builtin_amdgcn_wave_barrier();                     // the next chunk overwrites the list
        scan.advance();                                      // the destination and its partial sum carry over to the next chunk
    }
    if (cur != NONE) flush();
    cur = NONE;
    if (DET) {
        if (lane == 0) {
            a.side_v[2 * run] = wrote_head ? v_head : NONE;
            a.side_v[2 * run + 1] = wrote_tail ? v_tail : NONE;
        }
        wrote_head = wrote_tail = false;
        run += nw;
    } else {
        if ((unsigned long long)nw * per >= n_chunks) break;      // every run was somebody's first
        run = nw + rp_next_run(&a.ctr->pull_next[a.l], lane);
    }
    if (run >= n_runs) break;
    c_begin = run * per;
    c_end = min(n_chunks, c_begin + per);
    scan.begin(a, count, c_begin * cut.chunk, lane);
    v_head = (uint32_t)__shfl((int)scan.rv, 0);
    v_tail = a.list[rp_seg_search_wave(a.ioff, 0, count - 1, min(total, c_end * cut.chunk) - 1u)];
    }
    if (DET && lane == 0)                                         // the runs of this wavefront's numbers that do not exist
        for (; run < a.side_runs; run += nw) a.side_v[2 * run] = a.side_v[2 * run + 1] = NONE;
}

// The same hop from the list of its messages. A pull finds the messages by testing every in-neighbour of every vertex
// of A_l against the bitmap of A_{l-1}; when few of them carry a message (hop 2 of a large batch on the dense
// graph: 4.6 M of 110 M), those tests, each a request to the L2 that a compute unit can only have so many of in
// flight, are most of the hop; a push adds every number with an atomic of its own. The out-edge walk that marks A_l has every message
// in its hands and writes it down as a (destination, source) pair in the bucket of its destination (k_frontier_list); k_list_order puts
// every bucket's pairs in order, one bucket's behind the other's; and this kernel is the pull's inner part over that list: every
// wavefront takes a contiguous run of pairs, gathers the sources' rows G at a time and sums while the destination stays.
// Measured: hop 2 of 10,000 updates on the dense graph (4.6 M messages of 1 KB to 1.5 M rows) 0.33 ms for walk and list (pairs in edge
// order, then a radix sort) + 1.02 -> 0.15 + 1.02; hop 3 of 100 updates (3 M packed messages to 1 M rows) 0.48 (pushed) -> 0.07 + 0.18.
// A workgroup per bucket that orders it in LDS and sums it at once took 1.23 ms and 0.28 ms for the second part: while it
// orders, nothing is on its way.
struct ListArgs {
    const uint2 *pairs;
    uint2 *sorted;
    const float *pair_w;           // weighted sums: the edges' weights, beside the pairs
    float *sorted_w;
    uint32_t *cnt;
    ListCut cut;
    const uint32_t *m_count;       // |A_{l-1}| and, in the next word, the number of messages
    uint32_t cap;
    int force;
    const float *D;
    uint32_t ldd, d;
    uint32_t msg_bytes;            // packed messages: size of the table in bytes, below 4 GB
    float *X;
    DevCtr *ctr;
    uint32_t l;
    int mode, ratio, allow_disc;
    int attn;                      // an attention hop (rp_gat_listed)
};

// Whether the hop was listed at all (M: its messages), and whether the list is what moves them
__device__ __forceinline__ bool list_is_used(const ListArgs &a, uint32_t &M, bool &made) {
    const uint32_t cp = *a.m_count;
    M = cp ? a.m_count[1] : 0u;
    if (a.attn) {
        made = rp_gat_list_made(a.ctr, M, a.cap, a.force);
        return made && !a.ctr->pair_over[a.l];
    }
    const int hm = rp_hop_mode(a.ctr, a.l, a.d, a.mode, a.ratio, a.allow_disc);
    made = M > 0 && M <= a.cap && hm != RP_HOP_DISCOVER;
    return rp_hop_listed(a.ctr, a.l, a.d, M, a.cap, a.force, hm);
}

// A workgroup per bucket: its pairs counted per destination in LDS, then put in place behind the pairs of the buckets before it. The order
// within a destination is that in which the pairs come up.
template <int WT>
__global__ __launch_bounds__(256) void k_list_order(ListArgs a) {
    uint32_t M;
    bool made;
    if (!list_is_used(a, M, made)) return;
    __shared__ uint32_t s_at[RP_LIST_IDS];
    __shared__ uint32_t s_sum[4], s_before[4];
    constexpr int PER = 8;
    const uint32_t tid = threadIdx.x, bucket = blockIdx.x, ids = 1u << a.cut.shift, mask = ids - 1u;
    const uint32_t n = a.cnt[bucket];
    uint32_t before = 0;
    for (uint32_t b = tid; b < bucket; b += 256u) before += a.cnt[b];
    const uint2 *from = a.pairs + (size_t)bucket * a.cut.room;
    for (uint32_t i = tid; i < ids; i += 256u) s_at[i] = 0;
    __syncthreads();
    for (uint32_t c0 = tid; c0 < n; c0 += 256u * PER) {
        uint32_t v[PER];
#pragma unroll
        for (int k = 0; k < PER; ++k) v[k] = from[min(c0 + 256u * k, n - 1u)].x;
#pragma unroll
        for (int k = 0; k < PER; ++k)
            if (c0 + 256u * k < n) atomicAdd(&s_at[v[k] & mask], 1u);
    }
    __syncthreads();
    const uint32_t per = (ids + 255u) / 256u, i0 = min(ids, tid * per), i1 = min(ids, i0 + per);
    uint32_t mine = 0;
    for (uint32_t i = i0; i < i1; ++i) mine += s_at[i];
    const uint32_t incl = rp_wave_scan(mine);
    before = rp_wave_scan(before);
    if ((tid & 63u) == 63u) {
        s_sum[tid >> 6] = incl;
        s_before[tid >> 6] = before;
    }
    __syncthreads();
    uint32_t at = s_before[0] + s_before[1] + s_before[2] + s_before[3] + incl - mine;
    if (a.attn && bucket == gridDim.x - 1u && tid == 0) a.ctr->pairs[a.l] = s_before[0] + s_before[1] + s_before[2] + s_before[3] + n;
    for (uint32_t w = 0; w < (tid >> 6); ++w) at += s_sum[w];
    for (uint32_t i = i0; i < i1; ++i) {
        const uint32_t n_i = s_at[i];
        s_at[i] = at;
        at += n_i;
    }
    __syncthreads();
    for (uint32_t c0 = tid; c0 < n; c0 += 256u * PER) {
        uint2 p[PER];
        float w[PER];
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const uint32_t i = min(c0 + 256u * k, n - 1u);
            p[k] = from[i];
            w[k] = WT ? a.pair_w[(size_t)bucket * a.cut.room + i] : 1.0f;
        }
#pragma unroll
        for (int k = 0; k < PER; ++k)
            if (c0 + 256u * k < n) {
                const uint32_t to = atomicAdd(&s_at[p[k].x & mask], 1u);
                a.sorted[to] = p[k];
                if (WT) a.sorted_w[to] = w[k];
            }
    }
}

// the buckets' counts cleared for the next hop that is listed
__device__ __forceinline__ void list_clear(const ListArgs &a) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < a.cut.n) a.cnt[i] = 0;
}

template <int NJ, int WT>
__global__ __launch_bounds__(256) void k_scatter_list(ListArgs a) {
    uint32_t M;
    bool made;
    const bool used = list_is_used(a, M, made);
    if (made) list_clear(a);
    if (!used) return;
    if (blockIdx.x == 0 && threadIdx.x == 0) a.ctr->hop_mode[a.l] = 1u + RP_HOP_SORTED;
    constexpr int G = (NJ >= 8) ? 2 : 4;                    // message rows per round trip (and up to as many destination rows)
    constexpr uint32_t NONE = 0xFFFFFFFFu;
    const int lane = rp_lane();
    const uint32_t d = a.d;
    const uint32_t n_chunks = (M + 63u) / 64u;
    const uint32_t gw = (blockIdx.x * blockDim.x + threadIdx.x) >> 6, nw = (gridDim.x * blockDim.x) >> 6;
    const uint32_t per = (n_chunks + nw - 1) / nw;
    const uint32_t c_begin = min(n_chunks, gw * per), c_end = min(n_chunks, c_begin + per);
    if (c_begin >= c_end) return;
    // A destination whose pairs all lie inside this wavefront's run has no other writer: its row is read like one
    // more message when its first pair comes up, summed with the messages and stored with plain stores (a row of
    // float atomics costs the L2 one operation per number: 1.5 M rows of 256 took 0.9 ms that way, more than the
    // gathers). Only the destinations of the run's first and last pair can have pairs in a neighbour's run; their sums
    // go to memory as atomic additions.
    const uint32_t v_first = a.sorted[c_begin * 64u].x, v_last = a.sorted[min(M, c_end * 64u) - 1u].x;
    uint32_t cur = NONE;
    float acc[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[j] = 0.0f;
    auto flush = [&]() {
        float *xr = a.X + (size_t)cur * d;
        const bool shared = cur == v_first || cur == v_last;
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            const uint32_t col = lane + 64 * j;
            if (col < d) {
                if (!shared) xr[col] = acc[j];
                else if (acc[j] != 0.0f) unsafeAtomicAdd(&xr[col], acc[j]);
            }
        }
    };
    uint32_t e = c_begin * 64u + lane;
    uint2 nx = (e < M) ? a.sorted[e] : make_uint2(NONE, 0u);
    float nx_w = (WT && e < M) ? a.sorted_w[e] : 1.0f;
    for (uint32_t c = c_begin; c < c_end; ++c) {
        const uint2 my = nx;
        const float my_w = nx_w;
        const uint32_t n = min(64u, M - c * 64u);
        e += 64u;                                            // the next chunk's pairs are on their way during the gathers
        nx = (c + 1 < c_end && e < M) ? a.sorted[e] : make_uint2(NONE, 0u);
        if (WT) nx_w = (c + 1 < c_end && e < M) ? a.sorted_w[e] : 1.0f;
        for (uint32_t k0 = 0; k0 < n; k0 += G) {
            float r[G][NJ], rx[G][NJ], w[G];
            uint32_t vk[G];
            uint32_t prev = cur;                             // every pair before k0 has been summed: cur is pair k0 - 1's destination
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const int k = (int)min(k0 + g, 63u);
                const uint32_t uk = (uint32_t)__builtin_amdgcn_readlane((int)my.y, k);
                vk[g] = (uint32_t)__builtin_amdgcn_readlane((int)my.x, k);
                w[g] = WT ? __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(my_w), k)) : 1.0f;
                const bool live = k0 + g < n;
                const bool own = live && vk[g] != prev && vk[g] != v_first && vk[g] != v_last;   // first pair of an unshared destination
                prev = vk[g];
#pragma unroll
                for (int j = 0; j < NJ; ++j) {
                    const uint32_t col = lane + 64 * j;
                    r[g][j] = (live && col < d) ? a.D[(size_t)uk * a.ldd + col] : 0.0f;
                    rx[g][j] = (own && col < d) ? a.X[(size_t)vk[g] * d + col] : 0.0f;
                }
            }
#pragma unroll
            for (int g = 0; g < G; ++g) {
                if (k0 + g < n) {
                    if (vk[g] != cur) {
                        if (cur != NONE) flush();
                        cur = vk[g];
#pragma unroll
                        for (int j = 0; j < NJ; ++j) acc[j] = rx[g][j];
                    }
#pragma unroll
                    for (int j = 0; j < NJ; ++j) acc[j] = WT ? __builtin_fmaf(w[g], r[g][j], acc[j]) : acc[j] + r[g][j];
                }
            }
        }
    }
    if (cur != NONE) flush();
}

// The same hop for packed message rows (one 128-byte line each, see rp_msg_encode). Decoding a row costs a dozen
// vector instructions whatever the number of lanes that take part, and a wavefront's instruction rate, not the
// memory system, is what bounds a one-line gather; so a row is handled by 16 lanes (8 bytes = three columns
// each) and a wavefront works on four messages, a quad, at a time. The dirty in-edges of a chunk are first
// compacted (source, destination, weight) into LDS in edge order, i.e. sorted by destination; quad k is entries
// 4k .. 4k+3, one per 16-lane group. While all four belong to the destination being summed, every group adds its
// message to its own partial sums. A quad in which the destination changes is taken entry by entry; a change
// first adds the four groups' partial sums together and sends the row to memory as one 47-lane atomic addition
// (the atomic units take about three cycles per lane, so the number of such rows, not of instructions, is what
// counts). The destination and the partial sums carry over from chunk to chunk: a wavefront adds to a row once,
// however many chunks the row's in-edges span.
// Rows of up to 64 floats (not packed) are taken the same way, four columns per lane: 16, 8 or 4 lanes per row and 4, 8 or 16
// rows at a time. F names the form: 0 packed, else the lanes per row of floats.
// (A lane per column and a row per instruction before, 31 M edges, a discovering hop: 16 columns 700 us, 23 weighted ones 771, 60 737; now 411, 435, 585.)
template <int F>
struct RowForm {
    static constexpr int LANES = F ? F : 16;                // per row
    static constexpr int ROWS = 64 / LANES;                 // per load instruction
    static constexpr int LOADS = F == 4 ? 2 : 4;            // in flight per wavefront
    static constexpr int V = F ? 4 : 3;                     // columns per lane: 4 sub .. 4 sub + 3 (packed: sub, 16 + sub, 32 + sub)
};
typedef float floatx4u __attribute__((ext_vector_type(4), aligned(4)));   // (rows of floats begin at any multiple of four bytes)
// The groups' partial sums added up; what comes back is the column that this lane sends to memory (row_column), one per row of 16 lanes. Every
// step halves what a lane still has to add, and none goes through LDS: lanes 8 and 4 apart by rotations within a row, then two rows' columns
// trade places and are added (permlane16_swap and permlane32_swap: odd rows of the first operand, or its upper half, against even rows, or
// the lower half, of the second). With two or three shuffles per column in their place a sum of a few messages cost more than its gathers.
template <int F>
__device__ __forceinline__ float rows_sum(float (&acc)[RowForm<F>::V]) {
    constexpr int V = RowForm<F>::V, LANES = RowForm<F>::LANES;
#pragma unroll
    for (int j = 0; j < V; ++j) {
        if (LANES <= 8) acc[j] += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(acc[j]), 0x128, 0xf, 0xf, false));   // row_ror:8
        if (LANES <= 4) acc[j] += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(acc[j]), 0x124, 0xf, 0xf, false));   // row_ror:4
    }
    const float s = swap_add32(swap_add16(acc[0], acc[1]), swap_add16(acc[2], acc[V - 1]));   // (V = 3: the fourth row's is not used)
#pragma unroll
    for (int j = 0; j < V; ++j) acc[j] = 0.0f;
    return s;
}
template <int F>
__device__ __forceinline__ uint32_t row_column(uint32_t lane) {    // (beyond any row: nothing to send)
    const uint32_t row = lane >> 4, sub = lane & 15u;
    if (row >= (uint32_t)RowForm<F>::V || sub >= (uint32_t)RowForm<F>::LANES) return 0xFFFFFFFFu;
    return F ? 4u * sub + row : 16u * row + sub;
}
#define PULL4_PAD 0xFFFFFFFEu                               // destination of the entries that fill a chunk's last round
template <int F, int DISC, int WT, int DET>
__global__ __launch_bounds__(256) void k_scatter_pull4(PullArgs a) {
    static_assert(!DET || (!DISC && !WT && !F), "the deterministic form pulls into A_l, unweighted, packed rows");
    if constexpr (!DET)
        if (!pull_or_others<1, F ? 0 : 1, DISC, WT>(a)) return;
    const uint32_t count = *a.count_ptr;
    if (count == 0) return;
    if (blockIdx.x == 0 && threadIdx.x == 0) a.ctr->hop_mode[a.l] = 1u + (DISC ? RP_HOP_DISCOVER : RP_HOP_PULL);
    constexpr int T = PULL_CHUNK / 64;
    constexpr uint32_t NONE = 0xFFFFFFFFu;
    constexpr int LANES = RowForm<F>::LANES, ROWS = RowForm<F>::ROWS, LOADS = RowForm<F>::LOADS, V = RowForm<F>::V;
    constexpr uint32_t LIST = PULL_CHUNK + ROWS * LOADS;    // a round always reads ROWS * LOADS entries
    // per dirty in-edge: (packed: byte offset of the source's message row, else the source; destination); what the inner loop needs per
    // load is then one 8-byte LDS read and one addition (rows of floats: a multiplication as well) in front of it
    __shared__ uint2 s_e[4][LIST];
    __shared__ float s_w[WT ? 4 : 1][WT ? LIST : 1];
    const int lane = rp_lane(), wave = threadIdx.x >> 6;
    const uint32_t grp = (uint32_t)lane / LANES, sub = (uint32_t)lane & (LANES - 1u);
    const uint32_t d = a.d;
    const uint32_t total = a.ioff[count];
    const uint32_t gw = (blockIdx.x * blockDim.x + threadIdx.x) >> 6, nw = (gridDim.x * blockDim.x) >> 6;
    const RunCut cut = rp_run_cut(total, nw);
    const uint32_t n_chunks = cut.n_chunks;
    // runs of chunks: every nw-th one (DET) or fetched from a counter, see k_scatter_pull
    const uint32_t per = cut.per, n_runs = cut.n_runs;
    uint32_t run = gw;                                      // the first run needs no counter
    if (DET && n_runs > a.side_runs) {                      // cannot happen: the side entries are sized for the in-row pool
        if (gw == 0 && lane == 0) a.ctr->error = 9;
        return;
    }
    if (run >= n_runs) {
        if (DET && lane == 0)
            for (; run < a.side_runs; run += nw) a.side_v[2 * run] = a.side_v[2 * run + 1] = NONE;
        return;
    }
    uint32_t c_begin = run * per;
    uint32_t c_end = min(n_chunks, c_begin + per);
    // message rows through a buffer descriptor: 32-bit byte offsets (row offset from LDS + this lane's chunk)
    const __amdgpu_buffer_rsrc_t mres = __builtin_amdgcn_make_buffer_rsrc((void *)a.D, 0, a.msg_bytes, 0x00020000u);
    const uint32_t sub8 = 8u * sub;
    const float *frow = a.D + (4u * sub < d ? 4u * sub : 0u);   // rows of floats: lanes beyond the row repeat its first columns
    const uint32_t my_col = row_column<F>((uint32_t)lane);        // the column this lane sends to memory
    const bool sends = my_col < d;
    uint32_t cur = NONE;                                    // destination being summed (the same in all lanes)
    const bool rec = DET && a.bm_rec != nullptr;            // every destination is recomputed (see k_scatter_pull)
    float acc[V];                                           // this group's partial sums
#pragma unroll
    for (int j = 0; j < V; ++j) acc[j] = 0.0f;
    PullScan<T, WT> scan;
    scan.begin(a, count, c_begin * cut.chunk, lane);
    uint32_t v_head = NONE, v_tail = NONE;                  // DET: see k_scatter_pull
    bool wrote_head = false, wrote_tail = false;
    if (DET) {
        v_head = (uint32_t)__shfl((int)scan.rv, 0);
        v_tail = a.list[rp_seg_search_wave(a.ioff, 0, count - 1, min(total, c_end * cut.chunk) - 1u)];
    }
    auto flush = [&]() {
        const float mine = rows_sum<F>(acc);
        if (!DET) {
            if (sends && mine != 0.0f) unsafeAtomicAdd(&a.X[(size_t)cur * d + my_col], mine);
            if (DISC && lane == 0) atomicOr(&a.bm_cur[cur >> 5], 1u << (cur & 31));
        } else if (cur == v_head || cur == v_tail) {
            if (cur == v_head) wrote_head = true;
            else wrote_tail = true;
            if (sends) a.side_acc[(size_t)(2 * run + (cur == v_head ? 0u : 1u)) * d + my_col] = mine;
        } else if (sends) {
            float *x = &a.X[(size_t)cur * d + my_col];
            if (rec) *x = mine;
            else if (mine != 0.0f) unsafeAtomicAdd(x, mine);
        }
    };
    for (;;) {
    for (uint32_t c = c_begin; c < c_end; ++c) {
        const uint32_t e0 = c * cut.chunk, e1 = min(total, e0 + cut.chunk);
        uint32_t my_v[T], my_u[T];
        float my_w[WT ? T : 1];
        bool dirty[T];
        scan.chunk(a, count, e0, e1, lane, my_v, my_u, my_w, dirty);
        // compact the dirty edges, in edge order
        uint32_t n = 0;
#pragma unroll
        for (int t = 0; t < T; ++t) {
            if (DET) dirty[t] = dirty[t] || (rec && e0 + 64 * t + lane < e1);
            const unsigned long long mask = __ballot(dirty[t]);
            const uint32_t pos = n + __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
            if (dirty[t]) {
                s_e[wave][pos] = make_uint2(F ? my_u[t] : my_u[t] << 7, my_v[t]);
                if (WT) s_w[wave][pos] = my_w[t];
            }
            n += (uint32_t)__popcll(mask);
        }
        // the entries a round reads past the list's end: row 0 (valid memory), a destination that never matches
        if (lane < ROWS * LOADS) {
            s_e[wave][n + lane] = make_uint2(0u, PULL4_PAD);
            if (WT) s_w[wave][n + lane] = 0.0f;
        }
        // LDS accesses of one wavefront are executed in order, so the loads below see the stores above without a
        // workgroup barrier; the fence keeps the compiler from moving them across each other
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        for (uint32_t k0 = 0; k0 < n; k0 += ROWS * LOADS) {
            uint2 ent[LOADS];
            uint2 ch[LOADS];
            floatx4u fr[F ? LOADS : 1];
            float tv[DET ? LOADS : 1][3];                    // DET: the three columns of a recomputed row's source
#pragma unroll
            for (int r = 0; r < LOADS; ++r) {
                const uint32_t idx = k0 + ROWS * r + grp;
                ent[r] = s_e[wave][idx];
                if constexpr (F != 0) {
                    fr[r] = *(const floatx4u *)(frow + (size_t)ent[r].x * a.ldd);
                } else if (DET && rec) {
                    const float *t = a.R + (size_t)(ent[r].x >> 7) * a.ldr;
                    tv[DET ? r : 0][0] = t[sub];
                    tv[DET ? r : 0][1] = t[16u + sub];
                    tv[DET ? r : 0][2] = (32u + sub < d) ? t[32u + sub] : 0.0f;
                    ch[r] = make_uint2(0u, 0u);
                } else {
                    const uintx2 w2 = __builtin_bit_cast(uintx2, __builtin_amdgcn_raw_buffer_load_b64(mres, ent[r].x + sub8, 0, 0));
                    ch[r] = make_uint2(w2.x, w2.y);
                }
            }
#pragma unroll
            for (int r = 0; r < LOADS; ++r) {
                if (k0 + ROWS * r < n) {
                    // packed: the three columns as (integer, as a float) x (the chunk's power of two): one fused
                    // multiply-add per column takes them into the sums (the product is exact)
                    float q[V], f = 1.0f;
                    const float wk = WT ? s_w[wave][k0 + ROWS * r + grp] : 1.0f;   // (read again here: registers)
                    if constexpr (F != 0) {
#pragma unroll
                        for (int j = 0; j < V; ++j) q[j] = fr[r][j];
                        f = wk;
                    } else {
                        rp_msg_decode_parts(ch[r], q[0], q[1], q[2], f);
                        if (DET && rec) {
#pragma unroll
                            for (int j = 0; j < V; ++j) q[j] = tv[DET ? r : 0][j];
                            f = 1.0f;
                        }
                        if (WT) f *= wk;                     // a power of two times the weight: exact
                    }
                    auto add = [&]() {
#pragma unroll
                        for (int j = 0; j < V; ++j) acc[j] = (F && !WT) ? acc[j] + q[j] : __builtin_fmaf(q[j], f, acc[j]);
                    };
                    if (!__any(ent[r].y != cur)) {           // all of them go on
                        add();
                    } else {                                 // destination by destination (they are in order)
                        unsigned long long left = __ballot(ent[r].y != PULL4_PAD);
                        while (left) {
                            const int first = __ffsll((long long)left) - 1;
                            const uint32_t vg = (uint32_t)__builtin_amdgcn_readlane((int)ent[r].y, first);
                            if (vg != cur) {
                                if (cur != NONE) flush();
                                cur = vg;
                            }
                            const bool same = ent[r].y == vg;
                            if (same) add();
                            left &= ~__ballot(same);
                        }
                    }
                }
            }
        }
        __builtin_amdgcn_wave_barrier();                    // the next chunk overwrites the lists
        scan.advance();
    }
    if (cur != NONE) flush();
    cur = NONE;
    if (DET) {
        if (lane == 0) {
            a.side_v[2 * run] = wrote_head ? v_head : NONE;
            a.side_v[2 * run + 1] = wrote_tail ? v_tail : NONE;
        }
        wrote_head = wrote_tail = false;
        run += nw;
    } else {
        if ((unsigned long long)nw * per >= n_chunks) break;      // every run was somebody's first
        run = nw + rp_next_run(&a.ctr->pull_next[a.l], lane);
    }
    if (run >= n_runs) break;
    c_begin = run * per;
    c_end = min(n_chunks, c_begin + per);
    scan.begin(a, count, c_begin * cut.chunk, lane);
    if (DET) {
        v_head = (uint32_t)__shfl((int)scan.rv, 0);
        v_tail = a.list[rp_seg_search_wave(a.ioff, 0, count - 1, min(total, c_end * cut.chunk) - 1u)];
    }
    }
    if (DET && lane == 0)                                         // the runs of this wavefront's numbers that do not exist
        for (; run < a.side_runs; run += nw) a.side_v[2 * run] = a.side_v[2 * run + 1] = NONE;
}

// The list of a hop's messages (see k_scatter_list) where they are packed rows or rows of up to 64 floats: several at a time, like k_scatter_pull4. The
// destination's row, if no other run has pairs of it, is read with its first message and stored with the sum.
template <int F, int WT>
__global__ __launch_bounds__(256) void k_scatter_list4(ListArgs a) {
    uint32_t M;
    bool made;
    const bool used = list_is_used(a, M, made);
    if (made) list_clear(a);
    if (!used) return;
    if (blockIdx.x == 0 && threadIdx.x == 0) a.ctr->hop_mode[a.l] = 1u + RP_HOP_SORTED;
    constexpr uint32_t NONE = 0xFFFFFFFFu;
    constexpr int LANES = RowForm<F>::LANES, ROWS = RowForm<F>::ROWS, LOADS = RowForm<F>::LOADS, V = RowForm<F>::V;
    const int lane = rp_lane();
    const uint32_t d = a.d, grp = (uint32_t)lane / LANES, sub = (uint32_t)lane & (LANES - 1u);
    const uint32_t n_chunks = (M + 63u) / 64u;
    const uint32_t gw = (blockIdx.x * blockDim.x + threadIdx.x) >> 6, nw = (gridDim.x * blockDim.x) >> 6;
    const uint32_t per = (n_chunks + nw - 1) / nw;
    const uint32_t c_begin = min(n_chunks, gw * per), c_end = min(n_chunks, c_begin + per);
    if (c_begin >= c_end) return;
    const __amdgpu_buffer_rsrc_t mres = __builtin_amdgcn_make_buffer_rsrc((void *)a.D, 0, a.msg_bytes, 0x00020000u);
    const uint32_t col0 = 4u * sub < d ? 4u * sub : 0u;      // rows of floats: lanes beyond the row repeat its first columns
    const uint32_t my_col = row_column<F>((uint32_t)lane);        // the column this lane sends to memory
    const bool sends = my_col < d, has2 = 32u + sub < d;
    const uint32_t v_first = a.sorted[c_begin * 64u].x, v_last = a.sorted[min(M, c_end * 64u) - 1u].x;
    uint32_t cur = NONE;
    float acc[V];                                           // this group's partial sums
#pragma unroll
    for (int j = 0; j < V; ++j) acc[j] = 0.0f;
    auto flush = [&]() {
        const float mine = rows_sum<F>(acc);
        if (sends) {
            float *x = &a.X[(size_t)cur * d + my_col];
            if (cur != v_first && cur != v_last) *x = mine;
            else if (mine != 0.0f) unsafeAtomicAdd(x, mine);
        }
    };
    uint32_t e = c_begin * 64u + lane;
    uint2 nx = (e < M) ? a.sorted[e] : make_uint2(PULL4_PAD, 0u);
    float nx_w = (WT && e < M) ? a.sorted_w[e] : 0.0f;
    uint32_t before = NONE;                                 // the destination of the pair before the chunk
    for (uint32_t c = c_begin; c < c_end; ++c) {
        const uint2 my = nx;
        const float my_w = nx_w;
        const uint32_t n = min(64u, M - c * 64u);
        e += 64u;
        nx = (c + 1 < c_end && e < M) ? a.sorted[e] : make_uint2(PULL4_PAD, 0u);
        if (WT) nx_w = (c + 1 < c_end && e < M) ? a.sorted_w[e] : 0.0f;
        // which pairs are the first of a destination that nobody else writes
        uint32_t left = (uint32_t)__shfl_up((int)my.x, 1);
        left = lane == 0 ? before : left;
        const uint32_t first = my.x != left && my.x != v_first && my.x != v_last && my.x != PULL4_PAD ? 1u : 0u;
        before = (uint32_t)__shfl((int)my.x, 63);
        for (uint32_t k0 = 0; k0 < n; k0 += ROWS * LOADS) {
            uint32_t v[LOADS];
            uint2 ch[LOADS];
            floatx4u fr[F ? LOADS : 1];
            float x[LOADS][V], wk[LOADS];
#pragma unroll
            for (int r = 0; r < LOADS; ++r) {
                const int idx = (int)(k0 + ROWS * r + grp);  // below 64; past the list's end: row 0, no destination
                const uint32_t u = (uint32_t)__shfl((int)my.y, idx);
                v[r] = (uint32_t)__shfl((int)my.x, idx);
                wk[r] = WT ? __shfl(my_w, idx) : 1.0f;
                const bool own = __shfl((int)first, idx) != 0;
                if constexpr (F != 0) {
                    fr[r] = *(const floatx4u *)(a.D + (size_t)u * a.ldd + col0);
                    floatx4u old = {0.0f, 0.0f, 0.0f, 0.0f};
                    if (own) old = *(const floatx4u *)(a.X + (size_t)v[r] * d + col0);
#pragma unroll
                    for (int j = 0; j < V; ++j) x[r][j] = old[j];
                } else {
                    const uintx2 w2 = __builtin_bit_cast(uintx2, __builtin_amdgcn_raw_buffer_load_b64(mres, (u << 7) + 8u * sub, 0, 0));
                    ch[r] = make_uint2(w2.x, w2.y);
                    const float *xr = a.X + (size_t)v[r] * d + sub;
                    x[r][0] = own ? xr[0] : 0.0f;
                    x[r][1] = own ? xr[16] : 0.0f;
                    x[r][2] = own && has2 ? xr[32] : 0.0f;
                }
            }
#pragma unroll
            for (int r = 0; r < LOADS; ++r) {
                if (k0 + ROWS * r >= n) continue;
                float q[V], f;
                if constexpr (F != 0) {
#pragma unroll
                    for (int j = 0; j < V; ++j) q[j] = fr[r][j];
                    f = wk[r];
                } else {
                    rp_msg_decode_parts(ch[r], q[0], q[1], q[2], f);
                    if (WT) f *= wk[r];                      // a power of two times the weight: exact
                }
                if (!__any(v[r] != cur)) {                   // all of them go on
#pragma unroll
                    for (int j = 0; j < V; ++j) acc[j] = __builtin_fmaf(q[j], f, acc[j]);
                } else {                                     // destination by destination
                    unsigned long long left = __ballot(v[r] != PULL4_PAD);
                    while (left) {
                        const uint32_t vg = (uint32_t)__builtin_amdgcn_readlane((int)v[r], __ffsll((long long)left) - 1);
                        if (vg != cur) {
                            if (cur != NONE) flush();
                            cur = vg;
                        }
                        const bool same = v[r] == vg;
                        if (same)                            // (x is zero but for an unshared destination's first message)
#pragma unroll
                            for (int j = 0; j < V; ++j) acc[j] += __builtin_fmaf(q[j], f, x[r][j]);
                        left &= ~__ballot(same);
                    }
                }
            }
        }
    }
    if (cur != NONE) flush();
}

// Deterministic mode, after a DET pull: the side entries (two per run of chunks, in run order; entries of one
// destination are neighbours, apart from empty ones between them) are added up per destination in that order
// and the sum is added to the row, or replaces it if the row is recomputed. A wavefront per entry and all columns; the one that holds a
// destination's first entry does the work. The order of the additions is fixed, the reads are not: the entries around its own are read at once, then
// the old row and G parts of NB blocks of 64 columns are on their way at a time (one read per addition made the destination with the longest in-row,
// 40 entries of 256 columns, hold up the hop: 24 us; a wavefront per entry and block of columns, 60 K of them, took 17 us, now 14).
// Recomputed rows without any in-edge are zeroed here too: no in-edge, so the pull never met them.
template <int NB>
__global__ __launch_bounds__(256) void k_pull_fixup(PullArgs a, uint32_t n_entries, uint32_t pull_nw) {
    constexpr uint32_t NONE = 0xFFFFFFFFu;
    constexpr int G = NB <= 2 ? 16 : 32 / NB;
    const uint32_t count = *a.count_ptr;
    if (count == 0) return;
    n_entries = min(n_entries, 2u * rp_run_cut(a.ioff[count], pull_nw).n_runs);   // only the entries of runs that exist can hold anything
    const uint32_t lane = (uint32_t)rp_lane(), d = a.d;
    const uint32_t gw = (blockIdx.x * blockDim.x + threadIdx.x) >> 6, nw = (gridDim.x * blockDim.x) >> 6;
    for (uint32_t i = gw * 64u + lane; a.bm_rec && i < count; i += nw * 64u) {
        const uint32_t v = a.list[i];
        if (a.in_meta[v].y == 0 && rp_bit(a.bm_rec, v))
            for (uint32_t c = 0; c < d; ++c) a.X[(size_t)v * d + c] = 0.0f;
    }
    for (uint32_t k = gw; k < n_entries; k += nw) {
        uint32_t ahead = (k + lane < n_entries) ? a.side_v[k + lane] : NONE;         // lane 0: this entry
        uint32_t behind = (lane < k) ? a.side_v[k - 1u - lane] : NONE;               // lane 0: the nearest one
        const uint32_t v = (uint32_t)__builtin_amdgcn_readfirstlane((int)ahead);
        if (v == NONE) continue;
        // the nearest entry before k that is not empty: the same destination means k is not the first
        bool first = true;
        for (uint32_t b0 = k;;) {
            const unsigned long long m = __ballot(behind != NONE);
            if (m) first = (uint32_t)__shfl((int)behind, __ffsll((long long)m) - 1) != v;
            if (m || b0 <= 64u) break;
            b0 -= 64u;
            behind = (lane < b0) ? a.side_v[b0 - 1u - lane] : NONE;
        }
        if (!first) continue;
        const bool rec = a.bm_rec && rp_bit(a.bm_rec, v);
        float old[NB], t[NB];
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const uint32_t col = min(lane + 64u * b, d - 1u);
            old[b] = rec ? 0.0f : a.X[(size_t)v * d + col];
            t[b] = 0.0f;
        }
        for (uint32_t f0 = k;;) {
            unsigned long long same = __ballot(ahead == v);
            const unsigned long long other = __ballot(ahead != NONE && ahead != v);
            if (other) same &= (1ull << (__ffsll((long long)other) - 1)) - 1ull;     // entries past the first other destination are not ours
            while (same) {
                float part[G][NB];
                bool has[G];
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    has[g] = same != 0;
                    const uint32_t e = f0 + (uint32_t)(has[g] ? __ffsll((long long)same) - 1 : 0);
                    same &= same - 1;                                // (0 stays 0)
#pragma unroll
                    for (int b = 0; b < NB; ++b) part[g][b] = has[g] ? a.side_acc[(size_t)e * d + min(lane + 64u * b, d - 1u)] : 0.0f;
                }
#pragma unroll
                for (int g = 0; g < G; ++g)
#pragma unroll
                    for (int b = 0; b < NB; ++b)
                        if (has[g]) t[b] += part[g][b];
            }
            f0 += 64u;
            if (other || f0 >= n_entries) break;
            ahead = (f0 + lane < n_entries) ? a.side_v[f0 + lane] : NONE;
        }
#pragma unroll
        for (int b = 0; b < NB; ++b)
            if (lane + 64u * b < d) a.X[(size_t)v * d + lane + 64u * b] = old[b] + t[b];
    }
}

// discover = false: pull into A_l (the hop's list). true: scan every live vertex (c->all_list and
// c->ioff_all must have been produced by rp_launch_alive_list) and mark the receivers in bm[l].
// others: nothing else is launched to push the hop (discover = false), or to mark its set (true).
void rp_launch_scatter_pull(ripple_ctx *c, uint32_t l, bool discover, bool allow_disc, uint32_t pair_cap, bool others) {
    PullArgs a;
    a.others = others ? 1 : 0;
    a.out_list = c->list[l - 1];
    a.out_eoff = c->eoff[l - 1];
    a.out_meta = c->out_meta;
    a.out_pool = c->out_pool;
    a.mk = c->mk;
    a.m_count = &c->ctr->set[l - 1].a;
    a.sorted_cap = discover ? 0u : pair_cap;
    a.sorted_force = c->opt_sorted == 2;
    a.side_runs = 0;
    a.list = discover ? c->all_list : c->list[l];
    a.count_ptr = discover ? &c->ctr->n_all : &c->ctr->set[l].a;
    a.ioff = discover ? c->ioff_all : c->ioff[l];
    a.in_meta = c->in_meta;
    a.in_pool = c->in_pool;
    a.bm_prev = c->bm[l - 1];
    a.bm_cur = c->bm[l];
    const bool packed = c->layers[l - 1].proj && c->layers[l - 1].packed;
    a.D = packed ? (const float *)c->MSG : (c->layers[l - 1].proj ? c->PD : c->D[(l - 1) & 1]);
    a.d = c->xw[l];
    a.ldd = c->layers[l - 1].proj ? c->pd_ld : a.d;
    a.msg_bytes = (uint32_t)(c->n_cap * (RP_MSG_WORDS * 4u));   // packed layers exist below 2^25 vertices only
    a.X = c->X[l];
    a.ctr = c->ctr;
    a.l = l;
    a.mode = c->opt_scatter;
    a.ratio = c->opt_pull_ratio;
    a.allow_disc = allow_disc ? 1 : 0;
    dim3 grid(c->n_cu * 8), block(256);
    const bool wt = c->layers[l - 1].agg == RIPPLE_AGG_WSUM;
    a.in_w = wt ? c->in_w : nullptr;
    a.out_w = wt ? c->out_w : nullptr;
#define PULL_CASE(NJ)                                                                                      \
    do {                                                                                                   \
        if (discover && wt) hipLaunchKernelGGL((k_scatter_pull<NJ, 1, 1, 0>), grid, block, 0, c->stream, a);  \
        else if (discover) hipLaunchKernelGGL((k_scatter_pull<NJ, 1, 0, 0>), grid, block, 0, c->stream, a);   \
        else if (wt) hipLaunchKernelGGL((k_scatter_pull<NJ, 0, 1, 0>), grid, block, 0, c->stream, a);         \
        else hipLaunchKernelGGL((k_scatter_pull<NJ, 0, 0, 0>), grid, block, 0, c->stream, a);                 \
    } while (0)
#define PULL4_CASE(F)                                                                                      \
    do {                                                                                                   \
        if (discover && wt) hipLaunchKernelGGL((k_scatter_pull4<F, 1, 1, 0>), grid, block, 0, c->stream, a);  \
        else if (discover) hipLaunchKernelGGL((k_scatter_pull4<F, 1, 0, 0>), grid, block, 0, c->stream, a);   \
        else if (wt) hipLaunchKernelGGL((k_scatter_pull4<F, 0, 1, 0>), grid, block, 0, c->stream, a);         \
        else hipLaunchKernelGGL((k_scatter_pull4<F, 0, 0, 0>), grid, block, 0, c->stream, a);                 \
    } while (0)
    if (packed) PULL4_CASE(0);
    else if (a.d <= 16) PULL4_CASE(4);
    else if (a.d <= 32) PULL4_CASE(8);
    else if (a.d <= 64) PULL4_CASE(16);
    else if (a.d <= 128) PULL_CASE(2);
    else if (a.d <= 256) PULL_CASE(4);
    else if (a.d <= 512) PULL_CASE(8);
    else PULL_CASE(16);
#undef PULL_CASE
#undef PULL4_CASE
}

// About a thousand messages per bucket, so that a workgroup takes most of them in one round, and at most RP_LIST_IDS vertices (graphs of more
// than RP_LIST_BUCKETS times that have no lists)
ListCut rp_list_cut(const ripple_ctx *c, uint32_t messages) {
    uint32_t bits = 0, want = 8;
    while ((1ull << bits) < c->n_cap) ++bits;
    while ((1u << want) < RP_LIST_BUCKETS && ((messages >> want) > 1024u || (RP_LIST_IDS << want) < c->n_cap)) ++want;
    ListCut cut;
    cut.shift = bits > want ? bits - want : 0u;
    cut.n = ((c->n_cap - 1u) >> cut.shift) + 1u;
    cut.room = 2u * c->pair_cap / cut.n;
    return cut;
}

// From the list that k_frontier_list has made (the same pair_cap): nothing happens if it was not made or does not pay.
void rp_launch_list_order(ripple_ctx *c, uint32_t l, uint32_t pair_cap) {
    ListArgs a = {};
    a.attn = 1;
    a.pairs = c->pairs;
    a.sorted = c->pair_sorted;
    a.cnt = c->pair_cnt;
    a.cut = rp_list_cut(c, c->last_m[l] ? c->last_m[l] : pair_cap);
    a.m_count = &c->ctr->set[l - 1].a;
    a.cap = pair_cap;
    a.force = c->opt_sorted == 2;
    a.ctr = c->ctr;
    a.l = l;
    hipLaunchKernelGGL(k_list_order<0>, dim3(a.cut.n), dim3(256), 0, c->stream, a);
}
void rp_launch_scatter_list(ripple_ctx *c, uint32_t l, bool allow_disc, uint32_t pair_cap) {
    const LayerDev &ly = c->layers[l - 1];
    const bool packed = ly.proj && ly.packed;
    ListArgs a = {};
    a.pairs = c->pairs;
    a.sorted = c->pair_sorted;
    a.cnt = c->pair_cnt;
    a.cut = rp_list_cut(c, c->last_m[l] ? c->last_m[l] : pair_cap);
    a.m_count = &c->ctr->set[l - 1].a;
    a.cap = pair_cap;
    a.force = c->opt_sorted == 2;
    a.D = packed ? (const float *)c->MSG : (ly.proj ? c->PD : c->D[(l - 1) & 1]);
    a.d = c->xw[l];
    a.ldd = ly.proj ? c->pd_ld : a.d;
    a.msg_bytes = (uint32_t)(c->n_cap * (RP_MSG_WORDS * 4u));
    a.X = c->X[l];
    a.ctr = c->ctr;
    a.l = l;
    a.mode = c->opt_scatter;
    a.ratio = c->opt_pull_ratio;
    a.allow_disc = allow_disc ? 1 : 0;
    a.pair_w = c->pair_w;
    a.sorted_w = c->pair_w_sorted;
    const bool wt = ly.agg == RIPPLE_AGG_WSUM;
    if (wt) hipLaunchKernelGGL(k_list_order<1>, dim3(a.cut.n), dim3(256), 0, c->stream, a);
    else hipLaunchKernelGGL(k_list_order<0>, dim3(a.cut.n), dim3(256), 0, c->stream, a);
    const dim3 grid(c->n_cu * 8), block(256);
#define LIST_CASE(NJ)                                                                             \
    do {                                                                                          \
        if (wt) hipLaunchKernelGGL((k_scatter_list<NJ, 1>), grid, block, 0, c->stream, a);        \
        else hipLaunchKernelGGL((k_scatter_list<NJ, 0>), grid, block, 0, c->stream, a);           \
    } while (0)
#define LIST4_CASE(F)                                                                             \
    do {                                                                                          \
        if (wt) hipLaunchKernelGGL((k_scatter_list4<F, 1>), grid, block, 0, c->stream, a);        \
        else hipLaunchKernelGGL((k_scatter_list4<F, 0>), grid, block, 0, c->stream, a);           \
    } while (0)
    if (packed) LIST4_CASE(0);
    else if (a.d <= 16) LIST4_CASE(4);
    else if (a.d <= 32) LIST4_CASE(8);
    else if (a.d <= 64) LIST4_CASE(16);
    else if (a.d <= 128) LIST_CASE(2);
    else if (a.d <= 256) LIST_CASE(4);
    else if (a.d <= 512) LIST_CASE(8);
    else LIST_CASE(16);
#undef LIST_CASE
#undef LIST4_CASE
}

// Deterministic mode: the hop is pulled into A_l (bootstrap: into every live vertex, all of them recomputed;
// c->all_list and c->ioff_all must have been produced by rp_launch_alive_list), then the rows that more than
// one wavefront had in-edges of are finished.
void rp_launch_scatter_pull_det(ripple_ctx *c, uint32_t l, bool bootstrap) {
    const LayerDev &ly = c->layers[l - 1];
    PullArgs a = {};
    a.m_count = nullptr;
    a.sorted_cap = 0;
    a.sorted_force = 0;
    a.list = bootstrap ? c->all_list : c->list[l];
    a.count_ptr = bootstrap ? &c->ctr->n_all : &c->ctr->set[l].a;
    a.ioff = bootstrap ? c->ioff_all : c->ioff[l];
    a.in_meta = c->in_meta;
    a.in_pool = c->in_pool;
    a.in_w = nullptr;
    a.bm_prev = c->bm[l - 1];
    a.bm_cur = c->bm[l];
    const bool packed = ly.proj && ly.packed;
    a.D = packed ? (const float *)c->MSG : (ly.proj ? c->PD : c->D[(l - 1) & 1]);
    a.d = c->xw[l];
    a.ldd = ly.proj ? c->pd_ld : a.d;
    a.msg_bytes = (uint32_t)(c->n_cap * (RP_MSG_WORDS * 4u));
    a.X = c->X[l];
    a.ctr = c->ctr;
    a.l = l;
    a.mode = a.ratio = a.allow_disc = 0;
    a.bm_rec = bootstrap ? c->alive : nullptr;              // bootstrap: every listed vertex is recomputed; batches: none is
    a.Hprev = c->H[l - 1];
    a.R = ly.proj ? ly.T : nullptr;
    a.ldr = ly.ldt;
    a.store = c->store;
    a.side_v = c->side_v;
    a.side_acc = c->side_acc;
    dim3 grid(c->n_cu * 8), block(256);
    a.side_runs = c->side_runs;
    const uint32_t n_entries = 2u * c->side_runs;           // two per run
    const dim3 fix(std::min<uint32_t>(rp_div_up(n_entries, 4), c->n_cu * 8));
#define DET_CASE(NJ)                                                                                        \
    do {                                                                                                    \
        if (packed) hipLaunchKernelGGL((k_scatter_pull4<0, 0, 0, 1>), grid, block, 0, c->stream, a);        \
        else hipLaunchKernelGGL((k_scatter_pull<NJ, 0, 0, 1>), grid, block, 0, c->stream, a);               \
        hipLaunchKernelGGL(k_pull_fixup<NJ>, fix, block, 0, c->stream, a, n_entries, grid.x * 4u);          \
    } while (0)
    if (a.d <= 64) DET_CASE(1);
    else if (a.d <= 128) DET_CASE(2);
    else if (a.d <= 256) DET_CASE(4);
    else if (a.d <= 512) DET_CASE(8);
    else DET_CASE(16);
#undef DET_CASE
}

// ---------------------------------------------------------------------------------
// messages of a project-first layer
// ---------------------------------------------------------------------------------
// For every vertex u of A_{l-1}: P[u] = H^{l-1}[u] W_neigh has just been written to PD[u]. The message is what
// the receivers are still missing, m = P[u] - T[u], in the form it travels in: an fp32 row (left in PD[u];
// T[u] = P[u]) or a packed row (written to MSG[u]; T[u] += the values the packed numbers stand for, so what the
// rounding took away is part of u's next message). 16 lanes per row, three columns (c, 16 + c, 32 + c) each for
// packed rows; four rows per wavefront and step, two steps in flight.
__global__ __launch_bounds__(256) void k_messages(const uint32_t *list, const uint32_t *count_ptr, float *PD, uint32_t ldd,
                                                  float *T, uint32_t ldt, uint32_t d, uint32_t packed, uint32_t *MSG) {
    const uint32_t count = *count_ptr;
    const uint32_t lane = (uint32_t)rp_lane();
    const uint32_t gw = (blockIdx.x * blockDim.x + threadIdx.x) >> 6, nw = (gridDim.x * blockDim.x) >> 6;
    if (!packed) {                                          // any width: one wavefront per row, element by element
        constexpr int R = 8;
        for (uint32_t s0 = gw * R; s0 < count; s0 += nw * R) {
            uint32_t u[R];
#pragma unroll
            for (int r = 0; r < R; ++r) u[r] = list[min(s0 + r, count - 1u)];
            for (uint32_t col = lane; col < d; col += 64) {
                float p[R], t[R];
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    p[r] = PD[(size_t)u[r] * ldd + col];
                    t[r] = T[(size_t)u[r] * ldt + col];
                }
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    if (s0 + r >= count) continue;
                    PD[(size_t)u[r] * ldd + col] = p[r] - t[r];
                    T[(size_t)u[r] * ldt + col] = p[r];
                }
            }
        }
        return;
    }
    constexpr int R = 2;
    const uint32_t grp = lane >> 4, sub = lane & 15u;
    const bool has1 = 16u + sub < d, has2 = 32u + sub < d;
    for (uint32_t s0 = gw * 4u * R; s0 < count; s0 += nw * 4u * R) {
        uint32_t u[R];
        float p[R][3], t[R][3];
#pragma unroll
        for (int r = 0; r < R; ++r) u[r] = list[min(s0 + 4u * r + grp, count - 1u)];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const float *pr = PD + (size_t)u[r] * ldd;
            const float *tr = T + (size_t)u[r] * ldt;
            p[r][0] = pr[sub];
            t[r][0] = tr[sub];
            p[r][1] = has1 ? pr[16u + sub] : 0.0f;
            t[r][1] = has1 ? tr[16u + sub] : 0.0f;
            p[r][2] = has2 ? pr[32u + sub] : 0.0f;
            t[r][2] = has2 ? tr[32u + sub] : 0.0f;
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if (s0 + 4u * r + grp >= count) continue;
            float v0, v1, v2;
            const uint2 ch = rp_msg_encode(p[r][0] - t[r][0], p[r][1] - t[r][1], p[r][2] - t[r][2], v0, v1, v2);
            *(uint2 *)(MSG + (size_t)u[r] * RP_MSG_WORDS + 2u * sub) = ch;
            float *tr = T + (size_t)u[r] * ldt;
            tr[sub] = t[r][0] + v0;
            if (has1) tr[16u + sub] = t[r][1] + v1;
            if (has2) tr[32u + sub] = t[r][2] + v2;
        }
    }
}

void rp_launch_messages(ripple_ctx *c, uint32_t l) {
    const LayerDev &ly = c->layers[l - 1];
    const uint32_t hint = rp_rows_hint(c, l - 1);
    const uint32_t grid = std::max<uint32_t>(1u, std::min<uint32_t>(c->n_cu * 8, rp_div_up(hint, 4 * 8) + 1));
    hipLaunchKernelGGL(k_messages, dim3(grid), dim3(256), 0, c->stream, c->list[l - 1], &c->ctr->set[l - 1].a, c->PD, c->pd_ld,
                       ly.T, ly.ldt, c->xw[l], ly.packed, c->MSG);
}

// ---------------------------------------------------------------------------------
// max / min aggregation: keep, raise or recompute (Sec. 3.4.2)
// ---------------------------------------------------------------------------------
// A message carries the sender's old and new row. The owner of a candidate v (a vertex with a
// changed in-neighbour or a changed in-edge) decides, element by element:
//   * a new value that is at least as good as v's aggregate raises it (incremental case);
//   * an old value that equalled the aggregate and got worse may have been the one that set it; unless
//     another message reaches the aggregate again, the row is recomputed from all in-neighbours;
//   * anything else leaves the element alone.
// Recomputing is always right, so it is also taken where it is the cheaper way: for a created vertex
// and for a vertex with a short in-row whose in-edges changed, where reading the old and new rows of
// the changed in-neighbours would cost as much as reading every in-neighbour once, and as soon as one
// element is known to have lost its extreme. A vertex with a long in-row whose in-edges changed treats
// each changed edge as a message: an added edge sends its source's current row (no old value), a deleted
// one its source's pre-batch row as an old value that is gone.
// Rows whose aggregate ends up bit-equal to the old one are taken out of the hop's set again, so they
// are not transformed and send nothing on. There are no atomics on rows and the result does not
// depend on any order. One wavefront owns a candidate with up to long_min (at most MONO_LONG)
// in-neighbours; longer in-rows are queued and taken by a workgroup each, and a very long row that has
// to be recomputed is queued once more, in segments that a workgroup each reads.
#define MONO_LONG 256u
#define MONO_DIRTY_LIST 2048u     // changed in-neighbours of a long row remembered between counting and reading them
#define MONO_EDGE_HITS 1024u      // changed edges of one sink kept as messages; more: recompute
#define MONO_EDGE_SCAN 32768u     // longest list of changed edges a sink's workgroup searches; longer: recompute

struct MonoArgs {
    const uint32_t *list;          // candidates (ascending), or the queue of long rows
    const uint32_t *count_ptr;
    uint32_t *queue, *queue_count; // candidates with long in-rows, left to the workgroup kernel
    const uint2 *in_meta;
    const uint32_t *in_pool;
    const uint32_t *bm_prev;       // A_{l-1}: the in-neighbours whose row changed
    const uint32_t *bm_sink, *bm_vadd;
    uint32_t *bm_cur;              // the candidates on entry, the hop's set on exit
    const float *Dold;             // pre-batch rows of H^{l-1}, valid on A_{l-1}
    const void *Hprev;             // current H^{l-1}
    uint32_t d;
    float *X;
    int keep_prev;                 // the layer reads the vertex's own row: members of A_{l-1} stay in the set
    DevCtr *ctr;
    uint32_t l;
    // the batch's changed edges (source, sink, sign: < 0 deleted), read for sinks with long in-rows
    const uint32_t *st_src, *st_dst;
    const float *st_sign;
    uint32_t struct_cap;
    const uint32_t *alive;
    uint32_t long_min;             // in-rows longer than this (at most MONO_LONG) go to the workgroup kernel
    uint32_t split_min;            // in-rows of at least this many entries (at least ROW_SPLIT_MIN) are recomputed in segments
    uint32_t *out_list, *out_count; // small hops: the vertices that stay in the hop's set are appended here (or null)
    // very long rows that are recomputed: split into segments for k_scatter_mono_seg
    uint32_t *seg_v, *seg_done, *seg_base, *seg_r;
    float *seg_part;
    uint32_t big_cap, seg_cap, seg_ld;
};

template <int IS_MIN>
__device__ __forceinline__ bool mono_better(float a, float b) { return IS_MIN ? a < b : a > b; }

// Messages of the in-neighbours `mask` selects among the 64 ids held one per lane in my_u: inc becomes
// the best new value, lostm (bit j: column lane + 64 j) records elements whose old value equalled the
// aggregate and got worse. stop_early: return true as soon as such an element is not covered by inc.
template <int NJ, int IS_MIN, int STORE, int G>
__device__ __forceinline__ bool mono_messages(const MonoArgs &a, uint32_t my_u, unsigned long long mask, const float *xo,
                                              float *inc, uint32_t &lostm, bool stop_early) {
    const int lane = rp_lane();
    const uint32_t d = a.d;
    while (mask) {
        int kk[G];
        int n = 0;
#pragma unroll
        for (int g = 0; g < G; ++g) {
            kk[g] = 0;
            if (mask) {
                kk[g] = __ffsll((long long)mask) - 1;
                mask &= mask - 1;
                n = g + 1;
            }
        }
        float ro[G][NJ], rn[G][NJ];
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const uint32_t u = __shfl(my_u, kk[g]);
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                const uint32_t col = lane + 64 * j;
                const bool on = g < n && col < d;
                ro[g][j] = on ? a.Dold[(size_t)u * d + col] : 0.0f;
                rn[g][j] = on ? rp_load_h(a.Hprev, STORE, (size_t)u * d + col) : 0.0f;
            }
        }
        bool need = false;
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
#pragma unroll
            for (int g = 0; g < G; ++g) {
                if (g < n) {
                    if (mono_better<IS_MIN>(rn[g][j], inc[j])) inc[j] = rn[g][j];
                    if (ro[g][j] == xo[j] && mono_better<IS_MIN>(ro[g][j], rn[g][j])) lostm |= 1u << j;
                }
            }
            if (lane + 64 * j < (int)d && ((lostm >> j) & 1u) && mono_better<IS_MIN>(xo[j], inc[j])) need = true;
        }
        if (stop_early && __ballot(need) != 0ull) return true;
    }
    return false;
}

// Messages of changed in-edges of one sink, held one per lane (u = source, deleted = the edge went away)
// for the lanes in `mask`. A deleted edge sends its source's pre-batch row as a value that is gone: where
// it equalled the aggregate the element may have lost its extreme. An added edge sends the source's
// current row. Bit 31 of lostm: the pre-batch row is no longer there (the source was removed), recompute.
template <int NJ, int IS_MIN, int STORE>
__device__ __forceinline__ void mono_edge_messages(const MonoArgs &a, uint32_t my_u, bool my_deleted,
                                                   unsigned long long mask, const float *xo, float *inc, uint32_t &lostm) {
    const int lane = rp_lane();
    const uint32_t d = a.d;
    while (mask) {
        const int k = __ffsll((long long)mask) - 1;
        mask &= mask - 1;
        const uint32_t u = __shfl(my_u, k);
        const bool deleted = __shfl((int)my_deleted, k) != 0;
        if (deleted && !rp_bit(a.alive, u)) {
            lostm |= 1u << 31;
            continue;
        }
        const bool from_old = deleted && rp_bit(a.bm_prev, u);
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            const uint32_t col = lane + 64 * j;
            if (col >= d) continue;
            const float r = from_old ? a.Dold[(size_t)u * d + col] : rp_load_h(a.Hprev, STORE, (size_t)u * d + col);
            if (deleted) {
                if (r == xo[j]) lostm |= 1u << j;
            } else if (mono_better<IS_MIN>(r, inc[j])) {
                inc[j] = r;
            }
        }
    }
}

// best value per column over the rows of the `n_here` in-neighbours held one per lane in my_u, taken
// from lane `first` on in steps of `step`
template <int NJ, int IS_MIN, int STORE, int G>
__device__ __forceinline__ void mono_gather(const MonoArgs &a, uint32_t my_u, int n_here, float *xn) {
    const int lane = rp_lane();
    const uint32_t d = a.d;
    for (int k0 = 0; k0 < n_here; k0 += G) {
        float r[G][NJ];
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const bool on = k0 + g < n_here;
            const uint32_t u = __shfl(my_u, min(k0 + g, n_here - 1));
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                const uint32_t col = lane + 64 * j;
                r[g][j] = (on && col < d) ? rp_load_h(a.Hprev, STORE, (size_t)u * d + col) : xn[j];
            }
        }
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int j = 0; j < NJ; ++j)
                if (mono_better<IS_MIN>(r[g][j], xn[j])) xn[j] = r[g][j];
    }
}

// store the row if it differs from the old one, else take v out of the hop's set; returns "changed"
template <int NJ>
__device__ __forceinline__ bool mono_finish(const MonoArgs &a, uint32_t v, bool created, const float *xo, const float *xn) {
    const int lane = rp_lane();
    const uint32_t d = a.d;
    bool diff = false;
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        const uint32_t col = lane + 64 * j;
        if (col < d && xn[j] != xo[j]) diff = true;
    }
    const bool changed = __ballot(diff) != 0ull;
    if (changed) {
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            const uint32_t col = lane + 64 * j;
            if (col < d) a.X[(size_t)v * d + col] = xn[j];
        }
    }
    if (!changed && !created && !(a.keep_prev && rp_bit(a.bm_prev, v))) {
        if (lane == 0) atomicAnd(&a.bm_cur[v >> 5], ~(1u << (v & 31)));
    } else if (a.out_list && lane == 0) {
        a.out_list[atomicAdd(a.out_count, 1u)] = v;
    }
    return changed;
}

// wavefront gw of nw: the candidates gw, gw + nw, ... of the list
template <int NJ, int IS_MIN, int STORE>
__device__ __forceinline__ void mono_wave_role(const MonoArgs &a, uint32_t gw, uint32_t nw) {
    constexpr int GC = (NJ <= 4) ? 8 : 32 / NJ;                // senders in flight (two rows each)
    constexpr int GR = (NJ <= 2) ? 32 : 64 / NJ;               // rows in flight when recomputing: round trips pace a row
    constexpr int T = MONO_LONG / 64;
    const uint32_t count = *a.count_ptr;
    const int lane = rp_lane();
    const uint32_t d = a.d;
    const float ident = IS_MIN ? INFINITY : -INFINITY;
    uint32_t n_same = 0, n_inc = 0, n_rec = 0;
    for (uint32_t i = gw; i < count; i += nw) {
        const uint32_t v = a.list[i];
        const uint2 m = a.in_meta[v];
        if (m.y > a.long_min) {
            if (lane == 0) {
                if (a.queue) a.queue[atomicAdd(a.queue_count, 1u)] = v;
                else a.ctr->error = 9;                          // the long rows were meant to be sorted out already
            }
            continue;
        }
        const bool created = rp_bit(a.bm_vadd, v);
        float xo[NJ], xn[NJ];
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            const uint32_t col = lane + 64 * j;
            xo[j] = (col < d) ? a.X[(size_t)v * d + col] : 0.0f;
        }
        uint32_t my_u[T];
        unsigned long long dmask[T];
        uint32_t nd = 0;
#pragma unroll
        for (int t = 0; t < T; ++t) {
            const uint32_t e = 64 * t + lane;
            my_u[t] = (e < m.y) ? a.in_pool[m.x + e] : 0u;
            dmask[t] = __ballot(e < m.y && rp_bit(a.bm_prev, my_u[t]));
            nd += (uint32_t)__popcll(dmask[t]);
        }
        // reading old and new rows of nd senders against reading m.y rows once
        bool recompute = created || rp_bit(a.bm_sink, v) || 2 * nd >= m.y;
        if (!recompute) {
            float inc[NJ];
            uint32_t lostm = 0;
#pragma unroll
            for (int j = 0; j < NJ; ++j) inc[j] = ident;
#pragma unroll
            for (int t = 0; t < T; ++t)
                if (!recompute && dmask[t])
                    recompute = mono_messages<NJ, IS_MIN, STORE, GC>(a, my_u[t], dmask[t], xo, inc, lostm, true);
#pragma unroll
            for (int j = 0; j < NJ; ++j) xn[j] = mono_better<IS_MIN>(inc[j], xo[j]) ? inc[j] : xo[j];
        }
        if (recompute) {
#pragma unroll
            for (int j = 0; j < NJ; ++j) xn[j] = (m.y == 0) ? 0.0f : ident;     // no in-neighbours: zero
#pragma unroll
            for (int t = 0; t < T; ++t) {
                const int n_here = (int)min(64u, m.y - min(m.y, 64u * t));
                if (n_here > 0) mono_gather<NJ, IS_MIN, STORE, GR>(a, my_u[t], n_here, xn);
            }
        }
        const bool changed = mono_finish<NJ>(a, v, created, xo, xn);
        if (recompute) ++n_rec;
        else if (changed) ++n_inc;
        else ++n_same;
    }
    if (lane == 0) {
        if (n_same) atomicAdd(&a.ctr->mono[0][a.l], n_same);
        if (n_inc) atomicAdd(&a.ctr->mono[1][a.l], n_inc);
        if (n_rec) atomicAdd(&a.ctr->mono[2][a.l], n_rec);
    }
}

template <int NJ, int IS_MIN, int STORE>
__global__ __launch_bounds__(256) void k_scatter_mono(MonoArgs a) {
    mono_wave_role<NJ, IS_MIN, STORE>(a, (blockIdx.x * blockDim.x + threadIdx.x) >> 6, (gridDim.x * blockDim.x) >> 6);
}

// One workgroup of TEAM wavefronts per candidate with a long in-row: wavefront w takes the 64-entry
// blocks w, w + TEAM, ...; the wavefronts' partial results meet in LDS and wavefront 0 finishes the row.
// Workgroup bid of nb: the rows bid, bid + nb, ... of the queue.
template <int NJ, int IS_MIN, int STORE, int TEAM>
__device__ __forceinline__ void mono_team_role(const MonoArgs &a, uint32_t bid, uint32_t nb) {
    constexpr int GC = (NJ <= 4) ? 8 : 32 / NJ;
    constexpr int GR = (NJ <= 2) ? 32 : 64 / NJ;               // rows in flight: a long row is paced by round trips
    __shared__ float s_val[TEAM][NJ * 64];
    __shared__ uint32_t s_lost[TEAM][64];
    constexpr int IDS = 4;                                     // blocks of in-neighbour ids in flight while counting
    __shared__ uint32_t s_dirty[MONO_DIRTY_LIST];              // the changed in-neighbours of the row (while they fit)
    __shared__ uint32_t s_nd;
    __shared__ uint32_t s_flag;
    __shared__ uint32_t s_hit[MONO_EDGE_HITS];                 // the sink's entries in the list of changed edges
    __shared__ uint32_t s_nhit;
    __shared__ uint32_t s_base, s_slot;
    const uint32_t count = *a.count_ptr;
    const uint32_t n_st = a.ctr->n_struct;
    const int lane = rp_lane(), wave = threadIdx.x >> 6;
    const uint32_t d = a.d;
    const float ident = IS_MIN ? INFINITY : -INFINITY;
    for (uint32_t i = bid; i < count; i += nb) {
        const uint32_t v = a.list[i];
        const uint2 m = a.in_meta[v];
        const bool created = rp_bit(a.bm_vadd, v);
        float xo[NJ], xn[NJ];
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            const uint32_t col = lane + 64 * j;
            xo[j] = (col < d) ? a.X[(size_t)v * d + col] : 0.0f;
        }
        // the in-neighbours that changed: counted, and listed in LDS while they fit (several blocks of ids
        // are in flight per wavefront: the row is long and each block is two dependent reads)
        if (threadIdx.x == 0) {
            s_nd = 0;
            s_nhit = 0;
        }
        __syncthreads();
        for (uint32_t base = 64u * wave; base < m.y; base += 64u * TEAM * IDS) {
            uint32_t u[IDS];
            bool dirty[IDS];
#pragma unroll
            for (int t = 0; t < IDS; ++t) {
                const uint32_t e = base + 64u * TEAM * t + lane;
                u[t] = (e < m.y) ? a.in_pool[m.x + e] : 0u;
            }
#pragma unroll
            for (int t = 0; t < IDS; ++t) {
                const uint32_t e = base + 64u * TEAM * t + lane;
                dirty[t] = e < m.y && rp_bit(a.bm_prev, u[t]);
            }
#pragma unroll
            for (int t = 0; t < IDS; ++t) {
                const unsigned long long mask = __ballot(dirty[t]);
                if (!mask) continue;
                uint32_t pos = 0;
                if (lane == __ffsll((long long)mask) - 1) pos = atomicAdd(&s_nd, (uint32_t)__popcll(mask));
                pos = __shfl(pos, __ffsll((long long)mask) - 1) + (uint32_t)__popcll(mask & ((1ull << lane) - 1ull));
                if (dirty[t] && pos < MONO_DIRTY_LIST) s_dirty[pos] = u[t];
            }
        }
        __syncthreads();
        const uint32_t nd = s_nd;
        // A sink keeps its long row incremental when its changed edges can be looked up: each becomes a message.
        bool recompute = created;
        uint32_t ns = 0;
        if (!recompute && rp_bit(a.bm_sink, v)) {
            if (n_st > a.struct_cap || n_st > MONO_EDGE_SCAN) {
                recompute = true;
            } else {
                for (uint32_t s = threadIdx.x; s < n_st; s += TEAM * 64)
                    if (a.st_dst[s] == v && a.st_sign[s] != 0.0f) {
                        const uint32_t k = atomicAdd(&s_nhit, 1u);
                        if (k < MONO_EDGE_HITS) s_hit[k] = s;
                    }
                __syncthreads();
                ns = s_nhit;
                if (ns > MONO_EDGE_HITS) recompute = true;
            }
        }
        if (2 * (nd + ns) >= m.y) recompute = true;            // old and new rows of the senders against every row once
        if (!recompute) {                                      // every wavefront looks at its share of the messages
            float inc[NJ];
            uint32_t lostm = 0;
#pragma unroll
            for (int j = 0; j < NJ; ++j) inc[j] = ident;
            if (nd <= MONO_DIRTY_LIST) {
                for (uint32_t base = 64u * wave; base < nd; base += 64u * TEAM) {
                    const uint32_t k = base + lane;
                    const uint32_t u = (k < nd) ? s_dirty[k] : 0u;
                    mono_messages<NJ, IS_MIN, STORE, GC>(a, u, __ballot(k < nd), xo, inc, lostm, false);
                }
            } else {
                for (uint32_t base = 64u * wave; base < m.y; base += 64u * TEAM) {
                    const uint32_t e = base + lane;
                    const uint32_t u = (e < m.y) ? a.in_pool[m.x + e] : 0u;
                    const unsigned long long mask = __ballot(e < m.y && rp_bit(a.bm_prev, u));
                    if (mask) mono_messages<NJ, IS_MIN, STORE, GC>(a, u, mask, xo, inc, lostm, false);
                }
            }
            for (uint32_t base = 64u * wave; base < ns; base += 64u * TEAM) {
                const uint32_t k = base + lane;
                const uint32_t s = (k < ns) ? s_hit[k] : 0u;
                const uint32_t u = (k < ns) ? a.st_src[s] : 0u;
                const bool deleted = (k < ns) && a.st_sign[s] < 0.0f;
                mono_edge_messages<NJ, IS_MIN, STORE>(a, u, deleted, __ballot(k < ns), xo, inc, lostm);
            }
#pragma unroll
            for (int j = 0; j < NJ; ++j) s_val[wave][j * 64 + lane] = inc[j];
            s_lost[wave][lane] = lostm;
            __syncthreads();
            if (wave == 0) {
                lostm = 0;
                for (int w = 0; w < TEAM; ++w) lostm |= s_lost[w][lane];
                bool need = (lostm >> 31) != 0;
#pragma unroll
                for (int j = 0; j < NJ; ++j) {
                    float best = s_val[0][j * 64 + lane];
                    for (int w = 1; w < TEAM; ++w) {
                        const float x = s_val[w][j * 64 + lane];
                        if (mono_better<IS_MIN>(x, best)) best = x;
                    }
                    if (lane + 64 * j < (int)d && ((lostm >> j) & 1u) && mono_better<IS_MIN>(xo[j], best)) need = true;
                    xn[j] = mono_better<IS_MIN>(best, xo[j]) ? best : xo[j];
                }
                const bool rec = __ballot(need) != 0ull;
                if (lane == 0) s_flag = rec ? 1u : 0u;
            }
            __syncthreads();
            recompute = s_flag != 0;
            if (!recompute) {
                if (wave == 0) {
                    const bool changed = mono_finish<NJ>(a, v, created, xo, xn);
                    if (lane == 0) atomicAdd(&a.ctr->mono[changed ? 1 : 0][a.l], 1u);
                }
                __syncthreads();                               // the LDS arrays are reused by the next row
                continue;
            }
        }
        // recompute from all in-neighbours (m.y > long_min, so the row is not empty)
        if (m.y >= a.split_min) {
            // One compute unit reads a row of thousands of in-neighbours far too slowly: queue its segments,
            // a workgroup each takes one, the last to finish combines them (k_scatter_mono_seg).
            const uint32_t nseg = (m.y + ROW_SEG - 1) / ROW_SEG;
            if (threadIdx.x == 0) {
                const uint32_t r = atomicAdd(&a.ctr->n_big[a.l], 1u);
                const uint32_t base = atomicAdd(&a.ctr->n_seg[a.l], nseg);
                const bool fits = r < a.big_cap && base < a.seg_cap && nseg <= a.seg_cap - base;
                if (fits) {
                    a.seg_v[r] = v;
                    a.seg_done[r] = 0;
                    a.seg_base[r] = base;
                }
                s_base = base;
                s_slot = fits ? r : SEG_NONE;
            }
            __syncthreads();
            const uint32_t base = s_base, r = s_slot;
            for (uint32_t k = threadIdx.x; k < nseg; k += TEAM * 64)
                if (base < a.seg_cap && k < a.seg_cap - base) a.seg_r[base + k] = r;    // SEG_NONE: skipped there
            __syncthreads();
            if (r != SEG_NONE) continue;                       // (the capacities cover every row: not expected otherwise)
        }
#pragma unroll
        for (int j = 0; j < NJ; ++j) xn[j] = ident;
        const uint32_t chunk = (m.y <= 16u * 64u) ? 16u : 64u;  // shorter rows in finer pieces: every wavefront reads some
        for (uint32_t base = chunk * wave; base < m.y; base += chunk * TEAM) {
            const uint32_t e = base + lane;
            const uint32_t u = ((uint32_t)lane < chunk && e < m.y) ? a.in_pool[m.x + e] : 0u;
            mono_gather<NJ, IS_MIN, STORE, GR>(a, u, (int)min(chunk, m.y - base), xn);
        }
        __syncthreads();                                       // s_val may still be read by wavefront 0 (classification)
#pragma unroll
        for (int j = 0; j < NJ; ++j) s_val[wave][j * 64 + lane] = xn[j];
        __syncthreads();
        if (wave == 0) {
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                float best = s_val[0][j * 64 + lane];
                for (int w = 1; w < TEAM; ++w) {
                    const float x = s_val[w][j * 64 + lane];
                    if (mono_better<IS_MIN>(x, best)) best = x;
                }
                xn[j] = best;
            }
            mono_finish<NJ>(a, v, created, xo, xn);
            if (lane == 0) atomicAdd(&a.ctr->mono[2][a.l], 1u);
        }
        __syncthreads();
    }
}

template <int NJ, int IS_MIN, int STORE, int TEAM>
__global__ __launch_bounds__(TEAM * 64) void k_scatter_mono_long(MonoArgs a) {
    mono_team_role<NJ, IS_MIN, STORE, TEAM>(a, blockIdx.x, gridDim.x);
}

// Small hops, whose long rows were sorted out while the candidates were listed: both roles in one launch
// (the first team_blocks workgroups take a queued long row each, the wavefronts of the others a short
// candidate each), which saves one of the hop's dependent launches.
template <int NJ, int IS_MIN, int STORE, int TEAM>
__global__ __launch_bounds__(TEAM * 64) void k_scatter_mono_both(MonoArgs a, MonoArgs b, uint32_t team_blocks) {
    if (blockIdx.x < team_blocks) {
        mono_team_role<NJ, IS_MIN, STORE, TEAM>(b, blockIdx.x, team_blocks);
    } else {
        const uint32_t wb = blockIdx.x - team_blocks, nwb = gridDim.x - team_blocks;
        mono_wave_role<NJ, IS_MIN, STORE>(a, (wb * blockDim.x + threadIdx.x) >> 6, (nwb * blockDim.x) >> 6);
    }
}

// One workgroup per queued segment of a very long row that is recomputed: the extreme over the segment's
// ROW_SEG in-neighbours goes to the segment's partial row; the workgroup that finishes a row's last
// segment takes the extreme over the partial rows and finishes the row.
template <int NJ, int IS_MIN, int STORE, int TEAM>
__global__ __launch_bounds__(TEAM * 64) void k_scatter_mono_seg(MonoArgs a) {
    static_assert(TEAM * 64 == ROW_SEG, "one 64-entry block per wavefront");
    constexpr int GR = (NJ <= 2) ? 32 : 64 / NJ;
    __shared__ float s_val[TEAM][NJ * 64];
    const uint32_t n_seg = min(a.ctr->n_seg[a.l], a.seg_cap);
    const int lane = rp_lane(), wave = threadIdx.x >> 6;
    const uint32_t d = a.d;
    const float ident = IS_MIN ? INFINITY : -INFINITY;
    for (uint32_t e = blockIdx.x; e < n_seg; e += gridDim.x) {
        const uint32_t r = a.seg_r[e];
        if (r == SEG_NONE) continue;
        const uint32_t v = a.seg_v[r], first = a.seg_base[r];
        const uint2 m = a.in_meta[v];
        const uint32_t nseg = (m.y + ROW_SEG - 1) / ROW_SEG;
        const uint32_t lo = (e - first) * ROW_SEG, hi = min(m.y, lo + ROW_SEG);
        float xn[NJ];
#pragma unroll
        for (int j = 0; j < NJ; ++j) xn[j] = ident;
        const uint32_t b = lo + 64u * wave;
        if (b < hi) {
            const uint32_t u = (b + lane < hi) ? a.in_pool[m.x + b + lane] : 0u;
            mono_gather<NJ, IS_MIN, STORE, GR>(a, u, (int)min(64u, hi - b), xn);
        }
#pragma unroll
        for (int j = 0; j < NJ; ++j) s_val[wave][j * 64 + lane] = xn[j];
        __syncthreads();
        if (wave == 0) {
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                float best = s_val[0][j * 64 + lane];
                for (int w = 1; w < TEAM; ++w) {
                    const float x = s_val[w][j * 64 + lane];
                    if (mono_better<IS_MIN>(x, best)) best = x;
                }
                const uint32_t col = lane + 64 * j;
                if (col < d) a.seg_part[(size_t)e * a.seg_ld + col] = best;
            }
            __threadfence();                                   // the partial row is visible before the count moves
            uint32_t last = 0;
            if (lane == 0) last = (atomicAdd(&a.seg_done[r], 1u) == nseg - 1) ? 1u : 0u;
            last = __shfl(last, 0);
            if (last) {
                __threadfence();
                float xo[NJ];
#pragma unroll
                for (int j = 0; j < NJ; ++j) {
                    const uint32_t col = lane + 64 * j;
                    xo[j] = (col < d) ? a.X[(size_t)v * d + col] : 0.0f;
                    xn[j] = ident;
                }
                constexpr int GP = (NJ <= 4) ? 8 : 32 / NJ;     // partial rows requested per round trip
                for (uint32_t k0 = 0; k0 < nseg; k0 += GP) {
                    float x[GP][NJ];
#pragma unroll
                    for (int g = 0; g < GP; ++g) {
                        const float *part = a.seg_part + (size_t)(first + min(k0 + g, nseg - 1)) * a.seg_ld;
#pragma unroll
                        for (int j = 0; j < NJ; ++j) {          // written by other compute units: read past this one's cache
                            const uint32_t col = lane + 64 * j;
                            x[g][j] = (col < d) ? __hip_atomic_load(part + col, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : ident;
                        }
                    }
#pragma unroll
                    for (int g = 0; g < GP; ++g)
#pragma unroll
                        for (int j = 0; j < NJ; ++j)
                            if (mono_better<IS_MIN>(x[g][j], xn[j])) xn[j] = x[g][j];
                }
                mono_finish<NJ>(a, v, rp_bit(a.bm_vadd, v), xo, xn);
                if (lane == 0) atomicAdd(&a.ctr->mono[2][a.l], 1u);
            }
        }
        __syncthreads();
    }
}

static void launch_mono_direct(ripple_ctx *c, uint32_t l, const MonoArgs &h);

// A candidate escapes recomputation only if none of its columns' extremes was set by a changed in-neighbour and got worse. With
// m messages over the candidates' in-entries, a share m / entries of a row's in-neighbours has changed, so m * width / entries
// columns of it, on average, are in danger: from two on nearly every candidate would be recomputed after its messages have
// been read in vain. Judged by the previous batch; both ways are exact.
static bool mono_direct(const ripple_ctx *c, uint32_t l) {
    return c->hints_valid && c->last_m[l] && (uint64_t)c->last_m[l] * c->xw[l] >= 2ull * c->last_isum[l];
}

// candidates in c->all_list, *count_ptr of them (rp_launch_candidates[_sparse]); D[(l-1)&1] holds the pre-batch rows of A_{l-1}
void rp_launch_scatter_mono(ripple_ctx *c, uint32_t l, const uint32_t *count_ptr, bool listed) {
    MonoArgs a;
    const bool few = c->hints_valid && c->last_cand[l] <= 8192u;
    // few candidates: one wavefront would read a row of 100+ in-neighbours for tens of microseconds with the chip idle
    a.long_min = (few || listed) ? RP_MONO_LISTED_LONG : MONO_LONG;   // (a listed hop's long rows were sorted out with this limit)
    // a full chip is busy whichever workgroup reads a row: only the longest rows are split, so that none is left running
    // alone; in between (up to 128 K candidates) a row of a few thousand entries would still outlast everything else
    const bool some = c->hints_valid && c->last_cand[l] <= 131072u;
    a.split_min = few ? ROW_SPLIT_MIN : (some ? 4u : 64u) * ROW_SPLIT_MIN;
    a.list = c->all_list;
    a.count_ptr = count_ptr;
    // listed: the long rows are in c->eoff[l] already (rp_launch_candidates_sparse), nothing is queued here
    a.queue = listed ? nullptr : c->list[l];    // not written before the hop's set is final
    a.out_list = listed ? c->list[l] : nullptr;
    a.out_count = &c->ctr->set[l].a;                // zero since the batch began
    a.queue_count = &c->ctr->n_long[l];         // zero since the batch began
    a.in_meta = c->in_meta;
    a.in_pool = c->in_pool;
    a.bm_prev = c->bm[l - 1];
    a.bm_sink = c->bm_sink;
    a.bm_vadd = c->bm_vadd;
    a.bm_cur = c->bm[l];
    a.Dold = c->D[(l - 1) & 1];
    a.Hprev = c->H[l - 1];
    a.d = c->xw[l];
    a.X = c->X[l];
    a.keep_prev = c->layers[l - 1].self_mode != RIPPLE_SELF_NONE ? 1 : 0;
    a.ctr = c->ctr;
    a.l = l;
    a.st_src = c->st_src;
    a.st_dst = c->st_dst;
    a.st_sign = c->st_unit;                         // +1 added, -1 deleted, 0 re-weighted (nothing to a max / min layer)
    a.struct_cap = c->in_w ? 0u : c->struct_cap;   // weighted graphs: the sign carries the weight, sinks recompute
    a.alive = c->alive;
    a.seg_v = c->seg_v;
    a.seg_done = c->seg_done;
    a.seg_base = c->seg_base;
    a.seg_r = c->seg_r;
    a.seg_part = c->seg_part;
    a.big_cap = c->big_cap;
    a.seg_cap = std::min(c->seg_cap, c->seg_limit);
    a.seg_ld = c->seg_ld;
    if (!listed && mono_direct(c, l)) {
        launch_mono_direct(c, l, a);
        return;
    }
    MonoArgs b = a;
    b.list = listed ? c->eoff[l] : a.queue;
    b.count_ptr = &c->ctr->n_long[l];
    const bool is_min = c->layers[l - 1].agg == RIPPLE_AGG_MIN;
    // few candidates: every workgroup resident at once, so none waits for a slot behind one that holds a long chain of reads
    dim3 grid(c->n_cu * (few ? 4 : 8)), block(256);
#define MONO_PAIR(NJ, MN, ST, TEAM)                                                                          \
    do {                                                                                                     \
        if (listed) {                                                                                        \
            /* every workgroup resident at once: half the compute units' worth for each role */              \
            hipLaunchKernelGGL((k_scatter_mono_both<NJ, MN, ST, TEAM>), dim3(c->n_cu / 2 + (c->n_cu / 2) * (16 / TEAM)), \
                               dim3(TEAM * 64), 0, c->stream, a, b, c->n_cu / 2);                            \
        } else {                                                                                             \
            hipLaunchKernelGGL((k_scatter_mono<NJ, MN, ST>), grid, block, 0, c->stream, a);                  \
            hipLaunchKernelGGL((k_scatter_mono_long<NJ, MN, ST, TEAM>), dim3(c->n_cu * 2), dim3(TEAM * 64), 0, c->stream, b); \
        }                                                                                                    \
        hipLaunchKernelGGL((k_scatter_mono_seg<NJ, MN, ST, ROW_SEG / 64>), dim3(c->n_cu * 4), dim3(ROW_SEG), 0, c->stream, b); \
    } while (0)
#define MONO_CASE(NJ, TEAM)                                                                                  \
    do {                                                                                                     \
        if (is_min && c->store) MONO_PAIR(NJ, 1, 1, TEAM);                                                   \
        else if (is_min) MONO_PAIR(NJ, 1, 0, TEAM);                                                          \
        else if (c->store) MONO_PAIR(NJ, 0, 1, TEAM);                                                        \
        else MONO_PAIR(NJ, 0, 0, TEAM);                                                                      \
    } while (0)
    if (a.d <= 64) MONO_CASE(1, 16);
    else if (a.d <= 128) MONO_CASE(2, 16);
    else if (a.d <= 256) MONO_CASE(4, 16);
    else if (a.d <= 512) MONO_CASE(8, 16);
    else MONO_CASE(16, 8);
#undef MONO_CASE
#undef MONO_PAIR
}

// ---------------------------------------------------------------------------------
// bootstrap aggregation: X[v] = sum (op 0), max (1) or min (2) over u in in-row(v) of H_prev[u]
// ---------------------------------------------------------------------------------
// Bound by the gather of one row per in-edge. In-degrees are skewed (24 K entries in the longest in-row of a graph of
// 31 M edges), so the cut is over edges and not over rows: the flattened in-edge space of all live vertices is cut into
// runs of PULL_CHUNK-edge chunks, G rows are in flight per wavefront, and a destination whose in-edges all lie in one run is
// stored plainly. Sums of destinations that a run boundary cuts are left in parts and added up in run order by
// k_pull_all_close: a bootstrap of the same graph gives the same bits every time. Extremes do not depend on an order and are
// combined with atomics, onto the start value that k_pull_all_init puts there (together with the zeros of vertices without
// in-edges). One wavefront per row, one row in flight, is what this replaces: 34.0 / 15.6 / 8.3 ms for rows of 256 / 100 / 47
// floats over 31 M edges, most of it spent waiting for the few wavefronts with the longest rows; now 4.3 / 2.0 ms for 256 / 100 (7.4 and
// 6.2 TB/s of rows), 4.7 / 2.2 while sums and extremes were told apart in the inner loop. Sums of fp32 rows of up to 64 columns go through k_pull_all4
// (47 floats 0.95 ms, 1.2 here).
// The same cut serves the hops of max / min layers whose candidates are all recomputed (mono_direct): a candidate's new
// aggregate is compared with the old one when it is complete, stored if it differs and taken out of the hop's set if not;
// what a run boundary cuts is put together in XN and finished by k_mono_close.
struct PullAllArgs {
    PullArgs p;                    // list (live vertices or candidates), count_ptr, ioff, in_meta, in_pool, in_w, d, X
    const void *Hprev;
    uint32_t ldh;                  // its row stride
    int op;
    uint32_t n_cap;
    float *XN;                     // candidates: rows that a run boundary cuts [vertex x d]
    CutRows c;                     // sums: rows that a run boundary cuts
    uint32_t n_waves;              // wavefronts of the k_pull_all launch
};

__device__ __forceinline__ float pull_all_start(int op) { return op == 0 ? 0.0f : (op == 1 ? -INFINITY : INFINITY); }

// HOP: candidates of a max / min hop
template <int HOP>
__global__ __launch_bounds__(256) void k_pull_all_init(PullAllArgs a) {
    const int lane = rp_lane();
    const uint32_t gw = (blockIdx.x * blockDim.x + threadIdx.x) >> 6, nw = (gridDim.x * blockDim.x) >> 6;
    const uint32_t count = *a.p.count_ptr, d = a.p.d;
    const uint32_t total = count ? a.p.ioff[count] : 0u;
    const uint32_t span = rp_run_cut(total, a.n_waves).span();  // edges per run
    for (uint32_t base = gw * 64u; !HOP && base < a.n_cap; base += nw * 64u) {   // no in-edges (or not alive): zero
        const uint32_t v = base + (uint32_t)lane;
        unsigned long long m = __ballot(v < a.n_cap && a.p.in_meta[v].y == 0u);
        while (m) {
            const uint32_t w = base + (uint32_t)__ffsll((long long)m) - 1u;
            m &= m - 1ull;
            for (uint32_t col = lane; col < d; col += 64u) a.p.X[(size_t)w * d + col] = 0.0f;
        }
    }
    const uint32_t S = max(1u, min(64u, count / nw));       // vertices per wavefront and round
    for (uint32_t base = gw * S; a.op != 0 && base < count; base += nw * S) {   // extremes cut by a run boundary: the start value
        const uint32_t i = base + (uint32_t)lane;
        bool cut = false;
        uint32_t v = 0;
        if (i < count && (uint32_t)lane < S) {
            const uint32_t e0 = a.p.ioff[i], e1 = a.p.ioff[i + 1u];
            v = a.p.list[i];
            cut = e1 > e0 && e0 / span != (e1 - 1u) / span;
        }
        unsigned long long m = __ballot(cut);
        while (m) {
            const uint32_t w = (uint32_t)__shfl((int)v, __ffsll((long long)m) - 1);
            m &= m - 1ull;
            float *x = HOP ? a.XN : a.p.X;
            for (uint32_t col = lane; col < d; col += 64u) x[(size_t)w * d + col] = pull_all_start(a.op);
        }
    }
}

// x into *p by max (or min) without a lock: numbers >= 0 order like signed integers (and all of them above the negative
// ones), negative numbers among themselves like unsigned integers turned round. x is not a NaN.
__device__ __forceinline__ void rp_atomic_extreme(float *p, float x, bool is_max) {
    x += 0.0f;                                              // -0 -> +0
    const int i = __float_as_int(x);
    if (x >= 0.0f) (void)(is_max ? atomicMax((int *)p, i) : atomicMin((int *)p, i));
    else (void)(is_max ? atomicMin((unsigned int *)p, (unsigned int)i) : atomicMax((unsigned int *)p, (unsigned int)i));
}

// MODE 0: sums; 1: extremes (max / min) of the bootstrap; 2: extremes of a hop's candidates
template <int NJ, int STORE, int WT, int MODE>
__global__ __launch_bounds__(256) void k_pull_all(PullAllArgs a, MonoArgs h) {
    constexpr bool SUM = MODE == 0, HOP = MODE == 2;
    constexpr int G = (NJ >= 8) ? 2 : 16 / NJ;              // rows per round trip
    constexpr int T = PULL_CHUNK / 64;
    constexpr uint32_t NONE = 0xFFFFFFFFu;
    const uint32_t count = *a.p.count_ptr;
    if (count == 0) return;
    const int lane = rp_lane();
    const uint32_t d = a.p.d;
    const uint32_t total = a.p.ioff[count];
    const uint32_t gw = (blockIdx.x * blockDim.x + threadIdx.x) >> 6, nw = (gridDim.x * blockDim.x) >> 6;
    const RunCut cut = rp_run_cut(total, nw);
    const uint32_t n_chunks = cut.n_chunks;
    const uint32_t per = cut.per, n_runs = cut.n_runs;
    const float start = SUM ? 0.0f : pull_all_start(a.op);
    for (uint32_t run = gw; run < n_runs; run += nw) {
        const uint32_t c_begin = run * per, c_end = min(n_chunks, c_begin + per);
        PullScan<T, WT, 1> scan;
        scan.begin(a.p, count, c_begin * cut.chunk, lane);
        // the destinations of the run's first and last in-edge may have in-edges in other runs
        const uint32_t v_first = (uint32_t)__shfl((int)scan.rv, 0);
        const uint32_t e_end = min(total, c_end * cut.chunk);
        const uint32_t i_last = rp_seg_search_wave(a.p.ioff, 0, count - 1, e_end - 1u);
        const uint32_t v_last = a.p.list[i_last];
        const bool cut_first = a.p.ioff[scan.i_lo] < c_begin * cut.chunk;
        const uint32_t e_last = a.p.ioff[i_last + 1u];
        const bool cut_last = e_last > e_end;
        if (SUM && lane == 0)
            a.c.cut[run] = make_uint2(cut_last && !(v_last == v_first && cut_first) ? v_last : NONE, (e_last - 1u) / cut.span());
        uint32_t cur = NONE;
        float acc[NJ], xo[HOP ? NJ : 1];                     // HOP: the destination's old aggregate, requested with its first edge
#pragma unroll
        for (int j = 0; j < NJ; ++j) acc[j] = start;
        auto flush = [&]() {
            const bool began_before = cur == v_first && cut_first, shared = began_before || (cur == v_last && cut_last);
            float *xr = ((HOP && shared) ? a.XN : a.p.X) + (size_t)cur * d;
            if (SUM && shared) xr = a.c.part + (size_t)(2u * run + (began_before ? 0u : 1u)) * d;
            if constexpr (HOP) {
                if (!shared) {
                    mono_finish<NJ>(h, cur, rp_bit(h.bm_vadd, cur), xo, acc);
#pragma unroll
                    for (int j = 0; j < NJ; ++j) acc[j] = start;
                    return;
                }
            }
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                const uint32_t col = lane + 64 * j;
                if (col < d) {
                    if (SUM || !shared) xr[col] = acc[j];
                    else rp_atomic_extreme(&xr[col], acc[j], a.op == 1);
                }
                acc[j] = start;
            }
        };
        for (uint32_t c = c_begin; c < c_end; ++c) {
            const uint32_t e0 = c * cut.chunk, e1 = min(total, e0 + cut.chunk);
            uint32_t my_v[T], my_u[T];
            float my_w[WT ? T : 1];
            bool all[T];
            scan.chunk(a.p, count, e0, e1, lane, my_v, my_u, my_w, all);
#pragma unroll
            for (int t = 0; t < T; ++t) {
                const int n = (int)min(64u, e1 - min(e1, e0 + 64u * t));
                for (int k0 = 0; k0 < n; k0 += G) {
                    float r[G][NJ];
#pragma unroll
                    for (int g = 0; g < G; ++g) {
                        const uint32_t uk = (uint32_t)__builtin_amdgcn_readlane((int)my_u[t], min(k0 + g, n - 1));
#pragma unroll
                        for (int j = 0; j < NJ; ++j) {
                            const uint32_t col = min((uint32_t)lane + 64u * j, d - 1u);
                            r[g][j] = rp_load_h(a.Hprev, STORE, (size_t)uk * a.ldh + col);
                        }
                    }
#pragma unroll
                    for (int g = 0; g < G; ++g) {
                        if (k0 + g < n) {
                            const uint32_t vk = (uint32_t)__builtin_amdgcn_readlane((int)my_v[t], k0 + g);
                            if (vk != cur) {
                                if (cur != NONE) flush();
                                cur = vk;
                                if constexpr (HOP) {
#pragma unroll
                                    for (int j = 0; j < NJ; ++j) xo[j] = a.p.X[(size_t)vk * d + min((uint32_t)lane + 64u * j, d - 1u)];
                                }
                            }
                            const float wk = WT ? __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(my_w[WT ? t : 0]), k0 + g)) : 1.0f;
#pragma unroll
                            for (int j = 0; j < NJ; ++j) {
                                if (SUM) acc[j] = WT ? __builtin_fmaf(wk, r[g][j], acc[j]) : acc[j] + r[g][j];
                                else acc[j] = a.op == 1 ? fmaxf(acc[j], r[g][j]) : fminf(acc[j], r[g][j]);
                            }
                        }
                    }
                }
            }
            scan.advance();
        }
        if (cur != NONE) flush();
    }
}

// Sums of fp32 rows of up to 64 columns: several rows per load instruction and four columns per lane, as k_scatter_pull4 takes them. (A lane per
// column and a row per instruction takes 1,170 to 1,320 us for 47 columns and 31 M edges, depending on what the compiler makes of it; this 1,172, 64 G lines a second, and 950 with padded rows.)
template <int F, int WT>
__global__ __launch_bounds__(256) void k_pull_all4(PullAllArgs a) {
    constexpr int T = PULL_CHUNK / 64;
    constexpr uint32_t NONE = 0xFFFFFFFFu;
    constexpr int LANES = RowForm<F>::LANES, ROWS = RowForm<F>::ROWS, LOADS = RowForm<F>::LOADS;
    constexpr uint32_t LIST = PULL_CHUNK + ROWS * LOADS;
    __shared__ uint2 s_e[4][LIST];                          // per in-edge: source, destination
    __shared__ float s_w[WT ? 4 : 1][WT ? LIST : 1];
    const uint32_t count = *a.p.count_ptr;
    if (count == 0) return;
    const int lane = rp_lane(), wave = threadIdx.x >> 6;
    const uint32_t d = a.p.d, grp = (uint32_t)lane / LANES, sub = (uint32_t)lane & (LANES - 1u);
    const uint32_t total = a.p.ioff[count];
    const uint32_t gw = (blockIdx.x * blockDim.x + threadIdx.x) >> 6, nw = (gridDim.x * blockDim.x) >> 6;
    const RunCut cut = rp_run_cut(total, nw);
    const float *frow = (const float *)a.Hprev + (4u * sub < d ? 4u * sub : 0u);   // lanes beyond the row repeat its first columns
    const uint32_t my_col = row_column<F>((uint32_t)lane);
    for (uint32_t run = gw; run < cut.n_runs; run += nw) {
        const uint32_t c_begin = run * cut.per, c_end = min(cut.n_chunks, c_begin + cut.per);
        PullScan<T, WT, 1> scan;
        scan.begin(a.p, count, c_begin * cut.chunk, lane);
        const uint32_t v_first = (uint32_t)__shfl((int)scan.rv, 0);
        const uint32_t e_end = min(total, c_end * cut.chunk);
        const uint32_t i_last = rp_seg_search_wave(a.p.ioff, 0, count - 1, e_end - 1u);
        const uint32_t v_last = a.p.list[i_last];
        const bool cut_first = a.p.ioff[scan.i_lo] < c_begin * cut.chunk;
        const uint32_t e_last = a.p.ioff[i_last + 1u];
        const bool cut_last = e_last > e_end;
        if (lane == 0) a.c.cut[run] = make_uint2(cut_last && !(v_last == v_first && cut_first) ? v_last : NONE, (e_last - 1u) / cut.span());
        uint32_t cur = NONE;
        float acc[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[j] = 0.0f;
        auto flush = [&]() {
            const bool began_before = cur == v_first && cut_first, shared = began_before || (cur == v_last && cut_last);
            float *xr = shared ? a.c.part + (size_t)(2u * run + (began_before ? 0u : 1u)) * d : a.p.X + (size_t)cur * d;
            const float mine = rows_sum<F>(acc);
            if (my_col < d) xr[my_col] = mine;
        };
        for (uint32_t c = c_begin; c < c_end; ++c) {
            const uint32_t e0 = c * cut.chunk, e1 = min(total, e0 + cut.chunk), n = e1 - e0;
            uint32_t my_v[T], my_u[T];
            float my_w[WT ? T : 1];
            bool all[T];
            scan.chunk(a.p, count, e0, e1, lane, my_v, my_u, my_w, all);
#pragma unroll
            for (int t = 0; t < T; ++t)                      // (lanes past the chunk leave row 0 without a destination)
                if (64u * t < n) {
                    s_e[wave][64u * t + lane] = make_uint2(my_u[t], all[t] ? my_v[t] : PULL4_PAD);
                    if (WT) s_w[wave][64u * t + lane] = my_w[WT ? t : 0];
                }
            if (lane < ROWS * LOADS) {                       // entries a round reads past the list's end
                s_e[wave][n + lane] = make_uint2(0u, PULL4_PAD);
                if (WT) s_w[wave][n + lane] = 0.0f;
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");   // (LDS accesses of one wavefront are executed in order)
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            for (uint32_t k0 = 0; k0 < n; k0 += ROWS * LOADS) {
                uint2 ent[LOADS];
                floatx4u fr[LOADS];
                float wk[WT ? LOADS : 1];
#pragma unroll
                for (int r = 0; r < LOADS; ++r) {
                    ent[r] = s_e[wave][k0 + ROWS * r + grp];
                    if (WT) wk[WT ? r : 0] = s_w[wave][k0 + ROWS * r + grp];
                    fr[r] = *(const floatx4u *)(frow + (size_t)ent[r].x * a.ldh);
                }
#pragma unroll
                for (int r = 0; r < LOADS; ++r) {
                    if (k0 + ROWS * r >= n) continue;
                    auto add = [&]() {
#pragma unroll
                        for (int j = 0; j < 4; ++j) acc[j] = WT ? __builtin_fmaf(fr[r][j], wk[WT ? r : 0], acc[j]) : acc[j] + fr[r][j];
                    };
                    if (!__any(ent[r].y != cur)) {           // all of them go on
                        add();
                    } else {                                 // destination by destination (they are in order)
                        unsigned long long left = __ballot(ent[r].y != PULL4_PAD);
                        while (left) {
                            const uint32_t vg = (uint32_t)__builtin_amdgcn_readlane((int)ent[r].y, __ffsll((long long)left) - 1);
                            if (vg != cur) {
                                if (cur != NONE) flush();
                                cur = vg;
                            }
                            const bool same = ent[r].y == vg;
                            if (same) add();
                            left &= ~__ballot(same);
                        }
                    }
                }
            }
            __builtin_amdgcn_wave_barrier();                 // the next chunk overwrites the list
            scan.advance();
        }
        if (cur != NONE) flush();
    }
}

// Sums of destinations that a run boundary cuts, a wavefront per run: paced by three dependent reads and by the longest row's parts
// (31 M edges, 17 K runs: 11 / 13 / 10 us for rows of 100 / 256 / 47; 26 for 256 with one block of 64 columns after the other).
__global__ __launch_bounds__(256) void k_pull_all_close(PullAllArgs a) {
    const int lane = rp_lane();
    const uint32_t gw = (blockIdx.x * blockDim.x + threadIdx.x) >> 6, nw = (gridDim.x * blockDim.x) >> 6;
    const uint32_t count = *a.p.count_ptr, d = a.p.d;
    if (count == 0) return;
    const uint32_t n_runs = rp_run_cut(a.p.ioff[count], a.n_waves).n_runs;
    for (uint32_t r = gw; r < n_runs; r += nw) {
        const uint2 c = a.c.cut[r];
        for (uint32_t c0 = lane; c.x != 0xFFFFFFFFu && c0 < d; c0 += 64u * PARTS_B) {
            float t[PARTS_B];
            rp_sum_parts(a.c.part, d, r, c.y, c0, t);
#pragma unroll
            for (int b = 0; b < PARTS_B; ++b)
                if (c0 + 64u * b < d) a.p.X[(size_t)c.x * d + c0 + 64u * b] = t[b];
        }
    }
}

// Candidates without in-edges or cut by a run boundary: finished here, a wavefront each.
template <int NJ>
__global__ __launch_bounds__(256) void k_mono_close(PullAllArgs a, MonoArgs h) {
    const int lane = rp_lane();
    const uint32_t gw = (blockIdx.x * blockDim.x + threadIdx.x) >> 6, nw = (gridDim.x * blockDim.x) >> 6;
    const uint32_t count = *a.p.count_ptr, d = a.p.d;
    const uint32_t total = count ? a.p.ioff[count] : 0u;
    const uint32_t span = rp_run_cut(total, a.n_waves).span();
    const uint32_t S = max(1u, min(64u, count / nw));                    // vertices per wavefront and round (few of them: one each, most are cut)
    if (gw == 0 && lane == 0) h.ctr->mono[2][h.l] = count;               // all of them are recomputed
    for (uint32_t base = gw * S; base < count; base += nw * S) {
        const uint32_t i = base + (uint32_t)lane;
        uint32_t v = 0, e0 = 0, e1 = 1;
        bool todo = false;
        if (i < count && (uint32_t)lane < S) {
            e0 = a.p.ioff[i];
            e1 = a.p.ioff[i + 1u];
            v = a.p.list[i];
            todo = e1 == e0 || e0 / span != (e1 - 1u) / span;
        }
        unsigned long long m = __ballot(todo);
        while (m) {
            const int k = __ffsll((long long)m) - 1;
            m &= m - 1ull;
            const uint32_t w = (uint32_t)__shfl((int)v, k);
            const bool none = __shfl((int)(e1 - e0), k) == 0;
            float xo[NJ], xn[NJ];
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                const uint32_t col = min((uint32_t)lane + 64u * j, d - 1u);
                xo[j] = a.p.X[(size_t)w * d + col];
                xn[j] = none ? 0.0f : a.XN[(size_t)w * d + col];
            }
            mono_finish<NJ>(h, w, rp_bit(h.bm_vadd, w), xo, xn);
        }
    }
}

static PullAllArgs pull_all_args(ripple_ctx *c, uint32_t l) {
    const bool proj = c->layers[l - 1].proj != 0;
    PullAllArgs a = {};
    a.p.list = c->all_list;
    a.p.count_ptr = &c->ctr->n_all;
    a.p.ioff = c->ioff_all;
    a.p.in_meta = c->in_meta;
    a.p.in_pool = c->in_pool;
    a.p.in_w = (c->layers[l - 1].agg == RIPPLE_AGG_WSUM) ? c->in_w : nullptr;
    a.p.d = c->xw[l];
    a.p.X = c->X[l];
    a.Hprev = proj ? (const void *)c->layers[l - 1].T : c->H[l - 1];
    a.ldh = proj ? c->layers[l - 1].ldt : a.p.d;
    a.op = c->layers[l - 1].agg == RIPPLE_AGG_MAX ? 1 : (c->layers[l - 1].agg == RIPPLE_AGG_MIN ? 2 : 0);
    a.n_cap = c->n_cap;
    a.n_waves = c->n_cu * 8 * 4;
    return a;
}

// X^l[v] = sum over v's in-row of the previous layer's rows (of their projections, kept in the layer's T,
// for project-first layers). The live vertices and their in-degree prefix are in c->all_list and c->ioff_all.
void rp_launch_pull_all(ripple_ctx *c, uint32_t l) {
    const int store = c->layers[l - 1].proj ? 0 : c->store;
    PullAllArgs a = pull_all_args(c, l);
    a.c = rp_cut_rows(c->D[l & 1], c->max_runs);         // (no rows of changes during the bootstrap; load_model has made it large enough)
    const MonoArgs none = {};
    const dim3 grid(c->n_cu * 8), block(256);
    hipLaunchKernelGGL(k_pull_all_init<0>, grid, block, 0, c->stream, a);
#define PULL_CASE_W(NJ, STORE, WT) hipLaunchKernelGGL((k_pull_all<NJ, STORE, WT, 0>), grid, block, 0, c->stream, a, none)
#define PULL_CASE(NJ)                                  \
    do {                                               \
        if (a.op != 0 && store) hipLaunchKernelGGL((k_pull_all<NJ, 1, 0, 1>), grid, block, 0, c->stream, a, none); \
        else if (a.op != 0) hipLaunchKernelGGL((k_pull_all<NJ, 0, 0, 1>), grid, block, 0, c->stream, a, none);     \
        else if (store && a.p.in_w) PULL_CASE_W(NJ, 1, 1);  \
        else if (store) PULL_CASE_W(NJ, 1, 0);         \
        else if (a.p.in_w) PULL_CASE_W(NJ, 0, 1);      \
        else PULL_CASE_W(NJ, 0, 0);                    \
    } while (0)
#define PULL4_CASE(F)                                                                                       \
    do {                                                                                                    \
        if (a.p.in_w) hipLaunchKernelGGL((k_pull_all4<F, 1>), grid, block, 0, c->stream, a);                \
        else hipLaunchKernelGGL((k_pull_all4<F, 0>), grid, block, 0, c->stream, a);                         \
    } while (0)
    const bool quads = a.op == 0 && !store;
    if (quads && a.p.d <= 16) PULL4_CASE(4);
    else if (quads && a.p.d <= 32) PULL4_CASE(8);
    else if (quads && a.p.d <= 64) PULL4_CASE(16);
    else if (a.p.d <= 64) PULL_CASE(1);
    else if (a.p.d <= 128) PULL_CASE(2);
    else if (a.p.d <= 256) PULL_CASE(4);
    else if (a.p.d <= 512) PULL_CASE(8);
    else PULL_CASE(16);
#undef PULL_CASE
#undef PULL_CASE_W
#undef PULL4_CASE
    if (a.op == 0) hipLaunchKernelGGL(k_pull_all_close, dim3(c->n_cu * 16), block, 0, c->stream, a);
}

// All candidates of a max / min hop (in c->all_list with their in-degree prefix in c->ioff_all) recomputed; h: what mono_finish
// needs. The rows a run boundary cuts are put together in the buffer that the row update will fill afterwards.
static void launch_mono_direct(ripple_ctx *c, uint32_t l, const MonoArgs &h) {
    PullAllArgs a = pull_all_args(c, l);
    a.XN = c->D[l & 1];
    const dim3 grid(c->n_cu * 8), block(256);
    hipLaunchKernelGGL(k_pull_all_init<1>, dim3(c->n_cu * 2), block, 0, c->stream, a);
#define PULL_CASE(NJ)                                                                                                    \
    do {                                                                                                                 \
        if (c->store) hipLaunchKernelGGL((k_pull_all<NJ, 1, 0, 2>), grid, block, 0, c->stream, a, h);                    \
        else hipLaunchKernelGGL((k_pull_all<NJ, 0, 0, 2>), grid, block, 0, c->stream, a, h);                             \
        hipLaunchKernelGGL(k_mono_close<NJ>, dim3(c->n_cu * 4), block, 0, c->stream, a, h);                              \
    } while (0)
    if (a.p.d <= 64) PULL_CASE(1);
    else if (a.p.d <= 128) PULL_CASE(2);
    else if (a.p.d <= 256) PULL_CASE(4);
    else if (a.p.d <= 512) PULL_CASE(8);
    else PULL_CASE(16);
#undef PULL_CASE
}
