// Internal definitions shared by the host code and the gfx950 kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <hip/hip_bf16.h>
#include <stddef.h>
#include <stdint.h>
#include <string>
#include <vector>

#include "../../include/ripple.h"

#define RP_TOMB 0xFFFFFFFFu          // hole left in an adjacency row by a deletion
#define RP_WAVE 64

// per-vertex scratch bits kept in vstate[] while a batch is being applied
#define VS_TOUCH_OUT 1u              // out-row is on the touched list
#define VS_TOUCH_IN 2u
#define VS_ADDING 4u                 // created by this (sub-)batch
#define VS_DYING 8u                  // deleted by this (sub-)batch

// expanded edge of a deleted vertex
#define EXP_NONE 0u
#define EXP_OUT 1u                   // (w -> y): erase w from y's in-row
#define EXP_IN 2u                    // (x -> w): erase w from x's out-row
#define EXP_FIRST 4u                 // with one of the two: the first operation or edge to touch that row

#define READ_PIECES 8u               // pieces of rows that one launch writes to the host, of at most READ_FLOATS numbers each
#define READ_FLOATS 65536u

struct DevCtr {                      // device-resident counters, one instance per context
    // kept from batch to batch
    unsigned long long n_edges;
    uint32_t n_alive;
    uint32_t out_top, in_top;                 // first free pool entry
    uint32_t error;                           // sticky consistency error seen by a kernel
    uint32_t blocks_done;                     // workgroups of a kernel with a last-workgroup part that have finished (0 between launches)
    uint32_t n_all;                           // live vertices listed for a discovering hop
    uint32_t n_rec;                           // vertices with in-edges that the last listed attention hop recomputes
    uint32_t piece_done[READ_PIECES];         // workgroups that have written their part of a piece that the host reads (0 between launches)
    // from here on: zero when a batch begins (k_publish clears them once it has handed them to the host)
    struct alignas(8) Set {
        uint32_t a;                           // |A_l|
        uint32_t m;                           // out-edges of A_l: messages into layer l + 1
    } set[RIPPLE_MAX_LAYERS + 1];             // (eight bytes at a multiple of eight, so that small hops add to both at once)
    uint32_t touched[RIPPLE_MAX_LAYERS + 1];  // distinct live destinations of those edges
    uint32_t isum[RIPPLE_MAX_LAYERS + 1];     // sum of in-degrees over A_l
    uint32_t n_struct;
    uint32_t n_touch_out, n_touch_in;
    uint32_t n_exp;                           // expanded edges of deleted vertices
    uint32_t need_exp;                        // upper bound of n_exp computed while validating
    uint32_t n_applied, n_rejected;
    uint32_t n_add, n_del;                    // accepted edge adds / deletes (ops only)
    uint32_t n_gone;                          // edges that go with deleted vertices
    unsigned long long n_listed;              // touched out-rows (low half) and in-rows listed so far
    uint32_t n_entries;                       // entries of the touched rows' segments handed out so far
    uint32_t need_out, need_in;               // pool entries relocation will take
    uint32_t n_vadd;
    uint32_t abort_flag;                      // written by the capacity decision: 0 ok, bit0 pool, bit1 edges, bit2 scratch
    uint32_t n_long[RIPPLE_MAX_LAYERS + 1];   // max / min and attention hops: vertices with long in-rows queued for the workgroup kernel
    uint32_t cand[RIPPLE_MAX_LAYERS + 1];     // max / min hops: candidates listed while they were marked (small hops)
    uint32_t n_big[RIPPLE_MAX_LAYERS + 1];    // very long in-rows whose recomputation was split into segments
    uint32_t n_seg[RIPPLE_MAX_LAYERS + 1];    // segments queued for them
    uint32_t mono[3][RIPPLE_MAX_LAYERS + 1];  // max / min hops: candidates left unchanged / raised from the messages / recomputed
    uint32_t hop_mode[RIPPLE_MAX_LAYERS + 1]; // 1 + RP_HOP_* of the scatter kernel that moved hop l's messages (0: none ran, attention hops: no list)
    uint32_t range_rows;                      // attention layers: rows updated from sums that were not finite
    uint32_t pull_next[RIPPLE_MAX_LAYERS + 1];// pull scatter of hop l: runs of chunks handed out so far
    uint32_t pair_over[RIPPLE_MAX_LAYERS + 1];// a bucket of hop l's messages had no room for all of its own
    uint32_t pairs[RIPPLE_MAX_LAYERS + 1];    // attention hops: messages in the list (those of vertices that are not recomputed)
};
// buckets of a hop's messages: at most this many, each of at most this many consecutive vertices
#define RP_LIST_BUCKETS 8192u
#define RP_LIST_IDS 4096u
#define RP_CTR_WORDS ((uint32_t)(sizeof(DevCtr) / 4))
#define RP_CTR_BATCH ((uint32_t)(offsetof(DevCtr, set) / 4))   // first word that is zero when a batch begins

#define RP_MONO_LISTED_LONG 64u        // small max / min and attention hops: in-rows longer than this are queued for a workgroup while the hop's vertices are listed
#define ROW_SPLIT_MIN 512u
#define ROW_SEG 512u
#define ROW_SEG_MAX (1u << 18)           // segments queued at a time; rows that find the queue full are read by one workgroup
#define SEG_NONE 0xffffffffu

struct LayerDev {
    uint32_t d_in, d_hidden, d_out, K;        // K = rows of W0
    uint32_t agg, self_mode, act_inner, act_out;
    float eps;
    // weights padded to [Kpad x Npad] (Kpad multiple of 32, Npad multiple of 64), zero filled
    float *W0, *b0, *W1, *b1;
    __hip_bfloat16 *W0h, *W1h;                // bf16 copy of W0, transposed [N0pad x K0pad] (bf16 store only); W1h unused
    uint32_t K0pad, N0pad, K1pad, N1pad;
    // project-first layers: the cached aggregate holds sum_u H[u] W_neigh (d_out wide)
    uint32_t proj;
    // What the receivers of such a layer have been sent so far: T[u] (d_out floats) is the sum of all messages u
    // has ever sent, so the cached aggregate is X[v] = sum over v's in-neighbours of T[u] at all times. A message
    // is m = H[u] W_neigh - T[u] in the form it travels in (rounded to 19-bit block floating point when
    // the row is packed into one 128-byte line) and T[u] += m: what rounding takes away from one message is part
    // of the next, so nothing accumulates. Changed edges add or remove T[u] itself.
    float *T;
    uint32_t ldt;                             // row stride of T (sent_row_stride)
    uint32_t packed;                          // 0: messages travel as fp32 rows of PD; 1: as packed rows of MSG
    float *Wn;                                // neighbour weights padded to [roundup(d_in,32) x N0pad] (may alias W0)
    float *bzero;                             // N0pad zeros
    // concat layers with one linear map: PS[v] = H^{l-1}[v] W_self (d_out wide, fp32) is cached and
    // refreshed only where H^{l-1} changed, so the row transform multiplies the aggregate alone
    uint32_t selfc;
    float *PS;
    // project-first layers with a cached self term: [W_self | W_neigh] as one matrix [roundup(d_in,32) x 128] (W_neigh
    // from column 64 on) and 128 zeros, so that one pass over the rows of A_{l-1} yields both products; else null.
    float *Wc, *bzero_c;
    // attention layers: projected rows P[v] = H^{l-1}[v] W0 [n x d_out], scores a_src . P[v] and a_dst . P[v],
    // denominators of the softmax (the numerators are the layer's X rows); att = a_src then a_dst on the device
    float *att, *P, *ssrc, *sdst, *den;
    uint32_t ldp;                             // row stride of P: rows of up to 63 columns carry s_src behind them
    // the padded matrices once more with k by fours, [Kpad / 4][Npad][4] (wave_gemm); Wnq may alias W0q
    float *W0q, *Wnq, *W1q, *Wcq;
    // ... and as three bf16 parts each, in the order k_split_stream takes them (W0p: all K rows); Wnp may alias W0p
    unsigned short *W0p, *Wnp, *W1p, *Wcp;
    float lift0, lift1;                       // the powers of two that W0 (and what is cut out of it) and W1 are multiplied by first
};

// pieces of up to SMALL_OPS operations without vertex deletions: the Apply step in three launches (k_small_validate)
#define SMALL_WGS 128u
#define SMALL_OPS (4u * SMALL_WGS)

struct PhaseTimer;

struct ripple_ctx {
    int device = 0;
    hipStream_t stream = nullptr;
    std::string err;
    int state = 0;                             // 1 graph, 2 model, 3 inferred
    uint32_t n_cap = 0, n_words = 0;           // vertex capacity, bitmap words
    uint64_t e_cap = 0;
    uint64_t pool_cap = 0;
    int store = 0;                             // ripple_store
    uint32_t L = 0;
    uint32_t d[RIPPLE_MAX_LAYERS + 1] = {0};
    uint32_t dmax = 0, hmax = 0;               // widest layer / widest hidden
    LayerDev layers[RIPPLE_MAX_LAYERS];

    // graph store
    uint2 *out_meta = nullptr, *in_meta = nullptr;      // {start, len} per vertex
    uint32_t *out_capv = nullptr, *in_capv = nullptr;   // row capacity
    uint32_t *out_pool = nullptr, *in_pool = nullptr;
    float *in_w = nullptr, *out_w = nullptr;            // edge weights, parallel to in_pool and to out_pool (weighted graphs; out_w: from
                                                        // load_model on only with a weighted-sum layer)
    uint32_t *alive = nullptr;                          // bitmap
    uint32_t *vstate = nullptr;                         // VS_* bits, zero between batches
    uint32_t *pend_out = nullptr, *pend_in = nullptr;   // appended this batch
    uint32_t *dead_out = nullptr, *dead_in = nullptr;   // tombstones this batch
    uint32_t *hole_out = nullptr, *hole_in = nullptr;   // where a touched row's segment of seg_id / seg_x begins

    // embeddings and cached sums
    void *H[RIPPLE_MAX_LAYERS + 1] = {nullptr};
    float *X[RIPPLE_MAX_LAYERS + 1] = {nullptr};
    float *D[2] = {nullptr, nullptr};                   // delta rows D^l[v] (valid for v in A_l), ping-pong
    size_t max_runs = 0;                                // runs of chunks that the bootstrap and attention hops leave parts of cut rows for, in D
    float *tmp = nullptr;                               // hidden activations of two-stage updates
    float *PD = nullptr;                                // project-first layers: projected rows, then fp32 messages (by vertex)
    uint32_t *MSG = nullptr;                            // project-first layers with packed messages: 32 words per vertex
    // max / min (and attention) hops: in-rows of ROW_SPLIT_MIN entries or more are recomputed in segments of ROW_SEG
    // entries, one workgroup each. Per split row: vertex, segments finished, first segment; per segment: its row's
    // slot and its partial result (seg_ld floats)
    uint32_t *seg_v = nullptr, *seg_done = nullptr, *seg_base = nullptr, *seg_r = nullptr;
    float *seg_part = nullptr;
    uint32_t big_cap = 0, seg_cap = 0, seg_ld = 0;
    uint32_t seg_limit = 0xffffffffu;                   // RIPPLE_OPT_ROW_SEGMENTS: segments a hop may queue (<= seg_cap is used)
    float *gat_mag = nullptr;                           // attention hops: what a vertex's patches have added and taken away
    uint8_t *gat_rec = nullptr;                         // ... and whether it is recomputed (both valid for the hop's vertices)
    float *Pold = nullptr, *sold = nullptr;             // attention hops: projected rows / source scores of A_{l-1} before the batch
    uint32_t xw[RIPPLE_MAX_LAYERS + 1] = {0};           // width of X^l (d_{l-1}, or d_l when projected)
    uint32_t pd_ld = 0;                                 // row stride of PD (64-byte multiple)

    // frontier
    uint32_t *bm[RIPPLE_MAX_LAYERS + 1] = {nullptr};    // dirty bitmap per layer
    uint32_t *bm_sink = nullptr, *bm_vadd = nullptr;    // S and V_added
    uint8_t *mk = nullptr;                              // one byte per vertex: marks of the hop in progress (zero between hops)
    uint32_t *rep[RIPPLE_MAX_LAYERS + 1] = {nullptr};   // union over sub-batches (reporting)
    uint32_t *list[RIPPLE_MAX_LAYERS + 1] = {nullptr};  // A_l, ascending (l >= 1); op order for l = 0
    uint32_t *eoff[RIPPLE_MAX_LAYERS + 1] = {nullptr};  // exclusive scan of out-degrees over A_l, +1 entry
    uint32_t *part_cnt = nullptr, *part_deg = nullptr, *part_ideg = nullptr, *part_tch = nullptr, *part_rec = nullptr;  // per-block partial sums
    uint32_t *ioff[RIPPLE_MAX_LAYERS + 1] = {nullptr};  // exclusive scan of in-degrees over A_l, +1 entry
    uint32_t n_part = 0;
    uint32_t *all_list = nullptr;                       // scratch list (live vertices): full inference, discovering hops
    uint32_t *ioff_all = nullptr;                       // exclusive scan of in-degrees over all_list, +1 entry

    // batch staging
    uint32_t ops_cap = 0, feat_cap = 0;
    ripple_update *ops_d = nullptr;
    const float *payload = nullptr;                      // feature rows of the batch in progress: the caller's (device) or payload_pin
    uint32_t *op_status = nullptr, *op_pos_out = nullptr, *op_pos_in = nullptr;
    uint32_t *op_touch = nullptr;                        // per operation: accepted / add / first touch of its rows
    uint32_t *touch_out = nullptr, *touch_in = nullptr;  // touched row lists
    uint32_t touch_cap = 0;
    uint32_t exp_cap = 0;
    uint32_t *exp_kind = nullptr, *exp_a = nullptr, *exp_b = nullptr, *exp_pos = nullptr, *exp_rank = nullptr;
    uint32_t struct_cap = 0;
    uint32_t *st_src = nullptr, *st_dst = nullptr;
    float *st_sign = nullptr;                           // per changed edge: what its sink's weighted sums gain, +alpha / -alpha / alpha_new - alpha_old
    float *st_unit = nullptr;                           // the same for aggregates that ignore weights: +1 added, -1 deleted, 0 re-weighted
    uint32_t *op_rank_out = nullptr, *op_rank_in = nullptr;
    // a touched row's deletions and additions, the rows one after the other (2 ops_cap + exp_cap entries), and for the deterministic
    // mode the same in order
    uint32_t *seg_id = nullptr, *seg_x = nullptr, *srt_id = nullptr, *srt_x = nullptr;
    // deterministic mode: the pull kernels leave the sums of rows whose in-edges lie in more than one run of chunks here (two entries per run)
    uint32_t *side_v = nullptr;
    float *side_acc = nullptr;
    uint32_t side_runs = 0;                             // runs there is room for
    DevCtr *ctr = nullptr;
    DevCtr *ctr_host = nullptr;                         // pinned mirror, written by k_publish
    uint32_t *pub_flag = nullptr;                       // pinned: number of the last k_publish that has finished
    uint32_t pub_seq = 0;
    uint32_t *read_flag = nullptr;                      // pinned: number of the last launch that has written this piece, 16 words per piece
    uint32_t read_seq = 0;
    hipEvent_t idle = nullptr;                          // recorded behind the launches of a call that promises a synchronised stream
    bool ctr_dirty = false;                             // the per-batch counters are not zero (something ran after k_publish)
    ripple_update *ops_pin = nullptr;                   // pinned staging for ops
    float *payload_pin = nullptr;
    uint32_t pin_ops_cap = 0;
    uint32_t *made_pin = nullptr;                       // pinned: the vertices a small piece creates (SMALL_OPS entries)
    uint8_t *pin_block = nullptr;                       // pinned: ctr_host, pub_flag, io_pin, made_pin and the first ops_pin / payload_pin
    size_t pin_bytes = 0;
    // device arrays that share an allocation: the graph store's (but the pools), bitmaps and lists, batch scratch, messages as pairs, row segments, weights in parts
    uint8_t *graph_block = nullptr, *list_block = nullptr, *batch_block = nullptr, *pair_block = nullptr, *seg_block = nullptr, *part_block = nullptr;

    // gather staging for get_* calls; pinned: 16 words (a count), then ids, then rows
    uint32_t *io_pin = nullptr;
    float *gather_d = nullptr;
    uint32_t *gather_ids = nullptr;
    size_t gather_cap = 0, gather_ids_cap = 0;

    // last batch's sets (reporting)
    uint32_t last_a[RIPPLE_MAX_LAYERS + 1] = {0};
    bool hints_valid = false;                           // last_a / last_cand describe a batch (not the state after the bootstrap)
    uint32_t guess_a[RIPPLE_MAX_LAYERS + 1] = {0};      // |A_l| as the operations let expect it, where last_a says nothing
    uint32_t last_cand[RIPPLE_MAX_LAYERS + 1] = {0};
    uint32_t last_m[RIPPLE_MAX_LAYERS + 1] = {0};       // messages per hop of the last batch (a size hint)
    uint32_t last_isum[RIPPLE_MAX_LAYERS + 1] = {0};    // in-row entries a pull of that hop would have scanned
    uint32_t last_hop_mode[RIPPLE_MAX_LAYERS + 1] = {0};// 1 + RP_HOP_* of the kernel that moved that hop's messages
    // messages of a hop as (destination, source) pairs in buckets by destination (k_frontier_list), and how many each holds
    uint2 *pairs = nullptr, *pair_sorted = nullptr;     // ... and in order of destination
    float *pair_w = nullptr, *pair_w_sorted = nullptr;  // weighted graphs: the edges' weights, beside them
    uint32_t *pair_cnt = nullptr;                       // (zero between hops)
    uint32_t pair_cap = 0;                              // messages a listed hop may have; there is room for twice as many
    struct ListOver {                                   // hop l's last list that had a bucket run over (room 0: none since)
        uint32_t m = 0, room = 0, wait = 0;             // its messages, the entries a bucket had room for, batches until the next try
    } list_over[RIPPLE_MAX_LAYERS + 1];
    uint32_t list_room[RIPPLE_MAX_LAYERS + 1] = {0};    // what a bucket has room for in the batch in progress
    int opt_sorted = 1;                                 // 0 never, 1 where the last batch says it pays, 2 wherever it can be
    uint32_t last_n_ops = 0;                            // operations of the last single-piece batch    // candidates of the last batch's max / min hops (a size hint)
    bool last_from_rep = false;
    bool push_margin[RIPPLE_MAX_LAYERS + 1] = {false};  // last batch pushed at this hop by a wide margin
    bool disc_near[RIPPLE_MAX_LAYERS + 1] = {false};    // last batch's hop was within reach of the discovering mode

    // options
    int opt_timing = 0;
    int opt_scatter = 0;
    int opt_bf16_mfma = 1;                      // bf16 storage: multiply on the bf16 matrix cores
    int opt_project = 1;                        // allow project-first layers (read by load_model)
    int opt_selfcache = 1;                      // allow cached self projections (read by load_model)
    int opt_sparse = 1;                         // small frontiers are listed as they are marked (no bitmap scan)
    int opt_stream = 1;                         // products of many rows: persistent workgroups, tiles written while the next is multiplied (2: any size)
    int opt_split = 0;                          // products of few rows on the bf16 matrix cores as well, operands in three parts
    int opt_deterministic = 0;                  // bit-reproducible aggregation (owner kernels, no float atomics)
    int opt_pull_ratio = 1;                     // pull when messages * width * ratio >= scanned in-edges
    int opt_pack = 1;                           // project-first layers of 33..48 columns send one-line packed messages (read by load_model)
    ripple_stats stats;
    PhaseTimer *timer = nullptr;
    uint32_t n_cu = 256;
};

// ---- host helpers -----------------------------------------------------------------
#define RP_HIP(ctx, call)                                                              \
    do {                                                                               \
        hipError_t e__ = (call);                                                       \
        if (e__ != hipSuccess) {                                                       \
            (ctx)->err = std::string(#call) + ": " + hipGetErrorString(e__);          \
            return RIPPLE_EDEVICE;                                                     \
        }                                                                              \
    } while (0)

// |A_l| of the previous batch as a hint for launch shapes (tile sizes, grids, which compaction kernel); before
// the first batch nothing is known and the shapes for large sets are taken, which are never far off
static inline uint32_t rp_rows_hint(const ripple_ctx *c, uint32_t l) { return c->hints_valid ? c->last_a[l] : c->n_cap; }
// the same where a choice between kernels hangs on it that are each right for any size: without a previous batch, what the piece's operations reach
// on a graph of this mean degree. (First batch of a context: three hops of a few vertices each that were given persistent workgroups
// for every vertex took 20 us a product, tiles take 11.)
static inline uint32_t rp_rows_guess(const ripple_ctx *c, uint32_t l) { return c->hints_valid ? c->last_a[l] : c->guess_a[l]; }
static inline bool rp_layer_mono(const ripple_ctx *c, uint32_t l) {      // layer l (1-based) aggregates with max or min
    return l >= 1 && l <= c->L && (c->layers[l - 1].agg == RIPPLE_AGG_MAX || c->layers[l - 1].agg == RIPPLE_AGG_MIN);
}
static inline bool rp_layer_attn(const ripple_ctx *c, uint32_t l) {
    return l >= 1 && l <= c->L && c->layers[l - 1].agg == RIPPLE_AGG_ATTN;
}
static inline uint32_t rp_div_up(uint64_t a, uint64_t b) { return (uint32_t)((a + b - 1) / b); }
static inline uint32_t rp_round_up(uint32_t a, uint32_t b) { return (a + b - 1) / b * b; }

static inline bool rp_lists_allowed(const ripple_ctx *c) { return c->n_cap <= RP_LIST_BUCKETS * RP_LIST_IDS; }   // (pair_cap stays 0 else)

// ---- device helpers -----------------------------------------------------------------
#ifdef __HIPCC__
__device__ __forceinline__ int rp_lane() { return threadIdx.x & 63; }
__device__ __forceinline__ bool rp_bit(const uint32_t *bm, uint32_t v) { return (bm[v >> 5] >> (v & 31)) & 1u; }
__device__ __forceinline__ void rp_set_bit(uint32_t *bm, uint32_t v) {
    uint32_t m = 1u << (v & 31);
    if (!(bm[v >> 5] & m)) atomicOr(&bm[v >> 5], m);
}
__device__ __forceinline__ float rp_bf2f(__hip_bfloat16 x) { return __bfloat162float(x); }
__device__ __forceinline__ float rp_load_h(const void *H, int store, size_t idx) {
    return store ? __bfloat162float(((const __hip_bfloat16 *)H)[idx]) : ((const float *)H)[idx];
}
__device__ __forceinline__ uint32_t rp_row_cap(uint32_t need) {   // capacity given to a relocated row
    uint32_t c = need + (need >> 1) + 4u;
    return (c + 3u) & ~3u;
}
// largest i in [lo, hi] with off[i] <= e   (off is non-decreasing, off[lo] <= e)
__device__ __forceinline__ uint32_t rp_seg_search(const uint32_t *off, uint32_t lo, uint32_t hi, uint32_t e) {
    while (lo < hi) {
        const uint32_t mid = (lo + hi + 1) >> 1;
        if (off[mid] <= e) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}
// The same for a value that all 64 lanes share, found by the wavefront together: 64 probes per round
// trip instead of one, so a list of up to 4096 rows takes two dependent reads and not twelve. To be
// called by all 64 lanes.
__device__ __forceinline__ uint32_t rp_seg_search_wave(const uint32_t *off, uint32_t lo, uint32_t hi, uint32_t e) {
    const uint32_t lane = (uint32_t)rp_lane();
    while (hi - lo >= 64u) {
        const uint32_t step = (hi - lo) / 64u + 1u;        // probes at lo + step, lo + 2 step, ... (clipped to hi)
        const uint32_t p = min(hi, lo + (lane + 1u) * step);
        const uint32_t k = (uint32_t)__popcll(__ballot(off[p] <= e));   // the probes that are <= e come first
        const uint32_t nlo = k ? min(hi, lo + k * step) : lo;
        const uint32_t nhi = (k == 64u) ? hi : min(hi, lo + (k + 1u) * step) - 1u;
        lo = nlo;
        hi = max(nlo, nhi);
    }
    const uint32_t p = lo + lane;
    return lo + (uint32_t)__popcll(__ballot(p <= hi && p > lo && off[p] <= e));
}
// end of row i of the out-edge space of a listed set: eoff holds where each row begins, M is the total
__device__ __forceinline__ uint32_t rp_row_end(const uint32_t *eoff, uint32_t count, uint32_t M, uint32_t i) {
    return i + 1u < count ? eoff[i + 1u] : M;
}
// the same over [lo, last], for an answer expected close to lo: doubling steps, then bisection
__device__ __forceinline__ uint32_t rp_seg_forward(const uint32_t *off, uint32_t lo, uint32_t last, uint32_t e) {
    uint32_t step = 1;
    while (lo + step <= last && off[lo + step] <= e) {
        lo += step;
        step <<= 1;
    }
    return rp_seg_search(off, lo, min(last, lo + step), e);
}
// inclusive prefix sum over the 64 lanes (data-parallel primitives: shifts inside rows of 16 lanes, then row broadcasts)
__device__ __forceinline__ uint32_t rp_wave_scan(uint32_t x) {
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xf, 0xf, false);   // row_shr:1
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xf, 0xf, false);   // row_shr:2
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xf, 0xf, false);   // row_shr:4
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xf, 0xf, false);   // row_shr:8
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xa, 0xf, false);   // row_bcast:15 into rows 1 and 3
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xc, 0xf, false);   // row_bcast:31 into rows 2 and 3
    return x;
}
// number of lanes whose value b (ascending over the lanes) is <= e, found with shuffles; to be
// called by all 64 lanes together
__device__ __forceinline__ uint32_t rp_count_le(uint32_t b, uint32_t e) {
    const uint32_t top = __shfl(b, 63);
    uint32_t lo = 0;                                        // b of every lane below lo is <= e
#pragma unroll
    for (int s = 32; s > 0; s >>= 1) {
        const uint32_t v = __shfl(b, (int)(lo + s - 1));
        if (v <= e) lo += s;
    }
    if (lo == 63 && top <= e) lo = 64;
    return lo;
}

// true in the last of n workgroups to get here (all of what the others wrote is then visible; SYSTEM: to the host as well); called by whole
// workgroups. One wavefront of a workgroup passes the fence for all: it writes back the L2, and a fence in each of them made a launch of 64 workgroups
// that reports its end take 12.6 us until the host sees it (8.7 with one; a launch and k_report behind it 9.4).
template <bool SYSTEM = false>
__device__ __forceinline__ bool last_workgroup(DevCtr *ctr, uint32_t n) {
    __shared__ uint32_t s_last;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");        // this wavefront's stores and atomics have been performed: a barrier alone does not wait for them
    __syncthreads();
    if (threadIdx.x == 0) {
        if (SYSTEM) __threadfence_system();                 // results may lie in the host's memory
        else __threadfence();
        s_last = atomicAdd(&ctr->blocks_done, 1u) == n - 1u ? 1u : 0u;
        if (s_last) ctr->blocks_done = 0;
    }
    __syncthreads();
    if (!s_last) return false;
    __threadfence();
    return true;
}
// The same for a launch whose results the host waits for by looking at *flag (pinned memory) instead of waiting for the stream: the
// last workgroup stores `seq` there. flag null: nothing is reported. For launches of at most REPORT_WGS workgroups (each costs about 16 ns, one after
// the other: up to 96 of them take as long as k_report or less); after larger ones k_report does it.
#define REPORT_WGS 96u
struct HostFlag {
    uint32_t *flag;
    uint32_t seq;
    DevCtr *ctr;
};
__device__ __forceinline__ void report_done(const HostFlag &h, uint32_t n) {
    if (!h.flag) return;
    if (last_workgroup<true>(h.ctr, n) && threadIdx.x == 0) __hip_atomic_store(h.flag, h.seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// ---- packed messages ------------------------------------------------------------------
// A message row of 33..48 numbers as one 128-byte line of sixteen 8-byte chunks. Chunk c holds columns
// c, 16 + c and 32 + c as 19-bit two's-complement integers q (bits 0-18, 19-37, 38-56) that share a power of
// two: the 7-bit code E in bits 57-63 stands for the factor 2^(E - 82) (E = 0: the three numbers are zero). The
// largest of the three keeps 18 significant bits, so a number is off by at most 2^-19 of the largest in its
// chunk. A chunk is all a lane needs to decode its three columns: nothing is exchanged between lanes.
// Magnitudes of 2^63 and above are clipped; below 2^-82 they round to zero.
#define RP_MSG_WORDS 32u
#define RP_MSG_QBITS 19
static inline uint32_t rp_msg_packed(uint32_t d) { return (d > 32u && d <= 48u) ? 1u : 0u; }   // up to 32 floats are one line as they are
#ifdef __HIPCC__
// binary exponent of the factor of a chunk whose largest magnitude is `big`; and a number as its integer
__device__ __forceinline__ int rp_msg_exp(float big) {
    int e = 0;
    (void)frexpf(big, &e);                                  // big < 2^e
    return max(-81, min(45, e - (RP_MSG_QBITS - 1)));       // the factor is 2^se
}
__device__ __forceinline__ int rp_msg_q(float m, int se) {
    const int lim = (1 << (RP_MSG_QBITS - 1)) - 1;
    return max(-lim - 1, min(lim, __float2int_rn(ldexpf(m, -se))));
}
// what a number of such a chunk arrives as
__device__ __forceinline__ float rp_msg_round(float m, float big) {
    const int se = rp_msg_exp(big);
    return big > 0.0f ? (float)rp_msg_q(m, se) * ldexpf(1.0f, se) : 0.0f;
}
__device__ __forceinline__ uint2 rp_msg_encode(float m0, float m1, float m2, float &v0, float &v1, float &v2) {
    const float big = fmaxf(fabsf(m0), fmaxf(fabsf(m1), fabsf(m2)));
    const int se = rp_msg_exp(big);
    const bool zero = !(big > 0.0f);
    const int q0 = zero ? 0 : rp_msg_q(m0, se), q1 = zero ? 0 : rp_msg_q(m1, se), q2 = zero ? 0 : rp_msg_q(m2, se);
    const float f = ldexpf(1.0f, se);
    v0 = (float)q0 * f;                                     // the values the integers stand for (exact products)
    v1 = (float)q1 * f;
    v2 = (float)q2 * f;
    const unsigned long long mask = (1ull << RP_MSG_QBITS) - 1ull;
    const unsigned long long bits = ((unsigned long long)(uint32_t)q0 & mask) | (((unsigned long long)(uint32_t)q1 & mask) << 19) |
                                    (((unsigned long long)(uint32_t)q2 & mask) << 38) |
                                    ((unsigned long long)(zero ? 0u : (uint32_t)(se + 82)) << 57);
    return make_uint2((uint32_t)bits, (uint32_t)(bits >> 32));
}
__device__ __forceinline__ void rp_msg_decode(uint2 c, float &v0, float &v1, float &v2) {
    const float f = __uint_as_float(((c.y >> 25) + 45u) << 23);           // 2^(E - 82); E = 0 meets q = 0
    const int q0 = ((int)(c.x << 13)) >> 13;
    const int q1 = ((int)(__builtin_amdgcn_alignbit(c.y, c.x, 19) << 13)) >> 13;
    const int q2 = ((int)(c.y << 7)) >> 13;
    v0 = (float)q0 * f;
    v1 = (float)q1 * f;
    v2 = (float)q2 * f;
}
// the same in parts: the three integers as floats and the chunk's factor; (float)q * f is exact, so a fused
// multiply-add of the two into a sum rounds as the sum of the decoded value would
__device__ __forceinline__ void rp_msg_decode_parts(uint2 c, float &q0, float &q1, float &q2, float &f) {
    f = __uint_as_float(((c.y >> 25) + 45u) << 23);
    q0 = (float)(((int)(c.x << 13)) >> 13);
    q1 = (float)(((int)(__builtin_amdgcn_alignbit(c.y, c.x, 19) << 13)) >> 13);
    q2 = (float)(((int)(c.y << 7)) >> 13);
}
// column `col` alone (kernels that give every lane one column)
__device__ __forceinline__ float rp_msg_decode_col(uint2 c, uint32_t col) {
    float v0, v1, v2;
    rp_msg_decode(c, v0, v1, v2);
    return col < 16u ? v0 : (col < 32u ? v1 : v2);
}
#endif

// How hop l (1-based) moves its messages, decided on the device from the hop's own counters so
// that no host round trip is needed. 0 push: walk the out-edges of A_{l-1}, one atomic row update
// per message. 1 pull: scan the in-rows of A_l (index + dirty-bit probe per in-edge) and gather each
// message once. 2 discover: when A_{l-1} sends along a large share of all edges nearly every vertex
// is hit, so the in-rows of all live vertices are scanned once, which both gathers the messages and
// finds A_l, and the out-edge walk that would have marked A_l is skipped.
// mode: 0 automatic, 1 push, 2 pull, 3 discover wherever it is allowed.
#define RP_HOP_PUSH 0
#define RP_HOP_PULL 1
#define RP_HOP_DISCOVER 2
#define RP_HOP_SORTED 3                 // from the list of the hop's messages, sorted by destination (reported only)
__device__ __forceinline__ int rp_hop_mode(const DevCtr *ctr, uint32_t l, uint32_t d, int mode, int ratio, int allow_disc) {
    const unsigned long long m = ctr->set[l - 1].m;
    if (allow_disc && m > 0 && (mode == 3 || (mode == 0 && m * 8ull >= ctr->n_edges))) return RP_HOP_DISCOVER;
    if (mode == 1) return RP_HOP_PUSH;
    if (mode >= 2) return RP_HOP_PULL;
    return (m > 0 && m * d * 4ull * (unsigned long long)ratio >= 8ull * ctr->isum[l]) ? RP_HOP_PULL : RP_HOP_PUSH;
}

// A hop is taken from the list of its messages instead when the list was made (M fits the `cap` entries the host expected, no bucket
// has run over) and it pays (force: whenever the list was made). M: out-edges of A_{l-1}. In place of a pull: writing a message down and
// putting it in its place costs about what RP_LIST_FACTOR tests of an in-neighbour cost, and the launches what RP_LIST_FIXED of them cost. In
// place of a push: the M * d float atomics take longer from RP_LIST_NUMBERS on. All kernels of the hop but what both ways share, us:
//   pushed / listed, 31 M edges: 256 columns, 20 * 2^20 numbers 81 / 90, 32 127 / 96; 128 columns, 7.7 45 / 71, 21 87 / 77; 64 columns, 13 61 / 72, 19
//   83 / 74; 47 packed, 10 62 / 70, 15 88 / 72; 20 columns, 8.7 68 / 81, 15 105 / 105. 7 M edges: 256 columns, 20 98 / 126, 66 269 / 183; 64 columns, 18
//   101 / 107, 36 182 / 140.
//   pulled / listed, 64 columns: 2.1 M entries for 16 K messages 122 / 86, 1.4 M for 5 K 25 / 59; 30 M for 4.6 M 472 / 409; 128 columns, 30 M for
//   4.5 M 545 / 536; 256 columns, 29 M for 2.0 M 582 / 430, 2.0 M for 13 K 37 / 103, 2.8 M for 40 K 163 / 109.
// (Hops with more messages than an eighth of the edges discover: fewer than 6.5 entries per message, where both take as long, are rare.)
#define RP_LIST_FACTOR 4ull
#define RP_LIST_FIXED (2ull << 20)
#define RP_LIST_NUMBERS (16ull << 20)
static inline bool rp_list_pays_pull(unsigned long long m, unsigned long long in_entries) { return RP_LIST_FACTOR * m + RP_LIST_FIXED <= in_entries; }
__device__ __forceinline__ bool rp_hop_listed(const DevCtr *ctr, uint32_t l, uint32_t d, uint32_t M, uint32_t cap, int force, int hop_mode) {
    if (!cap || M == 0 || M > cap || ctr->pair_over[l] || hop_mode == RP_HOP_DISCOVER) return false;
    if (force) return true;
    return hop_mode == RP_HOP_PULL ? RP_LIST_FACTOR * M + RP_LIST_FIXED <= ctr->isum[l] : (unsigned long long)M * d >= RP_LIST_NUMBERS;
}

// An attention hop: its vertices that are recomputed read whole in-rows, the others take a message per changed in-neighbour. Those messages are found by
// testing every in-neighbour, or taken from a list that the out-edge walk writes, where that pays by the same measure (a set reached along M edges has
// about M mean in-degrees of in-neighbours, at most all edges). Decided before the set is known, from M alone: all of the hop's kernels agree.
// Not where M is more than a 64th of the edges: the messages' rows, two each, are then most of the work either way. Walk, compaction and scatter of a second
// hop, us, in-rows tested / messages listed, 0.6 M vertices and 31 M edges:
//   edges per message   47 columns     128 columns      256 columns
//         657           336 / 142      386 / 187        448 / 287
//         138           382 / 347      545 / 418        781 / 657
//          67           436 / 467      671 / 574      1,051 / 930
//          31           529 / 610      890 / 807      1,458 / 1,370
//          10           767 / 825    1,487 / 1,440    2,703 / 2,613
// Rows of up to 63 columns cross at about 100 edges per message, wider ones gain 3 to 9 % up to six times as many messages as the limit lets them have: one limit
// for both. On 0.4 M vertices and 4 M edges, where the second condition (a mean in-degree of ten) never lists, nothing is lost: 47 to 650 edges per message,
// 47 to 256 columns 60 to 222 us, listed 85 to 244.
#define RP_GAT_LIST_SHARE 64ull
__device__ __forceinline__ bool rp_gat_list_made(const DevCtr *ctr, uint32_t M, uint32_t cap, int force) {
    if (!cap || M == 0 || M > cap) return false;
    if (force) return true;
    const unsigned long long e = ctr->n_edges, n = ctr->n_alive ? ctr->n_alive : 1u;
    return RP_GAT_LIST_SHARE * M <= e && RP_LIST_FACTOR * M + RP_LIST_FIXED <= M * (e / n);
}
__device__ __forceinline__ bool rp_gat_listed(const DevCtr *ctr, uint32_t l, uint32_t cap, int force) {
    return cap && !ctr->pair_over[l] && rp_gat_list_made(ctr, ctr->set[l - 1].a ? ctr->set[l - 1].m : 0u, cap, force);
}
// a vertex of the hop's set is recomputed from all its in-neighbours
__device__ __forceinline__ bool rp_gat_recomputes(const uint32_t *bm_prev, const uint32_t *bm_sink, const uint32_t *bm_vadd, const uint2 *in_meta, uint32_t long_min, uint32_t v) {
    const uint32_t w = v >> 5, b = v & 31u, is = bm_prev[w] | bm_vadd[w], sink = bm_sink[w];    // (read together)
    return ((is >> b) & 1u) || (((sink >> b) & 1u) && in_meta[v].y <= long_min);
}

// position of `target` in row[0..len), searched by one wavefront; -1 when absent. Rows begin at multiples of four entries and
// have room for a multiple of four, so every lane reads four at a time, and long (hub) rows are read eight such blocks per round:
// a row of 24,000 entries takes 12 round trips (four bytes per lane and sixteen blocks took 24: 10,000 operations, a wavefront each, 80 us
// instead of 35).
template <int T>
__device__ __forceinline__ int rp_wave_find_blocks(const uint32_t *row, uint32_t base, uint32_t len, uint32_t target) {
    const int lane = rp_lane();
    uint4 v[T];
#pragma unroll
    for (int t = 0; t < T; ++t) {
        const uint32_t i = base + 256 * t + 4 * lane;
        v[t] = (i < len) ? *(const uint4 *)(row + i) : make_uint4(RP_TOMB, RP_TOMB, RP_TOMB, RP_TOMB);   // never a vertex id
    }
#pragma unroll
    for (int t = 0; t < T; ++t) {
        const uint32_t i = base + 256 * t + 4 * lane;
        const int k = v[t].x == target ? 0 : (v[t].y == target && i + 1 < len) ? 1 : (v[t].z == target && i + 2 < len) ? 2
                      : (v[t].w == target && i + 3 < len) ? 3 : 4;
        const unsigned long long m = __ballot(k < 4);
        if (m) {
            const int at = __ffsll((long long)m) - 1;
            return (int)(base + 256 * t + 4 * at + __shfl(k, at));
        }
    }
    return -1;
}
__device__ __forceinline__ int rp_wave_find(const uint32_t *row, uint32_t len, uint32_t target) {
    uint32_t base = 0;
    for (; base + 256 < len; base += 2048) {
        const int p = rp_wave_find_blocks<8>(row, base, len, target);
        if (p >= 0) return p;
    }
    return base < len ? rp_wave_find_blocks<1>(row, base, len, target) : -1;
}
#endif
