// GPU-resident graph store: out- and in-adjacency kept as per-vertex rows with
// slack inside two pools, built from a COO edge list, mutated by batches of
// updates (the Apply step of Sec. 3.3), and compacted when a pool fills up.
//
// A batch is applied in two phases. Validation decides, against the graph as
// it stands, which operations are accepted and how much pool space they need;
// nothing is modified. Only if everything fits does the commit phase run:
// deletions leave tombstones that one wavefront per touched row squeezes out,
// rows that would overflow move to fresh space at the pool's end, additions
// are appended. Deleting a vertex expands into deleting its incident edges
// (Sec. 3.2, vertex deletion). The host guarantees that operations inside one
// launch sequence never touch the same edge twice nor a vertex that the same
// sequence adds or deletes (other than a new vertex's own edges), so all
// operations can be handled in parallel without changing the array-order result.
#include "common.h"
#include "kernels.h"

// ---------------------------------------------------------------------------------
// exclusive scan over uint32 (two kernels: block sums, then per-block prefix + scan)
// ---------------------------------------------------------------------------------
#define SCAN_PER_BLOCK 1024

__device__ __forceinline__ uint32_t block_sum_256(uint32_t v, uint32_t *sh) {
    const int tid = threadIdx.x;
    for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o);
    if ((tid & 63) == 0) sh[tid >> 6] = v;
    __syncthreads();
    uint32_t t = sh[0] + sh[1] + sh[2] + sh[3];
    __syncthreads();
    return t;
}

__global__ __launch_bounds__(256) void k_scan_partial(const uint32_t *in, uint32_t n, uint32_t *part) {
    __shared__ uint32_t sh[4];
    uint32_t base = blockIdx.x * SCAN_PER_BLOCK + threadIdx.x * 4;
    uint32_t s = 0;
    for (int k = 0; k < 4; ++k)
        if (base + k < n) s += in[base + k];
    uint32_t t = block_sum_256(s, sh);
    if (threadIdx.x == 0) part[blockIdx.x] = t;
}

__global__ __launch_bounds__(256) void k_scan_final(const uint32_t *in, uint32_t *out, uint32_t n,
                                                    const uint32_t *part, uint32_t *total_out) {
    __shared__ uint32_t sh[4];
    __shared__ uint32_t wsum[4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    uint32_t pre = 0;
    for (uint32_t b = tid; b < blockIdx.x; b += 256) pre += part[b];
    pre = block_sum_256(pre, sh);
    uint32_t base = blockIdx.x * SCAN_PER_BLOCK + tid * 4;
    uint32_t v[4], s = 0;
    for (int k = 0; k < 4; ++k) {
        v[k] = (base + k < n) ? in[base + k] : 0u;
        s += v[k];
    }
    uint32_t incl = s;                                  // inclusive scan inside the wavefront
    for (int o = 1; o < 64; o <<= 1) {
        uint32_t t = __shfl_up(incl, o);
        if (lane >= o) incl += t;
    }
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    uint32_t woff = 0;
    for (int w = 0; w < wave; ++w) woff += wsum[w];
    uint32_t run = pre + woff + incl - s;
    for (int k = 0; k < 4; ++k) {
        if (base + k < n) out[base + k] = run;
        run += v[k];
    }
    if (total_out && blockIdx.x == gridDim.x - 1 && tid == 255) *total_out = run;
}

// out[i] = exclusive prefix of in[0..n); *total_out = sum. part: scratch of ceil(n/1024) words.
void rp_exclusive_scan(hipStream_t s, const uint32_t *in, uint32_t *out, uint32_t n, uint32_t *part,
                       uint32_t *total_out) {
    if (n == 0) return;
    uint32_t nb = rp_div_up(n, SCAN_PER_BLOCK);
    hipLaunchKernelGGL(k_scan_partial, dim3(nb), dim3(256), 0, s, in, n, part);
    hipLaunchKernelGGL(k_scan_final, dim3(nb), dim3(256), 0, s, in, out, n, part, total_out);
}

// ---------------------------------------------------------------------------------
// build from COO
// ---------------------------------------------------------------------------------
__global__ void k_degree_count(const uint32_t *src, const uint32_t *dst, uint64_t n_edges, uint32_t n_vertices,
                               uint32_t *deg_out, uint32_t *deg_in, uint32_t *err) {
    uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t e = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n_edges; e += stride) {
        uint32_t s = src[e], d = dst[e];
        if (s >= n_vertices || d >= n_vertices) {
            *err = 1;
            continue;
        }
        atomicAdd(&deg_out[s], 1u);
        atomicAdd(&deg_in[d], 1u);
    }
}

__global__ void k_fresh_caps(const uint32_t *len, const uint32_t *alive, uint32_t n_cap, uint32_t *capv) {
    uint32_t v = blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= n_cap) return;
    uint32_t l = len[v];
    bool live = rp_bit(alive, v);
    capv[v] = (live || l) ? ((l + (l >> 3) + 4u + 3u) & ~3u) : 0u;
}

__global__ void k_meta_len(const uint2 *meta, uint32_t n_cap, uint32_t *len) {
    uint32_t v = blockIdx.x * blockDim.x + threadIdx.x;
    if (v < n_cap) len[v] = meta[v].y;
}

__global__ void k_init_meta(const uint32_t *start, uint32_t n_cap, uint2 *meta) {
    uint32_t v = blockIdx.x * blockDim.x + threadIdx.x;
    if (v < n_cap) meta[v] = make_uint2(start[v], 0u);
}

__global__ void k_fill_rows(const uint32_t *key, const uint32_t *val, const float *wts, uint64_t n_edges,
                            uint2 *meta, uint32_t *pool, float *wpool) {
    uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t e = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n_edges; e += stride) {
        uint32_t k = key[e];
        uint32_t p = atomicAdd(&((uint32_t *)meta)[2 * (size_t)k + 1], 1u);
        pool[meta[k].x + p] = val[e];
        if (wpool) wpool[meta[k].x + p] = wts[e];
    }
}

// In-rows are filled in the order the edges were given (a stable sort by sink has put position e of the
// sorted sequence at offset e - first[sink] of the sink's row), so that their order is a function of the input.
__global__ void k_iota(uint32_t *out, uint64_t n) {
    uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t e = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += stride) out[e] = (uint32_t)e;
}

__global__ void k_fill_in_rows_ordered(const uint32_t *sorted_dst, const uint32_t *sorted_idx, const uint32_t *src,
                                       const float *wts, uint64_t n_edges, const uint32_t *first, const uint2 *meta,
                                       uint32_t *pool, float *wpool) {
    uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t e = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n_edges; e += stride) {
        const uint32_t k = sorted_dst[e], i = sorted_idx[e];
        const size_t at = (size_t)meta[k].x + ((uint32_t)e - first[k]);
        pool[at] = src[i];
        if (wpool) wpool[at] = wts[i];
    }
}

__global__ void k_set_len(uint2 *meta, const uint32_t *len, uint32_t n_cap) {
    uint32_t v = blockIdx.x * blockDim.x + threadIdx.x;
    if (v < n_cap) meta[v].y = len[v];
}

__global__ void k_set_alive_prefix(uint32_t *alive, uint32_t n_words, uint32_t n_vertices) {
    uint32_t w = blockIdx.x * blockDim.x + threadIdx.x;
    if (w >= n_words) return;
    uint32_t lo = w * 32u;
    uint32_t bits = 0;
    if (lo + 32u <= n_vertices) bits = 0xFFFFFFFFu;
    else if (lo < n_vertices) bits = (1u << (n_vertices - lo)) - 1u;
    alive[w] = bits;
}

ripple_status rp_build_graph(ripple_ctx *c, uint32_t n_vertices, uint64_t n_edges, const uint32_t *src_h,
                             const uint32_t *dst_h, const float *w_h) {
    hipStream_t s = c->stream;
    uint32_t *src_d = nullptr, *dst_d = nullptr, *tmp = nullptr, *err_d = nullptr;
    float *w_d = nullptr;
    size_t eb = (size_t)(n_edges ? n_edges : 1) * sizeof(uint32_t);
    RP_HIP(c, hipMalloc(&src_d, eb));
    RP_HIP(c, hipMalloc(&dst_d, eb));
    RP_HIP(c, hipMalloc(&tmp, (size_t)c->n_cap * 4 * 2 + 64));
    RP_HIP(c, hipMalloc(&err_d, 64));
    RP_HIP(c, hipMemsetAsync(err_d, 0, 64, s));
    if (n_edges) {
        RP_HIP(c, hipMemcpyAsync(src_d, src_h, eb, hipMemcpyHostToDevice, s));
        RP_HIP(c, hipMemcpyAsync(dst_d, dst_h, eb, hipMemcpyHostToDevice, s));
        if (w_h) {
            RP_HIP(c, hipMalloc(&w_d, eb));
            RP_HIP(c, hipMemcpyAsync(w_d, w_h, eb, hipMemcpyHostToDevice, s));
        }
    }
    uint32_t *deg_out = tmp, *deg_in = tmp + c->n_cap;
    RP_HIP(c, hipMemsetAsync(tmp, 0, (size_t)c->n_cap * 8, s));
    hipLaunchKernelGGL(k_set_alive_prefix, dim3(rp_div_up(c->n_words, 256)), dim3(256), 0, s, c->alive,
                       c->n_words, n_vertices);
    uint32_t gb = (uint32_t)std::min<uint64_t>(rp_div_up(n_edges ? n_edges : 1, 256), 65536);
    hipLaunchKernelGGL(k_degree_count, dim3(gb), dim3(256), 0, s, src_d, dst_d, n_edges, n_vertices, deg_out,
                       deg_in, err_d);
    uint32_t vb = rp_div_up(c->n_cap, 256);
    // caps -> starts, for both directions; pend_* serve as scratch for the scan output
    hipLaunchKernelGGL(k_fresh_caps, dim3(vb), dim3(256), 0, s, deg_out, c->alive, c->n_cap, c->out_capv);
    hipLaunchKernelGGL(k_fresh_caps, dim3(vb), dim3(256), 0, s, deg_in, c->alive, c->n_cap, c->in_capv);
    rp_exclusive_scan(s, c->out_capv, c->pend_out, c->n_cap, c->part_cnt, &c->ctr->out_top);
    rp_exclusive_scan(s, c->in_capv, c->pend_in, c->n_cap, c->part_deg, &c->ctr->in_top);
    hipLaunchKernelGGL(k_init_meta, dim3(vb), dim3(256), 0, s, c->pend_out, c->n_cap, c->out_meta);
    hipLaunchKernelGGL(k_init_meta, dim3(vb), dim3(256), 0, s, c->pend_in, c->n_cap, c->in_meta);
    uint32_t err_h = 0;
    RP_HIP(c, hipMemcpyAsync(&err_h, err_d, 4, hipMemcpyDeviceToHost, s));
    RP_HIP(c, hipMemcpyAsync(c->ctr_host, c->ctr, sizeof(DevCtr), hipMemcpyDeviceToHost, s));
    RP_HIP(c, hipStreamSynchronize(s));
    ripple_status rc = RIPPLE_OK;
    if (err_h) {
        c->err = "edge endpoint is not a live vertex (id >= n_vertices)";
        rc = RIPPLE_EINVAL;
    } else if (c->ctr_host->out_top > c->pool_cap || c->ctr_host->in_top > c->pool_cap) {
        c->err = "edge_capacity too small for the initial graph";
        rc = RIPPLE_ECAPACITY;
    } else if (n_edges) {
        hipLaunchKernelGGL(k_fill_rows, dim3(gb), dim3(256), 0, s, src_d, dst_d, (const float *)w_d, n_edges,
                           c->out_meta, c->out_pool, w_d ? c->out_w : (float *)nullptr);
        // in-rows: stable sort of the edge numbers by sink, then every edge knows its place
        uint32_t *ord = nullptr;
        unsigned key_bits = 1;
        while (key_bits < 32 && (1ull << key_bits) < (unsigned long long)n_vertices) ++key_bits;
        if (hipMalloc(&ord, 3 * eb + (size_t)c->n_cap * 4) != hipSuccess) {
            (void)hipGetLastError();
            c->err = "device allocation for the build failed";
            rc = RIPPLE_ENOMEM;
        } else {
            uint32_t *idx = ord, *sdst = ord + n_edges, *sidx = ord + 2 * n_edges, *first = ord + 3 * n_edges;
            hipLaunchKernelGGL(k_iota, dim3(gb), dim3(256), 0, s, idx, n_edges);
            rc = rp_stable_sort_pairs(c, dst_d, sdst, idx, sidx, (size_t)n_edges, key_bits);
            if (rc == RIPPLE_OK) {
                rp_exclusive_scan(s, deg_in, first, c->n_cap, c->part_deg, nullptr);
                hipLaunchKernelGGL(k_fill_in_rows_ordered, dim3(gb), dim3(256), 0, s, sdst, sidx, src_d, (const float *)w_d,
                                   n_edges, first, c->in_meta, c->in_pool, w_d ? c->in_w : (float *)nullptr);
                hipLaunchKernelGGL(k_set_len, dim3(vb), dim3(256), 0, s, c->in_meta, deg_in, c->n_cap);
            }
            hipStreamSynchronize(s);
            hipFree(ord);
        }
    }
    hipMemsetAsync(c->pend_out, 0, (size_t)c->n_cap * 4, s);
    hipMemsetAsync(c->pend_in, 0, (size_t)c->n_cap * 4, s);
    hipStreamSynchronize(s);
    hipFree(src_d);
    hipFree(dst_d);
    if (w_d) hipFree(w_d);
    hipFree(tmp);
    hipFree(err_d);
    if (rc == RIPPLE_OK) RP_HIP(c, hipGetLastError());
    return rc;
}

// ---------------------------------------------------------------------------------
// compaction: fresh caps, scan, copy every row into a new pool
// ---------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_copy_rows(uint2 *meta, const uint32_t *new_start, uint32_t n_cap,
                                                   const uint32_t *old_pool, uint32_t *new_pool, const float *old_w,
                                                   float *new_w) {
    const int lane = rp_lane();
    uint32_t gw = (blockIdx.x * blockDim.x + threadIdx.x) >> 6, nw = (gridDim.x * blockDim.x) >> 6;
    for (uint32_t v = gw; v < n_cap; v += nw) {
        uint2 m = meta[v];
        uint32_t ns = new_start[v];
        for (uint32_t i = lane; i < m.y; i += 64) new_pool[ns + i] = old_pool[m.x + i];
        if (old_w)
            for (uint32_t i = lane; i < m.y; i += 64) new_w[ns + i] = old_w[m.x + i];
        if (lane == 0) meta[v] = make_uint2(ns, m.y);
    }
}

static ripple_status compact_one(ripple_ctx *c, uint2 *meta, uint32_t *capv, uint32_t **pool, float **wpool,
                                 uint32_t *top_d, uint32_t *scratch_len, uint32_t *scratch_start) {
    hipStream_t s = c->stream;
    uint32_t vb = rp_div_up(c->n_cap, 256);
    uint32_t *new_pool = nullptr;
    float *new_w = nullptr;
    RP_HIP(c, hipMalloc(&new_pool, (size_t)c->pool_cap * 4));
    if (wpool && *wpool) RP_HIP(c, hipMalloc(&new_w, (size_t)c->pool_cap * 4));
    hipLaunchKernelGGL(k_meta_len, dim3(vb), dim3(256), 0, s, meta, c->n_cap, scratch_len);
    hipLaunchKernelGGL(k_fresh_caps, dim3(vb), dim3(256), 0, s, scratch_len, c->alive, c->n_cap, capv);
    rp_exclusive_scan(s, capv, scratch_start, c->n_cap, c->part_cnt, top_d);
    hipLaunchKernelGGL(k_copy_rows, dim3(c->n_cu * 8), dim3(256), 0, s, meta, scratch_start, c->n_cap, *pool,
                       new_pool, (const float *)(new_w ? *wpool : nullptr), new_w);
    RP_HIP(c, hipStreamSynchronize(s));
    hipFree(*pool);
    *pool = new_pool;
    if (new_w) {
        hipFree(*wpool);
        *wpool = new_w;
    }
    return RIPPLE_OK;
}

ripple_status rp_compact(ripple_ctx *c) {
    // pend_* / dead_* are zero between batches and serve as scratch here
    ripple_status rc = compact_one(c, c->out_meta, c->out_capv, &c->out_pool, &c->out_w, &c->ctr->out_top, c->pend_out,
                                   c->dead_out);
    if (rc != RIPPLE_OK) return rc;
    rc = compact_one(c, c->in_meta, c->in_capv, &c->in_pool, &c->in_w, &c->ctr->in_top, c->pend_in, c->dead_in);
    if (rc != RIPPLE_OK) return rc;
    hipStream_t s = c->stream;
    RP_HIP(c, hipMemsetAsync(c->pend_out, 0, (size_t)c->n_cap * 4, s));
    RP_HIP(c, hipMemsetAsync(c->pend_in, 0, (size_t)c->n_cap * 4, s));
    RP_HIP(c, hipMemsetAsync(c->dead_out, 0, (size_t)c->n_cap * 4, s));
    RP_HIP(c, hipMemsetAsync(c->dead_in, 0, (size_t)c->n_cap * 4, s));
    RP_HIP(c, hipStreamSynchronize(s));
    return RIPPLE_OK;
}

// ---------------------------------------------------------------------------------
// batch application
// ---------------------------------------------------------------------------------
struct MutArgs {
    const ripple_update *ops;
    uint32_t n_ops;
    const uint32_t *made;                        // small pieces: the vertices that the piece creates (pinned host memory)
    uint32_t n_made;
    const float *payload;
    uint32_t *status, *pos_out, *pos_in;
    uint32_t *rank_out, *rank_in;                // an edge operation's number among the row's additions or deletions
    uint32_t *op_touch;                          // bit 0 accepted edge op, 1 it is an add, 2 / 3 first touch of out-row(u) / in-row(v)
    uint2 *out_meta, *in_meta;
    uint32_t *out_capv, *in_capv;
    uint32_t *out_pool, *in_pool;
    float *in_w, *out_w;                         // edge weights parallel to in_pool and out_pool, or null
    uint32_t *alive, *vstate;
    uint32_t *pend_out, *pend_in, *dead_out, *dead_in;
    uint32_t *hole_out, *hole_in;                // where a touched row's segment of seg_id / seg_x begins
    uint32_t *seg_id, *seg_x;                    // per row: deletions (seg_x: position; in-rows, seg_id: source), then additions (seg_id:
                                                 // the other end; seg_x: the weight's bits)
    uint32_t *srt_id, *srt_x;                    // deterministic mode: long segments in order
    uint32_t *touch_out, *touch_in;
    uint32_t touch_cap;
    uint32_t *exp_kind, *exp_a, *exp_b;
    uint32_t *exp_pos, *exp_rank;                // where such an edge is in the row that stays, and its number among the row's deletions
    uint32_t exp_cap;
    uint32_t *st_src, *st_dst;
    float *st_sign, *st_unit;
    uint32_t struct_cap;
    uint32_t *bm0, *bm_sink, *bm_vadd;
    uint32_t *list0, *eoff0;
    float *D0;
    DevCtr *ctr;
    uint32_t n_cap;
    unsigned long long e_cap, pool_cap;
    int store;
    uint32_t L;
    uint32_t d[RIPPLE_MAX_LAYERS + 1];
    uint32_t xw[RIPPLE_MAX_LAYERS + 1];          // width of X^l
    void *H[RIPPLE_MAX_LAYERS + 1];
    float *X[RIPPLE_MAX_LAYERS + 1];
    float *T[RIPPLE_MAX_LAYERS + 1];             // project-first layers: what every vertex has sent so far (xw[l] floats per vertex), else null
    uint32_t ldt[RIPPLE_MAX_LAYERS + 1];         // its row stride
    uint32_t mono_mask;                          // bit l: layer l takes max / min or attention (no structural terms)
    uint32_t wsum_mask;                          // bit l: layer l aggregates with the edge weights
    int d0_old;                                  // layer 1 does: D0 receives the old feature row instead of the difference
    int det;                                     // deterministic mode
};

// slot in a global list for every lane with pred, one atomic per wavefront
__device__ __forceinline__ uint32_t wave_reserve(uint32_t *counter, bool pred) {
    unsigned long long m = __ballot(pred);
    if (!m) return 0;
    const int lane = rp_lane();
    int leader = __ffsll((long long)m) - 1;
    uint32_t base = 0;
    if (lane == leader) base = atomicAdd(counter, (uint32_t)__popcll(m));
    base = __shfl(base, leader);
    return base + (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
}

// The Apply step is paced by launches and by chains of dependent reads, not by bytes. Its launches are as few as its global
// dependencies allow: operations staged and vertex operations judged (k_stage), edge operations judged (k_validate, beside
// which the edges of deleted vertices are listed, then found by k_find_expanded), rows listed and measured and the decision
// taken (k_measure), edges (k_edges: tombstones, changed edges and structural terms, A_0) and rows
// (k_rows: feature rows, and every touched row finished by one wavefront). Small pieces do all that precedes k_edges in one
// launch (k_small_validate). 1,000 operations on the sparse graph took eleven to thirteen launches and 120 us of kernels.
//
// What an operation adds to or takes out of a row reaches the row's wavefront through a segment of two arrays: validation
// counts a row's additions and deletions (the counts' old values number them), the rows' segments are laid out one after
// the other (base in hole_out / hole_in: first the deletions, then the additions), and k_edges puts every operation's entry
// where its number says. So neither tombstones nor room for additions have to be searched for: squeezing two tombstones
// out of a row of ten thousand entries reads two entries and not all.

// operations from pinned host memory; vertex operations are judged on the way; bitmaps cleared
__global__ __launch_bounds__(256) void k_stage(MutArgs a, const ripple_update *src, ripple_update *dst, uint32_t *bitmaps, uint32_t n_bitmap_words) {
    const uint32_t stride = gridDim.x * 256u, t = blockIdx.x * 256u + threadIdx.x;
    for (uint32_t k = t; k < n_bitmap_words; k += stride) bitmaps[k] = 0;
    for (uint32_t i = t; i < a.n_ops; i += stride) {
        const ripple_update op = src[i];
        dst[i] = op;
        if (op.kind == RIPPLE_VERTEX_ADD) {
            const bool ok = !rp_bit(a.alive, op.u);
            if (ok) atomicOr(&a.vstate[op.u], VS_ADDING);
            a.status[i] = ok ? 1u : 0u;
        } else if (op.kind == RIPPLE_VERTEX_DEL) {
            const bool ok = rp_bit(a.alive, op.u);
            if (ok) {
                atomicOr(&a.vstate[op.u], VS_DYING);
                atomicAdd(&a.ctr->need_exp, a.out_meta[op.u].y + a.in_meta[op.u].y);
            }
            a.status[i] = ok ? 1u : 0u;
        }
    }
}

// Where `target` is in the row, searched by PARTS wavefronts that take blocks of 2,048 entries in turn; -1 if this wavefront does
// not find it
template <uint32_t PARTS>
__device__ __forceinline__ int find_part(const uint32_t *row, uint32_t len, uint32_t target, uint32_t part) {
    if (PARTS == 1) return rp_wave_find(row, len, target);
    if (len <= 256u) return part == 0 && len ? rp_wave_find_blocks<1>(row, 0, len, target) : -1;
    for (uint32_t base = part * 2048u; base < len; base += PARTS * 2048u) {
        const int p = rp_wave_find_blocks<8>(row, base, len, target);
        if (p >= 0) return p;
    }
    return -1;
}

// An accepted edge operation's number in its rows, and its flags: bit 0 accepted, 1 add, 2 / 3 first touch of out-row(u) /
// in-row(v). One lane.
__device__ __forceinline__ uint32_t count_edge(const MutArgs &a, const ripple_update &op, uint32_t i, int po, int pi) {
    const bool is_add = op.kind == RIPPLE_EDGE_ADD;
    // the four atomics are under way together: nothing waits for one before the next is sent
    const uint32_t to = atomicOr(&a.vstate[op.u], VS_TOUCH_OUT), ti = atomicOr(&a.vstate[op.v], VS_TOUCH_IN);
    const uint32_t ro = atomicAdd(is_add ? &a.pend_out[op.u] : &a.dead_out[op.u], 1u);
    const uint32_t ri = atomicAdd(is_add ? &a.pend_in[op.v] : &a.dead_in[op.v], 1u);
    if (!is_add) {
        a.pos_out[i] = (uint32_t)po;
        a.pos_in[i] = (uint32_t)pi;
    }
    a.rank_out[i] = ro;
    a.rank_in[i] = ri;
    const uint32_t flags = 1u | (is_add ? 2u : 0u) | ((to & VS_TOUCH_OUT) ? 0u : 4u) | ((ti & VS_TOUCH_IN) ? 0u : 8u);
    return flags;
}

// One operation, by W wavefronts that search its rows together (W = 1: one wavefront that shares nothing with the others of its
// workgroup). Thousands of wavefronts bumping the same few counters would queue up behind one another: only the rows' own bits
// and counts are set here, measure() makes the lists.
// SMALL: vertex operations are judged here too, and a vertex that is not alive may be one that this piece creates (a.made)
template <int W, int SMALL>
__device__ __forceinline__ void validate_op(const MutArgs &a, uint32_t i, const ripple_update &op, int *s_pos) {
    const int lane = rp_lane();
    const uint32_t wave = W == 1 ? 0u : threadIdx.x >> 6;
    const bool first = W == 1 ? lane == 0 : threadIdx.x == 0;
    const bool is_add = op.kind == RIPPLE_EDGE_ADD, is_edge = is_add || op.kind == RIPPLE_EDGE_DEL;
    if (W > 1) {
        if (threadIdx.x < 2) s_pos[threadIdx.x] = -1;
        __syncthreads();
    }
    uint32_t st = 0;
    bool judged = true;
    int po = -1, pi = -1;
    if (op.kind == RIPPLE_FEAT_UPDATE) {                   // needs the live flag only
        st = rp_bit(a.alive, op.u) ? 1u : 0u;
    } else if (op.kind == RIPPLE_VERTEX_ADD || op.kind == RIPPLE_VERTEX_DEL) {
        judged = SMALL;                                    // (otherwise by k_stage)
        if (SMALL) st = rp_bit(a.alive, op.u) ? 0u : 1u;   // (small pieces delete no vertices)
    } else {
        bool ok = true;
        const uint2 mo = a.out_meta[op.u], mi = a.in_meta[op.v];
        const bool live[2] = {rp_bit(a.alive, op.u), rp_bit(a.alive, op.v)};
        for (int side = 0; side < 2; ++side) {              // alive, or (edges) created by this piece
            const uint32_t w = side ? op.v : op.u;
            if (live[side]) continue;
            bool created = false;
            if (!SMALL) {
                created = is_edge && (a.vstate[w] & VS_ADDING);
            } else if (is_edge) {
                for (uint32_t k = lane; k < a.n_made; k += 64u) created |= a.made[k] == w;
                created = __ballot(created) != 0ull;
            }
            ok = ok && created;
        }
        if (ok) {                                           // the same for all wavefronts
            const uint32_t *ro = a.out_pool + mo.x, *ri = a.in_pool + mi.x;
            const uint32_t half = W / 2;
            if (is_add) {                                   // absent from the shorter of the two rows
                if (mo.y <= mi.y) po = find_part<W>(ro, mo.y, op.v, wave);
                else po = find_part<W>(ri, mi.y, op.u, wave);
            } else if (!is_edge && !a.out_w) {              // EDGE_REWEIGHT where only the in-row holds the weight (with weights in both rows: like a deletion)
                if (a.in_w) pi = find_part<W>(ri, mi.y, op.u, wave);
            } else if (W == 1) {
                po = find_part<1>(ro, mo.y, op.v, 0);
                if (po >= 0) pi = find_part<1>(ri, mi.y, op.u, 0);
            } else if (wave < half) {
                po = find_part<(W > 1 ? W / 2 : 1)>(ro, mo.y, op.v, wave);
            } else {
                pi = find_part<(W > 1 ? W / 2 : 1)>(ri, mi.y, op.u, wave - half);
            }
            if (W > 1 && lane == 0 && po >= 0) s_pos[0] = po;    // an entry occurs once: one wavefront finds it
            if (W > 1 && lane == 0 && pi >= 0) s_pos[1] = pi;
        }
        if (W > 1) {
            __syncthreads();
            po = s_pos[0];
            pi = s_pos[1];
        }
        if (ok && is_add) st = po < 0 ? 1u : 0u;
        else if (ok && !is_edge && !a.out_w) st = pi >= 0 ? 1u : 0u;
        else if (ok) {
            st = (po >= 0 && pi >= 0) ? 1u : 0u;
            if (first && (po >= 0) != (pi >= 0)) a.ctr->error = 3;     // the two adjacencies disagree
        }
        if (first && !is_edge && st) {
            a.pos_out[i] = (uint32_t)po;
            a.pos_in[i] = (uint32_t)pi;
        }
    }
    if (first) {
        if (judged) a.status[i] = st;
        a.op_touch[i] = (is_edge && st) ? count_edge(a, op, i, po, pi) : 0u;
    }
    if (W > 1) __syncthreads();                             // (s_pos is set anew)
}

#define EXPAND_OPS 16u
// The edges of the vertices that the piece deletes, a workgroup per 16 operations: it takes the vertices among them one after the other, all its
// wavefronts together, 1,024 entries of a row at a time. (A wavefront per vertex, 64 entries at a time: 100 deleted vertices on the dense
// graph, some with thousands of in-edges, held k_validate up for 142 us, now 104.)
__device__ __forceinline__ void list_expanded(const MutArgs &a, uint32_t bid, uint32_t nb, uint32_t *s_base) {
    if (a.ctr->need_exp > a.exp_cap) return;                // no room: the piece will not be committed
    constexpr int U = 4;
    const int lane = rp_lane();
    const uint32_t tid = threadIdx.x;
    for (uint32_t i0 = bid * EXPAND_OPS; i0 < a.n_ops; i0 += nb * EXPAND_OPS) {
        const uint32_t i = i0 + (uint32_t)lane, ic = min(i, a.n_ops - 1u);   // (the same operations in all wavefronts)
        const ripple_update op = a.ops[ic];
        const uint32_t st = a.status[ic];
        unsigned long long left = __ballot(lane < (int)EXPAND_OPS && i < a.n_ops && op.kind == RIPPLE_VERTEX_DEL && st != 0u);
        for (; left; left &= left - 1ull) {
            const uint32_t w = (uint32_t)__shfl((int)op.u, __ffsll((long long)left) - 1);
            const uint2 mo = a.out_meta[w], mi = a.in_meta[w];
            __syncthreads();
            if (tid == 0) *s_base = atomicAdd(&a.ctr->n_exp, mo.y + mi.y);
            __syncthreads();
            const uint32_t base = *s_base;
            for (uint32_t j0 = tid; j0 < mo.y; j0 += 256u * U) {
                uint32_t y[U], st[U];
#pragma unroll
                for (int t = 0; t < U; ++t) y[t] = a.out_pool[mo.x + min(j0 + 256u * t, mo.y - 1u)];
#pragma unroll
                for (int t = 0; t < U; ++t) st[t] = a.vstate[y[t]];
#pragma unroll
                for (int t = 0; t < U; ++t) {
                    const uint32_t j = j0 + 256u * t;
                    if (j >= mo.y) continue;
                    a.exp_kind[base + j] = (st[t] & VS_DYING) ? EXP_NONE : EXP_OUT;
                    a.exp_a[base + j] = w;
                    a.exp_b[base + j] = y[t];
                }
            }
            uint32_t gone = 0;
            for (uint32_t j0 = tid; j0 < mi.y; j0 += 256u * U) {
                uint32_t x[U], st[U];
#pragma unroll
                for (int t = 0; t < U; ++t) x[t] = a.in_pool[mi.x + min(j0 + 256u * t, mi.y - 1u)];
#pragma unroll
                for (int t = 0; t < U; ++t) st[t] = a.vstate[x[t]];
#pragma unroll
                for (int t = 0; t < U; ++t) {
                    const uint32_t j = j0 + 256u * t;
                    if (j >= mi.y) continue;
                    const bool keep = !(st[t] & VS_DYING);  // edges between two dying vertices count once
                    a.exp_kind[base + mo.y + j] = keep ? EXP_IN : EXP_NONE;
                    a.exp_a[base + mo.y + j] = x[t];
                    a.exp_b[base + mo.y + j] = w;
                    gone += keep ? 1u : 0u;
                }
            }
            gone = (uint32_t)__builtin_amdgcn_readlane((int)rp_wave_scan(gone), 63);
            if (tid == 0) gone += mo.y;                      // every out-edge disappears
            if (lane == 0 && gone) atomicAdd(&a.ctr->n_gone, gone);
        }
    }
}

// The first nd workgroups list the edges of deleted vertices, the others judge operations. A workgroup per operation (W = 4) while
// all of them are resident at once, a wavefront per operation above that. Averages of 40 to 60 launches, W = 4 and 1: 1,000
// operations on 1.2 M edges 10.0 and 11.1 us (single launches differ by 2.5), 1,777 on 31 M edges 16.2 and 21.4 (0.7), 10,000 on
// 124 M edges 53.6 and 34.7 (0.4).
#define WORKGROUP_OPS 2048u
template <int W>
__global__ __launch_bounds__(256) void k_validate(MutArgs a, uint32_t nd) {
    __shared__ int s_pos[2];
    __shared__ uint32_t s_base;
    if (blockIdx.x < nd) {
        list_expanded(a, blockIdx.x, nd, &s_base);
        return;
    }
    const uint32_t b = blockIdx.x - nd, nb = gridDim.x - nd;
    for (uint32_t i = W == 1 ? b * 4u + (threadIdx.x >> 6) : b; i < a.n_ops; i += W == 1 ? nb * 4u : nb)
        validate_op<W, 0>(a, i, a.ops[i], s_pos);
}

// where a deleted vertex's edges are in the rows of the vertices that stay
__global__ __launch_bounds__(256) void k_find_expanded(MutArgs a) {
    const int lane = rp_lane();
    const uint32_t gw = (blockIdx.x * blockDim.x + threadIdx.x) >> 6, nw = (gridDim.x * blockDim.x) >> 6;
    const uint32_t n = min(a.ctr->n_exp, a.exp_cap);
    for (uint32_t e = gw; e < n; e += nw) {
        const uint32_t kind = a.exp_kind[e];
        if (kind == EXP_NONE) continue;
        const bool from_in = kind == EXP_OUT;               // x -> y with x dying: x leaves y's in-row; else y leaves x's out-row
        const uint32_t x = a.exp_a[e], y = a.exp_b[e], row = from_in ? y : x;
        const uint2 m = from_in ? a.in_meta[row] : a.out_meta[row];
        const int p = rp_wave_find((from_in ? a.in_pool : a.out_pool) + m.x, m.y, from_in ? x : y);
        if (lane) continue;
        if (p < 0) {
            a.ctr->error = from_in ? 4 : 5;                 // the two adjacencies disagree
            a.exp_kind[e] = EXP_NONE;
            continue;
        }
        // (measure lists the rows: a counter that every newly touched row added to held 10,000 of them up: 97 us, now 21)
        const uint32_t bit = from_in ? VS_TOUCH_IN : VS_TOUCH_OUT, had = atomicOr(&a.vstate[row], bit);
        a.exp_rank[e] = atomicAdd(from_in ? &a.dead_in[row] : &a.dead_out[row], 1u);
        a.exp_pos[e] = (uint32_t)p;
        if (!(had & bit)) a.exp_kind[e] = kind | EXP_FIRST;
    }
}

// whether the batch may be committed at all
__device__ __forceinline__ uint32_t decide(const MutArgs &a) {
    const volatile DevCtr *c = a.ctr;                       // (all of it requested at once: one round trip and not five)
    const uint32_t need_out = c->need_out, need_in = c->need_in, out_top = c->out_top, in_top = c->in_top;
    const uint32_t n_add = c->n_add, n_del = c->n_del, need_exp = c->need_exp, error = c->error;
    const unsigned long long n_edges = c->n_edges;
    const unsigned long long changed = (unsigned long long)n_add + n_del + need_exp;
    uint32_t flag = 0;
    if ((unsigned long long)out_top + need_out > a.pool_cap || (unsigned long long)in_top + need_in > a.pool_cap) flag |= 1u;
    if (n_edges + n_add > a.e_cap + n_del) flag |= 2u;
    if (need_exp > a.exp_cap || changed > a.struct_cap || changed > a.touch_cap) flag |= 4u;
    if (error) flag |= 8u;
    return flag;
}

// Touched rows are listed and measured: the entries a row's segment takes, and the pool space that moving it takes. `j` is an
// operation whose flags say which rows it was the first to touch, or (EXPANDED) an edge of a deleted vertex. A few
// atomics per wavefront; the ones that hand out places and segments are under way together.
template <int EXPANDED>
__device__ __forceinline__ void measure(const MutArgs &a, const ripple_update *ops, uint32_t j) {
    const int lane = rp_lane();
    const unsigned long long below = (1ull << lane) - 1ull;
    uint32_t f = 0, u = 0, v = 0;
    if (EXPANDED) {
        if (j < min(a.ctr->n_exp, a.exp_cap)) {
            const uint32_t kind = a.exp_kind[j];
            if (kind == (EXP_IN | EXP_FIRST)) {
                f = 4u;
                u = a.exp_a[j];
            } else if (kind == (EXP_OUT | EXP_FIRST)) {
                f = 8u;
                v = a.exp_b[j];
            }
        }
    } else if (j < a.n_ops) {
        f = a.op_touch[j];
        u = ops[j].u;                                       // (v: of edge operations)
        v = ops[j].v;
    }
    const unsigned long long mo = __ballot((f & 4u) != 0), mi = __ballot((f & 8u) != 0);
    uint32_t eo = 0, ei = 0, no = 0, ni = 0;
    if (f & 4u) {
        const uint32_t pend = a.pend_out[u], dead = a.dead_out[u], need = a.out_meta[u].y - dead + pend, cap = a.out_capv[u];
        eo = dead + pend;
        if (pend && need > cap) no = rp_row_cap(need);
    }
    if (f & 8u) {
        const uint32_t pend = a.pend_in[v], dead = a.dead_in[v], need = a.in_meta[v].y - dead + pend, cap = a.in_capv[v];
        ei = dead + pend;
        if (pend && need > cap) ni = rp_row_cap(need);
    }
    const uint32_t incl = rp_wave_scan(eo + ei), sum_no = rp_wave_scan(no), sum_ni = rp_wave_scan(ni);
    const uint32_t adds = (uint32_t)__popcll(__ballot((f & 3u) == 3u)), dels = (uint32_t)__popcll(__ballot((f & 3u) == 1u));
    unsigned long long place = 0;
    uint32_t first = 0;
    if (lane == 63) {
        if (mo | mi) place = atomicAdd(&a.ctr->n_listed, ((unsigned long long)__popcll(mi) << 32) | (uint32_t)__popcll(mo));
        if (adds) atomicAdd(&a.ctr->n_add, adds);
        if (dels) atomicAdd(&a.ctr->n_del, dels);
        if (incl) first = atomicAdd(&a.ctr->n_entries, incl);
        if (sum_no) atomicAdd(&a.ctr->need_out, sum_no);
        if (sum_ni) atomicAdd(&a.ctr->need_in, sum_ni);
    }
    first = (uint32_t)__shfl((int)first, 63) + incl - eo - ei;
    if (f & 4u) a.hole_out[u] = first;
    if (f & 8u) a.hole_in[v] = first + eo;
    const uint32_t po = (uint32_t)__shfl((int)(uint32_t)place, 63) + (uint32_t)__popcll(mo & below);
    const uint32_t pi = (uint32_t)__shfl((int)(uint32_t)(place >> 32), 63) + (uint32_t)__popcll(mi & below);
    if (f & 4u) {
        if (po < a.touch_cap) a.touch_out[po] = u;
        else a.ctr->error = 2;
    }
    if (f & 8u) {
        if (pi < a.touch_cap) a.touch_in[pi] = v;
        else a.ctr->error = 2;
    }
}
// by one thread, when all rows have been measured
__device__ __forceinline__ void close_lists(const MutArgs &a) {
    const unsigned long long n = *(const volatile unsigned long long *)&a.ctr->n_listed;
    a.ctr->n_touch_out = (uint32_t)n;
    a.ctr->n_touch_in = (uint32_t)(n >> 32);
    a.ctr->abort_flag = decide(a);
}
// (one workgroup over 2,000 rows takes 17 us, four take 6: a compute unit has only so many reads under way)
__global__ __launch_bounds__(256) void k_measure(MutArgs a) {
    for (uint32_t start = blockIdx.x * 256u; start < a.n_ops; start += gridDim.x * 256u) measure<0>(a, a.ops, start + threadIdx.x);
    const uint32_t n_exp = min(a.ctr->n_exp, a.exp_cap);
    for (uint32_t start = blockIdx.x * 256u; start < n_exp; start += gridDim.x * 256u) measure<1>(a, a.ops, start + threadIdx.x);
    if (last_workgroup(a.ctr, gridDim.x) && threadIdx.x == 0) close_lists(a);
}

// All that precedes k_edges in one launch, for pieces of up to SMALL_OPS operations without vertex deletions. The first nb
// workgroups judge the operations, which they read from pinned host memory; the others clear the bitmaps. The last of the former
// makes the lists of touched rows, measures them and decides. Every workgroup that arrives there costs about 60 ns, one after the
// other, so they are at most SMALL_WGS: a workgroup per operation (W = 4) up to that number, a wavefront per operation (W = 1) above.
template <int W>
__global__ __launch_bounds__(256) void k_small_validate(MutArgs a, const ripple_update *src, ripple_update *dst, uint32_t nb,
                                                        uint32_t *bitmaps, uint32_t n_bitmap_words) {
    __shared__ int s_pos[2];
    const uint32_t tid = threadIdx.x;
    if (blockIdx.x >= nb) {
        const uint32_t stride = (gridDim.x - nb) * 256u;
        for (uint32_t k = (blockIdx.x - nb) * 256u + tid; k < n_bitmap_words; k += stride) bitmaps[k] = 0;
        return;
    }
    for (uint32_t i = W == 1 ? blockIdx.x * 4u + (tid >> 6) : blockIdx.x; i < a.n_ops; i += W == 1 ? nb * 4u : nb) {
        const ripple_update op = src[i];
        if (W == 1 ? (tid & 63u) == 0 : tid == 0) dst[i] = op;
        validate_op<W, 1>(a, i, op, s_pos);
    }
    if (!last_workgroup(a.ctr, nb)) return;
    for (uint32_t start = 0; start < a.n_ops; start += 256u) measure<0>(a, dst, start + tid);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");        // the counts have been added
    __syncthreads();
    if (tid == 0) close_lists(a);
}
// X^l[v] += sign * H^{l-1}[u] for one changed edge, while all H still hold their pre-batch values (Sec. 3.3.3: an added edge
// uses 0 as the source's old embedding, a deleted edge 0 as its new one). A project-first layer's aggregate is the sum of
// what its in-neighbours have sent (T), so a changed edge adds or removes T[u] itself.
__device__ __forceinline__ void struct_term(const MutArgs &a, uint32_t u, uint32_t v, uint32_t l, float sg, int lane) {
    const uint32_t w = a.T[l] ? a.xw[l] : a.d[l - 1];
    for (uint32_t c = lane; c < w; c += 256) {              // four reads on their way, then the additions
        float val[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const uint32_t col = min(c + 64u * t, w - 1u);
            val[t] = a.T[l] ? a.T[l][(size_t)u * a.ldt[l] + col] : rp_load_h(a.H[l - 1], a.store, (size_t)u * w + col);
        }
#pragma unroll
        for (int t = 0; t < 4; ++t)
            if (c + 64u * t < w && val[t] != 0.0f) unsafeAtomicAdd(&a.X[l][(size_t)v * w + c + 64u * t], sg * val[t]);
    }
}
// layers whose rows with a changed in-edge are recomputed have no such terms, and the deterministic mode orders them (k_det_terms)
__device__ __forceinline__ bool has_terms(const MutArgs &a, uint32_t l) { return !a.det && !((a.mono_mask >> l) & 1u); }

__device__ __forceinline__ void list_changed(const MutArgs &a, uint32_t s, uint32_t u, uint32_t v, float weighted, float unit) {
    if (s < a.struct_cap) {
        a.st_src[s] = u;
        a.st_dst[s] = v;
        a.st_sign[s] = weighted;
        a.st_unit[s] = unit;
    }
    rp_set_bit(a.bm_sink, v);
}

// One operation per thread: tombstones, the rows' segments, the list of changed edges, A_0 with its out-degree prefix
__device__ __forceinline__ void apply_op(const MutArgs &a, uint32_t i) {
    const bool in_range = i < a.n_ops;
    const uint32_t ic = min(i, a.n_ops - 1u), judged = a.status[ic], stop = a.ctr->abort_flag;
    ripple_update op = a.ops[ic];
    if (!in_range) op = ripple_update{99u, 0u, 0u, 0u};
    if (op.kind == RIPPLE_VERTEX_ADD || op.kind == RIPPLE_VERTEX_DEL) atomicAnd(&a.vstate[op.u], ~(VS_ADDING | VS_DYING));
    if (stop) return;
    const int lane = rp_lane();
    const bool acc = in_range && judged != 0;
    const unsigned long long ma = __ballot(acc), mr = __ballot(in_range && !acc);
    if (lane == 0) {
        if (ma) atomicAdd(&a.ctr->n_applied, (uint32_t)__popcll(ma));
        if (mr) atomicAdd(&a.ctr->n_rejected, (uint32_t)__popcll(mr));
    }
    const bool row = acc && (op.kind == RIPPLE_FEAT_UPDATE || op.kind == RIPPLE_VERTEX_ADD);
    const unsigned long long mrow = __ballot(row);
    if (mrow) {                                             // place and prefix come from the same addition
        const uint32_t dg = row ? a.out_meta[op.u].y - a.dead_out[op.u] + a.pend_out[op.u] : 0u;
        const uint32_t incl = rp_wave_scan(dg);
        unsigned long long old = 0;
        if (lane == 63)
            old = atomicAdd((unsigned long long *)&a.ctr->set[0], ((unsigned long long)incl << 32) | (uint32_t)__popcll(mrow));
        const uint32_t slot = (uint32_t)__shfl((int)(uint32_t)old, 63) + (uint32_t)__popcll(mrow & ((1ull << lane) - 1ull));
        const uint32_t first = (uint32_t)__shfl((int)(uint32_t)(old >> 32), 63);
        if (row) {
            a.list0[slot] = op.u;
            a.eoff0[slot] = first + incl - dg;
        }
    }
    const bool edge = acc && (op.kind == RIPPLE_EDGE_ADD || op.kind == RIPPLE_EDGE_DEL);
    const uint32_t s = wave_reserve(&a.ctr->n_struct, edge);
    if (!edge) return;
    float alpha = 1.0f;                                     // the edge's weight (1 on unweighted graphs)
    if (op.kind == RIPPLE_EDGE_DEL) {
        const uint32_t po = a.pos_out[i], pi = a.pos_in[i], si = a.hole_in[op.v] + a.rank_in[i];
        const size_t ri = (size_t)a.in_meta[op.v].x + pi;
        if (a.in_w) alpha = a.in_w[ri];
        a.seg_x[a.hole_out[op.u] + a.rank_out[i]] = po;
        a.seg_x[si] = pi;
        a.seg_id[si] = op.u;
        a.out_pool[a.out_meta[op.u].x + po] = RP_TOMB;
        a.in_pool[ri] = RP_TOMB;
        list_changed(a, s, op.u, op.v, -alpha, -1.0f);
    } else {
        const uint32_t si = a.hole_in[op.v] + a.dead_in[op.v] + a.rank_in[i], so = a.hole_out[op.u] + a.dead_out[op.u] + a.rank_out[i];
        if (a.in_w) alpha = __uint_as_float(op.feat_row);   // weighted graphs: EDGE_ADD carries the weight's bits there
        a.seg_id[so] = op.v;
        if (a.out_w) a.seg_x[so] = __float_as_uint(alpha);
        a.seg_id[si] = op.u;
        a.seg_x[si] = __float_as_uint(alpha);
        list_changed(a, s, op.u, op.v, alpha, 1.0f);
    }
}

// the edges of deleted vertices: the same, a thread per edge, then the terms, a wavefront per edge
__device__ __forceinline__ void apply_expanded(const MutArgs &a, uint32_t gw, uint32_t nw) {
    if (a.ctr->abort_flag) return;
    const int lane = rp_lane();
    const uint32_t n = min(a.ctr->n_exp, a.exp_cap);
    for (uint32_t e0 = gw * 64u; e0 < n; e0 += nw * 64u) {
        const uint32_t e = e0 + lane, kind = e < n ? a.exp_kind[e] & ~EXP_FIRST : EXP_NONE;
        const uint32_t s = wave_reserve(&a.ctr->n_struct, kind == EXP_OUT);
        if (kind == EXP_NONE) continue;
        const uint32_t x = a.exp_a[e], y = a.exp_b[e], p = a.exp_pos[e];
        if (kind == EXP_OUT) {
            const uint32_t si = a.hole_in[y] + a.exp_rank[e];
            const size_t ri = (size_t)a.in_meta[y].x + p;
            a.seg_id[si] = x;
            a.seg_x[si] = p;
            a.in_pool[ri] = RP_TOMB;
            list_changed(a, s, x, y, a.in_w ? -a.in_w[ri] : -1.0f, -1.0f);
        } else {
            a.seg_x[a.hole_out[x] + a.exp_rank[e]] = p;
            a.out_pool[a.out_meta[x].x + p] = RP_TOMB;
        }
    }
    if (a.det) return;
    for (unsigned long long t = gw; t < (unsigned long long)n * a.L; t += nw) {      // a wavefront per edge and layer
        const uint32_t e = (uint32_t)(t / a.L), l = (uint32_t)(t - (unsigned long long)e * a.L) + 1u;
        if ((a.exp_kind[e] & ~EXP_FIRST) != EXP_OUT || !has_terms(a, l)) continue;
        const uint32_t x = a.exp_a[e], y = a.exp_b[e];
        const float alpha = (a.in_w && ((a.wsum_mask >> l) & 1u)) ? a.in_w[a.in_meta[y].x + a.exp_pos[e]] : 1.0f;
        struct_term(a, x, y, l, -alpha, lane);
    }
}

// Three parts of one launch, none of which reads what another writes: a thread per operation (tb workgroups); the structural
// terms of the operations' edges, a wavefront per operation and layer, or on weighted graphs per operation (sb workgroups): that
// wavefront also gives a re-weighted edge its weight; the edges of deleted vertices (the rest).
__global__ __launch_bounds__(256) void k_edges(MutArgs a, uint32_t tb, uint32_t sb) {
    if (blockIdx.x < tb) {
        apply_op(a, blockIdx.x * 256u + threadIdx.x);
        return;
    }
    const uint32_t wave = threadIdx.x >> 6;
    if (blockIdx.x >= tb + sb) {
        apply_expanded(a, (blockIdx.x - tb - sb) * 4u + wave, (gridDim.x - tb - sb) * 4u);
        return;
    }
    const uint32_t stop = a.ctr->abort_flag;
    const int lane = rp_lane();
    const uint32_t per = a.in_w ? 1u : a.L;
    for (unsigned long long t = (blockIdx.x - tb) * 4u + wave; t < (unsigned long long)a.n_ops * per; t += sb * 4u) {
        const uint32_t i = (uint32_t)(t / per), l = (uint32_t)(t - (unsigned long long)i * per) + 1u;
        const uint32_t st = a.status[i];                    // (requested together, like all that does not depend on one another here)
        const ripple_update op = a.ops[i];
        if (!st || stop) continue;
        if (op.kind != RIPPLE_EDGE_ADD && op.kind != RIPPLE_EDGE_DEL && op.kind != RIPPLE_EDGE_REWEIGHT) continue;
        const float unit = op.kind == RIPPLE_EDGE_ADD ? 1.0f : (op.kind == RIPPLE_EDGE_DEL ? -1.0f : 0.0f);
        if (!a.in_w) {                                      // nothing is re-weighted, all layers see +1 / -1
            if (has_terms(a, l)) struct_term(a, op.u, op.v, l, unit, lane);
            continue;
        }
        const float given = __uint_as_float(op.feat_row);
        float *wp = op.kind == RIPPLE_EDGE_ADD ? nullptr : a.in_w + a.in_meta[op.v].x + a.pos_in[i];
        const float had = wp ? *wp : 0.0f;
        const float weighted = op.kind == RIPPLE_EDGE_ADD ? given : (op.kind == RIPPLE_EDGE_DEL ? -had : given - had);
        for (uint32_t k = 1; k <= a.L; ++k) {
            const float sg = ((a.wsum_mask >> k) & 1u) ? weighted : unit;
            if (sg != 0.0f && has_terms(a, k)) struct_term(a, op.u, op.v, k, sg, lane);   // (a new weight means nothing to layers that ignore weights)
        }
        if (op.kind == RIPPLE_EDGE_REWEIGHT && lane == 0) {  // the weighted sums of the sink gain (alpha_new - alpha_old) h_u
            *wp = given;
            if (a.out_w) a.out_w[a.out_meta[op.u].x + a.pos_out[i]] = given;
            list_changed(a, atomicAdd(&a.ctr->n_struct, 1u), op.u, op.v, weighted, 0.0f);
        }
    }
}

// Deterministic mode: the structural terms without atomics, and the order of appended in-row entries. A sum that walks a row in
// storage order is only a function of the graph if that order is one: the sinks' segments, filled in the order in which
// atomics were served, are put in ascending id order (a piece holds at most one operation per edge, so ids are distinct
// within a segment), the terms are added in it, with plain loads and stores by one owner per 64 columns, and k_rows appends
// the additions in it. With the rows built in the order the edges were given, and the fills of k_rows being functions of the row
// and the deleted positions alone, an in-row's order then depends on the batches that were applied and on nothing else.
// A workgroup per touched in-row; its wavefronts share the layers and columns, sixteen source rows are on their way at a time
// (one wavefront per sink, after a radix sort of all changed edges, took 77 us per 1,000 operations where this takes 15).
// Segments of up to DET_IDS entries are ranked in LDS. Longer ones (hubs in large batches) are ranked tile by tile and the tiles
// merged by the workgroup, `srt` and the segment itself taking turns; every entry finds its place in the other run by bisection.
// (All entries ranked against all others: batches of 2,000, 20,000 and 60,000 changes of one row took 1.5, 92 and 766 ms; now
// 0.69, 7.5 and 24.)
#define DET_IDS 1024u
#define DET_ADD 0x80000000u                 // an addition; ids are below 2^31

// Entries [0, cnt) of a tile, four per thread at most: ranked by id and written to the tile's places in `to_id` / `to_x` (which may be
// where they came from) with their kind; entries at or behind `dead` are additions. By the whole workgroup; cnt <= DET_IDS.
__device__ __forceinline__ void det_rank_tile(const uint32_t *id, const uint32_t *x, uint32_t cnt, uint32_t dead, uint32_t *s_in, uint32_t *to_id, uint32_t *to_x) {
    const uint32_t tid = threadIdx.x;
    uint32_t my[4], xv[4], rank[4];
    __syncthreads();
#pragma unroll
    for (uint32_t q = 0; q < 4; ++q) {
        const uint32_t i = tid + 256u * q;
        my[q] = i < cnt ? id[i] : 0u;
        xv[q] = i < cnt ? x[i] : 0u;
        rank[q] = 0;
        if (i < cnt) s_in[i] = my[q];
    }
    __syncthreads();
    for (uint32_t k = 0; k < cnt; ++k) {
        const uint32_t o = s_in[k];
#pragma unroll
        for (uint32_t q = 0; q < 4; ++q) rank[q] += o < my[q] ? 1u : 0u;
    }
#pragma unroll
    for (uint32_t q = 0; q < 4; ++q) {
        const uint32_t i = tid + 256u * q;
        if (i < cnt) {
            to_id[rank[q]] = my[q] | (i >= dead ? DET_ADD : 0u);
            to_x[rank[q]] = xv[q];
        }
    }
    __threadfence_block();
    __syncthreads();
}

// Runs of `run` entries (the last one shorter) merged in pairs from one pair of arrays to another. By the whole workgroup.
__device__ __forceinline__ void det_merge(const uint32_t *id, const uint32_t *x, uint32_t *to_id, uint32_t *to_x, uint32_t n, uint32_t run) {
    for (uint32_t i0 = 0; i0 < n; i0 += 1024u) {
        uint32_t e[4], lo[4], hi[4], at[4];                 // four bisections at a time: each step is a read that the next one waits for
#pragma unroll
        for (uint32_t q = 0; q < 4; ++q) {
            const uint32_t i = min(i0 + 256u * q + threadIdx.x, n - 1u);
            const uint32_t pair = i / (2u * run) * (2u * run), mid = min(n, pair + run), end = min(n, pair + 2u * run);
            e[q] = id[i];
            lo[q] = i < mid ? mid : pair;                   // the other run
            hi[q] = i < mid ? end : mid;
            at[q] = (i < mid ? i : pair + (i - mid)) - lo[q];   // + the place found there: where the entry goes (mod 2^32)
        }
        for (uint32_t left = run; left; left >>= 1)         // (`run` is a power of two; run entries take log2(run) + 1 steps)
#pragma unroll
            for (uint32_t q = 0; q < 4; ++q) {
                const uint32_t m = (lo[q] + hi[q]) >> 1;
                const bool open = lo[q] < hi[q], below = (id[min(m, n - 1u)] & ~DET_ADD) < (e[q] & ~DET_ADD);
                if (open && below) lo[q] = m + 1u;
                else if (open) hi[q] = m;
            }
#pragma unroll
        for (uint32_t q = 0; q < 4; ++q) {
            const uint32_t i = i0 + 256u * q + threadIdx.x;
            if (i < n) {
                to_id[at[q] + lo[q]] = e[q];
                to_x[at[q] + lo[q]] = x[i];
            }
        }
    }
    __threadfence_block();
    __syncthreads();
}

__global__ __launch_bounds__(256) void k_det_terms(MutArgs a) {
    constexpr int G = 16;
    __shared__ uint32_t s_in[DET_IDS], s_id[DET_IDS], s_x[DET_IDS], s_w[4];
    if (a.ctr->abort_flag) return;
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
    const uint32_t ni = min(a.ctr->n_touch_in, a.touch_cap);
    for (uint32_t j = blockIdx.x; j < ni; j += gridDim.x) {
        const uint32_t v = a.touch_in[j], base = a.hole_in[v], dead = a.dead_in[v], n = dead + a.pend_in[v];
        const bool in_lds = n <= DET_IDS;
        uint32_t *ids = in_lds ? s_id : a.srt_id + base, *xs = in_lds ? s_x : a.srt_x + base;
        if (in_lds) {
            det_rank_tile(a.seg_id + base, a.seg_x + base, n, dead, s_in, s_id, s_x);
        } else {
            uint32_t passes = 0;
            while ((DET_IDS << passes) < n) ++passes;       // (n is below 2^31)
            uint32_t *fi = (passes & 1u) ? a.seg_id + base : ids, *fx = (passes & 1u) ? a.seg_x + base : xs;   // the last pass ends in srt
            uint32_t *ti = (passes & 1u) ? ids : a.seg_id + base, *tx = (passes & 1u) ? xs : a.seg_x + base;
            for (uint32_t t0 = 0; t0 < n; t0 += DET_IDS)
                det_rank_tile(a.seg_id + base + t0, a.seg_x + base + t0, min(DET_IDS, n - t0), dead - min(dead, t0), s_in, fi + t0, fx + t0);
            for (uint32_t p = 0; p < passes; ++p) {
                det_merge(fi, fx, ti, tx, n, DET_IDS << p);
                uint32_t *s = fi;
                fi = ti;
                ti = s;
                s = fx;
                fx = tx;
                tx = s;
            }
        }
        uint32_t adds = 0;                                  // the additions, in order, back to their part of the segment
        for (uint32_t i0 = 0; i0 < n; i0 += 256u) {
            const uint32_t i = i0 + tid;
            const uint32_t id = i < n ? ids[i] : 0u;
            const unsigned long long m = __ballot((id & DET_ADD) != 0);
            if (lane == 0) s_w[wave] = (uint32_t)__popcll(m);
            __syncthreads();
            uint32_t before = adds + (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
            for (uint32_t k = 0; k < 4; ++k) {
                if (k < wave) before += s_w[k];
                adds += s_w[k];
            }
            if (id & DET_ADD) {
                a.seg_id[base + dead + before] = id & ~DET_ADD;
                a.seg_x[base + dead + before] = xs[i];
            } else if (!in_lds && i < n) {                  // (the merge went through the segment: the deletions' part is written again as well)
                a.seg_id[base + i - before] = id;
                a.seg_x[base + i - before] = xs[i];
            }
            __syncthreads();
        }
        uint32_t task = 0;
        for (uint32_t l = 1; l <= a.L; ++l) {
            if ((a.mono_mask >> l) & 1u) continue;
            const float *Tl = a.T[l];
            const uint32_t w = Tl ? a.xw[l] : a.d[l - 1];
            for (uint32_t c0 = 0; c0 < w; c0 += 64, ++task) {
                if ((task & 3u) != wave) continue;
                const uint32_t col = c0 + lane;
                float *xp = a.X[l] + (size_t)v * w + col;
                float x = (col < w) ? *xp : 0.0f;
                uint32_t next = lane < n ? ids[lane] : 0u;  // 64 entries, one per lane; the next 64 are under way meanwhile
                for (uint32_t j0 = 0; j0 < n; j0 += 64u) {
                    const uint32_t mine = next, cnt = min(64u, n - j0);
                    if (j0 + 64u + lane < n) next = ids[j0 + 64u + lane];
                    for (uint32_t k0 = 0; k0 < cnt; k0 += G) {
                        float val[G], sg[G];
#pragma unroll
                        for (int g = 0; g < G; ++g) {
                            val[g] = 0.0f;
                            if (k0 + (uint32_t)g >= cnt) continue;
                            const uint32_t id = (uint32_t)__builtin_amdgcn_readlane((int)mine, (int)(k0 + (uint32_t)g)), u = id & ~DET_ADD;
                            sg[g] = (id & DET_ADD) ? 1.0f : -1.0f;
                            if (col < w) val[g] = Tl ? Tl[(size_t)u * a.ldt[l] + col] : rp_load_h(a.H[l - 1], a.store, (size_t)u * w + col);
                        }
#pragma unroll
                        for (int g = 0; g < G; ++g)
                            if (k0 + (uint32_t)g < cnt) x += sg[g] * val[g];
                    }
                }
                if (col < w) *xp = x;
            }
        }
        __syncthreads();                                    // the next row's entries go to the same arrays
    }
}

// feature writes (with the hop-0 delta), vertex creation, vertex removal
__device__ __forceinline__ void apply_vertices(const MutArgs &a, uint32_t gw, uint32_t nw) {
    if (a.ctr->abort_flag) return;
    const int lane = rp_lane();
    const uint32_t d0 = a.d[0];
    for (uint32_t i = gw; i < a.n_ops; i += nw) {
        ripple_update op = a.ops[i];
        if (!a.status[i]) continue;
        uint32_t w = op.u;
        if (op.kind == RIPPLE_FEAT_UPDATE || op.kind == RIPPLE_VERTEX_ADD) {
            const float *row = a.payload + (size_t)op.feat_row * d0;
            for (uint32_t c = lane; c < d0; c += 64) {
                float nv = row[c];
                size_t idx = (size_t)w * d0 + c;
                float old;
                if (a.store) {
                    __hip_bfloat16 *h = (__hip_bfloat16 *)a.H[0];
                    old = __bfloat162float(h[idx]);
                    __hip_bfloat16 r = __float2bfloat16(nv);
                    nv = __bfloat162float(r);
                    h[idx] = r;
                } else {
                    float *h = (float *)a.H[0];
                    old = h[idx];
                    h[idx] = nv;
                }
                a.D0[idx] = a.d0_old ? old : nv - old;
            }
            if (lane == 0) {
                rp_set_bit(a.bm0, w);
                if (op.kind == RIPPLE_VERTEX_ADD) {
                    atomicOr(&a.alive[w >> 5], 1u << (w & 31));
                    rp_set_bit(a.bm_vadd, w);
                    atomicAdd(&a.ctr->n_alive, 1u);
                    atomicAdd(&a.ctr->n_vadd, 1u);
                }
            }
        } else if (op.kind == RIPPLE_VERTEX_DEL) {
            for (uint32_t l = 0; l <= a.L; ++l) {
                uint32_t dl = a.d[l];
                for (uint32_t c = lane; c < dl; c += 64) {
                    size_t idx = (size_t)w * dl + c;
                    if (a.store) ((__hip_bfloat16 *)a.H[l])[idx] = __float2bfloat16(0.0f);
                    else ((float *)a.H[l])[idx] = 0.0f;
                }
                if (l >= 1) {
                    uint32_t dp = a.xw[l];
                    for (uint32_t c = lane; c < dp; c += 64) a.X[l][(size_t)w * dp + c] = 0.0f;
                    if (a.T[l])                            // a vertex created under this id later has sent nothing yet
                        for (uint32_t c = lane; c < dp; c += 64) a.T[l][(size_t)w * a.ldt[l] + c] = 0.0f;
                }
            }
            if (lane == 0) {
                atomicAnd(&a.alive[w >> 5], ~(1u << (w & 31)));
                a.out_meta[w].y = 0;
                a.in_meta[w].y = 0;
                atomicSub(&a.ctr->n_alive, 1u);
            }
        }
    }
}

// Tombstones squeezed out of a row, by one wavefront: rows are unordered, so holes in the part that stays (the first
// keep = len - dead entries) take live entries of the part that goes: its k-th hole the tail's k-th live entry.
__device__ __forceinline__ void fill_holes(uint32_t *row, float *wrow, uint32_t keep, uint32_t len, const uint32_t *holes, uint32_t *s_live) {
    const int lane = rp_lane();
    const uint32_t dead = len - keep;
    const unsigned long long below = (1ull << lane) - 1ull;
    if (dead <= 64u) {                                      // the positions are known: nothing of the head is read
        const uint32_t hole = (uint32_t)lane < dead ? holes[lane] : 0xFFFFFFFFu;
        const uint32_t val = (uint32_t)lane < dead ? row[keep + lane] : RP_TOMB;
        const unsigned long long live = __ballot(val != RP_TOMB);
        if (val != RP_TOMB) s_live[__popcll(live & below)] = (uint32_t)lane;
        uint32_t rank = 0;
        for (uint32_t k = 0; k < dead; ++k) rank += (uint32_t)__shfl((int)hole, (int)k) < hole ? 1u : 0u;
        __builtin_amdgcn_wave_barrier();
        if (hole < keep) {                                  // as many as the tail has live entries
            const uint32_t from = keep + s_live[rank];
            row[hole] = row[from];
            if (wrow) wrow[hole] = wrow[from];
        }
        return;
    }
    // First the live entries of the tail are packed to its front, then the head is read sixteen blocks per round.
    uint32_t n_tail = 0;                                    // live entries packed at keep ..
    for (uint32_t base = keep; base < len; base += 64) {
        const uint32_t i = base + lane;
        const uint32_t val = (i < len) ? row[i] : RP_TOMB;
        const float wv = (wrow && i < len) ? wrow[i] : 0.0f;
        const bool live = val != RP_TOMB;
        const unsigned long long mask = __ballot(live);
        const uint32_t off = (uint32_t)__popcll(mask & below);
        if (live) {
            row[keep + n_tail + off] = val;
            if (wrow) wrow[keep + n_tail + off] = wv;
        }
        n_tail += (uint32_t)__popcll(mask);
    }
    uint32_t filled = 0;                                    // holes of the head filled so far
    for (uint32_t base = 0; base < keep && filled < n_tail; base += 1024) {
        uint32_t v[16];
#pragma unroll
        for (int t = 0; t < 16; ++t) {
            const uint32_t i = base + 64 * t + lane;
            v[t] = (i < keep) ? row[i] : 0u;
        }
#pragma unroll
        for (int t = 0; t < 16; ++t) {
            const uint32_t i = base + 64 * t + lane;
            const bool hole = i < keep && v[t] == RP_TOMB;
            const unsigned long long mask = __ballot(hole);
            const uint32_t k = filled + (uint32_t)__popcll(mask & below);
            if (hole && k < n_tail) {
                row[i] = row[keep + k];
                if (wrow) wrow[i] = wrow[keep + k];
            }
            filled += (uint32_t)__popcll(mask);
        }
    }
}

// one wavefront per touched row: tombstones squeezed out, the row moved if the additions do not fit, the additions appended,
// the row's scratch counters reset
__device__ __forceinline__ void finish_rows(const MutArgs &a, uint32_t gw, uint32_t nw, uint32_t *s_live) {
    const int lane = rp_lane();
    const bool aborted = a.ctr->abort_flag != 0;
    uint32_t no = min(a.ctr->n_touch_out, a.touch_cap), ni = min(a.ctr->n_touch_in, a.touch_cap);
    for (uint32_t j = gw; j < no + ni; j += nw) {
        const bool is_out = j < no;
        const uint32_t x = is_out ? a.touch_out[j] : a.touch_in[j - no];
        uint2 *meta = is_out ? a.out_meta : a.in_meta;
        uint32_t *capv = is_out ? a.out_capv : a.in_capv;
        uint32_t *pool = is_out ? a.out_pool : a.in_pool;
        float *wp = is_out ? a.out_w : a.in_w;             // weights travel with the rows' entries
        uint32_t *deadv = is_out ? a.dead_out : a.dead_in;
        uint32_t *pendv = is_out ? a.pend_out : a.pend_in;
        if (!aborted) {
            uint2 m = meta[x];
            const uint32_t dead = deadv[x], pend = pendv[x], cap = capv[x], seg = is_out ? a.hole_out[x] : a.hole_in[x];
            uint32_t len = m.y - min(dead, m.y);
            if (dead == 1 && m.y) {                         // the usual case: the last entry fills the hole
                const uint32_t hole = a.seg_x[seg];
                if (hole < len && lane == 0) {
                    pool[m.x + hole] = pool[m.x + len];
                    if (wp) wp[m.x + hole] = wp[m.x + len];
                }
            } else if (dead) {
                fill_holes(pool + m.x, wp ? wp + m.x : nullptr, len, m.y, a.seg_x + seg, s_live);
            }
            const uint32_t need = len + pend;
            bool room = true;
            if (pend && need > cap) {
                uint32_t ncap = rp_row_cap(need);
                uint32_t ns = 0;
                if (lane == 0) ns = atomicAdd(is_out ? &a.ctr->out_top : &a.ctr->in_top, ncap);
                ns = __shfl(ns, 0);
                if ((unsigned long long)ns + ncap <= a.pool_cap) {
                    for (uint32_t base = 0; base < len; base += 1024) {     // sixteen blocks in flight per round
                        uint32_t v[16];
#pragma unroll
                        for (int t = 0; t < 16; ++t) {
                            const uint32_t i = base + 64 * t + lane;
                            v[t] = (i < len) ? pool[m.x + i] : 0u;
                        }
#pragma unroll
                        for (int t = 0; t < 16; ++t) {
                            const uint32_t i = base + 64 * t + lane;
                            if (i < len) pool[ns + i] = v[t];
                        }
                    }
                    if (wp)
                        for (uint32_t i = lane; i < len; i += 64) wp[ns + i] = wp[m.x + i];
                    m.x = ns;
                    if (lane == 0) capv[x] = ncap;
                } else {
                    room = false;
                    if (lane == 0) a.ctr->error = 6;         // cannot happen: space was checked before commit
                }
            }
            for (uint32_t k = lane; room && k < pend; k += 64) {
                const uint32_t at = seg + dead + k;
                pool[m.x + len + k] = a.seg_id[at];
                if (wp) wp[m.x + len + k] = __uint_as_float(a.seg_x[at]);
            }
            if (lane == 0) meta[x] = make_uint2(m.x, room ? need : len);
        }
        if (lane == 0) {
            deadv[x] = 0;
            pendv[x] = 0;
            atomicAnd(&a.vstate[x], ~(is_out ? VS_TOUCH_OUT : VS_TOUCH_IN));
        }
    }
}

// Feature rows, created and deleted vertices (the first nb workgroups) and the touched rows (the others). The two parts meet
// nowhere: a deleted vertex's own rows are not touched ones.
__global__ __launch_bounds__(256) void k_rows(MutArgs a, uint32_t nb) {
    __shared__ uint32_t s_live[4][64];
    const uint32_t wave = threadIdx.x >> 6;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        a.eoff0[a.ctr->set[0].a] = a.ctr->set[0].m;
        if (!a.ctr->abort_flag)
            a.ctr->n_edges += (unsigned long long)a.ctr->n_add - (unsigned long long)a.ctr->n_del - (unsigned long long)a.ctr->n_gone;
    }
    if (blockIdx.x < nb) apply_vertices(a, blockIdx.x * 4u + wave, nb * 4u);
    else finish_rows(a, (blockIdx.x - nb) * 4u + wave, (gridDim.x - nb) * 4u, s_live[wave]);
}

__global__ void k_batch_reset(DevCtr *ctr, uint32_t *bitmaps, size_t n_bitmap_words) {
    size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n_bitmap_words; i += stride) bitmaps[i] = 0;
    if (blockIdx.x == 0)
        for (uint32_t k = RP_CTR_BATCH + threadIdx.x; k < RP_CTR_WORDS; k += blockDim.x) ((uint32_t *)ctr)[k] = 0;
}

// Hands the batch's counters to the host (pinned memory), clears those that a batch starts from zero and then says so: the
// host sees the number of this call in `flag`. One launch in place of a copy and the wait for a stream.
__global__ __launch_bounds__(256) void k_publish(DevCtr *ctr, DevCtr *host, HostFlag done) {
    for (uint32_t k = threadIdx.x; k < RP_CTR_WORDS; k += blockDim.x) {
        ((volatile uint32_t *)host)[k] = ((uint32_t *)ctr)[k];
        if (k >= RP_CTR_BATCH) ((uint32_t *)ctr)[k] = 0;
    }
    report_done(done, 1u);
}

// reports the end of the launches before it: for launches of more workgroups than should report by themselves
__global__ void k_report(HostFlag done) { report_done(done, 1u); }
void rp_launch_report(ripple_ctx *c) { hipLaunchKernelGGL(k_report, dim3(1), dim3(64), 0, c->stream, rp_host_flag(c)); }

void rp_launch_publish(ripple_ctx *c) {
    hipLaunchKernelGGL(k_publish, dim3(1), dim3(256), 0, c->stream, c->ctr, c->ctr_host, rp_host_flag(c));
    c->ctr_dirty = false;
}

static MutArgs make_args(ripple_ctx *c, uint32_t n_ops) {
    MutArgs a;
    a.ops = c->ops_d;
    a.n_ops = n_ops;
    a.made = c->made_pin;
    a.n_made = 0;
    a.payload = c->payload;
    a.status = c->op_status;
    a.hole_out = c->hole_out;
    a.hole_in = c->hole_in;
    a.rank_out = c->op_rank_out;
    a.rank_in = c->op_rank_in;
    a.seg_id = c->seg_id;
    a.seg_x = c->seg_x;
    a.srt_id = c->srt_id;
    a.srt_x = c->srt_x;
    a.eoff0 = c->eoff[0];
    a.op_touch = c->op_touch;
    a.pos_out = c->op_pos_out;
    a.pos_in = c->op_pos_in;
    a.out_meta = c->out_meta;
    a.in_meta = c->in_meta;
    a.out_capv = c->out_capv;
    a.in_capv = c->in_capv;
    a.out_pool = c->out_pool;
    a.in_pool = c->in_pool;
    a.in_w = c->in_w;
    a.out_w = c->out_w;
    a.alive = c->alive;
    a.vstate = c->vstate;
    a.pend_out = c->pend_out;
    a.pend_in = c->pend_in;
    a.dead_out = c->dead_out;
    a.dead_in = c->dead_in;
    a.touch_out = c->touch_out;
    a.touch_in = c->touch_in;
    a.touch_cap = c->touch_cap;
    a.exp_kind = c->exp_kind;
    a.exp_pos = c->exp_pos;
    a.exp_rank = c->exp_rank;
    a.exp_a = c->exp_a;
    a.exp_b = c->exp_b;
    a.exp_cap = c->exp_cap;
    a.st_src = c->st_src;
    a.st_dst = c->st_dst;
    a.st_sign = c->st_sign;
    a.st_unit = c->st_unit;
    a.struct_cap = c->struct_cap;
    a.bm0 = c->bm[0];
    a.bm_sink = c->bm_sink;
    a.bm_vadd = c->bm_vadd;
    a.list0 = c->list[0];
    a.D0 = c->D[0];
    a.ctr = c->ctr;
    a.n_cap = c->n_cap;
    a.e_cap = c->e_cap;
    a.pool_cap = c->pool_cap;
    a.store = c->store;
    a.L = c->L;
    for (uint32_t l = 0; l <= RIPPLE_MAX_LAYERS; ++l) {
        a.d[l] = c->d[l];
        a.xw[l] = c->xw[l];
        a.H[l] = c->H[l];
        a.X[l] = c->X[l];
        a.T[l] = (l >= 1 && l <= c->L && c->layers[l - 1].proj) ? c->layers[l - 1].T : nullptr;
        a.ldt[l] = a.T[l] ? c->layers[l - 1].ldt : 0u;
    }
    a.mono_mask = 0;
    a.wsum_mask = 0;
    for (uint32_t l = 1; l <= c->L; ++l) {
        if (rp_layer_mono(c, l) || rp_layer_attn(c, l)) a.mono_mask |= 1u << l;
        if (c->layers[l - 1].agg == RIPPLE_AGG_WSUM) a.wsum_mask |= 1u << l;
    }
    a.d0_old = rp_layer_mono(c, 1) ? 1 : 0;
    a.det = c->opt_deterministic;
    return a;
}

// counters and bitmaps cleared
void rp_launch_batch_reset(ripple_ctx *c) {
    // the per-layer bitmaps, S and V_added are one allocation starting at bm[0]
    const size_t words = (size_t)c->n_words * (c->L + 3);
    const uint32_t gb = std::min<uint32_t>(rp_div_up(words, 256), c->n_cu * 4);
    hipLaunchKernelGGL(k_batch_reset, dim3(gb), dim3(256), 0, c->stream, c->ctr, c->bm[0], words);
    c->ctr_dirty = false;
}

// Enqueues the whole Apply step for the n_ops operations at src (pinned host memory): bitmaps cleared, A_0 listed with its prefix.
void rp_launch_mutate(ripple_ctx *c, const ripple_update *src, uint32_t n_ops, bool has_vertex_del, bool has_vertex_or_feat) {
    if (c->ctr_dirty || n_ops == 0) rp_launch_batch_reset(c);
    if (n_ops == 0) return;
    hipStream_t s = c->stream;
    MutArgs a = make_args(c, n_ops);
    const uint32_t words = c->n_words * (c->L + 3), big = c->n_cu * 8, tb = rp_div_up(n_ops, 256);
    const bool small = n_ops <= SMALL_OPS && !has_vertex_del;
    if (small) {
        // Every wavefront with an endpoint that is not alive reads the created vertices over the bus: a list of their own, not all
        // operations (50 vertices with 8 edges each: a batch of 173 us -> 164)
        for (uint32_t i = 0; has_vertex_or_feat && i < n_ops; ++i)
            if (src[i].kind == RIPPLE_VERTEX_ADD) c->made_pin[a.n_made++] = src[i].u;
        const bool wide = n_ops <= SMALL_WGS;
        const uint32_t nb = wide ? n_ops : rp_div_up(n_ops, 4);
        const dim3 grid(nb + std::min<uint32_t>(rp_div_up(words, 1024), c->n_cu * 2));
        if (wide) hipLaunchKernelGGL(k_small_validate<4>, grid, dim3(256), 0, s, a, src, c->ops_d, nb, c->bm[0], words);
        else hipLaunchKernelGGL(k_small_validate<1>, grid, dim3(256), 0, s, a, src, c->ops_d, nb, c->bm[0], words);
    } else {
        const bool wide = n_ops <= WORKGROUP_OPS;
        const uint32_t nb = wide ? n_ops : std::min<uint32_t>(rp_div_up(n_ops, 4), c->n_cu * 32), nd = has_vertex_del ? std::min<uint32_t>(rp_div_up(n_ops, EXPAND_OPS), c->n_cu * 4) : 0u;
        hipLaunchKernelGGL(k_stage, dim3(std::min<uint32_t>(rp_div_up(std::max(words, n_ops), 256), c->n_cu * 4)), dim3(256), 0, s, a, src,
                           c->ops_d, c->bm[0], words);
        if (wide) hipLaunchKernelGGL(k_validate<4>, dim3(nb + nd), dim3(256), 0, s, a, nd);
        else hipLaunchKernelGGL(k_validate<1>, dim3(nb + nd), dim3(256), 0, s, a, nd);
        if (has_vertex_del) hipLaunchKernelGGL(k_find_expanded, dim3(big), dim3(256), 0, s, a);
        hipLaunchKernelGGL(k_measure, dim3(has_vertex_del ? SMALL_WGS : std::min<uint32_t>(tb, SMALL_WGS)), dim3(256), 0, s, a);
    }
    const bool terms = !a.det && (a.mono_mask >> 1) != (1u << c->L) - 1u;      // some layer has terms to be added here
    const uint32_t sb = (terms || c->in_w) ? std::min<uint32_t>(rp_div_up((uint64_t)n_ops * (c->in_w ? 1u : c->L), 4), big) : 0u;
    hipLaunchKernelGGL(k_edges, dim3(tb + sb + (has_vertex_del ? big : 0u)), dim3(256), 0, s, a, tb, sb);
    if (a.det) {
        int t = rp_timer_begin(c);
        hipLaunchKernelGGL(k_det_terms, dim3(has_vertex_del ? big : std::min<uint32_t>(n_ops, big)), dim3(256), 0, s, a);
        rp_timer_end(c, t, RIPPLE_PH_STRUCT, 0);
    }
    const uint32_t vb = has_vertex_or_feat ? std::min<uint32_t>(rp_div_up(n_ops, 4), c->n_cu * 2) : 0u;
    hipLaunchKernelGGL(k_rows, dim3(vb + (has_vertex_del ? big : std::min<uint32_t>(rp_div_up(2 * (uint64_t)n_ops, 4), big))), dim3(256), 0, s, a, vb);
}
