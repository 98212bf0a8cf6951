// Graph attention layers (Sec. 3.4.1, Eq. 3), hybrid-incremental.
//
// Layer l keeps, per vertex, the projected row P[v] = H^{l-1}[v] W, its two scores
// s_src[v] = a_src . P[v] and s_dst[v] = a_dst . P[v], and the un-normalised aggregate: the numerator
// X[v] = sum_u w_uv P[u] and the denominator den[v] = sum_u w_uv over v's in-neighbours u, with
// w_uv = exp(LeakyReLU(s_src[u] + s_dst[v])). The row transform is h_v = act(X[v] / den[v] + b).
// After a batch, a vertex of A_l that is itself in A_{l-1} (its own score moved, so every w_uv did)
// recomputes numerator and denominator from all its in-neighbours; any other vertex of A_l receives, per
// changed in-neighbour u, the message of the paper: <w_new P_new[u] - w_old P_old[u], w_new - w_old>.
// A vertex whose in-edges changed recomputes if its in-row is short; with a long in-row each changed edge
// is a message too (its pre-batch weight and row, added or taken away). Small hops have one owner per
// destination (a wavefront; a workgroup for long in-rows; a workgroup per 512-entry segment when a very long
// row is recomputed, the last of them adding the segments up in order), large ones are cut over edges.
#include "kernels.h"
#include "pull_scan.h"
#include <algorithm>

#define GAT_SLOPE 0.2f
#define GAT_LONG 256u
#define GAT_EDGE_HITS 1024u       // changed edges of one sink kept as messages; more: recompute
#define GAT_EDGE_SCAN 32768u      // longest list of changed edges a sink's workgroup searches; longer: recompute

struct GatArgs {
    const uint32_t *list;          // A_l, or a queue of rows
    const uint32_t *count_ptr;
    const uint2 *in_meta;
    const uint32_t *in_pool;
    const uint32_t *bm_prev;       // A_{l-1}
    const uint32_t *bm_sink, *bm_vadd;
    const float *P, *Pold;         // projected rows now / before the batch (the latter valid on A_{l-1}), row stride ldp
    uint32_t ldp;
    const float *ssrc, *sold, *sdst;
    uint32_t d;                    // d_out
    float *X, *den;
    int all;                       // recompute every listed row (the queue of cancelled rows)
    uint32_t long_min;             // in-rows longer than this are the workgroup role's
    uint32_t split_min;            // in-rows of at least this many entries are recomputed in segments (k_gat_scatter_seg)
    uint32_t *n_big, *n_seg;       // split rows / queued segments of this hop
    uint32_t *seg_v, *seg_done, *seg_base, *seg_r;
    float *seg_part;               // per segment: partial numerator (d floats), then the partial denominator
    uint32_t big_cap, seg_cap, seg_ld;
    // the batch's changed edges (source, sink, sign: < 0 deleted), read for sinks with long in-rows
    const uint32_t *st_src, *st_dst;
    const float *st_sign;
    const uint32_t *n_struct;
    uint32_t struct_cap;
};

__device__ __forceinline__ float gat_weight(float s_u, float t_v) {
    const float z = s_u + t_v;
    return __expf(z > 0.0f ? z : GAT_SLOPE * z);
}

// One block of up to 64 in-neighbours (id per lane in my_u, `valid` lanes hold one). recompute: all of them
// contribute w P[u]; otherwise the changed ones contribute w_new P[u] - w_old Pold[u]. acc: the wavefront's
// running numerator (column lane + 64 j); returns this lane's share of the denominator and adds the
// magnitude of what it patched (w_new + w_old) to mag.
template <int NJ, int G, bool recompute>
__device__ __forceinline__ float gat_block(const GatArgs &a, uint32_t my_u, bool valid, float t_v, float *acc, float &mag) {
    const int lane = rp_lane();
    const uint32_t d = a.d;
    const bool on = valid && (recompute || rp_bit(a.bm_prev, my_u));     // rp_bit is not evaluated when recomputing
    float wn = 0.0f, wo = 0.0f;
    if (on) {
        wn = gat_weight(a.ssrc[my_u], t_v);
        if (!recompute) wo = gat_weight(a.sold[my_u], t_v);
    }
    unsigned long long mask = __ballot(on);
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
        float rn[G][NJ], ro[recompute ? 1 : G][NJ];
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const uint32_t u = __shfl(my_u, kk[g]);
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                const uint32_t col = lane + 64 * j;
                const bool in = g < n && col < d;
                rn[g][j] = in ? a.P[(size_t)u * a.ldp + col] : 0.0f;
                if (!recompute) ro[g][j] = in ? a.Pold[(size_t)u * a.ldp + col] : 0.0f;
            }
        }
#pragma unroll
        for (int g = 0; g < G; ++g) {
            if (g < n) {
                const float wnk = __shfl(wn, kk[g]), wok = __shfl(wo, kk[g]);
#pragma unroll
                for (int j = 0; j < NJ; ++j) acc[j] += recompute ? wnk * rn[g][j] : wnk * rn[g][j] - wok * ro[g][j];
            }
        }
    }
    mag += wn + wo;
    return wn - wo;
}

// Messages of changed in-edges of one sink whose own score stayed (u = source, sgn = +1 added, -1 deleted,
// one per valid lane): the edge's weight and row as they were before the batch. For a deleted edge that
// is what goes away; for an added edge whose source also changed it cancels the old part of the
// changed-source message, which was never in the sums; for an added edge from an unchanged source it is
// the edge's contribution itself.
template <int NJ>
__device__ __forceinline__ float gat_edge_block(const GatArgs &a, uint32_t my_u, float my_sgn, bool valid, float t_v,
                                                float *acc, float &mag) {
    const int lane = rp_lane();
    const uint32_t d = a.d;
    bool from_old = false;
    float w = 0.0f;
    if (valid) {
        from_old = rp_bit(a.bm_prev, my_u);
        w = gat_weight(from_old ? a.sold[my_u] : a.ssrc[my_u], t_v);
    }
    unsigned long long mask = __ballot(valid);
    while (mask) {
        const int k = __ffsll((long long)mask) - 1;
        mask &= mask - 1;
        const uint32_t u = __shfl(my_u, k);
        const float wk = __shfl(w, k) * __shfl(my_sgn, k);
        const float *row = (__shfl((int)from_old, k) ? a.Pold : a.P) + (size_t)u * a.ldp;
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            const uint32_t col = lane + 64 * j;
            if (col < d) acc[j] += wk * row[col];
        }
    }
    mag += w;
    return w * my_sgn;
}

// A patched denominator that is tiny against what was added and taken away has lost its small terms
// (a weight e^z that dropped by many orders of magnitude leaves only rounding residue of itself): such a
// row is recomputed from all its in-neighbours instead.
#define GAT_CANCEL 1e-3f

__device__ __forceinline__ float gat_wave_sum(float x) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o);
    return x;
}

// wavefront gw of nw: the vertices gw, gw + nw, ... of the list
template <int NJ>
__device__ __forceinline__ void gat_wave_role(const GatArgs &a, uint32_t gw, uint32_t nw) {
    constexpr int G = (NJ <= 1) ? 8 : (NJ <= 2 ? 4 : (NJ <= 4 ? 2 : 1));
    constexpr int GR = (NJ <= 1) ? 16 : (NJ <= 16 ? 16 / NJ : 1);
    const uint32_t count = *a.count_ptr;
    const int lane = rp_lane();
    const uint32_t d = a.d;
    for (uint32_t i = gw; i < count; i += nw) {
        const uint32_t v = a.list[i];
        const uint2 m = a.in_meta[v];
        if (m.y > a.long_min) continue;                        // queued when the hop's vertices were listed
        bool recompute = rp_bit(a.bm_prev, v) || rp_bit(a.bm_sink, v) || rp_bit(a.bm_vadd, v);
        const float t_v = a.sdst[v];
        float acc[NJ];
        float dsum;
        for (;;) {                                             // a second pass only after a cancelled patch
#pragma unroll
            for (int j = 0; j < NJ; ++j) acc[j] = 0.0f;
            dsum = 0.0f;
            float mag = 0.0f;
            for (uint32_t base = 0; base < m.y; base += 64) {
                const uint32_t e = base + lane;
                const uint32_t my_u = (e < m.y) ? a.in_pool[m.x + e] : 0u;
                dsum += recompute ? gat_block<NJ, GR, true>(a, my_u, e < m.y, t_v, acc, mag)
                                  : gat_block<NJ, G, false>(a, my_u, e < m.y, t_v, acc, mag);
            }
            dsum = gat_wave_sum(dsum);
            if (recompute) break;
            mag = gat_wave_sum(mag);
            if (a.den[v] + dsum > GAT_CANCEL * mag) break;
            recompute = true;
        }
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            const uint32_t col = lane + 64 * j;
            if (col < d) {
                float *x = a.X + (size_t)v * d + col;
                *x = recompute ? acc[j] : *x + acc[j];
            }
        }
        if (lane == 0) a.den[v] = recompute ? dsum : a.den[v] + dsum;
    }
}

// one workgroup of TEAM wavefronts per long in-row; partial sums meet in LDS and are added in wavefront order.
// Workgroup bid of nb: the rows bid, bid + nb, ... of the queue.
template <int NJ, int TEAM>
__device__ __forceinline__ void gat_team_role(const GatArgs &a, uint32_t bid, uint32_t nb) {
    constexpr int G = (NJ <= 1) ? 8 : (NJ <= 2 ? 4 : (NJ <= 4 ? 2 : 1));
    constexpr int GR = (NJ <= 2) ? 16 : 32 / NJ;
    constexpr int IDS = 4;                                     // blocks of in-neighbour ids in flight while looking for changed ones
    __shared__ float s_val[TEAM][NJ * 64];
    __shared__ float s_den[TEAM], s_mag[TEAM];
    __shared__ uint32_t s_hit[GAT_EDGE_HITS];                  // the sink's entries in the list of changed edges
    __shared__ uint32_t s_nhit, s_base, s_slot;
    const uint32_t count = *a.count_ptr;
    const uint32_t n_st = *a.n_struct;
    const int lane = rp_lane(), wave = threadIdx.x >> 6;
    const uint32_t d = a.d;
    for (uint32_t i = bid; i < count; i += nb) {
        const uint32_t v = a.list[i];
        const uint2 m = a.in_meta[v];
        bool recompute = a.all || rp_bit(a.bm_prev, v) || rp_bit(a.bm_vadd, v);
        // a sink whose own score stayed keeps its long row incremental when its changed edges can be looked up
        uint32_t ns = 0;
        if (!recompute && rp_bit(a.bm_sink, v)) {
            if (n_st > a.struct_cap || n_st > GAT_EDGE_SCAN) {
                recompute = true;
            } else {
                if (threadIdx.x == 0) s_nhit = 0;
                __syncthreads();
                for (uint32_t s = threadIdx.x; s < n_st; s += TEAM * 64)
                    if (a.st_dst[s] == v && a.st_sign[s] != 0.0f) {
                        const uint32_t k = atomicAdd(&s_nhit, 1u);
                        if (k < GAT_EDGE_HITS) s_hit[k] = s;
                    }
                __syncthreads();
                ns = s_nhit;
                if (ns > GAT_EDGE_HITS || 2 * ns >= m.y) recompute = true;
            }
        }
        const float t_v = a.sdst[v];
        float acc[NJ];
        bool queued = false;
        for (;;) {                                             // a second pass only after a cancelled patch
            if (recompute && m.y >= a.split_min) {
                // One compute unit reads a row of thousands of in-neighbours far too slowly: queue its segments,
                // a workgroup each takes one, the last to finish adds them up (k_gat_scatter_seg).
                const uint32_t nseg = (m.y + ROW_SEG - 1) / ROW_SEG;
                if (threadIdx.x == 0) {
                    const uint32_t r = atomicAdd(a.n_big, 1u);
                    const uint32_t base = atomicAdd(a.n_seg, nseg);
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
                if (r != SEG_NONE) {                           // (the queue holds every row unless it is capped: then read it here)
                    queued = true;
                    break;
                }
            }
#pragma unroll
            for (int j = 0; j < NJ; ++j) acc[j] = 0.0f;
            float dsum = 0.0f, mag = 0.0f;
            if (recompute) {
                const uint32_t chunk = (m.y <= 16u * 64u) ? 16u : 64u;   // shorter rows in finer pieces: every wavefront reads some
                for (uint32_t base = chunk * wave; base < m.y; base += chunk * TEAM) {
                    const uint32_t e = base + lane;
                    const bool valid = (uint32_t)lane < chunk && e < m.y;
                    const uint32_t my_u = valid ? a.in_pool[m.x + e] : 0u;
                    dsum += gat_block<NJ, GR, true>(a, my_u, valid, t_v, acc, mag);
                }
            } else {
                for (uint32_t base = 64u * wave; base < m.y; base += 64u * TEAM * IDS) {
                    uint32_t u[IDS];
                    bool any[IDS];
#pragma unroll
                    for (int t = 0; t < IDS; ++t) {
                        const uint32_t e = base + 64u * TEAM * t + lane;
                        u[t] = (e < m.y) ? a.in_pool[m.x + e] : 0u;
                    }
#pragma unroll
                    for (int t = 0; t < IDS; ++t) {
                        const uint32_t e = base + 64u * TEAM * t + lane;
                        any[t] = __ballot(e < m.y && rp_bit(a.bm_prev, u[t])) != 0ull;
                    }
#pragma unroll
                    for (int t = 0; t < IDS; ++t) {
                        const uint32_t e = base + 64u * TEAM * t + lane;
                        if (any[t]) dsum += gat_block<NJ, G, false>(a, u[t], e < m.y, t_v, acc, mag);
                    }
                }
                for (uint32_t base = 64u * wave; base < ns; base += 64u * TEAM) {
                    const uint32_t k = base + lane;
                    const uint32_t s = (k < ns) ? s_hit[k] : 0u;
                    const uint32_t u = (k < ns) ? a.st_src[s] : 0u;
                    const float sgn = (k < ns && a.st_sign[s] < 0.0f) ? -1.0f : 1.0f;
                    dsum += gat_edge_block<NJ>(a, u, sgn, k < ns, t_v, acc, mag);
                }
            }
            dsum = gat_wave_sum(dsum);
            mag = gat_wave_sum(mag);
#pragma unroll
            for (int j = 0; j < NJ; ++j) s_val[wave][j * 64 + lane] = acc[j];
            if (lane == 0) {
                s_den[wave] = dsum;
                s_mag[wave] = mag;
            }
            __syncthreads();
            if (recompute) break;
            float dd = 0.0f, mm = 0.0f;                        // every thread takes the same decision
            for (int w = 0; w < TEAM; ++w) {
                dd += s_den[w];
                mm += s_mag[w];
            }
            if (a.den[v] + dd > GAT_CANCEL * mm) break;
            recompute = true;
            __syncthreads();                                   // the partial results are overwritten by the second pass
        }
        if (queued) continue;
        if (wave == 0) {
            float dd = 0.0f;
            for (int w = 0; w < TEAM; ++w) dd += s_den[w];
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                float t = 0.0f;
                for (int w = 0; w < TEAM; ++w) t += s_val[w][j * 64 + lane];
                const uint32_t col = lane + 64 * j;
                if (col < d) {
                    float *x = a.X + (size_t)v * d + col;
                    *x = recompute ? t : *x + t;
                }
            }
            if (lane == 0) a.den[v] = recompute ? dd : a.den[v] + dd;
        }
        __syncthreads();
    }
}

template <int NJ, int TEAM>
__global__ __launch_bounds__(TEAM * 64) void k_gat_scatter_long(GatArgs a) {
    gat_team_role<NJ, TEAM>(a, blockIdx.x, gridDim.x);
}

// Small hops, whose long rows were queued while the hop's vertices were listed: both roles in one launch
// (the first team_blocks workgroups take a long row each, the wavefronts of the others a short one each).
template <int NJ, int TEAM>
__global__ __launch_bounds__(TEAM * 64) void k_gat_scatter_both(GatArgs a, GatArgs b, uint32_t team_blocks) {
    if (blockIdx.x < team_blocks) {
        gat_team_role<NJ, TEAM>(b, blockIdx.x, team_blocks);
    } else {
        const uint32_t wb = blockIdx.x - team_blocks, nwb = gridDim.x - team_blocks;
        gat_wave_role<NJ>(a, (wb * blockDim.x + threadIdx.x) >> 6, (nwb * blockDim.x) >> 6);
    }
}

// One workgroup per queued segment of a very long row that is recomputed: numerator and denominator over
// the segment's ROW_SEG in-neighbours go to the segment's partial row; the workgroup that finishes a row's
// last segment adds the partial rows up in segment order and stores the row.
template <int NJ, int TEAM>
__global__ __launch_bounds__(TEAM * 64) void k_gat_scatter_seg(GatArgs a) {
    static_assert(TEAM * 64 == ROW_SEG, "one 64-entry block per wavefront");
    constexpr int GR = (NJ <= 2) ? 32 : 64 / NJ;
    __shared__ float s_val[TEAM][NJ * 64];
    __shared__ float s_den[TEAM];
    const uint32_t n_seg = min(*a.n_seg, a.seg_cap);
    const int lane = rp_lane(), wave = threadIdx.x >> 6;
    const uint32_t d = a.d;
    for (uint32_t e = blockIdx.x; e < n_seg; e += gridDim.x) {
        const uint32_t r = a.seg_r[e];
        if (r == SEG_NONE) continue;
        const uint32_t v = a.seg_v[r], first = a.seg_base[r];
        const uint2 m = a.in_meta[v];
        const uint32_t nseg = (m.y + ROW_SEG - 1) / ROW_SEG;
        const uint32_t lo = (e - first) * ROW_SEG, hi = min(m.y, lo + ROW_SEG);
        const float t_v = a.sdst[v];
        float acc[NJ];
#pragma unroll
        for (int j = 0; j < NJ; ++j) acc[j] = 0.0f;
        float dsum = 0.0f, mag = 0.0f;
        const uint32_t b = lo + 64u * wave;
        if (b < hi) {
            const bool valid = b + lane < hi;
            const uint32_t my_u = valid ? a.in_pool[m.x + b + lane] : 0u;
            dsum = gat_block<NJ, GR, true>(a, my_u, valid, t_v, acc, mag);
        }
        dsum = gat_wave_sum(dsum);
#pragma unroll
        for (int j = 0; j < NJ; ++j) s_val[wave][j * 64 + lane] = acc[j];
        if (lane == 0) s_den[wave] = dsum;
        __syncthreads();
        if (wave == 0) {
            float *part = a.seg_part + (size_t)e * a.seg_ld;
            float dd = 0.0f;
            for (int w = 0; w < TEAM; ++w) dd += s_den[w];
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                float t = 0.0f;
                for (int w = 0; w < TEAM; ++w) t += s_val[w][j * 64 + lane];
                const uint32_t col = lane + 64 * j;
                if (col < d) part[col] = t;
            }
            if (lane == 0) part[d] = dd;
            __threadfence();                                   // the partial row is visible before the count moves
            uint32_t last = 0;
            if (lane == 0) last = (atomicAdd(&a.seg_done[r], 1u) == nseg - 1) ? 1u : 0u;
            last = __shfl(last, 0);
            if (last) {
                __threadfence();
#pragma unroll
                for (int j = 0; j < NJ; ++j) acc[j] = 0.0f;
                dd = 0.0f;
                constexpr int GP = (NJ <= 4) ? 8 : 32 / NJ;     // partial rows requested per round trip
                for (uint32_t k0 = 0; k0 < nseg; k0 += GP) {   // written by other compute units: read past this one's cache
                    float x[GP][NJ], xd[GP];
#pragma unroll
                    for (int g = 0; g < GP; ++g) {
                        const bool on = k0 + g < nseg;
                        const float *p = a.seg_part + (size_t)(first + min(k0 + g, nseg - 1)) * a.seg_ld;
#pragma unroll
                        for (int j = 0; j < NJ; ++j) {
                            const uint32_t col = lane + 64 * j;
                            x[g][j] = (on && col < d) ? __hip_atomic_load(p + col, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0.0f;
                        }
                        xd[g] = on ? __hip_atomic_load(p + d, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0.0f;
                    }
#pragma unroll
                    for (int g = 0; g < GP; ++g) {              // in segment order
#pragma unroll
                        for (int j = 0; j < NJ; ++j) acc[j] += x[g][j];
                        dd += xd[g];
                    }
                }
#pragma unroll
                for (int j = 0; j < NJ; ++j) {
                    const uint32_t col = lane + 64 * j;
                    if (col < d) a.X[(size_t)v * d + col] = acc[j];
                }
                if (lane == 0) a.den[v] = dd;
            }
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------------
// large hops and the bootstrap: cut over edges
// ---------------------------------------------------------------------------------
// One owner per row leaves the wavefronts with long rows running when the others are done, and a wavefront waits for half a
// dozen dependent reads per row (81 K recomputed and 490 K patched rows of 47 over 31 M edges took 2.0 ms, a quarter of what
// the line gathers alone cost). Here the in-edge space of the listed vertices is cut into runs of chunks, handed out from a
// counter like a pull's. What an edge contributes is put into a list in LDS, in edge order, hence by destination: one entry
// for an in-neighbour of a recomputed vertex, two (the new term and the old one, taken away) for a changed in-neighbour of any
// other. The list is then summed like a pull's messages, one row per entry. A vertex whose in-edges lie in one run is
// written by that run alone; what a run boundary cuts is left in parts, which k_gat_close adds up in run order (see
// rp_sum_parts). Changed edges of a vertex that keeps its long row are added before (k_gat_edge_terms). A patched
// denominator that has cancelled (GAT_CANCEL) is found there too and its row recomputed by a workgroup.
struct GatEdgeArgs {
    PullArgs p;                    // list, count_ptr, ioff, in_meta, in_pool, bm_prev, d, X, ctr, l
    const uint32_t *bm_sink, *bm_vadd;
    const float *P, *Pold, *ssrc, *sold, *sdst;
    uint32_t ldp;
    CutRows c;                     // vertices that a run boundary cuts; a row: numerator (d), denominator, mag
    float *den, *mag;              // mag: what a vertex's patches have added and taken away (valid for listed vertices)
    uint8_t *rec;                  // per listed vertex: recomputed
    int all;                       // bootstrap
    uint32_t long_min;             // a sink with at most this many in-neighbours recomputes
    uint32_t n_waves;              // wavefronts of the k_gat_edges launch
    uint32_t *queue, *queue_count;
    const uint32_t *st_src, *st_dst, *n_struct;
    const float *st_sign;
    uint32_t struct_cap;
    // where the messages of the other vertices are listed (rp_gat_listed): the recomputed vertices that have in-edges, and p.ioff is over them
    const uint32_t *rec_list, *rec_count;
    uint32_t list_cap;             // 0: never listed
    int list_force;
};
// the vertices whose in-edges the hop reads, over which p.ioff is
__device__ __forceinline__ bool gat_rows(const GatEdgeArgs &a, const uint32_t *&list, uint32_t &count) {
    const bool listed = rp_gat_listed(a.p.ctr, a.p.l, a.list_cap, a.list_force);
    list = listed ? a.rec_list : a.p.list;
    count = listed ? *a.rec_count : *a.p.count_ptr;
    return listed;
}

__global__ __launch_bounds__(256) void k_gat_prepare(GatEdgeArgs a) {
    const int lane = rp_lane();
    const uint32_t gw = (blockIdx.x * blockDim.x + threadIdx.x) >> 6, nw = (gridDim.x * blockDim.x) >> 6;
    const uint32_t count = *a.p.count_ptr, d = a.p.d;
    for (uint32_t base = gw * 64u; base < count; base += nw * 64u) {
        const uint32_t i = base + (uint32_t)lane;
        bool zero = false;
        uint32_t v = 0;
        if (i < count) {
            v = a.p.list[i];
            const uint32_t deg = a.p.in_meta[v].y;
            const bool rec = a.all || rp_gat_recomputes(a.p.bm_prev, a.bm_sink, a.bm_vadd, a.p.in_meta, a.long_min, v);
            a.rec[v] = rec ? 1 : 0;
            a.mag[v] = 0.0f;
            zero = rec && deg == 0u;                        // no run meets it
            if (zero) a.den[v] = 0.0f;
        }
        unsigned long long m = __ballot(zero);
        while (m) {
            const uint32_t w = (uint32_t)__shfl((int)v, __ffsll((long long)m) - 1);
            m &= m - 1ull;
            for (uint32_t col = lane; col < d; col += 64u) a.p.X[(size_t)w * d + col] = 0.0f;
        }
    }
}

// changed edges of vertices that are not recomputed, as messages (see gat_edge_block); a wavefront each
__global__ __launch_bounds__(256) void k_gat_edge_terms(GatEdgeArgs a) {
    const int lane = rp_lane();
    const uint32_t gw = (blockIdx.x * blockDim.x + threadIdx.x) >> 6, nw = (gridDim.x * blockDim.x) >> 6;
    const uint32_t n = min(*a.n_struct, a.struct_cap), d = a.p.d;
    for (uint32_t s = gw; s < n; s += nw) {
        const uint32_t u = a.st_src[s], v = a.st_dst[s];
        const float sgn = a.st_sign[s];
        if (sgn == 0.0f || !rp_bit(a.bm_sink, v) || !rp_bit(a.p.bm_cur, v) || a.rec[v]) continue;   // (a deleted sink is in no set)
        const bool from_old = rp_bit(a.p.bm_prev, u);
        const float w = gat_weight(from_old ? a.sold[u] : a.ssrc[u], a.sdst[v]);
        const float *row = (from_old ? a.Pold : a.P) + (size_t)u * a.ldp;
        for (uint32_t col = lane; col < d; col += 64u) unsafeAtomicAdd(&a.p.X[(size_t)v * d + col], sgn * w * row[col]);
        if (lane == 0) {
            unsafeAtomicAdd(&a.den[v], sgn * w);
            unsafeAtomicAdd(&a.mag[v], w);
        }
    }
}

#define GAT_REC 0x80000000u                 // an entry's destination: it is recomputed
#define GAT_OLD 0x80000000u                 // an entry's source: the source's row as it was before the batch, taken away
// QUAD: rows of at most 63 columns that carry their score behind the last column (no read of its own): 16 lanes take a row, four
// columns each, so a wavefront sums four entries at a time (the rate of instructions, not memory, bounds a row of two
// cache lines otherwise). Else a wavefront per row, NJ columns per lane, weights made lane-parallel from the score array.
template <int NJ, bool QUAD>
__global__ __launch_bounds__(256) void k_gat_edges(GatEdgeArgs a) {
    constexpr int T = PULL_CHUNK / 64;
    constexpr int G = QUAD ? 4 : (NJ >= 8) ? 2 : 16 / NJ;   // quads / rows in flight
    constexpr uint32_t NONE = 0xFFFFFFFFu, PAD = 0x7FFFFFFEu, ITEMS = 2u * PULL_CHUNK + 16u;
    __shared__ uint32_t s_u[4][ITEMS], s_v[4][ITEMS];
    __shared__ float s_x[4][ITEMS];                         // QUAD: the destination's score; else the entry's weight
    uint32_t count;
    gat_rows(a, a.p.list, count);
    if (count == 0) return;
    const int lane = rp_lane(), wave = threadIdx.x >> 6;
    const uint32_t grp = (uint32_t)lane >> 4, sub = (uint32_t)lane & 15u;
    const uint32_t d = a.p.d, ldp = a.ldp;
    const uint32_t total = a.p.ioff[count];
    const uint32_t gw = (blockIdx.x * blockDim.x + threadIdx.x) >> 6, nw = (gridDim.x * blockDim.x) >> 6;
    const RunCut rc = rp_run_cut(total, nw);
    const uint32_t n_chunks = rc.n_chunks, per = rc.per, n_runs = rc.n_runs;
    uint32_t *su = s_u[wave], *sv = s_v[wave];
    float *sx = s_x[wave];
    for (uint32_t run = gw; run < n_runs;) {
        const uint32_t c_begin = run * per, c_end = min(n_chunks, c_begin + per);
        PullScan<T, 0, 1> scan;
        scan.begin(a.p, count, c_begin * rc.chunk, lane);
        const uint32_t e_end = min(total, c_end * rc.chunk);
        const uint32_t v_first = (uint32_t)__shfl((int)scan.rv, 0), i_last = rp_seg_search_wave(a.p.ioff, 0, count - 1, e_end - 1u);
        const uint32_t v_last = a.p.list[i_last];
        const uint32_t e_last = a.p.ioff[i_last + 1u];
        const bool cut_first = a.p.ioff[scan.i_lo] < c_begin * rc.chunk, cut_last = e_last > e_end;
        const bool goes_on = cut_last && !(v_last == v_first && cut_first);   // a vertex that begins here and ends in a later run
        if (lane == 0) a.c.cut[run] = make_uint2(goes_on ? v_last : NONE, (e_last - 1u) / rc.span());
        bool wrote_first = false, wrote_last = false;
        uint32_t cur = NONE;
        float acc[NJ], dsum = 0.0f, mag = 0.0f;
        float4 acq = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
#pragma unroll
        for (int j = 0; j < NJ; ++j) acc[j] = 0.0f;
        // A vertex's row and sums have one writer, so what is added to them is added by atomics that nothing waits for: with the old row read
        // first every patched vertex cost a wavefront a round trip to memory (139 K recomputed and 465 K patched rows of 47: 940 us -> 825).
        auto flush = [&]() {
            const uint32_t v = cur & ~GAT_REC;
            const bool began_before = v == v_first && cut_first, cut = began_before || (v == v_last && cut_last);
            const bool plain = cut || (cur & GAT_REC) != 0u;  // a part is stored plainly, like a recomputed row
            float *xr = cut ? a.c.part + (size_t)(2u * run + (began_before ? 0u : 1u)) * (d + 2u) : a.p.X + (size_t)v * d;
            wrote_first |= began_before;
            wrote_last |= cut && !began_before;
            float sums = lane == 0 ? dsum : mag;            // lane 0: the denominator's, lane 16: mag
            if (QUAD) {                                     // the four groups' sums together; lane (grp, sub) then has column 4 sub + grp
                acc[0] = swap_add32(swap_add16(acq.x, acq.y), swap_add16(acq.z, acq.w));
                const float dm = swap_add16(dsum, mag);
                sums = swap_add32(dm, dm);
                acq = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            }
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                const uint32_t col = QUAD ? 4u * sub + grp : (uint32_t)lane + 64u * j;
                if (col < d) {
                    if (plain) xr[col] = acc[j];
                    else unsafeAtomicAdd(&xr[col], acc[j]);
                }
                acc[j] = 0.0f;
            }
            if (lane == 0 || lane == 16) {
                float *to = cut ? xr + d + (lane ? 1u : 0u) : (lane ? a.mag : a.den) + v;
                if (cut || (plain && lane == 0)) *to = sums;
                else if (!plain) unsafeAtomicAdd(to, sums);
            }
            dsum = mag = 0.0f;
        };
        for (uint32_t c = c_begin; c < c_end; ++c) {
            const uint32_t e0 = c * rc.chunk, e1 = min(total, e0 + rc.chunk);
            uint32_t my_v[T], my_u[T];
            float no_w[1];
            bool valid[T], rec[T];
            scan.chunk(a.p, count, e0, e1, lane, my_v, my_u, no_w, valid);
            float t_v[T];
#pragma unroll
            for (int t = 0; t < T; ++t) {
                const uint32_t v = valid[t] ? my_v[t] : v_first;
                rec[t] = a.rec[v] != 0;
                t_v[t] = a.sdst[v];
            }
            uint32_t n = 0;
#pragma unroll
            for (int t = 0; t < T; ++t) {
                const bool one = valid[t] && (rec[t] || rp_bit(a.p.bm_prev, my_u[t]));
                const bool two = one && !rec[t];
                float wn = t_v[t], wo = t_v[t];
                if (!QUAD) {
                    wn = one ? gat_weight(a.ssrc[my_u[t]], t_v[t]) : 0.0f;
                    wo = two ? -gat_weight(a.sold[my_u[t]], t_v[t]) : 0.0f;
                }
                const unsigned long long m1 = __ballot(one), m2 = __ballot(two), below = (1ull << lane) - 1ull;
                const uint32_t at = n + (uint32_t)__popcll(m1 & below) + (uint32_t)__popcll(m2 & below);
                if (one) {
                    su[at] = my_u[t];
                    sv[at] = my_v[t] | (rec[t] ? GAT_REC : 0u);
                    sx[at] = wn;
                }
                if (two) {
                    su[at + 1u] = my_u[t] | GAT_OLD;
                    sv[at + 1u] = my_v[t];
                    sx[at + 1u] = wo;
                }
                n += (uint32_t)__popcll(m1) + (uint32_t)__popcll(m2);
            }
            if (lane < 16) {                                // entries that the last round reads past the end: row 0, no destination
                su[n + lane] = 0u;
                sv[n + lane] = PAD;
                sx[n + lane] = 0.0f;
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");   // (LDS accesses of one wavefront are executed in order)
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            if constexpr (QUAD) {
                for (uint32_t k0 = 0; k0 < n; k0 += 4u * G) {
                    uint32_t u[G], v[G];
                    float tv[G];
                    float4 r[G];
#pragma unroll
                    for (int g = 0; g < G; ++g) {
                        const uint32_t idx = min(k0 + 4u * g, n) + grp;      // at most n + 3
                        u[g] = su[idx];
                        v[g] = sv[idx];
                        tv[g] = sx[idx];
                        const float *row = ((u[g] & GAT_OLD) ? a.Pold : a.P) + (size_t)(u[g] & ~GAT_OLD) * ldp;
                        r[g] = 4u * sub < ldp ? *(const float4 *)(row + 4u * sub) : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                    }
#pragma unroll
                    for (int g = 0; g < G; ++g) {
                        if (k0 + 4u * g >= n) continue;
                        const float mine = (d & 3u) == 0u ? r[g].x : ((d & 3u) == 1u ? r[g].y : ((d & 3u) == 2u ? r[g].z : r[g].w));
                        const float w = gat_weight(__shfl(mine, (int)(16u * grp + d / 4u)), tv[g]);     // the row's score sits in lane d / 4
                        const float sw = (u[g] & GAT_OLD) ? -w : w;
                        if (!__any(v[g] != cur)) {
                            acq.x = __builtin_fmaf(sw, r[g].x, acq.x);
                            acq.y = __builtin_fmaf(sw, r[g].y, acq.y);
                            acq.z = __builtin_fmaf(sw, r[g].z, acq.z);
                            acq.w = __builtin_fmaf(sw, r[g].w, acq.w);
                            dsum += sw;
                            mag += w;
                        } else {                            // entry by entry (they are sorted by destination)
#pragma unroll
                            for (uint32_t q = 0; q < 4u; ++q) {
                                const uint32_t vq = (uint32_t)__builtin_amdgcn_readlane((int)v[g], 16 * (int)q);
                                if (vq == PAD) continue;
                                if (vq != cur) {
                                    if (cur != NONE) flush();
                                    cur = vq;
                                }
                                if (grp == q) {
                                    acq.x = __builtin_fmaf(sw, r[g].x, acq.x);
                                    acq.y = __builtin_fmaf(sw, r[g].y, acq.y);
                                    acq.z = __builtin_fmaf(sw, r[g].z, acq.z);
                                    acq.w = __builtin_fmaf(sw, r[g].w, acq.w);
                                    dsum += sw;
                                    mag += w;
                                }
                            }
                        }
                    }
                }
            } else {
                for (uint32_t k0 = 0; k0 < n; k0 += G) {
                    float r[G][NJ], w[G];
                    uint32_t v[G];
#pragma unroll
                    for (int g = 0; g < G; ++g) {
                        const uint32_t idx = min(k0 + (uint32_t)g, n - 1u);
                        const uint32_t u = (uint32_t)__builtin_amdgcn_readfirstlane((int)su[idx]);
                        v[g] = (uint32_t)__builtin_amdgcn_readfirstlane((int)sv[idx]);
                        w[g] = __uint_as_float((uint32_t)__builtin_amdgcn_readfirstlane((int)__float_as_uint(sx[idx])));
                        const float *row = ((u & GAT_OLD) ? a.Pold : a.P) + (size_t)(u & ~GAT_OLD) * ldp;
#pragma unroll
                        for (int j = 0; j < NJ; ++j) r[g][j] = row[min((uint32_t)lane + 64u * j, d - 1u)];
                    }
#pragma unroll
                    for (int g = 0; g < G; ++g) {
                        if (k0 + (uint32_t)g >= n) continue;
                        if (v[g] != cur) {
                            if (cur != NONE) flush();
                            cur = v[g];
                        }
#pragma unroll
                        for (int j = 0; j < NJ; ++j) acc[j] = __builtin_fmaf(w[g], r[g][j], acc[j]);
                        dsum += w[g];
                        mag += fabsf(w[g]);
                    }
                }
            }
            __builtin_amdgcn_wave_barrier();                // the next chunk overwrites the list
            scan.advance();
        }
        if (cur != NONE) flush();
        // nothing in this run changed for a vertex that it shares with others: its part is zero
        for (uint32_t col = lane; cut_first && !wrote_first && col < d + 2u; col += 64u) a.c.part[(size_t)(2u * run) * (d + 2u) + col] = 0.0f;
        for (uint32_t col = lane; goes_on && !wrote_last && col < d + 2u; col += 64u) a.c.part[(size_t)(2u * run + 1u) * (d + 2u) + col] = 0.0f;
        if ((unsigned long long)nw * per >= n_chunks) break;
        run = nw + rp_next_run(&a.p.ctr->pull_next[a.p.l], lane);
    }
}

// The messages of vertices that are not recomputed, from their list in order of destination (k_frontier_list, k_list_order): the old row taken away and
// the new one added per changed in-neighbour, a sum per destination. Rows of more than 63 columns whose pairs all lie in one wavefront's run have no other
// writer: their old row is read with the first message and stored with the sum. Narrow rows, and those at a run's ends, are added to by atomics. In
// place of testing all in-neighbours of those vertices for the few that changed (rp_gat_list_made): 209 K messages of 256 columns to 135 K of them,
// with 14 M in-neighbours, k_gat_edges 405 -> 285 us (650 -> 412 for twice the recomputed vertices) and 84 here; with atomics for every row 130.
template <int NJ, bool QUAD>
__global__ __launch_bounds__(256) void k_gat_list(GatEdgeArgs a, const uint2 *sorted, uint32_t cap, int force, uint32_t *cnt, uint32_t n_cnt) {
    const uint32_t M = a.p.ctr->set[a.p.l - 1u].a ? a.p.ctr->set[a.p.l - 1u].m : 0u;
    if (!rp_gat_list_made(a.p.ctr, M, cap, force)) return;
    {   // the buckets' counts for the next hop that is listed
        const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
        if (i < n_cnt) cnt[i] = 0;
    }
    if (a.p.ctr->pair_over[a.p.l]) return;
    if (blockIdx.x == 0 && threadIdx.x == 0) a.p.ctr->hop_mode[a.p.l] = 1u + RP_HOP_SORTED;
    constexpr uint32_t NONE = 0xFFFFFFFFu;
    constexpr int G = QUAD ? 4 : (NJ >= 8 ? 1 : 8 / NJ);    // quads / messages in flight, two rows each
    const uint32_t n_pairs = a.p.ctr->pairs[a.p.l];
    const int lane = rp_lane();
    const uint32_t d = a.p.d, ldp = a.ldp, grp = (uint32_t)lane >> 4, sub = (uint32_t)lane & 15u;
    const uint32_t gw = (blockIdx.x * blockDim.x + threadIdx.x) >> 6, nw = (gridDim.x * blockDim.x) >> 6;
    const uint32_t unit = n_pairs / 64u < nw ? 16u : 64u;   // pairs at a time: fewer where whole wavefronts would leave others without any
    const uint32_t n_chunks = (n_pairs + unit - 1u) / unit, per = (n_chunks + nw - 1u) / nw;
    const uint32_t c_begin = min(n_chunks, gw * per), c_end = min(n_chunks, c_begin + per);
    if (c_begin >= c_end) return;
    // destinations of the run's first and last pair may have pairs in a neighbour's run; all others have one writer
    const uint32_t v_first = sorted[c_begin * unit].x, v_last = sorted[min(n_pairs, c_end * unit) - 1u].x;
    uint32_t cur = NONE;
    float xo[NJ];                                           // the old row (not QUAD)
    float acc[NJ], dsum = 0.0f, mag = 0.0f;
    float4 acq = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[j] = xo[j] = 0.0f;
    auto flush = [&]() {
        float sums = lane == 0 ? dsum : mag;                // lane 0: the denominator's, lane 16: mag
        if (QUAD) {
            acc[0] = swap_add32(swap_add16(acq.x, acq.y), swap_add16(acq.z, acq.w));
            const float dm = swap_add16(dsum, mag);
            sums = swap_add32(dm, dm);
            acq = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        }
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            const uint32_t col = QUAD ? 4u * sub + grp : (uint32_t)lane + 64u * j;
            if (col < d) {
                float *x = &a.p.X[(size_t)cur * d + col];
                if (!QUAD && cur != v_first && cur != v_last) *x = xo[j] + acc[j];
                else unsafeAtomicAdd(x, acc[j]);
            }
            acc[j] = 0.0f;
        }
        if (lane == 0 || lane == 16) unsafeAtomicAdd((lane ? a.mag : a.den) + cur, sums);
        dsum = mag = 0.0f;
    };
    for (uint32_t c = c_begin; c < c_end; ++c) {
        const uint32_t e = c * unit + (uint32_t)lane, n = min(unit, n_pairs - c * unit);
        const bool in = (uint32_t)lane < n;
        const uint2 my = in ? sorted[e] : make_uint2(NONE, 0u);
        const float t_v = in ? a.sdst[my.x] : 0.0f;
        if constexpr (QUAD) {
            for (uint32_t k0 = 0; k0 < n; k0 += 4u * G) {
                uint32_t v[G];
                float tv[G];
                float4 rn[G], ro[G];
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    const int idx = (int)(k0 + 4u * g + grp); // below 64; past the list's end: row 0, no destination
                    const size_t at = (size_t)(uint32_t)__shfl((int)my.y, idx) * ldp + 4u * sub;
                    v[g] = (uint32_t)__shfl((int)my.x, idx);
                    tv[g] = __shfl(t_v, idx);
                    const bool col = 4u * sub < ldp;
                    rn[g] = col ? *(const float4 *)(a.P + at) : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                    ro[g] = col && v[g] != NONE ? *(const float4 *)(a.Pold + at) : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                }
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    if (k0 + 4u * g >= n) continue;
                    const uint32_t r = d & 3u;
                    const int from = (int)(16u * grp + d / 4u);   // the rows' scores sit in lane d / 4
                    const float wn = gat_weight(__shfl(r == 0u ? rn[g].x : (r == 1u ? rn[g].y : (r == 2u ? rn[g].z : rn[g].w)), from), tv[g]);
                    const float wo = gat_weight(__shfl(r == 0u ? ro[g].x : (r == 1u ? ro[g].y : (r == 2u ? ro[g].z : ro[g].w)), from), tv[g]);
                    auto add = [&]() {
                        acq.x += wn * rn[g].x - wo * ro[g].x;
                        acq.y += wn * rn[g].y - wo * ro[g].y;
                        acq.z += wn * rn[g].z - wo * ro[g].z;
                        acq.w += wn * rn[g].w - wo * ro[g].w;
                        dsum += wn - wo;
                        mag += wn + wo;
                    };
                    if (!__any(v[g] != cur)) {
                        add();
                    } else {                                // destination by destination (they are in order)
                        unsigned long long left = __ballot(v[g] != NONE);
                        while (left) {
                            const uint32_t vg = (uint32_t)__builtin_amdgcn_readlane((int)v[g], __ffsll((long long)left) - 1);
                            if (vg != cur) {
                                if (cur != NONE) flush();
                                cur = vg;
                            }
                            const bool same = v[g] == vg;
                            if (same) add();
                            left &= ~__ballot(same);
                        }
                    }
                }
            }
        } else {
            const float my_n = in ? gat_weight(a.ssrc[my.y], t_v) : 0.0f, my_o = in ? gat_weight(a.sold[my.y], t_v) : 0.0f;
            for (uint32_t k0 = 0; k0 < n; k0 += G) {
                float rn[G][NJ], ro[G][NJ], x[G][NJ];
                uint32_t before = cur;
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    const int kk = (int)min(k0 + (uint32_t)g, n - 1u);
                    const uint32_t u = (uint32_t)__builtin_amdgcn_readlane((int)my.y, kk), v = (uint32_t)__builtin_amdgcn_readlane((int)my.x, kk);
                    const bool own = v != before && v != v_first && v != v_last;
                    before = v;
#pragma unroll
                    for (int j = 0; j < NJ; ++j) {
                        const size_t at = (size_t)u * ldp + min((uint32_t)lane + 64u * j, d - 1u);
                        rn[g][j] = a.P[at];
                        ro[g][j] = a.Pold[at];
                        x[g][j] = own ? a.p.X[(size_t)v * d + min((uint32_t)lane + 64u * j, d - 1u)] : 0.0f;
                    }
                }
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    const int k = (int)(k0 + (uint32_t)g);
                    if (k >= (int)n) continue;
                    const uint32_t v = (uint32_t)__builtin_amdgcn_readlane((int)my.x, k);
                    const float wn = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(my_n), k));
                    const float wo = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(my_o), k));
                    if (v != cur) {
                        if (cur != NONE) flush();
                        cur = v;
#pragma unroll
                        for (int j = 0; j < NJ; ++j) xo[j] = x[g][j];
                    }
#pragma unroll
                    for (int j = 0; j < NJ; ++j) acc[j] += wn * rn[g][j] - wo * ro[g][j];
                    dsum += wn - wo;
                    mag += wn + wo;
                }
            }
        }
    }
    if (cur != NONE) flush();
}

uint32_t rp_gat_long_min(const ripple_ctx *c) { return c->in_w ? 0xFFFFFFFFu : GAT_LONG; }

// Vertices that a run boundary cuts: their parts added up, a wavefront per run (22 us for 256 columns and 12 K runs, 13 for 47 and
// 17 K). Then (hops) every patched denominator that has cancelled is queued: of the cut vertices by the wavefront that has just
// finished it, of the others, which this launch does not write, by a thread each.
__global__ __launch_bounds__(256) void k_gat_close(GatEdgeArgs a) {
    const int lane = rp_lane();
    const uint32_t gw = (blockIdx.x * blockDim.x + threadIdx.x) >> 6, nw = (gridDim.x * blockDim.x) >> 6;
    const uint32_t count = *a.p.count_ptr, d = a.p.d;
    if (count == 0) return;
    const uint32_t *rows;
    uint32_t n_rows;
    const bool listed = gat_rows(a, rows, n_rows);
    const RunCut rc = rp_run_cut(a.p.ioff[n_rows], a.n_waves);
    const uint32_t n_runs = rc.n_runs, span = rc.span();
    auto cancelled = [](float den, float mag) { return mag > 0.0f && !(den > GAT_CANCEL * mag); };
    for (uint32_t r = gw; r < n_runs; r += nw) {
        const uint2 c = a.c.cut[r];
        if (c.x == 0xFFFFFFFFu) continue;
        const uint32_t v = c.x;
        const bool rec = a.rec[v] != 0;
        float den = 0.0f, mag = 0.0f;                       // in the lanes of columns d and d + 1
        for (uint32_t c0 = lane; c0 < d + 2u; c0 += 64u * PARTS_B) {
            float old[PARTS_B], t[PARTS_B];
            float *to[PARTS_B];
#pragma unroll
            for (int b = 0; b < PARTS_B; ++b) {
                const uint32_t col = c0 + 64u * b;
                to[b] = col < d ? &a.p.X[(size_t)v * d + col] : (col == d ? &a.den[v] : &a.mag[v]);
                old[b] = (!rec && col < d + 2u) ? *to[b] : 0.0f;
            }
            rp_sum_parts(a.c.part, d + 2u, r, c.y, c0, t);
#pragma unroll
            for (int b = 0; b < PARTS_B; ++b) {
                const uint32_t col = c0 + 64u * b;
                const float x = old[b] + t[b];
                if (col <= d) *to[b] = x;                   // (mag is looked at here only)
                if (col == d) den = x;
                if (col == d + 1u) mag = x;
            }
        }
        den = __shfl(den, (int)(d & 63u));
        mag = __shfl(mag, (int)((d + 1u) & 63u));
        if (lane == 0 && !a.all && !rec && cancelled(den, mag)) a.queue[atomicAdd(a.queue_count, 1u)] = v;
    }
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; !a.all && i < count; i += gridDim.x * blockDim.x) {
        const uint32_t v = a.p.list[i], e0 = listed ? 0u : a.p.ioff[i], e1 = listed ? 0u : a.p.ioff[i + 1u];
        if (a.rec[v] || (e1 > e0 && e0 / span != (e1 - 1u) / span)) continue;
        if (cancelled(a.den[v], a.mag[v])) a.queue[atomicAdd(a.queue_count, 1u)] = v;
    }
}

// bootstrap: every live vertex (c->all_list, its in-degree prefix in c->ioff_all, count in ctr->n_all) is recomputed.
// listed: a small hop, whose vertices (and the long rows among them) were listed while they were marked: a wavefront or a
// workgroup per row in one launch, which is paced by the longest chain of reads; all other hops are cut over edges.
void rp_launch_gat_scatter(ripple_ctx *c, uint32_t l, bool bootstrap, bool listed, uint32_t pair_cap) {
    const LayerDev &ly = c->layers[l - 1];
    GatArgs a;
    a.list = c->list[l];
    a.count_ptr = &c->ctr->set[l].a;
    a.in_meta = c->in_meta;
    a.in_pool = c->in_pool;
    a.bm_prev = c->bm[l - 1];
    a.bm_sink = c->bm_sink;
    a.bm_vadd = c->bm_vadd;
    a.P = ly.P;
    a.Pold = c->Pold;
    a.ssrc = ly.ssrc;
    a.sold = c->sold;
    a.sdst = ly.sdst;
    a.ldp = ly.ldp;
    a.d = ly.d_out;
    a.X = c->X[l];
    a.den = ly.den;
    a.all = 0;
    a.long_min = RP_MONO_LISTED_LONG;                    // (the limit the long rows were queued with)
    a.split_min = ROW_SPLIT_MIN;
    a.n_big = &c->ctr->n_big[l];
    a.n_seg = &c->ctr->n_seg[l];
    a.seg_v = c->seg_v;
    a.seg_done = c->seg_done;
    a.seg_base = c->seg_base;
    a.seg_r = c->seg_r;
    a.seg_part = c->seg_part;
    a.big_cap = c->big_cap;
    a.seg_cap = std::min(c->seg_cap, c->seg_limit);
    a.seg_ld = c->seg_ld;
    a.st_src = c->st_src;
    a.st_dst = c->st_dst;
    a.st_sign = c->st_unit;                              // +1 added, -1 deleted, 0 re-weighted (attention ignores edge weights)
    a.n_struct = &c->ctr->n_struct;
    a.struct_cap = (c->in_w || bootstrap) ? 0u : c->struct_cap;   // weighted graphs: sinks recompute
    GatArgs b = a;                                       // the queue's side
    b.list = c->all_list;
    b.count_ptr = &c->ctr->n_long[l];
    const dim3 block(256);
    if (listed) {                                        // every workgroup resident at once: half the compute units' worth for each role
#define GAT_CASE(NJ, TEAM)                                                                                            \
    do {                                                                                                              \
        hipLaunchKernelGGL((k_gat_scatter_both<NJ, TEAM>), dim3(c->n_cu / 2 + (c->n_cu / 2) * (16 / TEAM)),           \
                           dim3(TEAM * 64), 0, c->stream, a, b, c->n_cu / 2);                                         \
        hipLaunchKernelGGL((k_gat_scatter_seg<NJ, ROW_SEG / 64>), dim3(c->n_cu * 4), dim3(ROW_SEG), 0, c->stream, b); \
    } while (0)
        if (a.d <= 64) GAT_CASE(1, 16);
        else if (a.d <= 128) GAT_CASE(2, 16);
        else if (a.d <= 256) GAT_CASE(4, 16);
        else if (a.d <= 512) GAT_CASE(8, 16);
        else GAT_CASE(16, 8);
#undef GAT_CASE
        return;
    }
    const dim3 grid(c->n_cu * 8);
    GatEdgeArgs e = {};
    e.p.list = bootstrap ? c->all_list : c->list[l];
    e.p.count_ptr = bootstrap ? &c->ctr->n_all : &c->ctr->set[l].a;
    e.p.ioff = bootstrap ? c->ioff_all : c->ioff[l];
    e.p.in_meta = c->in_meta;
    e.p.in_pool = c->in_pool;
    e.p.bm_prev = c->bm[l - 1];
    e.p.bm_cur = c->bm[l];
    e.p.d = ly.d_out;
    e.p.X = c->X[l];
    e.p.ctr = c->ctr;
    e.p.l = l;
    e.bm_sink = c->bm_sink;
    e.bm_vadd = c->bm_vadd;
    e.P = ly.P;
    e.Pold = c->Pold;
    e.ssrc = ly.ssrc;
    e.sold = c->sold;
    e.sdst = ly.sdst;
    e.ldp = ly.ldp;
    e.c = rp_cut_rows(c->D[l & 1], c->max_runs);                                // (free until the row update fills it; load_model has made it large enough)
    e.den = ly.den;
    e.mag = c->gat_mag;
    e.rec = c->gat_rec;
    e.all = bootstrap ? 1 : 0;
    e.long_min = rp_gat_long_min(c);
    e.n_waves = c->n_cu * 8 * 4;
    e.queue = c->all_list;
    e.queue_count = &c->ctr->n_long[l];
    e.st_src = c->st_src;
    e.st_dst = c->st_dst;
    e.st_sign = c->st_unit;
    e.n_struct = &c->ctr->n_struct;
    e.struct_cap = a.struct_cap;
    e.rec_list = c->ioff_all;
    e.rec_count = &c->ctr->n_rec;
    e.list_cap = pair_cap;
    e.list_force = c->opt_sorted == 2;
    hipLaunchKernelGGL(k_gat_prepare, grid, block, 0, c->stream, e);
    if (e.struct_cap) hipLaunchKernelGGL(k_gat_edge_terms, dim3(c->n_cu * 2), block, 0, c->stream, e);
    const uint32_t n_cnt = pair_cap ? rp_list_cut(c, c->last_m[l] ? c->last_m[l] : pair_cap).n : 0u;
    b.all = 1;                                           // rows whose patch has cancelled: read once more
    b.split_min = 0xFFFFFFFFu;
#define GAT_CASE(NJ, QUAD, TEAM)                                                                                              \
    do {                                                                                                                      \
        hipLaunchKernelGGL((k_gat_edges<NJ, QUAD>), grid, block, 0, c->stream, e);                                            \
        if (pair_cap) {                                                                                                       \
            rp_launch_list_order(c, l, pair_cap);                                                                             \
            hipLaunchKernelGGL((k_gat_list<NJ, QUAD>), grid, block, 0, c->stream, e, c->pair_sorted, pair_cap, c->opt_sorted == 2, c->pair_cnt, n_cnt); \
        }                                                                                                                     \
        hipLaunchKernelGGL(k_gat_close, dim3(c->n_cu * 16), block, 0, c->stream, e);                                                     \
        if (bootstrap) break;                                                                                                 \
        hipLaunchKernelGGL((k_gat_scatter_long<NJ, TEAM>), dim3(c->n_cu), dim3(TEAM * 64), 0, c->stream, b);                  \
    } while (0)
    if (e.ldp > e.p.d) GAT_CASE(1, true, 16);
    else if (e.p.d <= 64) GAT_CASE(1, false, 16);
    else if (e.p.d <= 128) GAT_CASE(2, false, 16);
    else if (e.p.d <= 256) GAT_CASE(4, false, 16);
    else if (e.p.d <= 512) GAT_CASE(8, false, 16);
    else GAT_CASE(16, false, 8);
#undef GAT_CASE
}

// before the projection of A_{l-1} is refreshed: keep the old rows and source scores for the messages
// 16 lanes per row, four columns each, eight rows per wavefront and round; with a row per wavefront, both kernels waited for one chain of two
// reads after another. A_2 of 300 updates on 31 M edges, rows of 47 columns: kept rows 69 -> 21 us, scores 44 -> 13.
#define GAT_ROWS_U 2
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx4u __attribute__((ext_vector_type(4), aligned(4)));
__global__ __launch_bounds__(256) void k_gat_save(const uint32_t *list, const uint32_t *count_ptr, const float *P,
                                                  const float *ssrc, uint32_t ldp, float *Pold, float *sold) {
    constexpr int U = GAT_ROWS_U;
    const uint32_t count = *count_ptr;
    const uint32_t lane = rp_lane(), grp = lane >> 4, sub = lane & 15u;
    const uint32_t gw = (blockIdx.x * blockDim.x + threadIdx.x) >> 6, nw = (gridDim.x * blockDim.x) >> 6;
    for (uint32_t i0 = gw * 4u * U; i0 < count; i0 += nw * 4u * U) {
        uint32_t v[U];
        float s[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = list[min(i0 + 4u * u + grp, count - 1u)];     // past the end: the last row again, not stored
#pragma unroll
        for (int u = 0; u < U; ++u) s[u] = ssrc[v[u]];
        for (uint32_t col = 4u * sub; col < ldp; col += 64u) {
            floatx4 x[U];
#pragma unroll
            for (int u = 0; u < U; ++u) x[u] = *(const floatx4u *)(P + (size_t)v[u] * ldp + col);   // (up to three numbers past the row: there is room)
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (i0 + 4u * u + grp >= count) continue;
                float *to = Pold + (size_t)v[u] * ldp + col;
                if (col + 4u <= ldp) {
                    *(floatx4u *)to = x[u];
                } else {
#pragma unroll
                    for (uint32_t k = 0; k < 3u; ++k)
                        if (col + k < ldp) to[k] = x[u][k];
                }
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (sub == 0u && i0 + 4u * u + grp < count) sold[v[u]] = s[u];
    }
}

// s_src[v] = a_src . P[v], s_dst[v] = a_dst . P[v] for the listed vertices (att: a_src then a_dst); rows with room keep s_src
// behind their last column as well
__global__ __launch_bounds__(256) void k_gat_scores(const uint32_t *list, const uint32_t *count_ptr, float *P, uint32_t ldp,
                                                    const float *att, uint32_t d, float *ssrc, float *sdst) {
    constexpr int U = GAT_ROWS_U;
    const uint32_t count = *count_ptr;
    const uint32_t lane = rp_lane(), grp = lane >> 4, sub = lane & 15u;
    const uint32_t gw = (blockIdx.x * blockDim.x + threadIdx.x) >> 6, nw = (gridDim.x * blockDim.x) >> 6;
    for (uint32_t i0 = gw * 4u * U; i0 < count; i0 += nw * 4u * U) {
        uint32_t v[U];
        float s[U], t[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            v[u] = list[min(i0 + 4u * u + grp, count - 1u)];
            s[u] = t[u] = 0.0f;
        }
        for (uint32_t col = 4u * sub; col < d; col += 64u) {
            const floatx4 as = *(const floatx4u *)(att + col), ad = *(const floatx4u *)(att + d + col);
            floatx4 x[U];
#pragma unroll
            for (int u = 0; u < U; ++u) x[u] = *(const floatx4u *)(P + (size_t)v[u] * ldp + col);
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (uint32_t k = 0; k < 4u; ++k) {
                    const bool in = col + k < d;
                    s[u] += in ? x[u][k] * as[k] : 0.0f;
                    t[u] += in ? x[u][k] * ad[k] : 0.0f;
                }
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int o = 1; o < 16; o <<= 1) {
                s[u] += __shfl_xor(s[u], o);
                t[u] += __shfl_xor(t[u], o);
            }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (sub == 0u && i0 + 4u * u + grp < count) {
                ssrc[v[u]] = s[u];
                sdst[v[u]] = t[u];
                if (ldp > d) P[(size_t)v[u] * ldp + d] = s[u];
            }
    }
}

void rp_launch_gat_save(ripple_ctx *c, uint32_t l, const uint32_t *list, const uint32_t *count_d) {
    const LayerDev &ly = c->layers[l - 1];
    hipLaunchKernelGGL(k_gat_save, dim3(c->n_cu * 8), dim3(256), 0, c->stream, list, count_d, ly.P, ly.ssrc, ly.ldp,
                       c->Pold, c->sold);
}

void rp_launch_gat_scores(ripple_ctx *c, uint32_t l, const uint32_t *list, const uint32_t *count_d) {
    const LayerDev &ly = c->layers[l - 1];
    hipLaunchKernelGGL(k_gat_scores, dim3(c->n_cu * 8), dim3(256), 0, c->stream, list, count_d, ly.P, ly.ldp, ly.att,
                       ly.d_out, ly.ssrc, ly.sdst);
}
