// The push scatter's inner part: messages along the out-edges of a hop's set, added to their destinations' rows with float
// atomics. Shared by k_scatter_push and the fused kernels of small hops.
#pragma once
#include "common.h"

#define PUSH_CHUNK 64

// A project-first layer's message element, lane = column, from what is to be sent: rounded as the packed row's chunk (columns c,
// 16 + c, 32 + c) would round it if the layer packs its rows. All 64 lanes together (lanes past the row pass zeros).
__device__ __forceinline__ float rp_message(float m, bool packed) {
    if (!packed) return m;
    float big = fabsf(m);
    big = fmaxf(big, __shfl_xor(big, 16));
    big = fmaxf(big, __shfl_xor(big, 32));
    return rp_msg_round(m, big);
}

// PK = 1 (NJ = 1 only): the message rows are packed 128-byte lines (D points at them). PK = 2: project-first layers of small
// hops, where no kernel has made the messages: D holds the sources' projected rows and T what they have sent; the message
// is made here, for every edge again (rp_message), and T is brought up to date by a later kernel.
// WT = 1: a message is multiplied by its edge's weight (out_w, parallel to out_pool: 4 bytes per edge, kept so that weighted sums need not
// walk every in-row of A_l for a few thousand messages: hop 1 of 1,777 updates on 31 M edges 283 -> 15 us, the whole batch 2.22 -> 1.67 ms;
// 13 updates on 43 M edges 0.69 -> 0.23).
template <int NJ, int PK, int WT>
__device__ __forceinline__ void push_edges(const uint32_t *list, const uint32_t *count_ptr, const uint32_t *eoff, const float *D,
                                           const float *T_sent, uint32_t ldt, uint32_t ldd, uint32_t d, const uint2 *out_meta,
                                           const uint32_t *out_pool, const float *out_w, float *X, uint32_t gw, uint32_t nw, bool packed = false) {
    constexpr int G = (NJ <= 2) ? 8 : (NJ <= 4 ? 4 : (NJ <= 8 ? 2 : 1));   // edges per round
    const uint32_t count = *count_ptr;
    if (count == 0) return;
    const int lane = rp_lane();
    const uint32_t M = count_ptr[1];
    // few messages: spread them over more wavefronts, very few: what one round takes (some hundred projected messages 7.8 -> 6.1 us)
    const uint32_t chunk = (M <= 2048u) ? (uint32_t)G : ((M <= 16384u) ? 16u : PUSH_CHUNK);
    const uint32_t n_chunks = (M + chunk - 1) / chunk;
    for (uint32_t c = gw; c < n_chunks; c += nw) {
        const uint32_t e0 = c * chunk, e1 = min(M, e0 + chunk);
        // the chunk's first row by the wavefront together; the 64 rows from there on (vertex, pool position,
        // end) one per lane, so an edge finds its row with shuffles instead of a chain of dependent reads
        const uint32_t i_lo = rp_seg_search_wave(eoff, 0, count - 1, e0);
        const uint32_t ri = min(count - 1, i_lo + (uint32_t)lane);
        const uint32_t rv = list[ri];
        const uint32_t rbase = out_meta[rv].x - eoff[ri];      // pool position of edge e: rbase + e (mod 2^32)
        const uint32_t bnd = rp_row_end(eoff, count, M, i_lo + (uint32_t)lane);
        const uint32_t e = min(e0 + (uint32_t)lane, e1 - 1);    // lanes past the chunk repeat its last edge (not used)
        const uint32_t k = rp_count_le(bnd, e);
        uint32_t my_i = i_lo + k, my_u = __shfl(rv, (int)min(k, 63u)), pos = __shfl(rbase, (int)min(k, 63u)) + e;
        if (k >= 64u) {                                         // more than 64 rows in 64 edges (rows without out-edges)
            my_i = rp_seg_search(eoff, i_lo + 64u, count - 1, e);
            my_u = list[my_i];
            pos = out_meta[my_u].x + (e - eoff[my_i]);
        }
        const uint32_t my_v = out_pool[pos];
        const float my_w = WT ? out_w[pos] : 1.0f;
        const int n_here = (int)(e1 - e0);
        // G edges per round: their sources' delta rows are requested together (consecutive edges mostly share
        // the source: the repeats are cache hits), then the additions go out
        for (int k0 = 0; k0 < n_here; k0 += G) {
            float dreg[G][NJ];
            uint32_t vk[G];
            if constexpr (PK == 1) {                           // lane = column: its chunk is lane mod 16
                uint2 ch[G];
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    const int k = min(k0 + g, n_here - 1);
                    const uint32_t uk = __shfl(my_u, k);
                    vk[g] = __shfl(my_v, k);
                    ch[g] = *(const uint2 *)((const uint32_t *)D + (size_t)uk * RP_MSG_WORDS + 2u * ((uint32_t)lane & 15u));
                }
#pragma unroll
                for (int g = 0; g < G; ++g) dreg[g][0] = ((uint32_t)lane < d) ? rp_msg_decode_col(ch[g], (uint32_t)lane) : 0.0f;
            } else {
                float sent[PK == 2 ? G : 1][NJ];
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    const int k = min(k0 + g, n_here - 1);
                    const uint32_t uk = __shfl(my_u, k);
                    vk[g] = __shfl(my_v, k);
#pragma unroll
                    for (int j = 0; j < NJ; ++j) {
                        const uint32_t col = lane + 64 * j;
                        dreg[g][j] = (col < d) ? D[(size_t)uk * ldd + col] : 0.0f;
                        if (PK == 2) sent[g][j] = (col < d) ? T_sent[(size_t)uk * ldt + col] : 0.0f;
                    }
                }
                if constexpr (PK == 2) {
#pragma unroll
                    for (int g = 0; g < G; ++g)
#pragma unroll
                        for (int j = 0; j < NJ; ++j) dreg[g][j] = rp_message(dreg[g][j] - sent[g][j], NJ == 1 && packed);
                }
            }
#pragma unroll
            for (int g = 0; g < G; ++g) {
                if (k0 + g < n_here) {
                    if (WT) {
                        const float wk = __shfl(my_w, k0 + g);
#pragma unroll
                        for (int j = 0; j < NJ; ++j) dreg[g][j] *= wk;
                    }
                    bool any = false;
#pragma unroll
                    for (int j = 0; j < NJ; ++j) any |= dreg[g][j] != 0.0f;
                    if (__ballot(any) != 0ull) {                // an all-zero delta changes nothing
                        float *xr = X + (size_t)vk[g] * d;
#pragma unroll
                        for (int j = 0; j < NJ; ++j) {
                            const uint32_t col = lane + 64 * j;
                            if (col < d) unsafeAtomicAdd(&xr[col], dreg[g][j]);
                        }
                    }
                }
            }
        }
    }
}
