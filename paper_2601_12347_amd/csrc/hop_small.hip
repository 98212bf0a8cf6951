// A small hop of a sum or mean layer in two launches (three when the layer is project-first), where the general path takes
// six to eight. Small hops are paced by launches and by chains of dependent reads, so what does not depend on one another
// runs side by side in one launch, and nothing that can be written on the way is made by a kernel of its own:
//   * the frontier of hop l (out-edge walk from A_{l-1} and roots; the list's degree prefix is written along with the list),
//   * the push of hop l's messages along the same out-edges (rows of D^{l-1}),
//   * the products of the previous embedding that the layer caches (self term; both products of a project-first layer),
// then, for project-first layers, the push of their messages, which the pushing wavefronts make themselves; then the row update.
#include "kernels.h"
#include "push.h"
#include "rows.h"
#include "walk.h"
#include <algorithm>

struct HopArgs {
    const uint32_t *list, *count_ptr, *eoff;       // A_{l-1}
    const uint2 *out_meta;
    const uint32_t *out_pool;
    const float *out_w;                            // weights beside the out-rows (WT: weighted sums; else null)
    SparseArgs sp;
    const float *D;                                // rows to push, or null
    uint32_t ldd, d;
    float *X;
    DevCtr *ctr;
    uint32_t l;
    uint32_t nb_walk, nb_push;                     // workgroups of the first two parts; the rest multiply
    TArgs g;                                       // (g.W null: no product)
};

template <int NJ, int STORE, int WT>
__global__ __launch_bounds__(256) void k_hop_small(HopArgs a) {
    const uint32_t wave = threadIdx.x >> 6;
    if (blockIdx.x < a.nb_walk) {
        const uint32_t gw = blockIdx.x * 4u + wave, nw = a.nb_walk * 4u;
        frontier_walk<true>(a.list, a.count_ptr, a.eoff, a.out_meta, a.out_pool, nullptr, a.sp, gw, nw);
        enter_roots(a.list, a.count_ptr, a.sp, gw, nw);
    } else if (blockIdx.x < a.nb_walk + a.nb_push) {
        if (blockIdx.x == a.nb_walk && threadIdx.x == 0 && a.count_ptr[1]) a.ctr->hop_mode[a.l] = 1u + RP_HOP_PUSH;
        push_edges<NJ, 0, WT>(a.list, a.count_ptr, a.eoff, a.D, nullptr, 0u, a.ldd, a.d, a.out_meta, a.out_pool, a.out_w, a.X,
                              (blockIdx.x - a.nb_walk) * 4u + wave, a.nb_push * 4u);
    } else {
        wave_gemm<4, STORE>(a.g, (blockIdx.x - a.nb_walk - a.nb_push) * 4u + wave, (gridDim.x - a.nb_walk - a.nb_push) * 4u);
    }
}

// messages of a project-first layer (PD: projected rows, T: what has been sent)
template <int NJ, int WT>
__global__ __launch_bounds__(256) void k_push_projected(HopArgs a, const float *PD, const float *T, uint32_t ldt, int packed) {
    if (blockIdx.x == 0 && threadIdx.x == 0 && a.count_ptr[1]) a.ctr->hop_mode[a.l] = 1u + RP_HOP_PUSH;
    push_edges<NJ, 2, WT>(a.list, a.count_ptr, a.eoff, PD, T, ldt, a.ldd, a.d, a.out_meta, a.out_pool, a.out_w, a.X, blockIdx.x * 4u + (threadIdx.x >> 6),
                          gridDim.x * 4u, packed != 0);
}

// Hop l from hints of the previous batch (the caller has made sure that they call for it): everything up to the row update,
// which the caller launches (rp_launch_small_addend for a project-first layer without a product left per row).
void rp_launch_hop_small(ripple_ctx *c, uint32_t l, bool self_term) {
    const LayerDev &ly = c->layers[l - 1];
    const uint32_t rows = c->last_a[l - 1], msgs = c->last_m[l];
    HopArgs a;
    a.list = c->list[l - 1];
    a.count_ptr = &c->ctr->set[l - 1].a;
    a.eoff = c->eoff[l - 1];
    a.out_meta = c->out_meta;
    a.out_pool = c->out_pool;
    a.out_w = ly.agg == RIPPLE_AGG_WSUM ? c->out_w : nullptr;
    a.sp = rp_sparse_args(c, l, c->list[l], &c->ctr->set[l].a, self_term);
    a.sp.eoff = c->eoff[l];
    a.d = c->xw[l];
    a.X = c->X[l];
    a.ctr = c->ctr;
    a.l = l;
    a.D = ly.proj ? nullptr : c->D[(l - 1) & 1];
    a.ldd = ly.proj ? c->pd_ld : a.d;
    a.nb_walk = std::min(16u + msgs / 128u, c->n_cu);
    const uint32_t nb_push = std::min(8u + msgs / (msgs <= 2048u ? 16u : 48u), c->n_cu * 4);
    a.nb_push = ly.proj ? 0u : nb_push;
    const bool both = rp_has_project_both(c, l);
    uint32_t nb_gemm = 0;
    a.g.W = nullptr;
    if (ly.proj || ly.selfc) {
        a.g = both ? rp_project_both_args(c, l, a.list, a.count_ptr, false)
                   : (ly.proj ? rp_project_args(c, l, a.list, a.count_ptr, false) : rp_self_project_args(c, l, a.list, a.count_ptr));
        if (c->opt_split || wave_gemm_waves(a.g, rows) > WAVE_GEMM_MAX) {   // many rows: launches of their own
            if (both) {
                rp_launch_project_both(c, l, a.list, a.count_ptr, false);
            } else {
                if (ly.proj) rp_launch_project(c, l, a.list, a.count_ptr, false);
                if (ly.selfc) rp_launch_self_project(c, l, a.list, a.count_ptr);
            }
            a.g.W = nullptr;
        } else {
            if (ly.proj && ly.selfc && !both) rp_launch_self_project(c, l, a.list, a.count_ptr);
            nb_gemm = std::min(rp_div_up(wave_gemm_waves(a.g, rows + rows / 2u), 4), c->n_cu * 2);
        }
    }
    const dim3 grid(a.nb_walk + a.nb_push + nb_gemm), block(256);
#define HOP_CASE(NJ)                                                                                    \
    do {                                                                                                \
        if (a.out_w && c->store) hipLaunchKernelGGL((k_hop_small<NJ, 1, 1>), grid, block, 0, c->stream, a); \
        else if (a.out_w) hipLaunchKernelGGL((k_hop_small<NJ, 0, 1>), grid, block, 0, c->stream, a);    \
        else if (c->store) hipLaunchKernelGGL((k_hop_small<NJ, 1, 0>), grid, block, 0, c->stream, a);   \
        else hipLaunchKernelGGL((k_hop_small<NJ, 0, 0>), grid, block, 0, c->stream, a);                 \
    } while (0)
    if (a.d <= 64) HOP_CASE(1);
    else if (a.d <= 128) HOP_CASE(2);
    else if (a.d <= 256) HOP_CASE(4);
    else if (a.d <= 512) HOP_CASE(8);
    else HOP_CASE(16);
#undef HOP_CASE
    if (!ly.proj) return;
#define PUSH_CASE(NJ)                                                                                                                     \
    do {                                                                                                                                  \
        if (a.out_w) hipLaunchKernelGGL((k_push_projected<NJ, 1>), dim3(nb_push), block, 0, c->stream, a, c->PD, ly.T, ly.ldt, (int)ly.packed);   \
        else hipLaunchKernelGGL((k_push_projected<NJ, 0>), dim3(nb_push), block, 0, c->stream, a, c->PD, ly.T, ly.ldt, (int)ly.packed);           \
    } while (0)
    if (a.d <= 64) PUSH_CASE(1);
    else if (a.d <= 128) PUSH_CASE(2);
    else if (a.d <= 256) PUSH_CASE(4);
    else PUSH_CASE(8);                                     // project-first layers at least halve the row: at most 512 columns
#undef PUSH_CASE
}
