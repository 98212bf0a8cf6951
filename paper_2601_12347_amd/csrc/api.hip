// C ABI of the library: context lifetime, model upload, bootstrap inference,
// the per-batch driver (host-side validation and conflict splitting, then the
// device pipeline Apply -> per layer {frontier, scatter, transform}), and the
// read-back calls the tests use.
#include "common.h"
#include "kernels.h"
#include "pull_scan.h"
#include "transform_args.h"

#include <chrono>
#include <cmath>
#include <cstring>
#include <new>

// ---------------------------------------------------------------------------------
// timing
// ---------------------------------------------------------------------------------
struct PhaseTimer {
    struct Rec {
        int phase, layer, e0, e1, counted;
    };
    std::vector<hipEvent_t> ev;
    std::vector<Rec> recs;
    int used = 0;
    int get(ripple_ctx *c) {
        if (used == (int)ev.size()) {
            hipEvent_t e;
            if (hipEventCreate(&e) != hipSuccess) return -1;
            ev.push_back(e);
        }
        return used++;
    }
};

int rp_timer_begin(ripple_ctx *c) {
    if (!c->opt_timing) return -1;
    int e = c->timer->get(c);
    if (e >= 0) hipEventRecord(c->timer->ev[e], c->stream);
    return e;
}

// counted = false: a second stretch of a phase already recorded for this hop (adds time, not a launch)
void rp_timer_end(ripple_ctx *c, int token, int phase, int layer, bool counted) {
    if (token < 0) return;
    int e = c->timer->get(c);
    if (e < 0) return;
    hipEventRecord(c->timer->ev[e], c->stream);
    c->timer->recs.push_back({phase, layer, token, e, counted ? 1 : 0});
}

static void timer_collect(ripple_ctx *c) {       // after the stream has been synchronised
    PhaseTimer *t = c->timer;
    for (const auto &r : t->recs) {
        float ms = 0.f;
        if (hipEventElapsedTime(&ms, t->ev[r.e0], t->ev[r.e1]) == hipSuccess) {
            c->stats.ms[r.phase][r.layer] += ms;
            c->stats.launches[r.phase][r.layer] += r.counted;
        }
    }
    t->recs.clear();
    t->used = 0;
}

// ---------------------------------------------------------------------------------
// small kernels
// ---------------------------------------------------------------------------------
__global__ void k_store_rows(const float *src, void *dst, size_t n, int store) {
    size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        if (store) ((__hip_bfloat16 *)dst)[i] = __float2bfloat16(src[i]);
        else ((float *)dst)[i] = src[i];
    }
}

// Rows of H (or X) as float32, four numbers per thread: bound by memory, so the rows' own widths decide the accesses (a row
// of 47 floats starts at any multiple of 4 bytes; 16-byte accesses take those), and `out` may be the caller's device
// memory or pinned host memory: nothing is written twice. (One number per thread into a staging array that was then copied:
// 0.54 ms for 2.45 M rows of 47; now 0.26.)
typedef float gfloatx4u __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t guintx2u __attribute__((ext_vector_type(2), aligned(2)));
// groups of four numbers i0, i0 + stride, ... of rows ids[0 .. n_rows) (no ids: first .. first + n_rows - 1)
template <int STORE>
__device__ __forceinline__ void gather_groups(const void *M, uint32_t d, const uint32_t *ids, uint32_t first, size_t n_rows, uint32_t n_cap, float *out,
                                              size_t i0, size_t stride) {
    const uint32_t groups = (d + 3u) / 4u;                   // of four numbers; a row's last one may be short
    const size_t total = n_rows * groups;
    for (size_t i = i0; i < total; i += stride) {
        const size_t r = total <= 0xFFFFFFFFull ? (size_t)((uint32_t)i / groups) : i / groups;
        const uint32_t col = (uint32_t)(i - r * groups) * 4u;
        const uint32_t id = ids ? ids[r] : (uint32_t)(first + r);
        gfloatx4u v = (gfloatx4u)(0.0f);
        if (id < n_cap) {                                    // up to three numbers past the row: the arrays have room behind them
            const size_t at = (size_t)id * d + col;
            if (STORE) {
                const guintx2u w = *(const guintx2u *)((const __hip_bfloat16 *)M + at);
                v.x = __uint_as_float(w.x << 16);
                v.y = __uint_as_float(w.x & 0xFFFF0000u);
                v.z = __uint_as_float(w.y << 16);
                v.w = __uint_as_float(w.y & 0xFFFF0000u);
            } else {
                v = *(const gfloatx4u *)((const float *)M + at);
            }
        }
        float *o = out + r * d + col;
        if (col + 4u <= d) {
            *(gfloatx4u *)o = v;
        } else {
            o[0] = v.x;
            if (col + 1u < d) o[1] = v.y;
            if (col + 2u < d) o[2] = v.z;
        }
    }
}
template <int STORE>
__global__ __launch_bounds__(256) void k_gather_rows(const void *M, uint32_t d, const uint32_t *ids, uint32_t first,
                                                     size_t n_rows, uint32_t n_cap, float *out, HostFlag done) {
    gather_groups<STORE>(M, d, ids, first, n_rows, n_cap, out, (size_t)blockIdx.x * 256u + threadIdx.x, (size_t)gridDim.x * 256u);
    report_done(done, gridDim.x);
}

// The same into pinned memory in pieces of `piece` rows, each at the front of READ_FLOATS numbers of its own; when piece p is there, `seq` goes to the word
// 64 * p bytes behind `flags`. Teams of PIECE_WGS workgroups take the pieces in turn (their 16,384 threads a piece's groups of four at once), so that one
// piece is on its way while the other team waits for its own to have arrived. `arrived`: a counter per piece, zero between launches.
#define PIECE_WGS 64u
#define PIECE_TEAMS 2u
template <int STORE>
__global__ __launch_bounds__(256) void k_gather_pieces(const void *M, uint32_t d, const uint32_t *ids, uint32_t first, uint32_t n_rows, uint32_t piece, uint32_t n_cap,
                                                       float *out, uint32_t *flags, uint32_t seq, uint32_t *arrived) {
    const uint32_t team = blockIdx.x / PIECE_WGS, wg = blockIdx.x % PIECE_WGS, n_pieces = (n_rows + piece - 1u) / piece;
    for (uint32_t p = team; p < n_pieces; p += PIECE_TEAMS) {
        const uint32_t r0 = p * piece;
        gather_groups<STORE>(M, d, ids ? ids + r0 : nullptr, first + r0, min(piece, n_rows - r0), n_cap, out + (size_t)p * READ_FLOATS, wg * 256u + threadIdx.x, PIECE_WGS * 256u);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");    // this wavefront's stores have been performed
        __syncthreads();
        if (threadIdx.x == 0) {
            __threadfence_system();
            if (atomicAdd(&arrived[p], 1u) == PIECE_WGS - 1u) {
                arrived[p] = 0;
                __hip_atomic_store(flags + 16u * p, seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
            }
        }
    }
}

// Numbers (or any 4-byte words) from one place to another, four per thread and load, four loads under way: whole tables on the device, and operations
// that are handed over on the device to the host. `from` and `to` start at multiples of four bytes.
__global__ __launch_bounds__(256) void k_copy_numbers(const float *from, float *to, size_t n, HostFlag done) {
    const size_t stride = (size_t)gridDim.x * 1024u, quads = n / 4u;
    for (size_t q0 = (size_t)blockIdx.x * 1024u + threadIdx.x; q0 < quads; q0 += stride) {
        gfloatx4u v[4];
#pragma unroll
        for (uint32_t k = 0; k < 4; ++k) v[k] = *(const gfloatx4u *)(from + 4u * min(q0 + 256u * k, quads - 1u));
#pragma unroll
        for (uint32_t k = 0; k < 4; ++k)
            if (q0 + 256u * k < quads) *(gfloatx4u *)(to + 4u * (q0 + 256u * k)) = v[k];
    }
    if (blockIdx.x == 0 && threadIdx.x < n % 4u) to[quads * 4u + threadIdx.x] = from[quads * 4u + threadIdx.x];
    report_done(done, gridDim.x);
}

__global__ void k_or_words(uint32_t *dst, const uint32_t *src, uint32_t n) {
    uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n && src[i]) dst[i] |= src[i];
}

__global__ void k_meta_len2(const uint2 *meta, uint32_t n_cap, uint32_t *len) {
    uint32_t v = blockIdx.x * blockDim.x + threadIdx.x;
    if (v < n_cap) len[v] = meta[v].y;
}

__global__ __launch_bounds__(256) void k_export_rows(const uint2 *meta, const uint32_t *pool, const uint32_t *off,
                                                     uint32_t n_cap, int direction, uint32_t *src_out,
                                                     uint32_t *dst_out) {
    const int lane = rp_lane();
    uint32_t gw = (blockIdx.x * blockDim.x + threadIdx.x) >> 6, nw = (gridDim.x * blockDim.x) >> 6;
    for (uint32_t v = gw; v < n_cap; v += nw) {
        uint2 m = meta[v];
        uint32_t o = off[v];
        for (uint32_t i = lane; i < m.y; i += 64) {
            uint32_t nb = pool[m.x + i];
            src_out[o + i] = direction ? nb : v;
            dst_out[o + i] = direction ? v : nb;
        }
    }
}

// ---------------------------------------------------------------------------------
// helpers
// ---------------------------------------------------------------------------------
// where a caller's memory is; a kernel of this context writes to FAR_GPU memory only with peer access
enum Place { ON_HOST, OWN_GPU, FAR_GPU };
static Place place_of(const ripple_ctx *c, const void *p) {
    hipPointerAttribute_t at;
    hipError_t e = hipPointerGetAttributes(&at, p);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        return ON_HOST;
    }
    if (at.type == hipMemoryTypeManaged) return OWN_GPU;
    return at.type != hipMemoryTypeDevice ? ON_HOST : (at.device == c->device ? OWN_GPU : FAR_GPU);
}
static bool is_device_ptr(const ripple_ctx *c, const void *p) { return place_of(c, p) != ON_HOST; }

#define RP_TRY(expr)                         \
    do {                                     \
        ripple_status rc__ = (expr);         \
        if (rc__ != RIPPLE_OK) return rc__;  \
    } while (0)

// every array has 16 bytes behind its end: the row transforms read rows in groups of four numbers
#define ARRAY_PAD 16
template <typename T>
static ripple_status dev_alloc(ripple_ctx *c, T **p, size_t count, bool zero) {
    size_t bytes = (count ? count : 1) * sizeof(T) + ARRAY_PAD;
    hipError_t e = hipMalloc((void **)p, bytes);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        c->err = "device allocation of " + std::to_string(bytes) + " bytes failed";
        *p = nullptr;
        return RIPPLE_ENOMEM;
    }
    if (zero) RP_HIP(c, hipMemsetAsync(*p, 0, bytes, c->stream));
    return RIPPLE_OK;
}

// Arrays that live and die together, in one allocation: hipMalloc of a few megabytes takes 50 to 300 us and every clearing memset
// is a launch, so a context of a small graph spent most of its preparation and half of its first batch on them.
struct Block {
    struct Part {
        void *p;                                             // where the array's address goes
        size_t at;
    } part[32];
    uint32_t n = 0;
    size_t bytes = 0;
    template <typename T>
    void add(T **p, size_t count) {
        part[n++] = {p, bytes};
        bytes += (std::max<size_t>(count, 1) * sizeof(T) + ARRAY_PAD + 255) & ~(size_t)255;
    }
};
static ripple_status block_alloc(ripple_ctx *c, const Block &b, uint8_t **base, bool zero) {
    RP_TRY(dev_alloc(c, base, b.bytes, zero));
    for (uint32_t i = 0; i < b.n; ++i) {
        void *at = *base + b.part[i].at;
        memcpy(b.part[i].p, &at, sizeof(at));
    }
    return RIPPLE_OK;
}

// What the host reads goes through pinned memory that the kernels write themselves (and read ids from). Rows leave in pieces of at most
// READ_FLOATS numbers: one launch writes up to READ_PIECES of them one after the other and says so after each, and while it writes the next ones the
// host copies; reads of more pieces take the two halves in turn. A read so takes little more than the slower of the two (kernels write to the host
// at 50 GB/s, a copy out of the pinned memory runs at 30 to 42). Rows of 47 numbers by ids, the runtime's copy to pageable memory / this, us: 66 K
// numbers 40 / 26, 235 K 67 / 59, 1.2 M 304 / 187, 9.4 M 2,249 / 1,407; 4 x 40 K to 4 x 300 K numbers behind a batch 76 to 319 / 43 to 186.
#define IO_PIN_IDS 131072u
// operations and feature rows of a batch that the pinned block has room for; larger batches get staging of their own
#define PIN_OPS 6144u
#define PIN_ROWS 1024u

static ripple_status fail(ripple_ctx *c, ripple_status rc, const char *msg);

HostFlag rp_host_flag(ripple_ctx *c) { return HostFlag{c->pub_flag, ++c->pub_seq, c->ctr}; }

// Waits until the launch that was given the last rp_host_flag has reported: it is the stream's last kernel, so the kernels before
// it have finished, and what it and they wrote is visible. Looking at a word of pinned memory costs less than a wait for the
// stream, which goes over every launch since the last one (a batch of twenty launches: 63 against 90 us). What takes longer than
// the limit gets the stream wait, which also is what reports a device error.
#define WAIT_SPIN_US 2000.0
static ripple_status wait_word(ripple_ctx *c, const uint32_t *word, uint32_t value) {
    RP_HIP(c, hipGetLastError());
    const auto t0 = std::chrono::steady_clock::now();
    for (uint32_t k = 0; __atomic_load_n(word, __ATOMIC_ACQUIRE) != value; ++k) {
        __builtin_ia32_pause();
        if ((k & 255u) == 255u && std::chrono::duration<double, std::micro>(std::chrono::steady_clock::now() - t0).count() > WAIT_SPIN_US) {
            RP_HIP(c, hipStreamSynchronize(c->stream));
            break;
        }
    }
    if (__atomic_load_n(word, __ATOMIC_ACQUIRE) != value) return fail(c, RIPPLE_EDEVICE, "a kernel did not report its end");
    return RIPPLE_OK;
}
ripple_status rp_wait_flag(ripple_ctx *c) { return wait_word(c, c->pub_flag, c->pub_seq); }

static size_t elem_size(const ripple_ctx *c) { return c->store ? 2 : 4; }

static ripple_status fail(ripple_ctx *c, ripple_status rc, const char *msg) {
    c->err = msg;
    return rc;
}

// ---------------------------------------------------------------------------------
// init / destroy
// ---------------------------------------------------------------------------------
static ripple_status init_graph(ripple_ctx **out, uint32_t n_vertices, uint32_t vertex_capacity, uint64_t n_edges,
                                uint64_t edge_capacity, const uint32_t *src, const uint32_t *dst, const float *weights,
                                const float *features, uint32_t d0, int store, void *hip_stream) {
    if (!out) return RIPPLE_EINVAL;
    *out = nullptr;
    if (vertex_capacity == 0 || n_vertices > vertex_capacity || vertex_capacity > (1u << 31) || d0 == 0 ||
        d0 > 1024 || n_edges > edge_capacity || (store != RIPPLE_STORE_F32 && store != RIPPLE_STORE_BF16) ||
        (n_edges && (!src || !dst)) || (n_vertices && !features))
        return RIPPLE_EINVAL;
    uint64_t pool_cap = edge_capacity + edge_capacity / 4 + 8ull * vertex_capacity + 1024;
    if (pool_cap >= (1ull << 32)) return RIPPLE_EINVAL;
    ripple_ctx *c = new (std::nothrow) ripple_ctx();
    if (!c) return RIPPLE_ENOMEM;
    *out = c;                                   // returned even on failure so that the error text can be read
    c->timer = new (std::nothrow) PhaseTimer();
    memset(&c->stats, 0, sizeof(c->stats));
    c->stream = (hipStream_t)hip_stream;
    RP_HIP(c, hipGetDevice(&c->device));
    RP_TRY(rp_static_scratch_init(c));
    RP_HIP(c, hipEventCreateWithFlags(&c->idle, hipEventDisableTiming));
    int cu = 0;
    RP_HIP(c, hipDeviceGetAttribute(&cu, hipDeviceAttributeMultiprocessorCount, c->device));
    c->n_cu = cu > 0 ? (uint32_t)cu : 256u;
    c->n_cap = vertex_capacity;
    c->n_words = rp_div_up(vertex_capacity, 32);
    c->e_cap = edge_capacity;
    c->pool_cap = pool_cap;
    c->store = store;
    c->d[0] = d0;
    const size_t n = c->n_cap;
    Block g;
    g.add(&c->out_meta, n);
    g.add(&c->in_meta, n);
    g.add(&c->out_capv, n);
    g.add(&c->in_capv, n);
    g.add(&c->vstate, n);
    g.add(&c->pend_out, n);
    g.add(&c->pend_in, n);
    g.add(&c->dead_out, n);
    g.add(&c->dead_in, n);
    g.add(&c->hole_out, n);
    g.add(&c->hole_in, n);
    g.add(&c->alive, (size_t)c->n_words);
    c->n_part = std::max(rp_div_up(n, 1024), rp_div_up(c->n_words, 256)) + 1;
    g.add(&c->part_cnt, (size_t)c->n_part);
    g.add(&c->part_deg, (size_t)c->n_part);
    g.add(&c->part_ideg, (size_t)c->n_part);
    g.add(&c->part_tch, (size_t)c->n_part);
    g.add(&c->part_rec, (size_t)c->n_part);
    g.add(&c->ctr, 1);
    RP_TRY(block_alloc(c, g, &c->graph_block, true));
    RP_TRY(dev_alloc(c, &c->out_pool, (size_t)pool_cap, false));
    RP_TRY(dev_alloc(c, &c->in_pool, (size_t)pool_cap, false));
    if (weights) {
        RP_TRY(dev_alloc(c, &c->in_w, (size_t)pool_cap, false));
        RP_TRY(dev_alloc(c, &c->out_w, (size_t)pool_cap, false));
    }
    {   // pinned memory, in one allocation (200 to 300 us each, whatever the size): counters, the flag, the staging of ordinary batches, read-back.
        // The room for rows comes last: what every batch uses lies close together (with 4 MB in between, the first batch took 10 to 50 us longer)
        const size_t ctr_at = 0, flag_at = (sizeof(DevCtr) + 63) & ~(size_t)63, piece_at = flag_at + 64, made_at = piece_at + 2 * READ_PIECES * 64;
        const size_t ops_at = made_at + SMALL_OPS * 4, rows_at = ops_at + PIN_OPS * sizeof(ripple_update), io_at = rows_at + (size_t)PIN_ROWS * d0 * 4;
        c->pin_bytes = io_at + (16 + IO_PIN_IDS + 2 * READ_PIECES * READ_FLOATS) * 4;
        RP_HIP(c, hipHostMalloc((void **)&c->pin_block, c->pin_bytes, hipHostMallocDefault));
        c->ctr_host = (DevCtr *)(c->pin_block + ctr_at);
        c->pub_flag = (uint32_t *)(c->pin_block + flag_at);
        c->io_pin = (uint32_t *)(c->pin_block + io_at);
        c->made_pin = (uint32_t *)(c->pin_block + made_at);
        c->ops_pin = (ripple_update *)(c->pin_block + ops_at);
        c->payload_pin = (float *)(c->pin_block + rows_at);
        c->pin_ops_cap = PIN_OPS;
        c->feat_cap = PIN_ROWS;
        memset(c->ctr_host, 0, sizeof(DevCtr));
        *c->pub_flag = 0;
        c->read_flag = (uint32_t *)(c->pin_block + piece_at);
        memset(c->read_flag, 0, 2 * READ_PIECES * 64);
    }
    {   // features
        void *h0 = nullptr;
        size_t bytes = n * d0 * elem_size(c);
        hipError_t e = hipMalloc(&h0, bytes + ARRAY_PAD);
        if (e != hipSuccess) return fail(c, RIPPLE_ENOMEM, "device allocation of the feature matrix failed");
        c->H[0] = h0;
        RP_HIP(c, hipMemsetAsync(h0, 0, bytes, c->stream));
        if (n_vertices) {
            size_t cnt = (size_t)n_vertices * d0;
            if (store == RIPPLE_STORE_F32) {
                RP_HIP(c, hipMemcpyAsync(h0, features, cnt * 4, hipMemcpyHostToDevice, c->stream));
            } else {
                float *tmp = nullptr;
                RP_TRY(dev_alloc(c, &tmp, cnt, false));
                RP_HIP(c, hipMemcpyAsync(tmp, features, cnt * 4, hipMemcpyHostToDevice, c->stream));
                hipLaunchKernelGGL(k_store_rows, dim3(c->n_cu * 8), dim3(256), 0, c->stream, tmp, h0, cnt, 1);
                RP_HIP(c, hipStreamSynchronize(c->stream));
                hipFree(tmp);
            }
        }
    }
    RP_TRY(rp_build_graph(c, n_vertices, n_edges, src, dst, weights));
    // counters that persist across batches
    c->ctr_host->n_alive = n_vertices;
    c->ctr_host->n_edges = n_edges;
    RP_HIP(c, hipMemcpyAsync(&c->ctr->n_alive, &c->ctr_host->n_alive, 4, hipMemcpyHostToDevice, c->stream));
    RP_HIP(c, hipMemcpyAsync(&c->ctr->n_edges, &c->ctr_host->n_edges, 8, hipMemcpyHostToDevice, c->stream));
    RP_HIP(c, hipStreamSynchronize(c->stream));
    c->state = 1;
    return RIPPLE_OK;
}

extern "C" ripple_status ripple_init_graph(ripple_ctx **out, uint32_t n_vertices, uint32_t vertex_capacity,
                                           uint64_t n_edges, uint64_t edge_capacity, const uint32_t *src,
                                           const uint32_t *dst, const float *features, uint32_t d0, int store,
                                           void *hip_stream) {
    return init_graph(out, n_vertices, vertex_capacity, n_edges, edge_capacity, src, dst, nullptr, features, d0, store,
                      hip_stream);
}

extern "C" ripple_status ripple_init_graph_weighted(ripple_ctx **out, uint32_t n_vertices, uint32_t vertex_capacity,
                                                    uint64_t n_edges, uint64_t edge_capacity, const uint32_t *src,
                                                    const uint32_t *dst, const float *edge_weights,
                                                    const float *features, uint32_t d0, int store, void *hip_stream) {
    if (!edge_weights) return RIPPLE_EINVAL;
    return init_graph(out, n_vertices, vertex_capacity, n_edges, edge_capacity, src, dst, edge_weights, features, d0,
                      store, hip_stream);
}

// staging that has not been replaced by a larger one of its own
static bool in_pin_block(const ripple_ctx *c, const void *p) {
    const uint8_t *q = (const uint8_t *)p, *end = c->pin_block + c->pin_bytes;
    return c->pin_block && q >= c->pin_block && q < end;
}

extern "C" void ripple_destroy(ripple_ctx *c) {
    if (!c) return;
    hipStreamSynchronize(c->stream);
    void *ptrs[] = {c->graph_block, c->list_block, c->batch_block, c->pair_block, c->part_block, c->out_pool, c->in_pool, c->in_w, c->out_w, c->D[0], c->D[1], c->tmp, c->PD,
                    c->MSG, c->side_v, c->side_acc, c->Pold, c->sold, c->gat_mag, c->gat_rec, c->seg_block, c->gather_d, c->gather_ids};
    for (void *p : ptrs)
        if (p) hipFree(p);
    for (uint32_t l = 0; l <= RIPPLE_MAX_LAYERS; ++l) {
        if (c->H[l]) hipFree(c->H[l]);
        if (c->X[l]) hipFree(c->X[l]);
    }
    for (uint32_t l = 0; l < c->L; ++l) {
        LayerDev &ly = c->layers[l];
        void *w[] = {ly.W0, ly.b0, ly.W1, ly.b1, ly.W0h, ly.W1h, ly.bzero, (ly.Wn != ly.W0) ? ly.Wn : nullptr, ly.PS,
                     ly.att, ly.P, ly.ssrc, ly.sdst, ly.den, ly.T, ly.Wc, ly.bzero_c, ly.W0q, (ly.Wnq != ly.W0q) ? ly.Wnq : nullptr, ly.W1q, ly.Wcq};
        for (void *p : w)
            if (p) hipFree(p);
    }
    if (c->ops_pin && !in_pin_block(c, c->ops_pin)) hipHostFree(c->ops_pin);
    if (c->payload_pin && !in_pin_block(c, c->payload_pin)) hipHostFree(c->payload_pin);
    if (c->pin_block) hipHostFree(c->pin_block);
    if (c->idle) hipEventDestroy(c->idle);
    if (c->timer) {
        for (hipEvent_t e : c->timer->ev) hipEventDestroy(e);
        delete c->timer;
    }
    delete c;
}

extern "C" const char *ripple_last_error(const ripple_ctx *c) { return c ? c->err.c_str() : ""; }

// ---------------------------------------------------------------------------------
// model
// ---------------------------------------------------------------------------------
static uint32_t pad_n(uint32_t n) { return n <= 64 ? 64u : (n <= 128 ? 128u : rp_round_up(n, 256)); }

// The padded matrix [Kpad x Npad] with k by fours (wave_gemm reads four consecutive k of a column at once), made on the device from
// the one that was uploaded: rearranged and copied by the host, the second layout took a quarter of ripple_load_model.
__global__ void k_quads(const float *w, float *q, uint32_t n, uint32_t Npad) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const uint32_t t = i & 3u, j = (i >> 2) % Npad, k4 = (i >> 2) / Npad;
    q[i] = w[(size_t)(4u * k4 + t) * Npad + j];
}
static ripple_status make_quads(ripple_ctx *c, const float *w, uint32_t Kpad, uint32_t Npad, float **out) {
    const uint32_t n = Kpad * Npad;                          // (at most 2048 x 1024; Kpad is a multiple of 32)
    RP_TRY(dev_alloc(c, out, n, false));
    hipLaunchKernelGGL(k_quads, dim3(rp_div_up(n, 256)), dim3(256), 0, c->stream, w, *out, n, Npad);
    return RIPPLE_OK;
}

static ripple_status upload_padded(ripple_ctx *c, const float *w, const float *b, uint32_t K, uint32_t N,
                                   uint32_t Kpad, uint32_t Npad, float **W_d, float **b_d, float **Wq_d) {
    std::vector<float> wp((size_t)Kpad * Npad, 0.0f), bp(Npad, 0.0f);
    for (uint32_t k = 0; k < K; ++k) memcpy(&wp[(size_t)k * Npad], &w[(size_t)k * N], (size_t)N * 4);
    memcpy(bp.data(), b, (size_t)N * 4);
    RP_TRY(dev_alloc(c, W_d, wp.size(), false));
    RP_TRY(dev_alloc(c, b_d, bp.size(), false));
    RP_HIP(c, hipMemcpy(*W_d, wp.data(), wp.size() * 4, hipMemcpyHostToDevice));
    RP_TRY(make_quads(c, *W_d, Kpad, Npad, Wq_d));
    RP_HIP(c, hipMemcpy(*b_d, bp.data(), bp.size() * 4, hipMemcpyHostToDevice));
    return RIPPLE_OK;
}

// Device scratch for batches of n_ops operations and want_exp edges of deleted vertices; what is there already is not made smaller
static ripple_status grow_scratch(ripple_ctx *c, uint32_t n_ops, uint32_t want_exp) {
    if (n_ops <= c->ops_cap && want_exp <= c->exp_cap) return RIPPLE_OK;
    RP_HIP(c, hipStreamSynchronize(c->stream));
    const uint32_t cap = n_ops <= c->ops_cap ? c->ops_cap : rp_round_up(n_ops <= PIN_OPS ? PIN_OPS : n_ops + n_ops / 2, 1024);
    const uint32_t exp = std::max(want_exp, c->exp_cap);
    if (c->batch_block) hipFree(c->batch_block);
    c->batch_block = nullptr;
    c->ops_cap = c->exp_cap = c->touch_cap = c->struct_cap = 0;
    const size_t both = (size_t)cap + exp, entries = 2 * (size_t)cap + exp;
    Block b;
    b.add(&c->ops_d, cap);
    b.add(&c->op_status, cap);
    b.add(&c->op_pos_out, cap);
    b.add(&c->op_pos_in, cap);
    b.add(&c->op_touch, cap);
    b.add(&c->op_rank_out, cap);
    b.add(&c->op_rank_in, cap);
    b.add(&c->touch_out, both);
    b.add(&c->touch_in, both);
    b.add(&c->exp_kind, exp);
    b.add(&c->exp_pos, exp);
    b.add(&c->exp_rank, exp);
    b.add(&c->exp_a, exp);
    b.add(&c->exp_b, exp);
    b.add(&c->st_src, both);
    b.add(&c->st_dst, both);
    b.add(&c->st_sign, both);
    b.add(&c->st_unit, both);
    b.add(&c->seg_id, entries);
    b.add(&c->seg_x, entries);
    if (c->opt_deterministic) {
        b.add(&c->srt_id, entries);
        b.add(&c->srt_x, entries);
    }
    RP_TRY(block_alloc(c, b, &c->batch_block, false));
    c->ops_cap = cap;
    c->exp_cap = exp;
    c->touch_cap = c->struct_cap = (uint32_t)both;
    return RIPPLE_OK;
}

// Pinned staging for n_ops operations and n_feat feature rows. Not to be called while a piece is under way: it reads them.
static ripple_status grow_staging(ripple_ctx *c, uint32_t n_ops, uint32_t n_feat) {
    if (n_ops <= c->pin_ops_cap && n_feat <= c->feat_cap) return RIPPLE_OK;
    RP_HIP(c, hipStreamSynchronize(c->stream));
    if (n_ops > c->pin_ops_cap) {
        if (c->ops_pin && !in_pin_block(c, c->ops_pin)) hipHostFree(c->ops_pin);
        c->ops_pin = nullptr;
        c->pin_ops_cap = 0;
        const uint32_t cap = rp_round_up(n_ops + n_ops / 2, 1024);
        RP_HIP(c, hipHostMalloc((void **)&c->ops_pin, (size_t)cap * sizeof(ripple_update), hipHostMallocDefault));
        c->pin_ops_cap = cap;
    }
    if (n_feat > c->feat_cap) {
        if (c->payload_pin && !in_pin_block(c, c->payload_pin)) hipHostFree(c->payload_pin);
        c->payload_pin = nullptr;
        c->feat_cap = 0;
        const uint32_t cap = rp_round_up(n_feat + n_feat / 2, 256);
        RP_HIP(c, hipHostMalloc((void **)&c->payload_pin, (size_t)cap * c->d[0] * 4, hipHostMallocDefault));
        c->feat_cap = cap;
    }
    return RIPPLE_OK;
}

// A matrix whose numbers are all below 2^-40 is lifted by 2^64 before it is split into bf16 parts (see PARTS_LIFT)
static float weight_lift(const float *w, size_t n) {
    float most = 0.0f;
    for (size_t i = 0; i < n; ++i)
        if (std::isfinite(w[i])) most = std::max(most, std::fabs(w[i]));
    return most < std::ldexp(1.0f, -40) ? std::ldexp(1.0f, 64) : 1.0f;
}

// Row stride of what vertices have sent (LayerDev::T), d columns. Every in-edge of the bootstrap gathers such a row, so what counts is how many lines of 128
// bytes a row touches (47 numbers at any multiple of four bytes 2.4 on average, at multiples of 64 bytes two: 31 M edges 1,172 / 950 us), and how much of
// the table the caches hold. Rows begin at multiples of 32 or 64 bytes where a tenth of the lines is saved, else one behind the other. Bootstrap of
// one layer, 600 K vertices, 20 M edges, us, unpadded / at multiples of 64 bytes:
//   2 columns 359 / 520, 3 400 / 525, 8 480 / 518 (the larger table misses); 6 columns 510 / 532, at multiples of 32 bytes 487;
//   10 columns 586 / 541, 13 652 / 544, 20 687 / 578, 23 778 / 592; 72 columns 1,530 / 1,537, 100 1,943 / 1,962 (no line saved).
static uint32_t sent_row_stride(uint32_t d) {
    auto lines = [d](uint32_t stride) {                  // of 32 rows, behind which the offsets repeat
        uint32_t n = 0;
        for (uint32_t r = 0; r < 32; ++r) n += (r * stride % 32u + d + 31u) / 32u;
        return n;
    };
    uint32_t best = d;
    for (uint32_t unit = 8; unit <= 16; unit *= 2)
        if (10u * lines(rp_round_up(d, unit)) <= 9u * lines(best)) best = rp_round_up(d, unit);
    return best;
}

extern "C" ripple_status ripple_load_model(ripple_ctx *c, uint32_t n_layers, const ripple_layer_desc *layers) {
    if (!c) return RIPPLE_EINVAL;
    if (c->state != 1) return fail(c, RIPPLE_ESTATE, "load_model needs a context fresh from init_graph");
    if (!layers || n_layers == 0 || n_layers > RIPPLE_MAX_LAYERS) return fail(c, RIPPLE_EINVAL, "bad layer count");
    uint32_t prev = c->d[0];
    for (uint32_t l = 0; l < n_layers; ++l) {
        const ripple_layer_desc &s = layers[l];
        if (s.d_in != prev || s.d_out == 0 || s.d_out > 1024 || s.d_hidden > 1024 || s.agg > RIPPLE_AGG_ATTN ||
            s.self_mode > RIPPLE_SELF_ADD || s.act_inner > RIPPLE_ACT_RELU || s.act_out > RIPPLE_ACT_RELU || !s.W0 ||
            !s.b0 || (s.d_hidden && (!s.W1 || !s.b1)))
            return fail(c, RIPPLE_EINVAL, "bad layer descriptor (widths must chain, dims <= 1024, pointers set)");
        if (s.agg == RIPPLE_AGG_WSUM && !c->in_w)
            return fail(c, RIPPLE_EINVAL, "weighted-sum layer on a graph that was built without edge weights");
        if (s.agg == RIPPLE_AGG_ATTN && (!s.att || s.self_mode != RIPPLE_SELF_NONE || s.d_hidden))
            return fail(c, RIPPLE_EINVAL, "attention layer: att must be set, self_mode none, d_hidden 0");
        if ((s.agg == RIPPLE_AGG_WSUM || s.agg >= RIPPLE_AGG_MAX) && c->opt_deterministic)
            return fail(c, RIPPLE_EINVAL, "the deterministic mode takes sum and mean layers only");
        prev = s.d_out;
    }
    c->L = n_layers;
    c->dmax = c->d[0];
    c->hmax = 0;
    for (uint32_t l = 0; l < n_layers; ++l) {
        const ripple_layer_desc &s = layers[l];
        LayerDev &ly = c->layers[l];
        memset(&ly, 0, sizeof(ly));
        ly.d_in = s.d_in;
        ly.d_hidden = s.d_hidden;
        ly.d_out = s.d_out;
        ly.K = (s.self_mode == RIPPLE_SELF_CONCAT) ? 2 * s.d_in : s.d_in;
        ly.agg = s.agg;
        ly.self_mode = s.self_mode;
        ly.act_inner = s.act_inner;
        ly.act_out = s.act_out;
        ly.eps = s.eps;
        uint32_t n0 = s.d_hidden ? s.d_hidden : s.d_out;
        ly.lift0 = weight_lift(s.W0, (size_t)ly.K * n0);
        ly.lift1 = s.d_hidden ? weight_lift(s.W1, (size_t)s.d_hidden * s.d_out) : 1.0f;
        ly.K0pad = rp_round_up(ly.K, 32);
        ly.N0pad = pad_n(n0);
        RP_TRY(upload_padded(c, s.W0, s.b0, ly.K, n0, ly.K0pad, ly.N0pad, &ly.W0, &ly.b0, &ly.W0q));
        if (c->store == RIPPLE_STORE_BF16) {               // transposed bf16 copy for the bf16 matrix cores
            std::vector<uint16_t> wt((size_t)ly.N0pad * ly.K0pad, 0);
            for (uint32_t k = 0; k < ly.K; ++k)
                for (uint32_t j = 0; j < n0; ++j) {
                    uint32_t bits;
                    memcpy(&bits, &s.W0[(size_t)k * n0 + j], 4);
                    bits += 0x7FFFu + ((bits >> 16) & 1u);      // round to nearest even
                    wt[(size_t)j * ly.K0pad + k] = (uint16_t)(bits >> 16);
                }
            RP_TRY(dev_alloc(c, &ly.W0h, wt.size(), false));
            RP_HIP(c, hipMemcpy(ly.W0h, wt.data(), wt.size() * 2, hipMemcpyHostToDevice));
        }
        // project first where the single linear map shrinks the row at least by half
        ly.proj = (c->opt_project && s.agg < RIPPLE_AGG_MAX && s.d_hidden == 0 && s.self_mode != RIPPLE_SELF_ADD && 2 * s.d_out <= s.d_in) ? 1u : 0u;
        ly.selfc = (c->opt_selfcache && s.d_hidden == 0 && s.self_mode == RIPPLE_SELF_CONCAT) ? 1u : 0u;
        if (s.agg == RIPPLE_AGG_ATTN) {
            RP_TRY(dev_alloc(c, &ly.att, (size_t)2 * s.d_out, false));
            RP_HIP(c, hipMemcpy(ly.att, s.att, (size_t)2 * s.d_out * 4, hipMemcpyHostToDevice));
            RP_TRY(dev_alloc(c, &ly.bzero, (size_t)ly.N0pad, true));
            ly.ldp = s.d_out <= 63 ? rp_round_up(s.d_out + 1, 16) : s.d_out;
            RP_TRY(dev_alloc(c, &ly.P, (size_t)c->n_cap * ly.ldp, true));
            RP_TRY(dev_alloc(c, &ly.ssrc, (size_t)c->n_cap, true));
            RP_TRY(dev_alloc(c, &ly.sdst, (size_t)c->n_cap, true));
            RP_TRY(dev_alloc(c, &ly.den, (size_t)c->n_cap, true));
        }
        if (ly.proj || ly.selfc) {
            std::vector<float> zeros(ly.N0pad, 0.0f);
            if (s.self_mode == RIPPLE_SELF_CONCAT) {           // rows d_in .. 2 d_in - 1 of W0
                RP_TRY(upload_padded(c, s.W0 + (size_t)s.d_in * s.d_out, zeros.data(), s.d_in, s.d_out,
                                     rp_round_up(s.d_in, 32), ly.N0pad, &ly.Wn, &ly.bzero, &ly.Wnq));
            } else {
                ly.Wn = ly.W0;
                ly.Wnq = ly.W0q;
                RP_TRY(dev_alloc(c, &ly.bzero, (size_t)ly.N0pad, true));
            }
        }
        if (ly.proj && ly.selfc && s.d_out <= 64 && s.d_in % 4 == 0) {
            const uint32_t kp = rp_round_up(s.d_in, 32);
            std::vector<float> wc((size_t)kp * 128, 0.0f);
            for (uint32_t k = 0; k < s.d_in; ++k)
                for (uint32_t j = 0; j < s.d_out; ++j) {
                    wc[(size_t)k * 128 + j] = s.W0[(size_t)k * s.d_out + j];                       // W_self
                    wc[(size_t)k * 128 + 64 + j] = s.W0[(size_t)(s.d_in + k) * s.d_out + j];       // W_neigh
                }
            RP_TRY(dev_alloc(c, &ly.Wc, wc.size(), false));
            RP_HIP(c, hipMemcpy(ly.Wc, wc.data(), wc.size() * 4, hipMemcpyHostToDevice));
            RP_TRY(make_quads(c, ly.Wc, kp, 128, &ly.Wcq));
            RP_TRY(dev_alloc(c, &ly.bzero_c, (size_t)128, true));
        }
        if (s.d_hidden) {
            ly.K1pad = rp_round_up(s.d_hidden, 32);
            ly.N1pad = pad_n(s.d_out);
            RP_TRY(upload_padded(c, s.W1, s.b1, s.d_hidden, s.d_out, ly.K1pad, ly.N1pad, &ly.W1, &ly.b1, &ly.W1q));
        }
        c->d[l + 1] = s.d_out;
        c->dmax = std::max(c->dmax, s.d_out);
        c->hmax = std::max(c->hmax, s.d_hidden);
    }
    {   // the weights in parts (fp32 rows; bf16 rows: where the products stay on fp32 numbers)
        Block b;
        struct Part {
            const float *w;
            uint32_t K, Npad;
            float lift;
            unsigned short **out;
        };
        std::vector<Part> parts;
        auto add = [&](const float *w, uint32_t K, uint32_t Npad, float lift, unsigned short **out) {
            if (!w) return;
            b.add(out, rp_weight_parts_size(K, Npad));
            parts.push_back({w, K, Npad, lift, out});
        };
        for (uint32_t l = 0; l < n_layers; ++l) {
            LayerDev &ly = c->layers[l];
            add(ly.W0, ly.K, ly.N0pad, ly.lift0, &ly.W0p);   // all rows: a product with W_self alone zeroes its rows from d_in on
            if (ly.Wn != ly.W0) add(ly.Wn, ly.d_in, ly.N0pad, ly.lift0, &ly.Wnp);
            add(ly.W1, ly.d_hidden, ly.N1pad, ly.lift1, &ly.W1p);
            add(ly.Wc, ly.d_in, 128u, ly.lift0, &ly.Wcp);
        }
        if (b.n) RP_TRY(block_alloc(c, b, &c->part_block, false));
        for (const Part &p : parts) rp_launch_weight_parts(c, p.w, p.K, p.Npad, p.lift, *p.out);
        for (uint32_t l = 0; l < n_layers; ++l)
            if (c->layers[l].Wn == c->layers[l].W0) c->layers[l].Wnp = c->layers[l].W0p;
    }
    const size_t n = c->n_cap;
    for (uint32_t l = 1; l <= c->L; ++l) {
        void *h = nullptr;
        size_t bytes = n * c->d[l] * elem_size(c);
        if (hipMalloc(&h, bytes + ARRAY_PAD) != hipSuccess) return fail(c, RIPPLE_ENOMEM, "device allocation of H failed");
        c->H[l] = h;
        RP_HIP(c, hipMemsetAsync(h, 0, bytes, c->stream));
        c->xw[l] = (c->layers[l - 1].proj || rp_layer_attn(c, l)) ? c->d[l] : c->d[l - 1];
        RP_TRY(dev_alloc(c, &c->X[l], n * c->xw[l], true));
        if (c->layers[l - 1].selfc) RP_TRY(dev_alloc(c, &c->layers[l - 1].PS, n * c->d[l], true));
        if (c->layers[l - 1].proj) {
            c->layers[l - 1].ldt = sent_row_stride(c->d[l]);
            RP_TRY(dev_alloc(c, &c->layers[l - 1].T, n * c->layers[l - 1].ldt, true));
            // packed rows are addressed with 32-bit byte offsets (vertex id * 128): below 2^25 vertices
            c->layers[l - 1].packed = (c->opt_pack && n < (1u << 25)) ? rp_msg_packed(c->d[l]) : 0u;
        }
    }
    {
        uint32_t aw = 0;                                 // widest attention layer
        for (uint32_t l = 1; l <= c->L; ++l)
            if (rp_layer_attn(c, l)) aw = std::max(aw, c->layers[l - 1].ldp);
        if (aw) {
            RP_TRY(dev_alloc(c, &c->Pold, n * aw, true));
            RP_TRY(dev_alloc(c, &c->sold, n, true));
            RP_TRY(dev_alloc(c, &c->gat_mag, n, true));
            RP_TRY(dev_alloc(c, &c->gat_rec, n, true));
        }
    }
    {
        uint32_t mw = 0;                                 // widest max / min aggregate, widest attention numerator and its denominator
        for (uint32_t l = 1; l <= c->L; ++l) {
            if (rp_layer_mono(c, l)) mw = std::max(mw, c->xw[l]);
            if (rp_layer_attn(c, l)) mw = std::max(mw, c->d[l] + 1);
        }
        if (mw) {                                        // in-rows sum to at most the pool: that bounds rows and segments
            c->big_cap = (uint32_t)std::min<uint64_t>(c->pool_cap / ROW_SPLIT_MIN + 1, ROW_SEG_MAX);
            c->seg_cap = (uint32_t)std::min<uint64_t>(c->pool_cap / ROW_SEG + c->big_cap, ROW_SEG_MAX);
            c->seg_ld = rp_round_up(mw, 32);             // partial rows share no 128-byte line
            Block b;
            b.add(&c->seg_v, c->big_cap);
            b.add(&c->seg_done, c->big_cap);
            b.add(&c->seg_base, c->big_cap);
            b.add(&c->seg_r, c->seg_cap);
            b.add(&c->seg_part, (size_t)c->seg_cap * c->seg_ld);
            RP_TRY(block_alloc(c, b, &c->seg_block, false));
        }
    }
    {   // rows of changes; the bootstrap and attention hops leave the parts of cut rows there before (two per run of chunks)
        size_t part = 0;
        for (uint32_t l = 1; l <= c->L && !c->opt_deterministic; ++l)
            if (!rp_layer_mono(c, l)) part = std::max<size_t>(part, c->xw[l] + (rp_layer_attn(c, l) ? 2u : 0u));
        c->max_runs = rp_max_runs(c->pool_cap, c->n_cu * 8 * 4);
        part = part ? 2 * c->max_runs * (1 + part) : 0;
        RP_TRY(dev_alloc(c, &c->D[0], std::max(n * c->dmax, part), false));
        RP_TRY(dev_alloc(c, &c->D[1], std::max(n * c->dmax, part), false));
    }
    if (c->hmax) RP_TRY(dev_alloc(c, &c->tmp, n * c->hmax, false));
    {
        uint32_t pw = 0;
        for (uint32_t l = 1; l <= c->L; ++l)
            if (c->layers[l - 1].proj) pw = std::max(pw, c->d[l]);
        c->pd_ld = pw <= 32 ? 32 : rp_round_up(pw, 16);  // up to 32 columns: one 128-byte line per row; else 64-byte multiples
        if (pw) RP_TRY(dev_alloc(c, &c->PD, n * c->pd_ld, true));
        bool packed = false;
        for (uint32_t l = 1; l <= c->L; ++l) packed |= c->layers[l - 1].proj && c->layers[l - 1].packed;
        if (packed) RP_TRY(dev_alloc(c, &c->MSG, n * RP_MSG_WORDS, true));
    }
    if (c->opt_deterministic) {                          // two side entries per run of chunks of the pull kernels
        uint32_t xmax = 1;
        for (uint32_t l = 1; l <= c->L; ++l) xmax = std::max(xmax, c->xw[l]);
        // runs: up to four per wavefront of the grid while a run is shorter than eight chunks, else an eighth of the chunks
        // (256 in-row entries each) that the in-row pool can hold
        const size_t nw = (size_t)c->n_cu * 8 * 4;
        c->side_runs = (uint32_t)std::max<size_t>(4 * nw, c->pool_cap / (256 * 8) + 2);
        const size_t entries = 2 * (size_t)c->side_runs;
        RP_TRY(dev_alloc(c, &c->side_v, entries, false));
        RP_TRY(dev_alloc(c, &c->side_acc, entries * xmax, false));
    }
    bool weighted = false;
    for (uint32_t l = 1; l <= c->L; ++l) weighted |= c->layers[l - 1].agg == RIPPLE_AGG_WSUM;
    bool sums = false, attn = false;                     // some hop from the second on is one of sums, of attention
    for (uint32_t l = 2; l <= c->L; ++l) {
        attn |= rp_layer_attn(c, l);
        sums |= !rp_layer_mono(c, l) && !rp_layer_attn(c, l);
    }
    if ((sums || attn) && !c->opt_deterministic && rp_lists_allowed(c)) {
        // (destination, source) pairs of a hop's messages: room for twice a quarter of the edge capacity, at most 2^26 (a hop with
        // more messages than that quarter is pulled, pushed or discovers). Attention hops list at most a 64th of the edges (RP_GAT_LIST_SHARE):
        // room for twice a sixteenth of them, so that a bucket may hold eight times what the average one does. 24 bytes per message:
        // 0.81 GB on the graph of 124 M edges, 0.27 where only attention lists.
        c->pair_cap = (uint32_t)std::min<uint64_t>(std::max<uint64_t>(c->pool_cap / (sums ? 4 : 16), 1u << 14), 1u << 25);
        Block b;
        b.add(&c->pairs, 2 * (size_t)c->pair_cap);
        b.add(&c->pair_sorted, c->pair_cap);
        if (weighted) {                                  // ... and the edges' weights
            b.add(&c->pair_w, 2 * (size_t)c->pair_cap);
            b.add(&c->pair_w_sorted, c->pair_cap);
        }
        RP_TRY(block_alloc(c, b, &c->pair_block, false));
    }
    // bitmaps: layers 0..L, then S, then V_added, contiguous; reporting copies separately
    uint32_t *bmall = nullptr, *repall = nullptr, *lists = nullptr, *eoffs = nullptr, *ioffs = nullptr;
    Block b;
    b.add(&bmall, (size_t)c->n_words * (c->L + 3));
    b.add(&repall, (size_t)c->n_words * (c->L + 1));
    b.add(&lists, (n + 1) * (c->L + 1));
    b.add(&eoffs, (n + 1) * (c->L + 1));
    b.add(&ioffs, (n + 1) * (c->L + 1));
    b.add(&c->all_list, n + 1);
    b.add(&c->mk, (size_t)c->n_words * 32);
    b.add(&c->ioff_all, n + 1);
    b.add(&c->pair_cnt, RP_LIST_BUCKETS);
    RP_TRY(block_alloc(c, b, &c->list_block, true));
    for (uint32_t l = 0; l <= c->L; ++l) {
        c->bm[l] = bmall + (size_t)l * c->n_words;
        c->rep[l] = repall + (size_t)l * c->n_words;
        c->list[l] = lists + (size_t)l * (n + 1);
        c->eoff[l] = eoffs + (size_t)l * (n + 1);
        c->ioff[l] = ioffs + (size_t)l * (n + 1);
    }
    c->bm_sink = bmall + (size_t)(c->L + 1) * c->n_words;
    c->bm_vadd = bmall + (size_t)(c->L + 2) * c->n_words;
    RP_TRY(grow_scratch(c, PIN_OPS, 0));
    RP_HIP(c, hipStreamSynchronize(c->stream));
    if (!weighted && c->out_w) {                         // no layer sends weighted messages: given back, and a new weight need not be looked up
        hipFree(c->out_w);                               // in the out-row either
        c->out_w = nullptr;
    }
    c->state = 2;
    return RIPPLE_OK;
}

static ripple_status range_error(ripple_ctx *c, uint32_t rows) {
    c->err = "attention exponentials overflowed the float range: " + std::to_string(rows) +
             " row updates used sums that were not finite (scores must stay below about 88)";
    return RIPPLE_ERANGE;
}

// ---------------------------------------------------------------------------------
// bootstrap inference
// ---------------------------------------------------------------------------------
extern "C" ripple_status ripple_full_infer(ripple_ctx *c) {
    if (!c) return RIPPLE_EINVAL;
    if (c->state < 2) return fail(c, RIPPLE_ESTATE, "full_infer needs init_graph and load_model first");
    // all live vertices as one list (the alive bitmap itself is the source)
    hipLaunchKernelGGL(k_or_words, dim3(rp_div_up(c->n_words, 256)), dim3(256), 0, c->stream, c->bm[0], c->alive,
                       c->n_words);
    rp_launch_bitmap_to_list(c, c->bm[0], c->all_list, 0xFFFFFFFFu, &c->ctr->set[0].a);
    rp_launch_alive_list(c);                               // the same list once more, with its in-degree prefix
    for (uint32_t l = 1; l <= c->L; ++l) {
        if (rp_layer_attn(c, l)) {
            rp_launch_gat_project(c, l, c->all_list, &c->ctr->set[0].a);
            rp_launch_gat_scores(c, l, c->all_list, &c->ctr->set[0].a);
            rp_launch_gat_scatter(c, l, true);
            rp_launch_transform(c, l, c->all_list, &c->ctr->set[0].a, false);
            continue;
        }
        if (rp_has_project_both(c, l)) {
            rp_launch_project_both(c, l, c->all_list, &c->ctr->set[0].a, true);
        } else {
            if (c->layers[l - 1].proj) rp_launch_project(c, l, c->all_list, &c->ctr->set[0].a, true);
            if (c->layers[l - 1].selfc) rp_launch_self_project(c, l, c->all_list, &c->ctr->set[0].a);
        }
        if (c->opt_deterministic) rp_launch_scatter_pull_det(c, l, true);  // same summation order as the batches use
        else rp_launch_pull_all(c, l);
        rp_launch_transform(c, l, c->all_list, &c->ctr->set[0].a, false);
    }
    RP_HIP(c, hipMemcpyAsync(c->ctr_host, c->ctr, sizeof(DevCtr), hipMemcpyDeviceToHost, c->stream));
    rp_launch_batch_reset(c);
    RP_HIP(c, hipStreamSynchronize(c->stream));
    RP_HIP(c, hipGetLastError());
    const uint32_t range_rows = c->ctr_host->range_rows;
    for (uint32_t l = 0; l <= c->L; ++l) c->last_a[l] = 0;
    c->hints_valid = false;
    c->last_n_ops = 0;
    c->last_from_rep = false;
    c->state = 3;
    if (range_rows) return range_error(c, range_rows);
    return RIPPLE_OK;
}

// ---------------------------------------------------------------------------------
// per-batch driver
// ---------------------------------------------------------------------------------
// Flat hash over the keys a sub-batch has touched: edge (u,v) -> present,
// vertex w -> flags. Entries are valid only for the current generation.
struct TouchTable {
    std::vector<uint64_t> keys;
    std::vector<uint32_t> gen;
    std::vector<uint8_t> val;
    uint32_t cur = 1;
    size_t mask = 0;
    void reserve(size_t n_keys) {
        size_t want = 64;
        while (want < n_keys * 4) want <<= 1;
        if (want > keys.size()) {
            keys.assign(want, 0);
            gen.assign(want, 0);
            val.assign(want, 0);
            cur = 1;
        }
        mask = keys.size() - 1;
    }
    void next_generation() {
        if (++cur == 0) {
            std::fill(gen.begin(), gen.end(), 0);
            cur = 1;
        }
    }
    uint8_t *find(uint64_t key, bool insert) {
        size_t h = (size_t)((key * 0x9E3779B97F4A7C15ull) >> 20) & mask;
        for (;;) {
            if (gen[h] != cur) {
                if (!insert) return nullptr;
                gen[h] = cur;
                keys[h] = key;
                val[h] = 0;
                return &val[h];
            }
            if (keys[h] == key) return &val[h];
            h = (h + 1) & mask;
        }
    }
};

#define TF_EDGE_REF 1
#define TF_FEAT 2
#define TF_VADD 4
#define TF_VDEL 8

struct SubBatch {
    uint32_t begin, end;
    bool has_vdel, has_vertex_or_feat;
};

// Cut the batch where an operation depends on an earlier one of the same piece, so that every
// piece can be applied in parallel with the same result as applying it in array order.
static void split_batch(const ripple_update *ops, uint32_t n, TouchTable &tt, std::vector<SubBatch> &out) {
    out.clear();
    tt.reserve((size_t)n * 3 + 16);
    tt.next_generation();
    SubBatch cur{0, 0, false, false};
    const uint64_t VKEY = 0x8000000000000000ull;
    for (uint32_t i = 0; i < n; ++i) {
        const ripple_update &op = ops[i];
        for (int attempt = 0; attempt < 2; ++attempt) {
            bool conflict = false;
            if (op.kind == RIPPLE_EDGE_ADD || op.kind == RIPPLE_EDGE_DEL || op.kind == RIPPLE_EDGE_REWEIGHT) {
                uint64_t ek = ((uint64_t)op.u << 32) | op.v;
                uint8_t *fu = tt.find(VKEY | op.u, false), *fv = tt.find(VKEY | op.v, false);
                if (tt.find(ek, false) || (fu && (*fu & TF_VDEL)) || (fv && (*fv & TF_VDEL))) conflict = true;
                else {
                    *tt.find(ek, true) = 1;
                    *tt.find(VKEY | op.u, true) |= TF_EDGE_REF;
                    *tt.find(VKEY | op.v, true) |= TF_EDGE_REF;
                }
            } else {
                uint8_t *f = tt.find(VKEY | op.u, false);
                uint8_t flags = f ? *f : 0;
                if (op.kind == RIPPLE_FEAT_UPDATE) {
                    if (flags & (TF_FEAT | TF_VADD | TF_VDEL)) conflict = true;
                    else *tt.find(VKEY | op.u, true) |= TF_FEAT;
                } else {
                    if (flags) conflict = true;
                    else *tt.find(VKEY | op.u, true) |= (op.kind == RIPPLE_VERTEX_ADD ? TF_VADD : TF_VDEL);
                }
            }
            if (!conflict) break;
            cur.end = i;                       // close the piece before this operation and start afresh
            out.push_back(cur);
            cur = SubBatch{i, i, false, false};
            tt.next_generation();
        }
        if (op.kind == RIPPLE_VERTEX_DEL) cur.has_vdel = true;
        if (op.kind >= RIPPLE_VERTEX_ADD && op.kind <= RIPPLE_FEAT_UPDATE) cur.has_vertex_or_feat = true;
    }
    cur.end = n;
    if (cur.end > cur.begin || out.empty()) out.push_back(cur);
}

static bool ops_in_range(const ripple_update *ops, uint32_t n_ops, uint32_t n_cap, uint32_t n_feat_rows) {
    for (uint32_t i = 0; i < n_ops; ++i) {
        const ripple_update &op = ops[i];
        bool bad = op.kind > RIPPLE_EDGE_REWEIGHT || op.u >= n_cap;
        if (!bad && (op.kind <= RIPPLE_EDGE_DEL || op.kind == RIPPLE_EDGE_REWEIGHT)) bad = op.v >= n_cap;
        if (!bad && (op.kind == RIPPLE_VERTEX_ADD || op.kind == RIPPLE_FEAT_UPDATE)) bad = op.feat_row >= n_feat_rows;
        if (bad) return false;
    }
    return true;
}

extern "C" ripple_status ripple_plan_batch(const ripple_update *ops, uint32_t n_ops, uint32_t vertex_capacity,
                                           uint32_t n_feat_rows, uint32_t *piece_end, uint32_t cap, uint32_t *n_pieces) {
    if ((n_ops && !ops) || !n_pieces || (cap && !piece_end)) return RIPPLE_EINVAL;
    if (!ops_in_range(ops, n_ops, vertex_capacity, n_feat_rows)) return RIPPLE_EINVAL;
    *n_pieces = 0;
    if (n_ops == 0) return RIPPLE_OK;
    TouchTable tt;
    std::vector<SubBatch> pieces;
    split_batch(ops, n_ops, tt, pieces);
    for (size_t p = 0; p < pieces.size(); ++p)
        if (p < cap) piece_end[p] = pieces[p].end;
    *n_pieces = (uint32_t)pieces.size();
    return RIPPLE_OK;
}

// A_{l-1} is part of A_l: the layer reads the vertex's own row (a self term, or its attention score)
#define SPARSE_MAX_ROWS 4096u
#define SPARSE_MAX_EDGES 65536u

// Hop l + 1 forwards D^l = new - old rows of layer l, unless its layer is handled project-first: that one
// sends H^l W_neigh minus what it has sent before and never looks at the difference.
static bool next_reads_delta(const ripple_ctx *c, uint32_t l) { return l < c->L && !c->layers[l].proj; }

static bool layer_self(const ripple_ctx *c, uint32_t l) {
    return c->layers[l - 1].self_mode != RIPPLE_SELF_NONE || rp_layer_attn(c, l);
}

// Hop l's set (and the previous hop's) was small in the previous batch, which was of about this size: the
// hop lists its vertices while marking them instead of scanning the bitmap. Only a choice between two
// correct paths.
static bool small_frontier(const ripple_ctx *c, uint32_t l, uint32_t n_ops, bool multi) {
    return c->opt_sparse && !multi && c->last_a[l] <= SPARSE_MAX_ROWS && c->last_a[l - 1] <= SPARSE_MAX_ROWS &&
           c->last_m[l] <= SPARSE_MAX_EDGES && c->last_n_ops && n_ops <= 2 * c->last_n_ops;
}

// Hop l of a sum or mean layer was so small that it pushes and is launched whole (rp_launch_hop_small): the same hint with
// limits of its own. The push costs an atomic per number sent (3e11 a second), so the numbers are bounded to what takes
// about as long as the launches saved; twice the vertices of small_frontier, because no single workgroup goes over the list here.
#define TINY_MAX_ROWS 16384u
#define TINY_MAX_NUMBERS (4u << 20)
static bool tiny_hop(const ripple_ctx *c, uint32_t l, uint32_t n_ops, bool multi) {
    const LayerDev &ly = c->layers[l - 1];
    if (ly.proj && ly.self_mode == RIPPLE_SELF_CONCAT && !ly.selfc) return false;      // (a product per row is left in the row update)
    return c->opt_sparse && !multi && c->opt_scatter <= 1 && c->opt_sorted < 2 && c->last_n_ops && n_ops <= 2 * c->last_n_ops &&
           c->last_a[l] <= TINY_MAX_ROWS && c->last_a[l - 1] <= TINY_MAX_ROWS &&
           (uint64_t)c->last_m[l] * c->xw[l] <= TINY_MAX_NUMBERS;
}

// Hop l's list had a bucket run over, and would again: the hop has not become much smaller and its buckets have no more room than they had. A
// graph whose hubs lie in one bucket would pay for the walk that writes the list (0.12 ms for 4.6 M messages instead of 0.09) and two empty
// launches at every batch. Edges come and go: every LIST_OVER_WAIT batches it is tried all the same.
#define LIST_OVER_WAIT 64u
static bool list_runs_over(ripple_ctx *c, uint32_t l, uint32_t pair_cap) {
    c->list_room[l] = rp_list_cut(c, c->last_m[l] ? c->last_m[l] : pair_cap).room;
    ripple_ctx::ListOver &o = c->list_over[l];
    if (!o.room || c->last_m[l] < o.m / 2u || c->list_room[l] > o.room || o.wait == 0u) {
        o.room = 0;
        return false;
    }
    --o.wait;
    return true;
}

// |A_l| where no previous batch says it: a replaced row reaches its out-neighbours, any other operation one or two vertices, every hop
// after it multiplies by the mean degree. Below some thousand rows the kernels do not differ enough to trust a guess with.
#define GUESS_MIN_ROWS 4096u
static void guess_rows(ripple_ctx *c, const ripple_update *ops, uint32_t n) {
    uint64_t feat = 0;
    for (uint32_t i = 0; i < n; ++i) feat += ops[i].kind == RIPPLE_FEAT_UPDATE || ops[i].kind == RIPPLE_VERTEX_ADD;
    const uint64_t reach = c->e_cap / c->n_cap + 2;
    uint64_t rows = feat;
    for (uint32_t l = 0; l <= c->L; ++l) {
        c->guess_a[l] = (uint32_t)std::min<uint64_t>(c->n_cap, std::max<uint64_t>(rows, GUESS_MIN_ROWS));
        rows = std::min<uint64_t>(c->n_cap, rows * reach + (l == 0 ? 2ull * (n - feat) : 0ull));
    }
}

// Enqueue one conflict-free piece: Apply, then hop by hop frontier / scatter / transform.
static void enqueue_piece(ripple_ctx *c, const SubBatch &sb, bool multi) {
    const uint32_t n = sb.end - sb.begin;
    int t = rp_timer_begin(c);
    const ripple_update *ops = c->ops_pin + sb.begin;
    rp_launch_mutate(c, ops, n, sb.has_vdel, sb.has_vertex_or_feat);
    rp_timer_end(c, t, RIPPLE_PH_INGEST, 0);
    if (!c->hints_valid) guess_rows(c, ops, n);
    if (multi)
        hipLaunchKernelGGL(k_or_words, dim3(rp_div_up(c->n_words, 256)), dim3(256), 0, c->stream, c->rep[0], c->bm[0],
                           c->n_words);
    bool have_all = false;                              // live-vertex list of this piece exists
    if (c->opt_deterministic) {                         // one owner per aggregate row, fixed summation order
        for (uint32_t l = 1; l <= c->L; ++l) {
            t = rp_timer_begin(c);
            rp_launch_frontier_mark(c, l, false);
            rp_timer_end(c, t, RIPPLE_PH_FRONTIER, (int)l);
            t = rp_timer_begin(c);
            rp_launch_frontier_compact(c, l, layer_self(c, l), l < c->L, true, multi);
            rp_timer_end(c, t, RIPPLE_PH_COMPACT, (int)l);
            if (c->layers[l - 1].proj || c->layers[l - 1].selfc) {
                t = rp_timer_begin(c);
                if (rp_has_project_both(c, l)) {
                    rp_launch_project_both(c, l, c->list[l - 1], &c->ctr->set[l - 1].a, false);
                } else {
                    if (c->layers[l - 1].proj) rp_launch_project(c, l, c->list[l - 1], &c->ctr->set[l - 1].a, false);
                    if (c->layers[l - 1].selfc) rp_launch_self_project(c, l, c->list[l - 1], &c->ctr->set[l - 1].a);
                }
                if (c->layers[l - 1].proj) rp_launch_messages(c, l);
                rp_timer_end(c, t, RIPPLE_PH_OTHER, (int)l);
            }
            t = rp_timer_begin(c);
            rp_launch_scatter_pull_det(c, l, false);
            rp_timer_end(c, t, RIPPLE_PH_SCATTER, (int)l);
            t = rp_timer_begin(c);
            rp_launch_transform(c, l, c->list[l], &c->ctr->set[l].a, next_reads_delta(c, l));
            rp_timer_end(c, t, RIPPLE_PH_TRANSFORM, (int)l);
        }
        return;
    }
    for (uint32_t l = 1; l <= c->L; ++l) {
        if (rp_layer_mono(c, l)) {                     // max / min: keep, raise or recompute, then prune (Sec. 3.4.2)
            const bool listed = small_frontier(c, l, n, multi) && c->last_cand[l] <= SPARSE_MAX_ROWS;
            t = rp_timer_begin(c);
            if (listed) rp_launch_candidates_sparse(c, l, layer_self(c, l), RP_MONO_LISTED_LONG);
            else rp_launch_frontier_mark(c, l, false);
            rp_timer_end(c, t, RIPPLE_PH_FRONTIER, (int)l);
            if (!listed) {
                t = rp_timer_begin(c);
                rp_launch_candidates(c, l);
                rp_timer_end(c, t, RIPPLE_PH_COMPACT, (int)l, false);
            }
            if (c->layers[l - 1].selfc) {
                t = rp_timer_begin(c);
                rp_launch_self_project(c, l, c->list[l - 1], &c->ctr->set[l - 1].a);
                rp_timer_end(c, t, RIPPLE_PH_OTHER, (int)l);
            }
            t = rp_timer_begin(c);
            rp_launch_scatter_mono(c, l, listed ? &c->ctr->cand[l] : &c->ctr->n_all, listed);
            rp_timer_end(c, t, RIPPLE_PH_SCATTER, (int)l);
            t = rp_timer_begin(c);
            if (listed) rp_launch_list_offsets(c, l, l < c->L);  // the aggregation kernels listed what stays
            else rp_launch_frontier_compact(c, l, layer_self(c, l), l < c->L, false, multi, true);
            rp_timer_end(c, t, RIPPLE_PH_COMPACT, (int)l);
            t = rp_timer_begin(c);
            rp_launch_transform(c, l, c->list[l], &c->ctr->set[l].a, next_reads_delta(c, l));
            rp_timer_end(c, t, RIPPLE_PH_TRANSFORM, (int)l);
            have_all = false;                          // the candidates went through the live-vertex list's buffer
            continue;
        }
        if (rp_layer_attn(c, l)) {                     // attention: recompute or numerator / denominator deltas (Sec. 3.4.1)
            t = rp_timer_begin(c);
            rp_launch_gat_save(c, l, c->list[l - 1], &c->ctr->set[l - 1].a);
            rp_launch_gat_project(c, l, c->list[l - 1], &c->ctr->set[l - 1].a);
            rp_launch_gat_scores(c, l, c->list[l - 1], &c->ctr->set[l - 1].a);
            rp_timer_end(c, t, RIPPLE_PH_OTHER, (int)l);
            const bool listed = small_frontier(c, l, n, multi);
            uint32_t pair_cap = 0;
            if (listed) {
                t = rp_timer_begin(c);
                rp_launch_frontier_sparse(c, l, true, l < c->L, RP_MONO_LISTED_LONG);
                rp_timer_end(c, t, RIPPLE_PH_FRONTIER, (int)l);
            } else {
                // messages listed as they are marked, where the last batch says that this pays (the kernels decide)
                if (l >= 2 && c->pair_cap && c->opt_sorted) {
                    const uint64_t m = c->last_m[l], e = c->ctr_host->n_edges, nv = std::max(1u, c->ctr_host->n_alive);
                    if (c->opt_sorted == 2 || (c->hints_valid && RP_GAT_LIST_SHARE * m <= e && rp_list_pays_pull(m, m * (e / nv)))) pair_cap = c->pair_cap;
                    if (pair_cap && list_runs_over(c, l, pair_cap)) pair_cap = 0;
                }
                t = rp_timer_begin(c);
                rp_launch_frontier_mark(c, l, false, pair_cap);
                rp_timer_end(c, t, RIPPLE_PH_FRONTIER, (int)l);
                t = rp_timer_begin(c);
                rp_launch_frontier_compact(c, l, true, l < c->L, true, multi, false, pair_cap);
                rp_timer_end(c, t, RIPPLE_PH_COMPACT, (int)l);
            }
            t = rp_timer_begin(c);
            rp_launch_gat_scatter(c, l, false, listed, pair_cap);
            rp_timer_end(c, t, RIPPLE_PH_SCATTER, (int)l);
            t = rp_timer_begin(c);
            rp_launch_transform(c, l, c->list[l], &c->ctr->set[l].a, next_reads_delta(c, l));
            rp_timer_end(c, t, RIPPLE_PH_TRANSFORM, (int)l);
            have_all = false;                          // the long-row queue and the recomputed vertices went through the live-vertex list's buffers
            continue;
        }
        // hop 1 always pushes: hop-0 rows are in operation order, not ranked by vertex id. Where the
        // previous batch pushed with a wide margin the pull kernel is not even enqueued (pushing is
        // always correct; the prediction only saves a launch). The same goes for the discovering
        // mode: its kernels are enqueued only where the previous batch came near its threshold.
        if (tiny_hop(c, l, n, multi)) {       // two or three launches for the whole hop
            t = rp_timer_begin(c);
            rp_launch_hop_small(c, l, layer_self(c, l));
            rp_timer_end(c, t, RIPPLE_PH_FRONTIER, (int)l);
            t = rp_timer_begin(c);
            const LayerDev &ly = c->layers[l - 1];
            if (ly.proj) rp_launch_small_addend(c, l, next_reads_delta(c, l));
            else rp_launch_transform(c, l, c->list[l], &c->ctr->set[l].a, next_reads_delta(c, l));
            rp_timer_end(c, t, RIPPLE_PH_TRANSFORM, (int)l);
            continue;
        }
        const bool may_pull = l >= 2 && c->opt_scatter != 1 && !(c->opt_scatter == 0 && c->push_margin[l]);
        const bool may_disc = l >= 2 && may_pull && (c->opt_scatter == 3 || (c->opt_scatter == 0 && c->disc_near[l]));
        // a frontier that was small last time (and a batch of about the same size) is listed as it is marked
        const bool sparse = !may_disc && small_frontier(c, l, n, multi);
        t = rp_timer_begin(c);
        if (may_disc && !have_all) {
            rp_launch_alive_list(c);
            have_all = true;
        }
        // A hop that the last batch moved a good many messages at without discovering its set is taken from the list of them
        // (k_scatter_list) where that pays: in place of a pull through in-rows that hold enough entries, or of a push of enough numbers.
        // The out-edge walk writes the list, of up to eight times the last batch's messages: batches differ by the hubs they meet, and one that is pulled
        // because it has more than was expected costs more than the walk (100 updates on the dense graph that meet a hub, hop 3: 165 us of walk and 1,115 pulled, 210 and 460 listed).
        // The kernels make sure on the device that the list is only used if it still pays; else the hop is pulled or pushed.
        uint32_t pair_cap = 0;
        if (l >= 2 && !sparse && c->pair_cap && c->opt_sorted && c->opt_scatter != 1 && c->opt_scatter != 3) {
            const uint64_t m = c->last_m[l];
            const bool pulls = c->opt_scatter == 2 || m * c->xw[l] * 4ull * (unsigned)c->opt_pull_ratio >= 8ull * c->last_isum[l];
            if (c->opt_sorted == 2) pair_cap = c->pair_cap;
            else if (c->hints_valid && m && m <= c->pair_cap && c->last_hop_mode[l] != 1u + RP_HOP_DISCOVER &&
                     (pulls ? rp_list_pays_pull(m, c->last_isum[l]) : m * c->xw[l] >= RP_LIST_NUMBERS))
                pair_cap = (uint32_t)std::min<uint64_t>(8 * m + 4096, c->pair_cap);
            if (pair_cap && list_runs_over(c, l, pair_cap)) pair_cap = 0;
        }
        if (sparse) rp_launch_frontier_sparse(c, l, layer_self(c, l), l < c->L);
        else if (!may_disc || pair_cap) rp_launch_frontier_mark(c, l, may_disc, pair_cap);   // (else by the launch that discovers or marks)
        rp_timer_end(c, t, RIPPLE_PH_FRONTIER, (int)l, !may_disc || pair_cap);
        const bool both = rp_has_project_both(c, l);
        if (c->layers[l - 1].proj) {                   // what travels is already multiplied by W_neigh
            t = rp_timer_begin(c);
            if (both) rp_launch_project_both(c, l, c->list[l - 1], &c->ctr->set[l - 1].a, false);   // and the self terms in the same pass
            else rp_launch_project(c, l, c->list[l - 1], &c->ctr->set[l - 1].a, false);
            rp_launch_messages(c, l);
            rp_timer_end(c, t, RIPPLE_PH_OTHER, (int)l);
        }
        if (c->layers[l - 1].selfc && !both) {         // H^{l-1} changed exactly on A_{l-1}
            t = rp_timer_begin(c);
            rp_launch_self_project(c, l, c->list[l - 1], &c->ctr->set[l - 1].a);
            rp_timer_end(c, t, RIPPLE_PH_OTHER, (int)l, !c->layers[l - 1].proj);
        }
        if (may_disc) {                                // scatters and marks A_l in one scan of all in-rows
            t = rp_timer_begin(c);
            rp_launch_scatter_pull(c, l, true, true, 0, !pair_cap);
            rp_timer_end(c, t, RIPPLE_PH_SCATTER, (int)l, false);
        }
        if (!sparse) {
            t = rp_timer_begin(c);
            rp_launch_frontier_compact(c, l, layer_self(c, l), l < c->L, true, multi);
            rp_timer_end(c, t, RIPPLE_PH_COMPACT, (int)l);
        }
        t = rp_timer_begin(c);
        if (!may_pull) rp_launch_scatter_push(c, l, pair_cap);
        if (pair_cap) rp_launch_scatter_list(c, l, may_disc, pair_cap);
        if (may_pull) rp_launch_scatter_pull(c, l, false, may_disc, pair_cap, c->opt_scatter < 2);
        rp_timer_end(c, t, RIPPLE_PH_SCATTER, (int)l);
        t = rp_timer_begin(c);
        rp_launch_transform(c, l, c->list[l], &c->ctr->set[l].a, next_reads_delta(c, l));
        rp_timer_end(c, t, RIPPLE_PH_TRANSFORM, (int)l);
    }
}

// The counters to the host, and the end of everything enqueued before.
static ripple_status publish_and_wait(ripple_ctx *c) {
    rp_launch_publish(c);
    return rp_wait_flag(c);
}

// Stage, enqueue and wait for one piece; on a full adjacency pool or a full scratch buffer the piece (which
// aborts on the device before it changes anything) is retried after compaction / growth. On return with
// RIPPLE_OK the pinned mirror of the counters describes the piece.
static ripple_status run_piece(ripple_ctx *c, const SubBatch &sb, bool multi, uint32_t *compactions) {
    for (int attempt = 0;; ++attempt) {
        enqueue_piece(c, sb, multi);
        RP_TRY(publish_and_wait(c));
        const DevCtr &h = *c->ctr_host;
        if (!h.abort_flag) return RIPPLE_OK;
        if (h.abort_flag & 8u) {
            c->err = "graph store consistency error " + std::to_string(h.error);
            return RIPPLE_EDEVICE;
        }
        if (h.abort_flag & 2u) return fail(c, RIPPLE_ECAPACITY, "edge capacity exceeded");
        if (attempt >= 2) return fail(c, RIPPLE_ECAPACITY, "adjacency pool exhausted even after compaction");
        if (h.abort_flag & 4u) {
            uint32_t want = h.need_exp + h.need_exp / 2 + 1024;
            RP_TRY(grow_scratch(c, 0, want));
        }
        if (h.abort_flag & 1u) {
            ++*compactions;
            RP_TRY(rp_compact(c));
        }
    }
}

extern "C" ripple_status ripple_apply_updates(ripple_ctx *c, const ripple_update *ops, uint32_t n_ops,
                                              const float *feat_payload, uint32_t n_feat_rows,
                                              ripple_batch_result *res) {
    if (!c) return RIPPLE_EINVAL;
    if (c->state != 3) return fail(c, RIPPLE_ESTATE, "apply_updates needs full_infer first");
    if ((n_ops && !ops) || (n_feat_rows && !feat_payload)) return fail(c, RIPPLE_EINVAL, "null batch pointer");
    if (res) memset(res, 0, sizeof(*res));
    static thread_local TouchTable tt;
    static thread_local std::vector<SubBatch> pieces;
    hipStream_t s = c->stream;
    int t_total = rp_timer_begin(c);

    const bool rows_on_host = n_feat_rows && !is_device_ptr(c, feat_payload);
    RP_TRY(grow_staging(c, n_ops, rows_on_host ? n_feat_rows : 0u));
    // operations are needed on the host (validation, conflict analysis)
    const ripple_update *hops = ops;
    const Place ops_place = n_ops ? place_of(c, ops) : ON_HOST;
    if (ops_place == OWN_GPU) {                            // by a kernel that reports its end: the runtime's copy and the wait for the stream take 15 us more
        const uint32_t gb = rp_div_up(n_ops, 256 * 4);
        const HostFlag done = gb <= REPORT_WGS ? rp_host_flag(c) : HostFlag{nullptr, 0u, nullptr};
        hipLaunchKernelGGL(k_copy_numbers, dim3(gb), dim3(256), 0, s, (const float *)ops, (float *)c->ops_pin, (size_t)n_ops * 4, done);
        if (!done.flag) rp_launch_report(c);
        RP_TRY(rp_wait_flag(c));
        hops = c->ops_pin;
    } else if (ops_place == FAR_GPU) {
        RP_HIP(c, hipMemcpyAsync(c->ops_pin, ops, (size_t)n_ops * sizeof(ripple_update), hipMemcpyDeviceToHost, s));
        RP_HIP(c, hipStreamSynchronize(s));
        hops = c->ops_pin;
    }
    if (!ops_in_range(hops, n_ops, c->n_cap, n_feat_rows))
        return fail(c, RIPPLE_EINVAL, "operation with unknown kind, vertex id or payload row out of range");
    if (n_ops == 0) {                              // nothing to do: the affected sets become empty
        rp_launch_batch_reset(c);
        RP_TRY(publish_and_wait(c));
        for (uint32_t l = 0; l <= c->L; ++l) c->last_a[l] = 0;
        c->last_from_rep = false;
        if (res) {
            res->n_sub_batches = 0;
            res->n_alive = c->ctr_host->n_alive;
            res->n_edges = c->ctr_host->n_edges;
        }
        return RIPPLE_OK;
    }
    split_batch(hops, n_ops, tt, pieces);
    const bool multi = pieces.size() > 1;
    // room for the edges of deleted vertices only where there are any; what turns out too small grows (run_piece)
    bool deletes = false;
    for (const SubBatch &sb : pieces) deletes |= sb.has_vdel;
    RP_TRY(grow_scratch(c, n_ops, deletes ? std::max<uint32_t>(c->exp_cap, (uint32_t)std::min<uint64_t>(1u << 20, 2 * c->e_cap + 1)) : 0u));
    if (hops != c->ops_pin) memcpy(c->ops_pin, hops, (size_t)n_ops * sizeof(ripple_update));

    if (multi)
        RP_HIP(c, hipMemsetAsync(c->rep[0], 0, (size_t)c->n_words * (c->L + 1) * 4, s));
    // feature rows: used in place when they already live on the device
    c->payload = feat_payload;
    if (rows_on_host) {                                    // the kernel that applies them reads each row once, over the bus
        memcpy(c->payload_pin, feat_payload, (size_t)n_feat_rows * c->d[0] * 4);
        c->payload = c->payload_pin;
    }

    ripple_status rc = RIPPLE_OK;
    uint32_t applied = 0, rejected = 0, n_struct = 0, compactions = 0, ops_done = 0, range_rows = 0;
    uint64_t msgs[RIPPLE_MAX_LAYERS + 1] = {0}, tchd[RIPPLE_MAX_LAYERS + 1] = {0};
    uint32_t mono[3][RIPPLE_MAX_LAYERS + 1] = {{0}};
    uint32_t hop_mode[RIPPLE_MAX_LAYERS + 1] = {0};
    for (size_t p = 0; p < pieces.size() && rc == RIPPLE_OK; ++p) {
        const SubBatch &sb = pieces[p];
        const uint32_t n = sb.end - sb.begin;
        rc = run_piece(c, sb, multi, &compactions);
        if (rc != RIPPLE_OK) break;
        ops_done = sb.end;
        const DevCtr &h = *c->ctr_host;
        applied += h.n_applied;
        rejected += h.n_rejected;
        n_struct += h.n_struct;
        range_rows += h.range_rows;
        for (uint32_t l = 1; l <= c->L; ++l) {
            msgs[l] += h.set[l - 1].m;
            tchd[l] += h.touched[l];
            c->last_m[l] = h.set[l - 1].m;
            c->last_isum[l] = h.isum[l];
            c->last_hop_mode[l] = h.hop_mode[l];
            if (h.pair_over[l]) c->list_over[l] = {h.set[l - 1].m, c->list_room[l], LIST_OVER_WAIT};
            hop_mode[l] = h.hop_mode[l];
            for (int k = 0; k < 3; ++k) mono[k][l] += h.mono[k][l];
            c->last_cand[l] = h.mono[0][l] + h.mono[1][l] + h.mono[2][l];
            // pull wins when m * row_bytes * ratio >= 8 * in-edges; remember if push won by a factor of 16
            const unsigned long long lhs = (unsigned long long)h.set[l - 1].m * c->xw[l] * 4ull * (unsigned)c->opt_pull_ratio * 16ull;
            c->push_margin[l] = lhs < 8ull * h.isum[l];
            c->disc_near[l] = (unsigned long long)h.set[l - 1].m * 64ull >= h.n_edges;     // threshold: m * 8 >= edges
        }
        if (!multi)
            for (uint32_t l = 0; l <= c->L; ++l) c->last_a[l] = h.set[l].a;
        c->last_n_ops = multi ? 0u : n;
        c->hints_valid = !multi;
    }
    c->payload = nullptr;                          // never leave the caller's buffer in the context
    if (rc != RIPPLE_OK) {
        // Pieces before the failing one stay applied and fully propagated (the state is that of the batch's
        // first ops_done operations); the failing piece changed nothing. Say how far the batch got.
        (void)hipStreamSynchronize(s);
        c->timer->recs.clear();
        c->timer->used = 0;
        c->hints_valid = false;
        if (res) {
            res->n_ops = n_ops;
            res->n_ops_done = ops_done;
            res->n_applied = applied;
            res->n_rejected = rejected;
            res->n_sub_batches = (uint32_t)pieces.size();
            res->n_compactions = compactions;
            res->n_structural = n_struct;
            if (ops_done) {                        // counters of the last piece that went through
                res->n_alive = c->ctr_host->n_alive;
                res->n_edges = c->ctr_host->n_edges;
            }
        }
        if (multi && ops_done) {                   // the sets reported are those of the applied pieces
            for (uint32_t l = 0; l <= c->L; ++l) rp_launch_bitmap_to_list(c, c->rep[l], c->all_list, 0xFFFFFFFFu, &c->ctr->set[l].a);
            c->ctr_dirty = true;
            if (hipMemcpyAsync(c->ctr_host, c->ctr, sizeof(DevCtr), hipMemcpyDeviceToHost, s) == hipSuccess &&
                hipStreamSynchronize(s) == hipSuccess)
                for (uint32_t l = 0; l <= c->L; ++l) {
                    c->last_a[l] = c->ctr_host->set[l].a;
                    if (res) res->affected[l] = c->last_a[l];
                }
            c->last_from_rep = true;
        }
        return rc;
    }
    RP_HIP(c, hipGetLastError());
    if (multi) {                                   // sizes of the united sets
        for (uint32_t l = 0; l <= c->L; ++l) rp_launch_bitmap_to_list(c, c->rep[l], c->all_list, 0xFFFFFFFFu, &c->ctr->set[l].a);
        c->ctr_dirty = true;
        RP_HIP(c, hipMemcpyAsync(c->ctr_host, c->ctr, sizeof(DevCtr), hipMemcpyDeviceToHost, s));
        RP_HIP(c, hipStreamSynchronize(s));
        for (uint32_t l = 0; l <= c->L; ++l) c->last_a[l] = c->ctr_host->set[l].a;
    }
    c->last_from_rep = multi;
    rp_timer_end(c, t_total, RIPPLE_PH_TOTAL, 0);
    if (c->opt_timing) {
        RP_HIP(c, hipStreamSynchronize(s));
        timer_collect(c);
        c->stats.batches += 1;
        for (uint32_t l = 0; l <= c->L; ++l) {
            c->stats.rows[l] += c->last_a[l];
            c->stats.msgs[l] += msgs[l];
            c->stats.touched[l] += tchd[l];
        }
    }
    if (res) {
        res->n_ops = n_ops;
        res->n_ops_done = n_ops;
        res->n_applied = applied;
        res->n_rejected = rejected;
        res->n_sub_batches = (uint32_t)pieces.size();
        res->n_compactions = compactions;
        res->n_alive = c->ctr_host->n_alive;
        res->n_edges = c->ctr_host->n_edges;
        res->n_structural = n_struct;
        for (uint32_t l = 0; l <= c->L; ++l) {
            res->affected[l] = c->last_a[l];
            res->messages[l] = msgs[l];
            res->mono_unchanged[l] = mono[0][l];
            res->mono_incremental[l] = mono[1][l];
            res->mono_recomputed[l] = mono[2][l];
            res->hop_mode[l] = hop_mode[l];
        }
    }
    if (range_rows) return range_error(c, range_rows);      // the batch is applied; res describes it
    return RIPPLE_OK;
}

// ---------------------------------------------------------------------------------
// read-back
// ---------------------------------------------------------------------------------
static ripple_status gather_rows(ripple_ctx *c, const void *M, int store, uint32_t d, const uint32_t *ids,
                                 uint32_t n_ids, float *out) {
    if (n_ids == 0) return RIPPLE_OK;
    if (!out) return fail(c, RIPPLE_EINVAL, "null output pointer");
    hipStream_t s = c->stream;
    if (!ids && n_ids > c->n_cap) return fail(c, RIPPLE_EINVAL, "more rows requested than vertex_capacity");
    const uint32_t *ids_d = nullptr;
    if (ids) {
        if (is_device_ptr(c, ids)) {
            ids_d = ids;
        } else {
            for (uint32_t i = 0; i < n_ids; ++i)
                if (ids[i] >= c->n_cap) return fail(c, RIPPLE_EINVAL, "vertex id out of range");
            if (n_ids <= IO_PIN_IDS) {
                memcpy(c->io_pin + 16, ids, (size_t)n_ids * 4);
                ids_d = c->io_pin + 16;
            } else {
                if (n_ids > c->gather_ids_cap) {
                    if (c->gather_ids) hipFree(c->gather_ids);
                    c->gather_ids = nullptr;
                    c->gather_ids_cap = 0;
                    RP_TRY(dev_alloc(c, &c->gather_ids, (size_t)n_ids, false));
                    c->gather_ids_cap = n_ids;
                }
                RP_HIP(c, hipMemcpyAsync(c->gather_ids, ids, (size_t)n_ids * 4, hipMemcpyHostToDevice, s));
                ids_d = c->gather_ids;
            }
        }
    }
    const Place place = place_of(c, out);
    const size_t total = (size_t)n_ids * d;
    if (!ids && !store && place != ON_HOST) {                // contiguous float32 rows
        if (place == OWN_GPU) {                              // (4.6 M numbers 26 us with the runtime's copy and the wait for the stream, 14 so)
            const uint32_t gb = (uint32_t)std::min<size_t>((total + 4095) / 4096, c->n_cu * 8);
            const HostFlag done = gb <= REPORT_WGS ? rp_host_flag(c) : HostFlag{nullptr, 0u, nullptr};
            hipLaunchKernelGGL(k_copy_numbers, dim3(gb), dim3(256), 0, s, (const float *)M, out, total, done);
            if (!done.flag) rp_launch_report(c);
            return rp_wait_flag(c);
        }
        RP_HIP(c, hipMemcpyAsync(out, M, total * 4, hipMemcpyDefault, s));
        RP_HIP(c, hipStreamSynchronize(s));
        return RIPPLE_OK;
    }
    auto launch = [&](size_t r0, size_t rows, float *to, bool report) {
        const uint32_t gb = (uint32_t)std::min<size_t>((rows * ((d + 3) / 4) + 255) / 256, c->n_cu * 16);
        const uint32_t *from = ids_d ? ids_d + r0 : nullptr;
        const HostFlag done = (report && gb <= REPORT_WGS) ? rp_host_flag(c) : HostFlag{nullptr, 0u, nullptr};
        if (store) hipLaunchKernelGGL(k_gather_rows<1>, dim3(gb), dim3(256), 0, s, M, d, from, (uint32_t)r0, rows, c->n_cap, to, done);
        else hipLaunchKernelGGL(k_gather_rows<0>, dim3(gb), dim3(256), 0, s, M, d, from, (uint32_t)r0, rows, c->n_cap, to, done);
        if (report && !done.flag) rp_launch_report(c);
    };
    if (place == OWN_GPU) {
        launch(0, n_ids, out, true);
        return rp_wait_flag(c);
    }
    if (place == ON_HOST) {
        float *pinned = (float *)(c->io_pin + 16 + IO_PIN_IDS);
        if (total <= READ_FLOATS) {
            launch(0, n_ids, pinned, true);
            RP_TRY(rp_wait_flag(c));
            memcpy(out, pinned, total * 4);
            return RIPPLE_OK;
        }
        const uint32_t piece = READ_FLOATS / d, half = piece * READ_PIECES;          // rows (of at most 1,024 numbers)
        uint32_t seq[2];
        auto fill = [&](uint32_t k) {                       // rows k * half .. into half k % 2
            const uint32_t r0 = k * half, rows = std::min(half, n_ids - r0), h = k % 2u;
            seq[h] = ++c->read_seq;
            const auto kernel = store ? k_gather_pieces<1> : k_gather_pieces<0>;
            hipLaunchKernelGGL(kernel, dim3(PIECE_WGS * std::min(PIECE_TEAMS, rp_div_up(rows, piece))), dim3(256), 0, s, M, d, ids_d ? ids_d + r0 : nullptr, r0, rows, piece, c->n_cap,
                               pinned + (size_t)h * READ_PIECES * READ_FLOATS, c->read_flag + h * READ_PIECES * 16u, seq[h], c->ctr->piece_done);
        };
        const uint32_t n_halves = rp_div_up(n_ids, half);
        for (uint32_t k = 0; k < std::min(n_halves, 2u); ++k) fill(k);
        for (uint32_t k = 0; k < n_halves; ++k) {
            const uint32_t h = k % 2u;
            for (uint32_t p = 0, r = k * half; p < READ_PIECES && r < n_ids; ++p, r += piece) {
                RP_TRY(wait_word(c, c->read_flag + (h * READ_PIECES + p) * 16u, seq[h]));
                memcpy(out + (size_t)r * d, pinned + (size_t)(h * READ_PIECES + p) * READ_FLOATS, (size_t)std::min(piece, n_ids - r) * d * 4);
            }
            if (k + 2u < n_halves) fill(k + 2u);
        }
        return RIPPLE_OK;
    }
    const size_t chunk_rows = std::max<size_t>(1, ((size_t)64 << 20) / d);
    const size_t need = std::min<size_t>(chunk_rows, n_ids) * d;
    if (need > c->gather_cap) {
        if (c->gather_d) hipFree(c->gather_d);
        c->gather_d = nullptr;
        c->gather_cap = 0;
        RP_TRY(dev_alloc(c, &c->gather_d, need, false));
        c->gather_cap = need;
    }
    for (size_t r0 = 0; r0 < n_ids; r0 += chunk_rows) {
        size_t rows = std::min<size_t>(chunk_rows, n_ids - r0);
        launch(r0, rows, c->gather_d, false);
        RP_HIP(c, hipMemcpyAsync(out + r0 * d, c->gather_d, rows * d * 4, hipMemcpyDefault, s));   // another GPU's
        RP_HIP(c, hipStreamSynchronize(s));
    }
    return RIPPLE_OK;
}

extern "C" ripple_status ripple_get_embeddings(ripple_ctx *c, uint32_t layer, const uint32_t *ids, uint32_t n_ids,
                                               float *out) {
    if (!c) return RIPPLE_EINVAL;
    if (c->state < 1 || (layer > 0 && c->state < 3)) return fail(c, RIPPLE_ESTATE, "embeddings not computed yet");
    if (layer > c->L) return fail(c, RIPPLE_EINVAL, "layer out of range");
    return gather_rows(c, c->H[layer], c->store, c->d[layer], ids, n_ids, out);
}

extern "C" ripple_status ripple_get_aggregates(ripple_ctx *c, uint32_t layer, const uint32_t *ids, uint32_t n_ids,
                                               float *out) {
    if (!c) return RIPPLE_EINVAL;
    if (c->state < 3) return fail(c, RIPPLE_ESTATE, "aggregates not computed yet");
    if (layer == 0 || layer > c->L) return fail(c, RIPPLE_EINVAL, "layer out of range");
    return gather_rows(c, c->X[layer], 0, c->xw[layer], ids, n_ids, out);
}

extern "C" ripple_status ripple_get_layer_info(ripple_ctx *c, uint32_t layer, uint32_t *aggregate_width,
                                                int *projected) {
    if (!c) return RIPPLE_EINVAL;
    if (c->state < 2) return fail(c, RIPPLE_ESTATE, "no model loaded");
    if (layer == 0 || layer > c->L) return fail(c, RIPPLE_EINVAL, "layer out of range");
    if (aggregate_width) *aggregate_width = c->xw[layer];
    if (projected)
        *projected = (int)(c->layers[layer - 1].proj | (c->layers[layer - 1].selfc << 1) |
                           ((c->layers[layer - 1].proj && c->layers[layer - 1].packed) ? 4u : 0u));
    return RIPPLE_OK;
}

extern "C" ripple_status ripple_get_affected(ripple_ctx *c, uint32_t layer, uint32_t *ids_out, uint32_t cap,
                                             uint32_t *n_out) {
    if (!c) return RIPPLE_EINVAL;
    if (c->state != 3) return fail(c, RIPPLE_ESTATE, "no batch has been applied");
    if (layer > c->L || !n_out || (cap && !ids_out)) return fail(c, RIPPLE_EINVAL, "bad argument");
    uint32_t *bitmap = c->last_from_rep ? c->rep[layer] : c->bm[layer];
    const bool direct = cap <= IO_PIN_IDS;         // the ids go straight to pinned host memory
    rp_launch_bitmap_to_list(c, bitmap, direct ? c->io_pin + 16 : c->all_list, cap, c->io_pin, true);
    RP_TRY(rp_wait_flag(c));
    const uint32_t n = c->io_pin[0];
    *n_out = n;
    uint32_t m = std::min(n, cap);
    if (direct) memcpy(ids_out, c->io_pin + 16, (size_t)m * 4);
    else if (m) RP_HIP(c, hipMemcpy(ids_out, c->all_list, (size_t)m * 4, hipMemcpyDeviceToHost));
    return RIPPLE_OK;
}

extern "C" ripple_status ripple_get_affected_static(ripple_ctx *c, uint32_t layer, uint32_t *ids_out, uint32_t cap,
                                                    uint32_t *n_out) {
    if (!c) return RIPPLE_EINVAL;
    if (c->state != 3) return fail(c, RIPPLE_ESTATE, "no batch has been applied");
    if (layer > c->L || !n_out || (cap && !ids_out)) return fail(c, RIPPLE_EINVAL, "bad argument");
    if (!is_device_ptr(c, n_out) || (cap && !is_device_ptr(c, ids_out)))
        return fail(c, RIPPLE_EINVAL, "ids_out and n_out must be device memory");
    return rp_launch_affected_static(c, c->last_from_rep ? c->rep[layer] : c->bm[layer], ids_out, cap, n_out);
}

extern "C" ripple_status ripple_export_edges(ripple_ctx *c, int direction, uint32_t *src_out, uint32_t *dst_out,
                                             uint64_t cap, uint64_t *n_out) {
    if (!c) return RIPPLE_EINVAL;
    if (c->state < 1) return fail(c, RIPPLE_ESTATE, "no graph");
    if (!n_out || (direction != 0 && direction != 1)) return fail(c, RIPPLE_EINVAL, "bad argument");
    hipStream_t s = c->stream;
    const uint2 *meta = direction ? c->in_meta : c->out_meta;
    const uint32_t *pool = direction ? c->in_pool : c->out_pool;
    uint32_t *len = nullptr, *off = nullptr, *total_d = nullptr, *sd = nullptr, *dd = nullptr;
    RP_TRY(dev_alloc(c, &len, (size_t)c->n_cap, false));
    RP_TRY(dev_alloc(c, &off, (size_t)c->n_cap, false));
    RP_TRY(dev_alloc(c, &total_d, 16, true));
    uint32_t vb = rp_div_up(c->n_cap, 256);
    hipLaunchKernelGGL(k_meta_len2, dim3(vb), dim3(256), 0, s, meta, c->n_cap, len);
    rp_exclusive_scan(s, len, off, c->n_cap, c->part_cnt, total_d);
    uint32_t total = 0;
    RP_HIP(c, hipMemcpyAsync(&total, total_d, 4, hipMemcpyDeviceToHost, s));
    RP_HIP(c, hipStreamSynchronize(s));
    *n_out = total;
    ripple_status rc = RIPPLE_OK;
    if (total && total <= cap) {
        if (!src_out || !dst_out) rc = fail(c, RIPPLE_EINVAL, "null output pointer");
        else {
            rc = dev_alloc(c, &sd, (size_t)total, false);
            if (rc == RIPPLE_OK) rc = dev_alloc(c, &dd, (size_t)total, false);
            if (rc == RIPPLE_OK) {
                hipLaunchKernelGGL(k_export_rows, dim3(c->n_cu * 8), dim3(256), 0, s, meta, pool, off, c->n_cap,
                                   direction, sd, dd);
                hipMemcpyAsync(src_out, sd, (size_t)total * 4, hipMemcpyDeviceToHost, s);
                hipMemcpyAsync(dst_out, dd, (size_t)total * 4, hipMemcpyDeviceToHost, s);
                if (hipStreamSynchronize(s) != hipSuccess) rc = fail(c, RIPPLE_EDEVICE, "export failed");
            }
        }
    }
    hipFree(len);
    hipFree(off);
    hipFree(total_d);
    if (sd) hipFree(sd);
    if (dd) hipFree(dd);
    return rc;
}

extern "C" ripple_status ripple_get_degrees(ripple_ctx *c, int direction, uint32_t *deg_out, uint8_t *alive_out) {
    if (!c) return RIPPLE_EINVAL;
    if (c->state < 1) return fail(c, RIPPLE_ESTATE, "no graph");
    if (direction != 0 && direction != 1) return fail(c, RIPPLE_EINVAL, "bad direction");
    hipStream_t s = c->stream;
    if (deg_out) {
        uint32_t *len = nullptr;
        RP_TRY(dev_alloc(c, &len, (size_t)c->n_cap, false));
        hipLaunchKernelGGL(k_meta_len2, dim3(rp_div_up(c->n_cap, 256)), dim3(256), 0, s,
                           direction ? c->in_meta : c->out_meta, c->n_cap, len);
        hipMemcpyAsync(deg_out, len, (size_t)c->n_cap * 4, hipMemcpyDeviceToHost, s);
        hipError_t e = hipStreamSynchronize(s);
        hipFree(len);
        if (e != hipSuccess) return fail(c, RIPPLE_EDEVICE, "degree read-back failed");
    }
    if (alive_out) {
        std::vector<uint32_t> bm(c->n_words);
        RP_HIP(c, hipMemcpy(bm.data(), c->alive, (size_t)c->n_words * 4, hipMemcpyDeviceToHost));
        for (uint32_t v = 0; v < c->n_cap; ++v) alive_out[v] = (bm[v >> 5] >> (v & 31)) & 1u;
    }
    return RIPPLE_OK;
}

extern "C" ripple_status ripple_compact(ripple_ctx *c) {
    if (!c) return RIPPLE_EINVAL;
    if (c->state < 1) return fail(c, RIPPLE_ESTATE, "no graph");
    return rp_compact(c);
}

extern "C" ripple_status ripple_set_option(ripple_ctx *c, int option, int64_t value) {
    if (!c) return RIPPLE_EINVAL;
    switch (option) {
    case RIPPLE_OPT_TIMING: c->opt_timing = value ? 1 : 0; return RIPPLE_OK;
    case RIPPLE_OPT_SCATTER_MODE:
        if (value < 0 || value > 3) return fail(c, RIPPLE_EINVAL, "scatter mode must be 0, 1, 2 or 3");
        c->opt_scatter = (int)value;
        return RIPPLE_OK;
    case RIPPLE_OPT_DETERMINISTIC:
        if (c->state != 1) return fail(c, RIPPLE_ESTATE, "the deterministic mode is chosen before load_model");
        c->opt_deterministic = value ? 1 : 0;
        return RIPPLE_OK;
    case RIPPLE_OPT_SELF_CACHE:
        if (c->state != 1) return fail(c, RIPPLE_ESTATE, "the self-projection cache is chosen before load_model");
        c->opt_selfcache = value ? 1 : 0;
        return RIPPLE_OK;
    case RIPPLE_OPT_SPLIT_MFMA:
        if (c->state != 1) return fail(c, RIPPLE_ESTATE, "RIPPLE_OPT_SPLIT_MFMA must be set before load_model");
        c->opt_split = value ? 1 : 0;
        return RIPPLE_OK;
    case RIPPLE_OPT_BF16_MFMA:
        c->opt_bf16_mfma = value ? 1 : 0;
        return RIPPLE_OK;
    case RIPPLE_OPT_SPARSE_FRONTIER:
        c->opt_sparse = value ? 1 : 0;
        return RIPPLE_OK;
    case RIPPLE_OPT_ROW_SEGMENTS:
        if (value < 0) return fail(c, RIPPLE_EINVAL, "the number of row segments cannot be negative");
        c->seg_limit = (uint32_t)std::min<long long>(value, 0xffffffffll);
        return RIPPLE_OK;
    case RIPPLE_OPT_PROJECT_FIRST:
        if (c->state != 1) return fail(c, RIPPLE_ESTATE, "project-first must be chosen before load_model");
        c->opt_project = value ? 1 : 0;
        return RIPPLE_OK;
    case RIPPLE_OPT_PACKED_MESSAGES:
        if (c->state != 1) return fail(c, RIPPLE_ESTATE, "packed messages must be chosen before load_model");
        c->opt_pack = value ? 1 : 0;
        return RIPPLE_OK;
    case RIPPLE_OPT_STREAM_TRANSFORM:
        if (value < 0 || value > 2) return fail(c, RIPPLE_EINVAL, "RIPPLE_OPT_STREAM_TRANSFORM must be 0, 1 or 2");
        c->opt_stream = (int)value;
        return RIPPLE_OK;
    case RIPPLE_OPT_SORTED_MESSAGES:
        if (value < 0 || value > 2) return fail(c, RIPPLE_EINVAL, "RIPPLE_OPT_SORTED_MESSAGES must be 0, 1 or 2");
        c->opt_sorted = (int)value;
        return RIPPLE_OK;
    case RIPPLE_OPT_PULL_RATIO:
        if (value < 1 || value > 1024) return fail(c, RIPPLE_EINVAL, "pull ratio must be in 1..1024");
        c->opt_pull_ratio = (int)value;
        return RIPPLE_OK;
    default: return fail(c, RIPPLE_EINVAL, "unknown option");
    }
}

extern "C" ripple_status ripple_get_stats(ripple_ctx *c, ripple_stats *out, int reset) {
    if (!c || !out) return RIPPLE_EINVAL;
    *out = c->stats;
    if (reset) memset(&c->stats, 0, sizeof(c->stats));
    return RIPPLE_OK;
}
