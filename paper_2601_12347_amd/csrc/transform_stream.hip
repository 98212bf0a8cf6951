#include "kernels.h"
#include "rows.h"

// Row transform of many rows (the Compute step of Sec. 3.3 in re-apply form, and the products of the previous embedding that a
// layer caches), fp32 numbers on the bf16 matrix cores.
//
// A product of fp32 numbers: x = x0 + x1 + x2 and w = w0 + w1 + w2 with bf16 numbers, each the rounding of what the ones before it
// leave (exact to 2^-26 of x), and x w is the six largest of the nine products; the three left out are below 2^-24 x w together.
// x0 w0 and the five others go to two accumulators, so the small terms are not rounded to the large sum's last bit on the way.
// Against 64-bit sums the rows are closer than a chain of fp32 products: 2-norm of the error over that of the result, K = 256,
// normal / rectified rows: 8.5e-8 / 6.6e-8 (fp32 matrix cores 2.9e-7 / 2.0e-7; K = 32: 3.9e-8 against 1.0e-7; K = 96 and 128 in between).
// What bounds it: six products of a bf16 rate of 1.7 to 2.1 PFLOP/s (dense matrix products of numbers that are not zero lower the clock;
// 2.4 with zeros) and memory, neither at its limit: 1.5 M rows 256 -> 256 with a cached row keep the matrix cores busy 42 % of the cycles, at
// 2.0 GHz, and move 3.6 TB/s, because a compute unit's one workgroup converts, stores and waits at its slices' barriers in between; fp32
// products reach 138 TFLOP/s, 3/8 of that in the end. Measured, fp32 products
// (persistent workgroups for 256 -> 256, 32 x 128 tiles otherwise) -> now: 1.5 M rows 256 -> 256 with a cached row 1.66 -> 1.35 ms
// (4.6 GB moved), 612 K rows 0.68 -> 0.53, without it 0.84 -> 0.46, 100 -> 256 0.49 -> 0.32 and 0.55 -> 0.38, both products of 256 -> 47
// 1.5 M rows 0.73 -> 0.71 and 612 K 0.28 -> 0.27; 1.5 M bf16 rows 256 -> 47 0.53 -> 0.29. fp32 rows to at most 64 columns stay with the
// tiles of k_transform_split: tiles / this kernel, 256 -> 47, 65,536 rows 27.7 / 29.6 us, 98,304 rows 39.3 / 44.1, 131,072 rows 50.2 / 46.8, 262,144
// rows 103 / 83 (not taken: the bootstrap and the largest hops of such a layer would gain).
// Other shapes of the same kernel: two workgroups of four wavefronts without a parked tile 1.50 ms for the first of these, four
// wavefronts that only fetch and eight that only multiply 1.6, products of 16 x 16 x 32 no difference.
// Rows stored in bf16 are exact as they are: three products.
// What a sum of finite products cannot show: infinities and NaNs of the rows or the weights, and numbers that bf16 rounds to
// infinity, leave a sum that is not finite (x1 = x - x0 is a NaN then). Such an element is stored as a NaN, beside it the old value, and made
// again on the fp32 matrix cores once the wavefront has no tile left: in the loop it would cost registers that the loop does not have
// (the parked tile's sums and the next tile's are all live there).
//
// A workgroup of eight wavefronts per compute unit is persistent and owns tiles of BM rows by all N columns; a wavefront has 64 rows
// by 32 columns of one. No part of a tile waits for memory on its own:
//  * the weights never pass through LDS: they come from the L2 in the order in which the matrix cores take them (k by eights), 16
//    bytes per lane and part, two steps of 16 k ahead;
//  * the gathered rows pass through a double-buffered LDS slice of 32 or 64 k (one barrier per slice), split as they are written there from
//    registers requested two slices earlier, also across the tile boundary;
//  * the finished tile's sums are parked in registers and leave for memory in eight chunks during the slices of the next tile; the
//    cached / old values that a chunk is combined with are requested two slices before the chunk is finished;
//  * the mean's 1/deg is applied to the finished row.
// Every array is addressed through a buffer descriptor with 32-bit offsets (as flat addresses the unrolled slices kept dozens of
// 64-bit pointers alive): arrays of less than 4 GB.
struct StreamArgs {
    TArgs t;
    uint32_t x_row, x_bytes;       // gathered rows: stride and extent in bytes
    uint32_t o_row, o_bytes;       // rows written (H, D, addend / tmp_out): stride and extent in bytes
    uint32_t o2_row, o2_bytes;     // tmp_out2
};

// Sums that were not finite (see above): a wavefront goes over its blocks of 32 x 32 once more, and those that hold a NaN are multiplied again as
// fp32 numbers. A lane looks at the elements it has stored itself; where the sum was finite after all and only what it was added to was
// not, the same NaN comes out. Bootstrap of 169 K rows, 128 -> 256 -> 256 -> 40, SAGE: 1.06 ms with finite features, 1.32 with a NaN at the
// largest hub, 2.6 with an infinity in every row; with the products made one after the other where the sum was finished 1.68 and 28 ms, and
// 1 to 14 registers spilled in most of the shapes.
template <int BM, int TM, int WN, int MODE, int STORE, int OUT, bool ADD, bool DELTA>
__device__ __forceinline__ void blocks_again(const StreamArgs &sa) {
    const TArgs &a = sa.t;
    const uint32_t count = *a.count_ptr, n_tiles = (count + BM - 1) / BM, lane = threadIdx.x & 63u, wave = threadIdx.x >> 6, wn = wave % WN, wm = wave / WN;
    const uint32_t col = wn * 32u + (lane & 31u);
    const bool second = OUT == 0 && a.split_col && wn * 32u >= a.split_col;
    const uint32_t ocol = second ? col - a.split_col : col, ld = OUT == 1 ? a.N : (second ? a.tmp_out2_ld : a.tmp_out_ld);
    const uint32_t lim = OUT == 0 && a.split_col ? (second ? a.N - a.split_col : a.N1) : a.N;
    float *out = OUT == 1 ? (float *)a.Hout : (second ? a.tmp_out2 : a.tmp_out);
    const float bias = a.bias[col];
#pragma unroll 1
    for (uint32_t tile = blockIdx.x; tile < n_tiles; tile += gridDim.x)
#pragma unroll 1
        for (uint32_t i = 0; i < (uint32_t)TM; ++i) {
            const uint32_t row0 = tile * BM + (wm * TM + i) * 32u;
            size_t at[16];                                 // where this lane's elements lie; not stored: `there` clear
            uint32_t there = 0, nans = 0;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const uint32_t slot = row0 + (uint32_t)(r >> 2) * 8u + (lane >> 5) * 4u + (r & 3), s = min(slot, count - 1u);
                at[r] = (size_t)(OUT == 0 && a.out_mode == 0 ? s : a.list[s]) * ld + min(ocol, lim - 1u);
                there |= (slot < count && ocol < lim ? 1u : 0u) << r;
            }
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const float z = out[at[r]];
                nans |= (z != z ? 1u : 0u) << r;
            }
            nans &= there;
            if (!__any(nans != 0u)) continue;
            const uint32_t slot = min(row0 + (lane & 31u), count - 1u), v = a.list[slot], deg = a.mean ? a.in_meta[v].y : 1u;
            const floatx16 sum = fp32_block<MODE, STORE>(a, slot, v, 1.0f / (float)(deg > 1u ? deg : 1u), col, (int)lane);
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                if (!(nans >> r & 1u)) continue;
                float z = sum[r] + bias;
                if (ADD) z += a.addend[at[r]];
                if (a.act == RIPPLE_ACT_RELU) z = z > 0.0f ? z : 0.0f;
                out[at[r]] = z;
                if (DELTA && !a.d_old) a.D[at[r]] = z - a.D[at[r]];   // the old value is there
            }
        }
}

// SW: k per slice, KS slices (K <= SW KS); WN: wavefronts side by side (32 WN columns); MODE, STORE: see fetch_raw (MODE 0, 2, 3, 4).
// OUT 0: the product goes to tmp_out (and tmp_out2). 1: H is updated; ADD: plus an unscaled cached row, DELTA: the delta row is written too.
template <int SW, int KS, int WN, int MODE, int STORE, int OUT, bool ADD, bool DELTA>
__global__ __launch_bounds__(512, 2) void k_split_stream(StreamArgs sa) {
    static_assert(OUT == 1 || (!ADD && !DELTA), "products are stored as they are");
    constexpr int WM = 8 / WN, TM = 2, BM = 32 * TM * WM;                     // a wavefront: TM blocks of 32 x 32
    constexpr int TPR = SW / 4, RPP = 512 / TPR, NA = BM / RPP;               // staging: threads per row, rows at a time, groups of four per thread and slice
    constexpr int NC = 4 * TM, SPS = SW / 16, STEPS = SPS * KS, EVERY = STEPS / NC;           // chunks of a tile; steps of 16 k of a slice and a tile, steps per chunk
    constexpr int LEAD = 2;                                // chunks requested ahead
    constexpr int PL = STORE ? 1 : 3;                      // parts of a row number
    constexpr int BQ = 2;                                  // steps whose weights are held or on their way
    constexpr int LD = SW + 8;                             // LDS row stride in bf16 (eight rows cover all banks)
    constexpr bool TWO = MODE == 2;
    static_assert(EVERY >= 1 && STEPS % BQ == 0 && NC % LEAD == 0, "schedule");
    __shared__ __attribute__((aligned(16))) unsigned short As[2][PL][BM][LD];
    __shared__ uint32_t s_again[8];                        // a wavefront has stored NaNs in place of sums that have to be made again
    __shared__ uint32_t s_row[2][BM];                      // output row of every slot of the tile
    __shared__ float s_scale[MODE == 0 ? 2 : 1][MODE == 0 ? BM : 1];

    const TArgs &a = sa.t;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, wn = wave % WN, wm = wave / WN;
    const uint32_t count = *a.count_ptr;
    const uint32_t n_tiles = (count + BM - 1) / BM;
    uint32_t tile = blockIdx.x;
    if (tile >= n_tiles) return;

    if (tid < 8) s_again[tid] = 0;
    constexpr uint32_t RSRC3 = 0x00020000u, NOWHERE = 0xFFFFF000u;        // beyond every array: nothing is stored there
    const uint32_t plane = a.wp_k * a.Npad * 2u;           // bytes of one part of the weights
    const __amdgpu_buffer_rsrc_t wres = __builtin_amdgcn_make_buffer_rsrc((void *)a.Wp, 0, 3u * plane, RSRC3);
    const void *xsrc = MODE == 0 ? (const void *)a.X : (MODE == 3 ? (const void *)a.tmp_in : a.Hprev);
    const __amdgpu_buffer_rsrc_t xres = __builtin_amdgcn_make_buffer_rsrc((void *)xsrc, 0, sa.x_bytes, RSRC3);
    const __amdgpu_buffer_rsrc_t qres = __builtin_amdgcn_make_buffer_rsrc((void *)(TWO ? (const void *)a.X : xsrc), 0, sa.x_bytes, RSRC3);
    const bool second = OUT == 0 && a.split_col && wn * 32u >= a.split_col;   // this wavefront's columns are the second product's
    const uint32_t out_row = second ? sa.o2_row : sa.o_row;
    const __amdgpu_buffer_rsrc_t ores = __builtin_amdgcn_make_buffer_rsrc(
        OUT == 1 ? a.Hout : (void *)(second ? a.tmp_out2 : a.tmp_out), 0, second ? sa.o2_bytes : sa.o_bytes, RSRC3);
    const __amdgpu_buffer_rsrc_t pres = __builtin_amdgcn_make_buffer_rsrc((void *)(ADD ? a.addend : a.X), 0, ADD ? sa.o_bytes : 0u, RSRC3);
    const __amdgpu_buffer_rsrc_t dres = __builtin_amdgcn_make_buffer_rsrc((void *)(DELTA ? a.D : (float *)a.X), 0, DELTA ? sa.o_bytes : 0u, RSRC3);

    const uint32_t c4a = tid % TPR * 4u;
    const uint32_t r_own = tid / TPR;                      // this thread stages rows r_own + RPP i of every slice
    const uint32_t col = wn * 32u + (lane & 31u);
    const uint32_t ocol = second ? col - a.split_col : col;                   // column of the array it is stored in
    const uint32_t lim = OUT == 0 && a.split_col ? (second ? a.N - a.split_col : a.N1) : a.N;
    const bool stored = ocol < lim;                        // (padding columns are not)
    const uint32_t colb = ocol * 4u;
    const uint32_t wvo = ((lane >> 5) * a.Npad + col) * 16u;                  // weights: eight k of one column
    const float bias = a.bias[col];                        // (padded)
    const float up = PL == 3 ? PARTS_LIFT : 1.0f, down = 1.0f / (up * a.wp_lift), eps_up = a.one_plus_eps * up;   // (see PARTS_LIFT)
    constexpr uint32_t XB = STORE && MODE != 3 ? 2u : 4u;  // bytes of a gathered number
    const uint32_t k_last = (a.K - 1u) & ~3u;              // first k of a row's last group of four
    const uint32_t kstep = 2u * a.Npad * 16u;              // bytes of the weights of 16 k

    auto row_scale = [&](uint32_t v) {
        const uint32_t deg = a.in_meta[v].y;
        return a.mean ? 1.0f / (float)(deg > 1u ? deg : 1u) : 1.0f;
    };
    // the rows this thread stages, of the current tile and the next two; slots past the end repeat the last one and are never stored
    constexpr bool SCALE = MODE == 0 || TWO;
    uint32_t v_cur[NA], v_nxt[NA], v_far[NA];
    float sc_cur[SCALE ? NA : 1], sc_nxt[SCALE ? NA : 1];
    auto slot_of = [&](uint32_t t, int i) { return min(t * BM + r_own + (uint32_t)RPP * i, count - 1u); };
#pragma unroll
    for (int i = 0; i < NA; ++i) {
        v_cur[i] = a.list[slot_of(tile, i)];
        v_nxt[i] = a.list[slot_of(tile + gridDim.x, i)];
        if constexpr (SCALE) sc_cur[i] = row_scale(v_cur[i]) * (TWO ? up : down);
        if (c4a == 0) {                                    // nothing is parked yet: its rows only have to be valid
            s_row[1][r_own + RPP * i] = (OUT == 0 && a.out_mode == 0) ? 0u : v_cur[i];
            if (MODE == 0) s_scale[1][r_own + RPP * i] = 1.0f;
        }
    }
    floatx4 ra[2][NA], rq[TWO ? 2 : 1][TWO ? NA : 1];
    // (bf16 rows of odd width begin at multiples of two bytes only: a buffer load takes those, like a global one)
    auto load_x = [&](int buf, int i, uint32_t t, uint32_t v, int slice) {
        const uint32_t off = (MODE == 3 ? slot_of(t, i) : v) * sa.x_row + min((uint32_t)slice * SW + c4a, k_last) * XB;
        if (XB == 2u) {
            const uintx2 w = __builtin_bit_cast(uintx2, __builtin_amdgcn_raw_buffer_load_b64(xres, off, 0, 0));
            ra[buf][i].x = __uint_as_float(w.x);
            ra[buf][i].y = __uint_as_float(w.y);
        } else {
            ra[buf][i] = __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(xres, off, 0, 0));
        }
        if constexpr (TWO) rq[buf][i] = __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(qres, off, 0, 0));
    };
    auto stage_x = [&](int buf, int slice, int i, float sc) {                 // slice `slice` from ra[buf] into As[buf]
        floatx4 x = ra[buf][i];
        const uint32_t k = (uint32_t)slice * SW + c4a;
        uintx2 part[PL];
        if (XB == 2u) {                                    // bf16 rows: as they are
            uint32_t w0 = __float_as_uint(x.x), w1 = __float_as_uint(x.y);
            w0 = k + 1u < a.K ? w0 : (k < a.K ? w0 & 0xFFFFu : 0u);
            w1 = k + 3u < a.K ? w1 : (k + 2u < a.K ? w1 & 0xFFFFu : 0u);
            part[0].x = w0;
            part[0].y = w1;
        } else {
            if constexpr (TWO) x = x * eps_up + rq[buf][i] * sc;
            else x = x * up;
            x.x = k < a.K ? x.x : 0.0f;                    // padding, and what was read past the row's end
            x.y = k + 1u < a.K ? x.y : 0.0f;
            x.z = k + 2u < a.K ? x.z : 0.0f;
            x.w = k + 3u < a.K ? x.w : 0.0f;
            split_parts<PL>(x, part);
        }
#pragma unroll
        for (int p = 0; p < PL; ++p) *(uintx2 *)&As[buf][p][r_own + RPP * i][c4a] = part[p];
    };
    uintx4 bq[BQ][3];                                      // weights of step g in bq[g % BQ]
    auto load_w = [&](int g) {
#pragma unroll
        for (int p = 0; p < 3; ++p)
            bq[g % BQ][p] = __builtin_bit_cast(uintx4, __builtin_amdgcn_raw_buffer_load_b128(wres, wvo, (uint32_t)(g % STEPS) * kstep + p * plane, 0));
    };
    bf16x8 av[2][TM][PL];                                  // row operands of step g in av[g & 1]
    auto read_a = [&](int g) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int p = 0; p < PL; ++p)
                av[g & 1][i][p] = __builtin_bit_cast(bf16x8, *(const uintx4 *)&As[(g / SPS) & 1][p][(wm * TM + i) * 32 + (lane & 31)][g % SPS * 16 + (lane >> 5) * 8]);
    };
#pragma unroll
    for (int i = 0; i < NA; ++i) load_x(0, i, tile, v_cur[i], 0);
#pragma unroll
    for (int g = 0; g < BQ; ++g) load_w(g);
#pragma unroll
    for (int i = 0; i < NA; ++i) load_x(1, i, tile, v_cur[i], 1);
#pragma unroll
    for (int i = 0; i < NA; ++i) stage_x(0, 0, i, TWO ? sc_cur[TWO ? i : 0] : 1.0f);
    if (KS > 2)                                            // (KS = 2: the next tile's first slice, requested in this tile's)
#pragma unroll
        for (int i = 0; i < NA; ++i) load_x(0, i, tile, v_cur[i], 2);

    floatx16 acc[TM], cor[TM], done[TM];                   // large terms, small terms, the parked tile's sums
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][r] = cor[i][r] = done[i][r] = 0.0f;
    uint32_t prev_rows = 0;                                // the parked tile's valid rows (0: nothing parked)
    int par = 0;                                           // s_row / s_scale [par]: the current tile, [par ^ 1]: the parked one
    float pa[LEAD][4], po[LEAD][4];                        // cached-row and old values of the chunks in flight
#pragma unroll
    for (int q = 0; q < LEAD; ++q)
#pragma unroll
        for (int j = 0; j < 4; ++j) pa[q][j] = po[q][j] = 0.0f;

    // Chunk c of a tile: sums 4 (c & 3) .. + 3 of block c >> 2, four rows (j) of this lane's column. `buf`: the tile's entry in s_row.
    auto chunk_row = [&](int c, int j) { return (uint32_t)((wm * TM + (c >> 2)) * 32 + (c & 3) * 8 + (lane >> 5) * 4 + j); };
    auto request_chunk = [&](int c, int buf) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t off = stored ? s_row[buf][chunk_row(c, j)] * sa.o_row + colb : NOWHERE;
            if (ADD) pa[c % LEAD][j] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(pres, off, 0, 0));
            if (DELTA) po[c % LEAD][j] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(ores, off, 0, 0));
        }
    };
    auto finish_chunk = [&](int c, int buf) {
        float sum[4];
        uint32_t off[4];
        bool bad = false;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t lr = chunk_row(c, j);
            off[j] = stored && lr < prev_rows ? s_row[buf][lr] * out_row + colb : NOWHERE;
            sum[j] = done[c >> 2][(c & 3) * 4 + j];
            if constexpr (MODE == 0) sum[j] *= s_scale[buf][lr];
            else sum[j] *= down;
            bad |= !__builtin_isfinite(sum[j]);
            float z = sum[j] + bias + (ADD ? pa[c % LEAD][j] : 0.0f);
            if (a.act == RIPPLE_ACT_RELU) z = z > 0.0f ? z : 0.0f;
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(z), ores, off[j], 0, 0);
            if (DELTA) __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(a.d_old ? po[c % LEAD][j] : z - po[c % LEAD][j]), dres, off[j], 0, 0);
        }
        if (__builtin_expect(__any(bad), 0)) {             // (see blocks_again)
            s_again[wave] = 1u;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (__builtin_isfinite(sum[j])) continue;
                __builtin_amdgcn_raw_buffer_store_b32(0x7FC00000u, ores, off[j], 0, 0);
                if (DELTA) __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(po[c % LEAD][j]), dres, off[j], 0, 0);
            }
        }
    };

    for (;;) {
        const uint32_t tile_n = tile + gridDim.x;
#pragma unroll
        for (int i = 0; i < NA; ++i) v_far[i] = a.list[slot_of(tile_n + gridDim.x, i)];
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            // every wavefront is done with slice s - 1 (As[(s + 1) & 1] may be overwritten) and has written its part of slice s
            __syncthreads();
            read_a(SPS * s);
            if (s == 0) {
                if (c4a == 0)                              // this tile's rows, for when it is written out
#pragma unroll
                    for (int i = 0; i < NA; ++i) {
                        s_row[par][r_own + RPP * i] = (OUT == 0 && a.out_mode == 0) ? slot_of(tile, i) : v_cur[i];
                        if constexpr (MODE == 0) s_scale[par][r_own + RPP * i] = sc_cur[i];
                    }
                if constexpr (SCALE)
#pragma unroll
                    for (int i = 0; i < NA; ++i) sc_nxt[i] = row_scale(v_nxt[i]) * (TWO ? up : down);
                if (KS == 2)
#pragma unroll
                    for (int i = 0; i < NA; ++i) load_x(0, i, tile_n, v_nxt[i], 0);
            }
#pragma unroll
            for (int kk = 0; kk < SPS; ++kk) {
                const int g = SPS * s + kk, now = g & 1;
                if (kk + 1 < SPS) read_a(g + 1);                // (the next slice's are read behind the barrier)
                __builtin_amdgcn_sched_barrier(0);
                bf16x8 bv[3];
#pragma unroll
                for (int p = 0; p < 3; ++p) bv[p] = __builtin_bit_cast(bf16x8, bq[g % BQ][p]);
#define TERM(dst, x, w)                                                                                        \
    _Pragma("unroll") for (int i = 0; i < TM; ++i)                                                             \
        dst[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[now][i][x], bv[w], dst[i], 0, 0, 0)
                TERM(cor, 0, 2);
                if constexpr (PL == 3) {
                    TERM(cor, 2, 0);
                    TERM(cor, 1, 1);
                    TERM(cor, 1, 0);
                }
                TERM(cor, 0, 1);
                TERM(acc, 0, 0);
#undef TERM
                __builtin_amdgcn_sched_barrier(0);         // (the scheduler would sink the requests to their use)
                load_w(g + BQ);                            // past the tile's end: the next tile's first steps
                // a chunk of the parked tile, requested LEAD chunks ago, is finished; the one LEAD on is requested (of the tile being
                // multiplied, once the parked one has none left)
                if (g % EVERY == 0) {
                    const int c = g / EVERY;
                    finish_chunk(c, par ^ 1);
                    if (ADD || DELTA) request_chunk((c + LEAD) % NC, c + LEAD < NC ? par ^ 1 : par);
                }
                // slice s + 1 into the other LDS buffer, slice s + 3 into the registers it came from
#pragma unroll
                for (int i = 0; i < NA; ++i)
                    if (i * SPS / NA == kk) {
                        stage_x((s + 1) & 1, (s + 1) % KS, i, TWO ? (s + 1 < KS ? sc_cur[TWO ? i : 0] : sc_nxt[TWO ? i : 0]) : 1.0f);
                        if (KS > 2 || s == 0) load_x((s + 1) & 1, i, s + 3 < KS ? tile : tile_n, s + 3 < KS ? v_cur[i] : v_nxt[i], (s + 3) % KS);
                    }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                done[i][r] = acc[i][r] + cor[i][r];
                acc[i][r] = cor[i][r] = 0.0f;
            }
        prev_rows = min((uint32_t)BM, count - tile * BM);
        par ^= 1;
#pragma unroll
        for (int i = 0; i < NA; ++i) {
            v_cur[i] = v_nxt[i];
            v_nxt[i] = v_far[i];
            if constexpr (SCALE) sc_cur[i] = sc_nxt[i];
        }
        tile = tile_n;
        if (tile >= n_tiles) break;
    }
    // the last tile: its first LEAD chunks are on their way already
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        finish_chunk(c, par ^ 1);
        if ((ADD || DELTA) && c + LEAD < NC) request_chunk(c + LEAD, par ^ 1);
    }
    if (s_again[wave]) {
        auto *args = __builtin_amdgcn_kernarg_segment_ptr();
        asm volatile("" : "+s"(args));                     // read again from memory: nothing of this is kept during the loop
        blocks_again<BM, TM, WN, MODE, STORE, OUT, ADD, DELTA>(*(const StreamArgs *)args);
    }
}

// The weights, times `lift`, as the kernel takes them: three parts, each [Kp / 8][Npad][8] bf16, zero rows from K on
__global__ void k_weight_parts(const float *w, uint32_t K, uint32_t Kp, uint32_t Npad, float lift, unsigned short *out) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= Kp / 8u * Npad) return;
    const uint32_t n = i % Npad, k8 = i / Npad * 8u;
    floatx4 x[2];
#pragma unroll
    for (uint32_t t = 0; t < 8u; ++t) {
        const uint32_t k = k8 + t;
        const float f = k < K ? w[(size_t)k * Npad + n] * lift : 0.0f;
        x[t >> 2][t & 3u] = f;
    }
    uintx2 lo[3], hi[3];
    split_parts<3>(x[0], lo);
    split_parts<3>(x[1], hi);
#pragma unroll
    for (int p = 0; p < 3; ++p) {
        uintx4 q;
        q.x = lo[p].x;
        q.y = lo[p].y;
        q.z = hi[p].x;
        q.w = hi[p].y;
        *(uintx4 *)(out + ((size_t)p * (Kp / 8u) * Npad + i) * 8u) = q;
    }
}

size_t rp_weight_parts_size(uint32_t K, uint32_t Npad) { return (size_t)3 * rp_round_up(K, 128) * Npad; }
void rp_launch_weight_parts(ripple_ctx *c, const float *w, uint32_t K, uint32_t Npad, float lift, unsigned short *out) {
    const uint32_t kp = rp_round_up(K, 128);
    hipLaunchKernelGGL(k_weight_parts, dim3(rp_div_up(kp / 8u * Npad, 256)), dim3(256), 0, c->stream, w, K, kp, Npad, lift, out);
}

// K: 128 or 256, the rows of the weights' parts. Slices of 64 k where the tile has 64 rows; tiles of 128 and 256 rows have no room for
// them in registers and LDS.
template <int K>
static bool launch_k(ripple_ctx *c, const StreamArgs &s) {
    const TArgs &a = s.t;
    const dim3 grid(c->opt_stream == 2 ? 2u : c->n_cu), block(512);   // 2: small products cross tile boundaries too
#define GO(WN, ...) hipLaunchKernelGGL((k_split_stream<(WN == 8 ? 64 : 32), K / (WN == 8 ? 64 : 32), WN, __VA_ARGS__>), grid, block, 0, c->stream, s)
    if (a.a_mode == 4) {
        if (a.Npad == 256 && !a.store) GO(8, 4, 0, 0, false, false);
        else if (a.Npad == 128 && !a.store) GO(4, 4, 0, 0, false, false);
        else if (a.Npad == 128) GO(4, 4, 1, 0, false, false);
        else if (a.Npad == 64) GO(2, 4, 1, 0, false, false);
        else return false;
    } else if (a.a_mode == 0) {
#define ROWS(WN)                                                       \
    do {                                                               \
        if (a.addend && a.D) GO(WN, 0, 0, 1, true, true);              \
        else if (a.addend) GO(WN, 0, 0, 1, true, false);               \
        else if (a.D) GO(WN, 0, 0, 1, false, true);                    \
        else GO(WN, 0, 0, 1, false, false);                            \
    } while (0)
        if (a.Npad == 256) ROWS(8);
        else ROWS(4);
#undef ROWS
    } else if (a.a_mode == 2) {
        GO(8, 2, 0, 0, false, false);
    } else {
        if (a.D) GO(8, 3, 0, 1, false, true);
        else GO(8, 3, 0, 1, false, false);
    }
#undef GO
    return true;
}

// Enough rows for every persistent workgroup to see two tiles (of 64 rows at 256 padded columns, 128 at 128, 256 at 64): about 14 to 19 us go by
// before the first tile is out, whatever the number of rows, and where only some workgroups have a second tile the others wait. Kernel
// time, tiles of k_transform_split / this kernel, us: 256 -> 256, 8,192 rows 13.2 / 16.7, 16,384 rows (one tile each) 23.7 / 18.9, 24,576 rows
// 30.8 / 28.6, 32,768 rows (two) 39.0 / 31.3; with a cached row 24.8 / 21.7, 31.8 / 33.7 and 40.2 / 36.0; GIN sums 26.3 / 22.8, 37.1 / 34.2 and
// 47.0 / 36.0; both products of 256 -> 47, 49,152 rows (one and a half) 32.6 / 35.7, 65,536 rows (two) 41.4 / 38.1, from bf16 rows 26.6 / 26.6 and
// 33.4 / 27.8; 256 -> 47 from bf16 rows, 98,304 rows 27.0 / 29.3, 131,072 rows (two) 33.9 / 30.9. (One tile each would be 10 to 20 % faster
// here too, but a set a little larger than the previous batch's would be slower.) RIPPLE_OPT_STREAM_TRANSFORM = 2: any number.
#define STREAM_MIN_TILES 2u
bool rp_launch_stream(ripple_ctx *c, const TArgs &a, uint32_t rows_hint) {
    if (!c->opt_stream || !a.Wp || a.K > 256u || a.Npad > 256u || a.Npad < 64u) return false;
    const bool shape = a.a_mode == 4   ? a.out_mode == 2 && (a.Npad == 128u || (a.Npad == 64u) == (a.store != 0))
                       : a.a_mode == 0 ? a.out_mode == 1 && !a.store && !(a.addend && a.addend_scaled) && a.Npad >= 128u
                       : a.a_mode == 2 ? a.out_mode == 0 && !a.store && a.Npad == 256u
                       : a.a_mode == 3 ? a.out_mode == 1 && !a.store && !a.addend && a.Npad == 256u
                                       : false;
    if (!shape) return false;
    if (c->opt_stream != 2 && rows_hint < STREAM_MIN_TILES * c->n_cu * (64u * 256u / a.Npad)) return false;
    StreamArgs s;
    s.t = a;
    uint64_t most = 0;                                     // rows are addressed with 32-bit byte offsets, the top 4 KB kept free
    auto extent = [&](uint64_t row, uint32_t &row_out, uint32_t &bytes) {
        const uint64_t b = (uint64_t)c->n_cap * row + 16u; // (every array has 16 bytes behind its end)
        most = std::max(most, b);
        row_out = (uint32_t)row;
        bytes = (uint32_t)b;
    };
    extent(a.a_mode == 3 ? (uint64_t)a.tmp_ld * 4u : (uint64_t)a.d_in * (a.a_mode == 4 && a.store ? 2u : 4u), s.x_row, s.x_bytes);
    extent(a.out_mode == 1 ? (uint64_t)a.N * 4u : (uint64_t)a.tmp_out_ld * 4u, s.o_row, s.o_bytes);
    s.o2_row = s.o2_bytes = 0;
    if (a.split_col) extent((uint64_t)a.tmp_out2_ld * 4u, s.o2_row, s.o2_bytes);
    if (most > 0xFFFFF000ull) return false;
    return a.K <= 128u ? launch_k<128>(c, s) : launch_k<256>(c, s);
}
