// How the row transforms read and write rows: shared by the tiled kernels and the one for few rows.
#pragma once
#include "transform_args.h"

typedef uint32_t uintx4 __attribute__((ext_vector_type(4)));
typedef uint32_t uintx2 __attribute__((ext_vector_type(2)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ float bf_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf_hi(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }

__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {     // round to nearest even
    const __hip_bfloat16 a = __float2bfloat16(lo), b = __float2bfloat16(hi);
    return (uint32_t)__builtin_bit_cast(unsigned short, a) | ((uint32_t)__builtin_bit_cast(unsigned short, b) << 16);
}

// Rows of any width: a row of 190 or 47 floats starts at a multiple of 4 bytes only, which a 16-byte global load takes all
// the same. The last group of a row may read up to three numbers past its end (the next row's, or, behind the last row,
// the padding dev_alloc puts behind every array); they are zeroed or dropped later.
typedef float floatx4u __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t uintx2u __attribute__((ext_vector_type(2), aligned(2)));    // four bf16 numbers
__device__ __forceinline__ uint32_t last_group(uint32_t n) { return (n - 1u) & ~3u; }   // first column of a row's last group of four

// Raw 16 (or 8) bytes for four consecutive k of one gathered row; no arithmetic on the data.
// MODE 1 with bf16 embeddings and MODE 2 need two sources (p: own embedding, q: aggregate). MODE 1 takes rows whose width
// is a multiple of four only (a group must not straddle the two halves).
template <int MODE, int STORE>
__device__ __forceinline__ void fetch_raw(const TArgs &a, uint32_t v, uint32_t slot, uint32_t k, floatx4 &p, floatx4 &q) {
    const uint32_t kc = min(k, last_group(a.K));
    const size_t row = (size_t)v * a.d_in;
    auto bf4 = [](const void *h, size_t i) {
        const uintx2u r = *(const uintx2u *)((const __hip_bfloat16 *)h + i);
        floatx4 f = (floatx4)(0.0f);
        f.x = __uint_as_float(r.x);
        f.y = __uint_as_float(r.y);
        return f;
    };
    if (MODE == 0) {
        p = *(const floatx4u *)(a.X + row + kc);
    } else if (MODE == 3) {
        p = *(const floatx4u *)(a.tmp_in + (size_t)slot * a.tmp_ld + kc);
    } else if (MODE == 4) {
        if (STORE) p = bf4(a.Hprev, row + kc);
        else p = *(const floatx4u *)((const float *)a.Hprev + row + kc);
    } else if (MODE == 2) {
        q = *(const floatx4u *)(a.X + row + kc);
        if (STORE) p = bf4(a.Hprev, row + kc);
        else p = *(const floatx4u *)((const float *)a.Hprev + row + kc);
    } else {                                                  // MODE 1: k < d_in own embedding, else aggregate
        if (STORE) {
            const uint32_t kh = min(kc, a.d_in - 4u), kx = kc >= a.d_in ? kc - a.d_in : 0u;
            p = bf4(a.Hprev, row + kh);
            q = *(const floatx4u *)(a.X + row + kx);
        } else {
            const float *src = (kc < a.d_in) ? (const float *)a.Hprev + row + kc : a.X + row + (kc - a.d_in);
            p = *(const floatx4u *)src;
        }
    }
}

template <int MODE, int STORE>
__device__ __forceinline__ floatx4 finish_raw(const TArgs &a, floatx4 p, floatx4 q, uint32_t k, float scale) {
    floatx4 h = p;
    if (STORE && (MODE == 1 || MODE == 2 || MODE == 4)) {
        const uint32_t w0 = __float_as_uint(p.x), w1 = __float_as_uint(p.y);
        h.x = bf_lo(w0);
        h.y = bf_hi(w0);
        h.z = bf_lo(w1);
        h.w = bf_hi(w1);
    }
    floatx4 r;
    if (MODE == 0) {
        r = p * scale;
    } else if (MODE == 3) {
        r = p;
    } else if (MODE == 4) {
        r = h;
    } else if (MODE == 2) {
        r = h * a.one_plus_eps + q * scale;
    } else {
        const floatx4 x = STORE ? q : p;
        r = (k < a.d_in) ? h : x * scale;
    }
    if (k + 4u > a.K) {                                       // padding, and what was read past the row's end
        r.x = k < a.K ? r.x : 0.0f;
        r.y = k + 1u < a.K ? r.y : 0.0f;
        r.z = k + 2u < a.K ? r.z : 0.0f;
        r.w = k + 3u < a.K ? r.w : 0.0f;
    }
    return r;
}

// ---------------------------------------------------------------------------------
// fp32 numbers as bf16 parts
// ---------------------------------------------------------------------------------
__device__ __forceinline__ uint32_t to_bf16x2(float a, float b) {
    floatx2 f;
    f.x = a;
    f.y = b;
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, bf16x2));     // to nearest even
}
// The parts of a number below 2^-109 would reach into bf16's subnormal numbers and lose bits (rows of 1e-36: sums off by 2.5e-5 of their
// norm, fp32 products by 1.3e-7). So the rows are multiplied by PARTS_LIFT before they are split, and matrices of such numbers by a power of
// two of their own (wp_lift), and the sums are brought back: exact both ways. Sums of 2^110 and more (1e33) run over and are made again.
#define PARTS_LIFT 131072.0f                                // 2^17
// four numbers as PL bf16 numbers each, four to eight bytes per part
template <int PL>
__device__ __forceinline__ void split_parts(floatx4 x, uintx2 (&part)[PL]) {
#pragma unroll
    for (int p = 0; p < PL; ++p) {
        part[p].x = to_bf16x2(x.x, x.y);
        part[p].y = to_bf16x2(x.z, x.w);
        if (p + 1 < PL) {                                  // what is left: exact
            x.x -= __uint_as_float(part[p].x << 16);
            x.y -= __uint_as_float(part[p].x & 0xFFFF0000u);
            x.z -= __uint_as_float(part[p].y << 16);
            x.w -= __uint_as_float(part[p].y & 0xFFFF0000u);
        }
    }
}

// A block of 32 rows by 32 columns on the fp32 matrix cores, straight from memory: for the blocks whose sums of parts are not finite. slot, v,
// scale: of row lane % 32 of the block; col: this lane's column (of the padded matrix). Eight k per step: the lower half of the wavefront
// has the first four, product i takes number i of both halves. The sums lie as those of any 32 x 32 product do.
template <int MODE, int STORE>
__device__ __forceinline__ floatx16 fp32_block(const TArgs &a, uint32_t slot, uint32_t v, float scale, uint32_t col, int lane) {
    const floatx4 *Wq = (const floatx4 *)a.Wq;
    floatx16 sum;
#pragma unroll
    for (int r = 0; r < 16; ++r) sum[r] = 0.0f;
#pragma unroll 4
    for (uint32_t k0 = 0; k0 < a.Kpad; k0 += 8u) {
        const uint32_t k = k0 + 4u * ((uint32_t)lane >> 5);
        floatx4 p, q = (floatx4)(0.0f), w = Wq[(size_t)(k >> 2) * a.Npad + col];
        fetch_raw<MODE, STORE>(a, v, slot, k, p, q);
        const floatx4 x = finish_raw<MODE, STORE>(a, p, q, k, scale);
#pragma unroll
        for (int i = 0; i < 4; ++i) sum = __builtin_amdgcn_mfma_f32_32x32x2f32(x[i], k + i < a.K ? w[i] : 0.0f, sum, 0, 0, 0);
    }
    return sum;
}

// ---------------------------------------------------------------------------------
// few rows
// ---------------------------------------------------------------------------------
// A hop of some hundred or thousand rows leaves most of the chip idle and is paced by the chain of dependent steps: list entry,
// row, products, store. Here every wavefront has one 16 x 16 block of the output to itself (MFMA 16x16x4, fp32): a K of 256 is
// 64 products one after the other, a microsecond, where a 32 x 32 block takes four; there is no LDS and no barrier, so a
// wavefront waits for its own loads only; rows and weights are requested five steps of 16 k ahead. A lane holds four
// consecutive k of its row (one 16-byte load), which the four products of a step take one each, so a step's k are
// numbered lane group first: k = 4 * (lane / 16) + i for product i; the weights lie in that order in a.Wq (k by fours).
// What bounds more rows is the L2, 32 KB per block at a K of 256, and that a SIMD's second wavefront starts behind its first.
template <int MODE, int STORE>
__device__ __forceinline__ void wave_gemm(const TArgs &a, uint32_t gw, uint32_t nw) {
    constexpr int STAGES = 6;
    static_assert(MODE != 2, "sums of two rows go through the tiles");
    constexpr bool TWO = MODE == 1 && STORE == 1;
    const uint32_t count = *a.count_ptr;
    const int lane = (int)(threadIdx.x & 63u);
    const uint32_t sub = (uint32_t)lane & 15u, grp = (uint32_t)lane >> 4;
    const uint32_t n_ct = (a.N + 15u) / 16u, n_tiles = (count + 15u) / 16u * n_ct;
    const floatx4 *Wq = (const floatx4 *)a.Wq;
    for (uint32_t tile = gw; tile < n_tiles; tile += nw) {
        const uint32_t row0 = tile / n_ct * 16u, col = tile % n_ct * 16u + sub;
        const uint32_t slot = min(row0 + sub, count - 1u), v = a.list[slot];
        floatx4 ra[STAGES], rq[TWO ? STAGES : 1], rb[STAGES];
        auto request = [&](uint32_t k0, int s) {
            const uint32_t k = min(k0, a.Kpad - 16u) + 4u * grp;     // past the end: the last step once more, not used
            rb[s] = Wq[(size_t)(k >> 2) * a.Npad + col];
            floatx4 q = (floatx4)(0.0f);
            fetch_raw<MODE, STORE>(a, v, slot, k, ra[s], q);
            if constexpr (TWO) rq[s] = q;
        };
#pragma unroll
        for (int s = 0; s < STAGES; ++s) request(16u * s, s);
        const uint32_t deg = a.mean ? a.in_meta[v].y : 1u;
        const float scale = 1.0f / (float)(deg > 1u ? deg : 1u);
        // what this lane stores (four rows, one column) is combined with other rows: requested up front
        uint32_t ov[4];
        float add[4], old[4], osc[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) ov[r] = a.list[min(row0 + 4u * grp + r, count - 1u)];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const uint32_t dg = (a.mean && a.addend && a.addend_scaled) ? a.in_meta[ov[r]].y : 1u;
            osc[r] = 1.0f / (float)(dg > 1u ? dg : 1u);
            const size_t at = (size_t)ov[r] * a.N + min(col, a.N - 1u);
            add[r] = (a.out_mode == 1 && a.addend) ? a.addend[at] : 0.0f;
            old[r] = (a.out_mode == 1 && a.D) ? rp_load_h(a.Hout, a.store, at) : 0.0f;
        }
        const float bias = a.bias[col];
        floatx4 even = (floatx4)(0.0f), odd = (floatx4)(0.0f);   // two sums, so that the products do not wait for one another
        for (uint32_t kb = 0; kb < a.Kpad; kb += 16u * STAGES) {
#pragma unroll
            for (int s = 0; s < STAGES; ++s) {
                const uint32_t k0 = kb + 16u * s;
                if (k0 >= a.Kpad) break;
                floatx4 q = (floatx4)(0.0f);
                if constexpr (TWO) q = rq[s];
                const floatx4 x = finish_raw<MODE, STORE>(a, ra[s], q, k0 + 4u * grp, scale);
                even = __builtin_amdgcn_mfma_f32_16x16x4f32(x.x, rb[s].x, even, 0, 0, 0);
                odd = __builtin_amdgcn_mfma_f32_16x16x4f32(x.y, rb[s].y, odd, 0, 0, 0);
                even = __builtin_amdgcn_mfma_f32_16x16x4f32(x.z, rb[s].z, even, 0, 0, 0);
                odd = __builtin_amdgcn_mfma_f32_16x16x4f32(x.w, rb[s].w, odd, 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);           // (the scheduler would sink the requests to their use)
                request(k0 + 16u * STAGES, s);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if (col >= a.N || (a.split_col && col >= a.N1 && col < a.split_col)) continue;   // padding columns
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const uint32_t os = row0 + 4u * grp + r;
            if (os >= count) continue;
            float z = even[r] + odd[r] + bias + add[r] * osc[r];
            if (a.act == RIPPLE_ACT_RELU) z = z > 0.0f ? z : 0.0f;
            if (a.out_mode != 1) {
                const size_t orow = a.out_mode == 0 ? os : ov[r];
                if (a.split_col && col >= a.split_col) a.tmp_out2[orow * a.tmp_out2_ld + (col - a.split_col)] = z;
                else a.tmp_out[orow * a.tmp_out_ld + col] = z;
                continue;
            }
            const size_t at = (size_t)ov[r] * a.N + col;
            if (a.store) {
                const __hip_bfloat16 zr = __float2bfloat16(z);
                z = __bfloat162float(zr);
                ((__hip_bfloat16 *)a.Hout)[at] = zr;
            } else {
                ((float *)a.Hout)[at] = z;
            }
            if (a.D) a.D[at] = a.d_old ? old[r] : z - old[r];
        }
    }
}
// wavefronts (= 16 x 16 blocks) that `rows` rows take
static inline uint32_t wave_gemm_waves(const TArgs &a, uint32_t rows) { return rp_div_up(rows ? rows : 1u, 16u) * rp_div_up(a.N, 16u); }
// Within a launch that has other work too (k_hop_small) a launch is saved as well: up to two wavefronts per SIMD.
#define WAVE_GEMM_MAX 2048u
// On its own, against the tiles of k_transform_split (kernel time, wavefront each / tiles, us): 256 -> 256, 64 rows 7.0 / 9.5, 1,024 rows (a
// wavefront per SIMD) 7.4 / 10.1, 1,536 rows 10.2 / 10.4, 2,048 rows 10.4 / 10.4, 3,072 rows 13.8 / 10.8; 100 -> 256, 2,048 rows 7.2 / 8.0, 3,072
// rows 8.8 / 8.2; both products of 256 -> 47, 2,048 rows (0.9 per SIMD) 7.5 / 9.5, 3,072 rows (1.3) 11.0 / 9.6, from bf16 rows 7.6 / 8.0 and 11.5 /
// 7.9; 100 -> 60, 8,192 rows (2) 6.7 / 7.1, 12,288 rows 8.2 / 7.6. So: up to two wavefronts per SIMD, one with bf16 rows. (fp32 rows are nearly
// even between one and two, and the number expected is the previous batch's: on 1.2 M edges sets differ by a factor of two from batch
// to batch, and where a limit of one took the tiles they were slower: 12.2 us against 11.3 for 100 updates, 10.7 against 9.2 for 100 of a
// max layer's narrow products.) Rows that are added up from two places take a wavefront each longer at any number: 256 -> 256, 16 rows
// 10.8 / 7.2, 1,024 rows 10.0 / 8.3.
static inline bool wave_gemm_pays(const TArgs &a, uint32_t rows) {
    return a.a_mode != 2 && wave_gemm_waves(a, rows) <= (a.store && a.a_mode == 4 ? 1024u : 2048u);
}
