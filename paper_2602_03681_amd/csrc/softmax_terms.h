// Products to fp32 accuracy on the bf16 matrix instruction (internal header).
//
// An fp32 number is exactly the sum of three bf16 numbers, each the one before's remainder rounded to nearest.  A product of
// two matrices is then the sum of products of their terms, each at the bf16 rate, 16 times the fp32 rate of
// this chip: 3 products where one operand is bf16 already (exact up to the fp32 accumulation), 6 where neither is.  The
// three left out are together at most 2^-23 of the operands' product (second terms reach 2^-8 of the power of two of the
// number, third ones 2^-16) and have either sign.  (Cut off instead of rounded, the terms after the first reach 2^-7 and
// 2^-15, all of the number's sign: up to 2^-21, a bias; the carried states of a 512-token recurrence were then 1.1e-7 off,
// now 7e-8, as in a recurrence of fp32 multiply-adds.)  Against one fp32 matrix instruction that is 5 and 2.7
// times the rate, and there are no fp16 range limits anywhere.
#pragma once
#include "mfma_util.h"
#include "nats_common.h"

namespace nats {

constexpr int N_TERMS = 3;   // bf16 terms of an fp32 number

template <typename T>
constexpr int terms_of() { return sizeof(T) == 2 ? 1 : N_TERMS; }

__device__ __forceinline__ f32x4 mfma_bf16(u32x4 a, u32x4 b, f32x4 c) {
    typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c,
                                                   0, 0, 0);
}
// c += (sum of the terms of a) (sum of the terms of b), the smallest products first
template <int NA, int NB>
__device__ __forceinline__ f32x4 mfma_terms(const u32x4 (&a)[NA], const u32x4 (&b)[NB], f32x4 c) {
#pragma unroll
    for (int s = N_TERMS - 1; s >= 0; --s)
#pragma unroll
        for (int i = 0; i < NA; ++i) {
            const int j = s - i;
            if (j >= 0 && j < NB) c = mfma_bf16(a[i], b[j], c);
        }
    return c;
}

// The same with everything but the leading product in a sum of its own, to be added at the end: an accumulation rounds at the
// size of what it adds onto, and of 6 instructions per step one then adds onto the large sum.
template <int NA, int NB>
__device__ __forceinline__ void mfma_terms(const u32x4 (&a)[NA], const u32x4 (&b)[NB], f32x4& lead, f32x4& rest) {
#pragma unroll
    for (int s = N_TERMS - 1; s > 0; --s)
#pragma unroll
        for (int i = 0; i < NA; ++i) {
            const int j = s - i;
            if (j >= 0 && j < NB) rest = mfma_bf16(a[i], b[j], rest);
        }
    lead = mfma_bf16(a[0], b[0], lead);
}
// the terms of the negated numbers
template <int N>
__device__ __forceinline__ void negate(u32x4 (&t)[N]) {
#pragma unroll
    for (int i = 0; i < N; ++i) t[i] ^= 0x80008000u;
}

// Two floats -> their bf16 terms, the first float's in the low halves.  Each term is rounded to nearest: what is left is exact in
// fp32, at most half of the term's last place, and of either sign.
__device__ __forceinline__ void split_pair(float x, float y, uint32_t (&t)[N_TERMS]) {
#pragma unroll
    for (int i = 0; i < N_TERMS; ++i) {
        t[i] = pack_bf16x2(x, y);
        if (i == N_TERMS - 1) break;
        x -= __uint_as_float(t[i] << 16);
        y -= __uint_as_float(t[i] & 0xffff0000u);
    }
}
// 8 floats -> their bf16 terms
__device__ __forceinline__ void split_terms(const float (&x)[8], u32x4 (&t)[N_TERMS]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        uint32_t p[N_TERMS];
        split_pair(x[2 * i], x[2 * i + 1], p);
#pragma unroll
        for (int n = 0; n < N_TERMS; ++n) t[n][i] = p[n];
    }
}

// 8 consecutive elements as they come from memory, and their terms
template <typename T>
struct Raw8 {
    u32x4 w[sizeof(T) / 2];
    __device__ __forceinline__ void load(const T* p) {
#pragma unroll
        for (int i = 0; i < (int)sizeof(T) / 2; ++i) w[i] = reinterpret_cast<const u32x4*>(p)[i];
    }
    __device__ __forceinline__ void zero() {
#pragma unroll
        for (int i = 0; i < (int)sizeof(T) / 2; ++i) w[i] = u32x4{0u, 0u, 0u, 0u};
    }
    __device__ __forceinline__ void floats(float (&x)[8]) const {
        if constexpr (sizeof(T) == 2) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                x[2 * i] = __uint_as_float(w[0][i] << 16);
                x[2 * i + 1] = __uint_as_float(w[0][i] & 0xffff0000u);
            }
        } else {
#pragma unroll
            for (int i = 0; i < 8; ++i) x[i] = __uint_as_float(w[i / 4][i % 4]);
        }
    }
    __device__ __forceinline__ void terms(u32x4 (&t)[terms_of<T>()]) const {
        if constexpr (sizeof(T) == 2) {
            t[0] = w[0];
        } else {
            float x[8];
            floats(x);
            split_terms(x, t);
        }
    }
};

// 4 floats -> their bf16 terms
__device__ __forceinline__ void split_terms(const float (&x)[4], uint2 (&t)[N_TERMS]) {
    uint32_t lo[N_TERMS], hi[N_TERMS];
    split_pair(x[0], x[1], lo);
    split_pair(x[2], x[3], hi);
#pragma unroll
    for (int n = 0; n < N_TERMS; ++n) t[n] = make_uint2(lo[n], hi[n]);
}

// A tile of 64 rows of D elements in LDS: one plane [64][D + PAD] of bf16 per term.  Operand of a product over the
// columns: 16-byte reads along a row (rows()).  Operand of a product over the rows: the transposing read of gfx950
// (cols()), so that no transposed copy is made.
template <int D, int N, int ROWS = 64, int PAD = LDS_PAD>
struct TermTile {
    static constexpr int RS = D + PAD, PLANE = ROWS * RS, BYTES = N * PLANE * 2;
    using Terms = u32x4[N];
    uint16_t* p;
    __device__ __forceinline__ void put(int row, int col, const u32x4 (&t)[N]) const {
#pragma unroll
        for (int i = 0; i < N; ++i) *reinterpret_cast<u32x4*>(p + i * PLANE + row * RS + col) = t[i];
    }
    __device__ __forceinline__ void put(int row, int col, const uint2 (&t)[N]) const {   // four elements
#pragma unroll
        for (int i = 0; i < N; ++i) *reinterpret_cast<uint2*>(p + i * PLANE + row * RS + col) = t[i];
    }
    // row `row`, columns col .. col + 7 (16x16x32 operand with the columns as contraction index: row l16, col + 8 lq)
    __device__ __forceinline__ void rows(int row, int col, u32x4 (&t)[N]) const {
#pragma unroll
        for (int i = 0; i < N; ++i) t[i] = *reinterpret_cast<const u32x4*>(p + i * PLANE + row * RS + col);
    }
    // operand with the rows as contraction index: this lane (l16, lq) gets column col + l16, rows r0 + 4 lq + j in its
    // slots j < 4 and rows r0 + 16 + 4 lq + j - 4 in the others: the order in which two result tiles of 16 rows lie in
    // a lane's registers.  The read hands a group of 16 lanes, each of which names 4 elements of one row, the 4 x 16
    // block transposed: lane 4 m + n of the group names columns 4 n .. 4 n + 3 of row m and receives column 4 m + n.
    __device__ __forceinline__ void cols(int r0, int col, int l16, int lq, u32x4 (&t)[N]) const {
        cols_from<4, 16>(r0, col, l16, lq, t);
    }
    // the same with rows r0 + 8 lq + j in slots j < 8: the order in which rows() reads the other operand
    __device__ __forceinline__ void cols_in_order(int r0, int col, int l16, int lq, u32x4 (&t)[N]) const {
        cols_from<8, 4>(r0, col, l16, lq, t);
    }
    template <int STEP, int HI>   // slots j < 4: rows r0 + STEP lq + j; the others: HI rows further
    __device__ __forceinline__ void cols_from(int r0, int col, int l16, int lq, u32x4 (&t)[N]) const {
        typedef short s16x4 __attribute__((ext_vector_type(4)));
        typedef __attribute__((address_space(3))) s16x4* lds_s16x4;
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const uint16_t* a = p + i * PLANE + (r0 + STEP * lq + (l16 >> 2)) * RS + col + 4 * (l16 & 3);
            const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)a);
            const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)(a + HI * RS));
            const uint2 l2 = __builtin_bit_cast(uint2, lo), h2 = __builtin_bit_cast(uint2, hi);
            t[i] = u32x4{l2.x, l2.y, h2.x, h2.y};
        }
    }
};

}  // namespace nats
