// fp32 products on the bf16 matrix pipe, by the method of Henry, Tang and Heinecke ("Leveraging the bfloat16 artificial
// intelligence datatype for higher-precision computations", ARITH 2019).  A float is cut into three bfloat16 parts, each rounded
// to nearest,
//     x = h + m + l   (8 + 8 + 8 significand bits with signed remainders: the three parts hold x exactly where 2^-110 <= |x|
//                      <= 3.39e38, the largest bfloat16; below, the low parts run out of exponent and x is held to 2^-134),
// and a product of two such sums is taken as the six part products down to 2^-18 of the whole,
//     x y ~ h h' + (h m' + m h') + (m m' + h l' + l h'),
// each exact in the fp32 accumulator's input.  What is left out (m l', l m', l l') is at most 2^-25 of |x y|, half a
// unit in the last place of an fp32 product.  One 16x16x32 bf16 instruction takes 16 cycles where the eight 16x16x4
// fp32 instructions of the same depth take 256: six of them need 96, so a contraction bound by the fp32 matrix pipe
// has 2.7 times its rate here.  Cutting costs 5.5 vector instructions per element, so it pays where an element, once
// cut, meets at least a few tens of others.
// A part of an infinity, of a NaN or of a finite number above the largest bfloat16 is a NaN, and so is every sum in which it
// takes part: the callers compute sums that came out as NaN once more in plain fp32, the training kernels with
// plain_products below, the ranking kernel (which has no registers left for it) one after the other.
#pragma once

#include <hip/hip_runtime.h>

namespace legend {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32v2 __attribute__((ext_vector_type(2)));
typedef float f32v4 __attribute__((ext_vector_type(4)));

// the eight consecutive contraction elements that a lane hands to one 16x16x32 instruction, in three parts
struct Split8 {
    uint4 h, m, l;
};

__device__ inline uint32_t bf16_pair(float a, float b) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32v2{a, b}, bf16x2));
}

__device__ inline void split_pair(float a, float b, uint32_t& h, uint32_t& m, uint32_t& l) {
    h = bf16_pair(a, b);
    a -= __uint_as_float(h << 16);
    b -= __uint_as_float(h & 0xffff0000u);
    m = bf16_pair(a, b);
    a -= __uint_as_float(m << 16);
    b -= __uint_as_float(m & 0xffff0000u);
    l = bf16_pair(a, b);
}

__device__ inline Split8 split8(const float (&x)[8]) {
    Split8 s;
    split_pair(x[0], x[1], s.h.x, s.m.x, s.l.x);
    split_pair(x[2], x[3], s.h.y, s.m.y, s.l.y);
    split_pair(x[4], x[5], s.h.z, s.m.z, s.l.z);
    split_pair(x[6], x[7], s.h.w, s.m.w, s.l.w);
    return s;
}

__device__ inline f32v4 mfma_bf16(uint4 a, uint4 b, f32v4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// LDS tile of one operand: [part][8-element group kg of the slice][row][8], the rows of a kg block padded by two, so that
// the four groups a store instruction touches and the sixteen rows a load touches fall into different banks.
// Lane (l15, g) of a wave reads elements 8g..8g+7 of row l15: one 128-bit read per part.
template <int ROWS, int KGS = 4>
struct SplitTile {
    static constexpr int KG_BYTES = (ROWS + 2) * 16;
    static constexpr int PART_BYTES = KGS * KG_BYTES;
    static constexpr int BYTES = 3 * PART_BYTES;
    __device__ static void store(char* base, int row, int kg, const Split8& s) {
        char* p = base + kg * KG_BYTES + row * 16;
        *reinterpret_cast<uint4*>(p) = s.h;
        *reinterpret_cast<uint4*>(p + PART_BYTES) = s.m;
        *reinterpret_cast<uint4*>(p + 2 * PART_BYTES) = s.l;
    }
    __device__ static Split8 load(const char* base, int row, int kg) {
        const char* p = base + kg * KG_BYTES + row * 16;
        Split8 s;
        s.h = *reinterpret_cast<const uint4*>(p);
        s.m = *reinterpret_cast<const uint4*>(p + PART_BYTES);
        s.l = *reinterpret_cast<const uint4*>(p + 2 * PART_BYTES);
        return s;
    }
};

// acc[a][b] += A[a] B[b]^T over 32 contraction elements: six passes over the RA x RB blocks, so that consecutive
// instructions never wait for each other's accumulator
template <int RA, int RB>
__device__ inline void split_mfma(const Split8 (&A)[RA], const Split8 (&B)[RB], f32v4 (&acc)[RA][RB]) {
#pragma unroll
    for (int p = 0; p < 6; ++p)
#pragma unroll
        for (int a = 0; a < RA; ++a)
#pragma unroll
            for (int b = 0; b < RB; ++b) {
                const uint4 x = p == 1 || p == 4 ? A[a].m : p == 0 ? A[a].l : A[a].h;
                const uint4 y = p == 1 || p == 3 ? B[b].m : p == 2 ? B[b].l : B[b].h;
                acc[a][b] = mfma_bf16(x, y, acc[a][b]);
            }
}

// Once more in plain fp32 what came out as NaN: acc[a][b] = sum over k < n of A(a, k) B(b, k) for the blocks of 16 x 16 of a
// wave, on the fp32 matrix instructions, operands straight from memory.  A(a, k) and B(b, k) are element k of this lane's row l15 of
// a block of either operand.  Only NaNs are replaced, so that a finite sum does not depend on what else is in its block.
// A wave calls this as one, where any of its sums is a NaN.  A batch over a diverged table (5 000 edges, 1000 negatives, d = 256)
// takes 1.08 times as long as one over a finite table; with a loop for each such sum it took 10 times as long.
template <int RA, int RB, class LA, class LB>
__device__ __forceinline__ void plain_products(int n, LA A, LB B, f32v4 (&acc)[RA][RB]) {
    const int g = (threadIdx.x & 63) >> 4;
#pragma unroll
    for (int b = 0; b < RB; ++b) {
        f32v4 c[RA];
#pragma unroll
        for (int a = 0; a < RA; ++a) c[a] = f32v4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
        for (int k0 = 0; k0 < n; k0 += 16) {      // lane group g: elements k0 + 4g .. k0 + 4g + 3
            float x[RA][4], y[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const int k = k0 + 4 * g + t, kc = k < n ? k : n - 1;
                const float yk = B(b, kc);
                y[t] = k < n ? yk : 0.f;
#pragma unroll
                for (int a = 0; a < RA; ++a) {
                    const float xk = A(a, kc);
                    x[a][t] = k < n ? xk : 0.f;
                }
            }
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int a = 0; a < RA; ++a) c[a] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[a][t], y[t], c[a], 0, 0, 0);
            bool all = true;                      // NaN already: nothing more to come
#pragma unroll
            for (int a = 0; a < RA; ++a)
#pragma unroll
                for (int v = 0; v < 4; ++v) all = all & (c[a][v] != c[a][v]);
            if (__all(all)) break;
        }
#pragma unroll
        for (int a = 0; a < RA; ++a)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                float s = acc[a][b][v];
                asm volatile("" : "+v"(s));      // compared here and not in front of the loop, where the masks would spill
                acc[a][b][v] = s != s ? c[a][v] : s;
            }
    }
}

}  // namespace legend
