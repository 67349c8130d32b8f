// fp32 products on the bf16 matrix pipe.  A float is cut into three bfloat16 parts, each rounded to nearest,
//     x = h + m + l   (8 + 8 + 8 significand bits with signed remainders: the three parts hold x exactly),
// and a product of two such sums is taken as the six part products down to 2^-18 of the whole,
//     x y ~ h h' + (h m' + m h') + (m m' + h l' + l h'),
// each exact in the fp32 accumulator's input.  What is left out (m l', l m', l l') is at most 2^-25 of |x y|, half a
// unit in the last place of an fp32 product.  One 16x16x32 bf16 instruction takes 16 cycles where the eight 16x16x4
// fp32 instructions of the same depth take 256: six of them need 96, so a contraction bound by the fp32 matrix pipe
// has 2.7 times its rate here.  Cutting costs 5.5 vector instructions per element, so it pays where an element, once
// cut, meets at least a few tens of others.
// A part of an infinity or a NaN is a NaN: a sum in which an infinity takes part comes out as NaN, and the callers
// recompute such a sum in plain fp32.
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

}  // namespace legend
