// Batch computation of the product scores up to 128 dimensions on the bf16 matrix pipe (paper Sec. 2.1 stage 5, Sec. 6): gather, scores,
// loss and backward of one row tile of one chunk and one corrupted side per workgroup, every fp32 product as six bf16 products of
// three-part splits (split_bf16.h), at 2.7 times the rate of the fp32 matrix instructions.
//
// Eight waves, one workgroup per compute unit.  Softmax losses take two sweeps over the chunk's negatives, the others one:
//   sweep 1   sums of exp(S - reference) per row, tiles of 32 negatives dealt to the waves, which take their operand of the scores
//             from memory in the order the instruction wants it; the composed rows Q stand in LDS in parts.  Nothing is shared
//             between waves: no barrier.
//   sweep 2   in steps of 64 negatives.  Waves 0 to 3 (producers) form scores again and weights W, and write W and the negatives to LDS
//             in parts; waves 4 to 7 (consumers), one step behind, multiply: G_Q += W Neg and G_neg = W^T Q, each for its
//             own columns, with its part of Q in registers.  A SIMD has one wave of either kind, so that one's vector
//             instructions run beside the other's matrix instructions.
// The operand that is transposed comes out of the same LDS tile by the transposing read.  The weights' order of registers after a score
// product is already the order of an operand with the positives as contraction index.
//
// What bounds it: issue and latency at two waves a SIMD (a wave issues one vector instruction per five cycles; the producers' chain sets the
// pace of sweep 2).  The matrix pipe needs 130 us of a batch of 50 000 edges, 1000 negatives, d = 100, and is busy a quarter of the
// time; memory is read twice, 1.1 GB.  That batch takes 0.48 ms by itself (0.52 while the sums of G_Q spilled), 0.53 with
// fp32 instructions and a single sweep; both sides and complex products 0.94 (1.21).  Against the two-sweep kernel on fp32 instructions:
// d = 50, both sides, chunks of 100, 0.56 ms (0.95); logistic at d = 128, 20 011 edges, 333 negatives, 0.131 ms (0.24).
// Against 64 bits the gradients are closer than with fp32 instructions in each of 19 shapes (2-norm over one batch, source rows and the
// others apart; d = 64 to 128, softmax, logistic and margin losses, scores from 0.1 to beyond 100, eight seeds each).
//
// Tried: the operand of the scores loaded by neighbouring lanes and exchanged between lanes in registers (216 more vector instructions a
// tile, no faster); the gradient rows staged in LDS with three barriers a step (0.48 ms, but d = 50 0.67); the consumers bringing the
// negatives into LDS (they become the slower half); loads of the first tile ahead of the positives' rows (they are waited for first: slower).
#include <type_traits>

#include "chunk_common.h"
#include "split_bf16.h"

#ifndef LEGEND_SPLIT_NJ
#define LEGEND_SPLIT_NJ 0
#endif

namespace legend {

typedef short s16x4 __attribute__((ext_vector_type(4)));

constexpr int kSThreads = 512;
constexpr int kSWaves = kSThreads / kWave;
constexpr int kSRow = 64;                   // positives per workgroup (padded), and negatives per step
constexpr int kSWPart = 16 * kSRow * 8;     // bytes of one part of a weight tile
constexpr int kSWTile = 3 * kSWPart;
constexpr float kSMasked = -1e30f;          // score of a column past the chunk's negatives

// exp(x) * 2^-58 for x <= 110 without overflow: 2^(h/2) is scaled by 2^-29 and squared.
__device__ inline float exp_lifted(float x) {
    const float L2E_HI = 1.44269502162933349609375f;
    const float L2E_LO = 1.925963033500011e-8f;
    const float hi = x * L2E_HI;
    float lo = fmaf(x, L2E_HI, -hi);
    lo = fmaf(x, L2E_LO, lo);
    const float r = __builtin_amdgcn_exp2f(0.5f * hi) * 1.862645149230957e-9f;     // 2^-29
    const float r2 = r * r;
    return fmaf(r2, lo * 0.6931471805599453f, r2);
}

// sum * exp(x) for a sum against one reference taken to another: a sum may hold exp(110) times what its reference stands for, and x may lie
// below -87, where exp(x) by itself is below fp32's normal range and comes out as 0.
__device__ inline float times_exp(float sum, float x) {
    const float half = fast_exp(0.5f * x);
    return (sum * half) * half;
}

// split_mfma with the five smaller part products in a sum of their own.  The matrix pipe rounds what an instruction adds to nearest, without a
// bias, where its products are of the accumulator's size; products far below it are rounded down at the accumulator's size.  Measured
// on random rows of 128 elements against 64 bits, in 2^-24 of the scores' root mean square: rounding error 1.09 and mean 0.00 with the small
// products apart, 2.57 and -0.12 in one sum, 3.42 and 0.00 with fp32 instructions.  A mean is what a loss over many scores keeps.
template <int RA, int RB>
__device__ __forceinline__ void split_mfma_low(const Split8 (&A)[RA], const Split8 (&B)[RB], f32v4 (&acc)[RA][RB], f32v4 (&low)[RA][RB]) {
#pragma unroll
    for (int p = 0; p < 6; ++p)
#pragma unroll
        for (int a = 0; a < RA; ++a)
#pragma unroll
            for (int b = 0; b < RB; ++b) {
                const uint4 x = p == 1 || p == 4 ? A[a].m : p == 0 ? A[a].l : A[a].h;
                const uint4 y = p == 1 || p == 3 ? B[b].m : p == 2 ? B[b].l : B[b].h;
                if (p < 5) low[a][b] = mfma_bf16(x, y, low[a][b]);
                else acc[a][b] = mfma_bf16(x, y, acc[a][b]);
            }
}

// Both LDS layouts are made of 8-byte chunks, four bf16 of one part: the composed rows as [part][chunk of 4 columns][64 rows], a
// weight tile as [part][chunk of 4 rows][64 negatives].  A lane reads two chunks of its row for an operand whose contraction index
// is the chunked one, and the transposing read (16 lanes: 4 rows x 4 chunks) serves the other direction.  The row index is
// crossed with the chunk number so that both kinds of read, and the stores, touch every bank once: chunk bit 0 flips row
// bits 2 and 4, chunk bit 1 row bit 3.
__device__ __forceinline__ int chunk_cross(int chunk) { return (chunk & 1) * 20 ^ ((chunk >> 1) & 1) * 8; }

__device__ __forceinline__ uint2 lds_b64(const char* p) { return *reinterpret_cast<const uint2*>(p); }
__device__ __forceinline__ uint2 lds_tr(const char* p) {
    typedef __attribute__((address_space(3))) s16x4* lds_p;
    return __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_p)(const_cast<char*>(p))));
}
// over the 16 lanes of a row, by rotations
template <class F>
__device__ __forceinline__ float row16(float x, F&& f) {
    x = f(x, __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0x128, 0xf, 0xf, true)));
    x = f(x, __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0x124, 0xf, 0xf, true)));
    x = f(x, __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0x122, 0xf, 0xf, true)));
    return f(x, __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0x121, 0xf, 0xf, true)));
}
__device__ __forceinline__ float row16_sum(float x) { return row16(x, [](float a, float b) { return a + b; }); }
__device__ __forceinline__ float row16_max(float x) { return row16(x, [](float a, float b) { return fmaxf(a, b); }); }
// A softmax reference: the nearest multiple of 2^-12.  A score far above it (100 above 30) then loses nothing when the reference is taken
// away.  With a reference of more bits the difference was rounded at its own size, for the sum of the row's terms and not for its weights,
// which then did not add up to 1.  Error of the source rows' gradients, scores in the tens, some of 100 (d = 100, N = 1000): 7.9e-7 with references
// as they come, 4.0e-7 so.
__device__ __forceinline__ float softmax_ref(float x) { return fabsf(x) < 4096.f ? rintf(x * 4096.f) * (1.f / 4096.f) : x; }
__device__ __forceinline__ uint4 minus(uint4 x) { return make_uint4(x.x ^ 0x80008000u, x.y ^ 0x80008000u, x.z ^ 0x80008000u, x.w ^ 0x80008000u); }
__device__ __forceinline__ Split8 minus(Split8 x) { return Split8{minus(x.h), minus(x.m), minus(x.l)}; }
__device__ __forceinline__ uint4 join(uint2 a, uint2 b) { return make_uint4(a.x, a.y, b.x, b.y); }

template <int NJ>
struct SplitShape {
    static constexpr bool packed_tail = NJ == 7;            // d = 97..100: three slices of 32 and four elements more
    static constexpr int KS = NJ / 2;                       // slices of 32 contraction elements
    static constexpr int NCH = 4 * NJ;
    static constexpr int q_part = NCH * kSRow * 8;
    static constexpr int q_bytes = 3 * q_part;
    static constexpr int GS = 16 * NJ + 4;                  // row stride of G_Q
    static constexpr int small_floats = 6 * kSRow + 2 * kSWaves * kSRow + 2 * kSRow + 16;
    static constexpr size_t lds_bytes = (size_t)2 * q_bytes + 2 * kSWTile + sizeof(int32_t) * kIdsLds + sizeof(float) * small_floats;
    // column blocks of consumer c: G_Q blocks q0(c) .. + qn(c), G_neg blocks n0(c) .. + nn(c); with two blocks in all the
    // four consumers share them by halves of the rows and of the negatives
    static constexpr int halves = NJ == 2 ? 2 : 1;
    static constexpr int q0(int c) { return NJ == 2 ? c & 1 : NJ == 4 ? c : NJ == 6 ? (c < 2 ? 2 * c : 2 + c) : 2 * c; }
    static constexpr int qn(int c) { return NJ <= 4 ? 1 : NJ == 6 ? (c < 2 ? 2 : 1) : NJ == 7 ? (c < 3 ? 2 : 1) : 2; }
    static constexpr int n0(int c) { return NJ == 2 ? c & 1 : NJ == 4 ? c : NJ == 6 ? (c < 2 ? c : 2 * c - 2) : NJ == 7 ? (c ? 2 * c - 1 : 0) : 2 * c; }
    static constexpr int nn(int c) { return NJ <= 4 ? 1 : NJ == 6 ? (c < 2 ? 1 : 2) : NJ == 7 ? (c ? 2 : 1) : 2; }
    static constexpr int most = NJ <= 4 ? 1 : 2;
    static_assert(lds_bytes <= 160 * 1024, "LDS");
};

template <int NJ, int VW, int LOSS>
__global__ void __launch_bounds__(kSThreads, 2)
k_chunk_split(BatchGeom g, BucketParams bp, const int32_t* __restrict__ neg_ids, float* __restrict__ grad,
              double* __restrict__ loss_partial, uint32_t* __restrict__ redo, unsigned long long* __restrict__ redo_total,
              float limit, int rescale_allowed) {
    using Sh = SplitShape<NJ>;
    constexpr int KS = Sh::KS;
    constexpr bool TAIL = Sh::packed_tail;
    constexpr bool SOFT = LOSS == LEGEND_LOSS_SOFTMAX;
    constexpr bool LOW = NJ < 8;              // the small products of a score in a sum of their own
    // Above 100 dimensions there are no registers for that.  There the first half of the slices is summed with the opposite sign and the
    // sum turned round before the second half, so that what is rounded down in either half nearly cancels.
    auto turned = [](int ks) { return !LOW && ks < KS / 2; };
    constexpr int PB = Sh::q_part;

    extern __shared__ __align__(16) char sm[];
    char* Qt = sm;                            // composed rows; in the second sweep two tiles of negatives, at its end G_Q
    char* Wt = sm + 2 * Sh::q_bytes;          // two weight tiles
    float* f_s = reinterpret_cast<float*>(Wt + 2 * kSWTile);      // [64] positive scores
    float* ref_s = f_s + kSRow;
    float* low_s = ref_s + kSRow;             // [64] log-sum-exp: ref_s + low_s
    float* lse_s = low_s + kSRow;             // [64] loss of the row: log-sum-exp - f
    float* a_s = lse_s + kSRow;               // [64] dL/df
    float* rowloss_s = a_s + kSRow;           // [64]
    float* Lw = rowloss_s + kSRow;            // [8][64] every wave's row sums (margin: counts)
    float* Rw = Lw + kSWaves * kSRow;         // [8][64] the references they were taken against
    float* mx_s = Rw + kSWaves * kSRow;       // [2][64] row maxima of the first 64 negatives
    uint32_t* flag_s = reinterpret_cast<uint32_t*>(mx_s + 2 * kSRow);      // [0] not finite, [1] a reference was raised; [8..15]:
    double* wave_loss = reinterpret_cast<double*>(flag_s + 8);             // [4] the producers' sums of the negatives' losses
    int32_t* ids_s = reinterpret_cast<int32_t*>(flag_s + 16);

    const int d = bp.dim;
    const int tid = threadIdx.x;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63;
    const int l15 = lane & 15;
    const int gq = lane >> 4;

    int wg = blockIdx.x;
    const int t_row = wg % g.T;  wg /= g.T;
    const int c = wg % g.nchunks;
    const int si = wg / g.nchunks;
    const int side = g.side_id[si];
    const int chunk_rows = min(g.C, g.P - c * g.C);
    const int row0 = t_row * g.rows_tile;
    const int nrows = max(0, min(g.rows_tile, chunk_rows - row0));
    const int64_t e0 = (int64_t)c * g.C + row0;
    const int32_t* eb = bp.edges + (bp.batch_lo + e0) * 3;
    const float* Ex = side == 0 ? bp.E_src : bp.E_dst;
    const float* Ey = side == 0 ? bp.E_dst : bp.E_src;
    const float* En = Ey;
    const int xcol = side == 0 ? 0 : 2;
    const int ycol = 2 - xcol;
    const int N = g.N;
    const int32_t* my_negs = neg_ids + ((int64_t)si * g.nchunks + c) * N;
    const int64_t side_base = (int64_t)si * g.per_side;
    const int64_t neg_base = side_base + (int64_t)g.roles * g.P + ((int64_t)c * g.T + t_row) * N;
    const bool upper = nrows > 32;            // uniform: row blocks 2 and 3 hold something
    const int h = d >> 1;

    // endpoints and relations of the wave's eight rows w, w + 8, ...: lanes 3 u .. 3 u + 2 hold those of the u-th
    constexpr int RPW = kSRow / kSWaves;
    const int eids = lane < 3 * RPW && w + kSWaves * (lane / 3) < nrows ? eb[(w + kSWaves * (lane / 3)) * 3 + lane % 3] : 0;
    const int T64 = (N + 63) >> 6;
    const int ntiles = 2 * T64;
    for (int k = tid; k < min(N, kIdsLds); k += kSThreads) ids_s[k] = my_negs[k];
    if (tid < 16) flag_s[tid] = 0;

    // ---- negatives: column k of 64-tile t is negative k T + t (every tile is an even sample of the chunk's negatives, so that
    // the first tile's row maxima are a good softmax reference); a wave's tile i is one half of 64-tile i / 2 -----------------
    auto neg_at = [&](int i, int k) __attribute__((always_inline)) { return (32 * (i & 1) + k) * T64 + (i >> 1); };
    auto live = [&](int i) __attribute__((always_inline)) { return i < ntiles && neg_at(i, 0) < N; };
    const bool ids_in_lds = N <= kIdsLds;
    auto id_of = [&](int n) __attribute__((always_inline)) {
        n = min(n, N - 1);
        typedef __attribute__((address_space(3))) const int32_t* lds_ids_t;
        return ids_in_lds ? ((lds_ids_t)ids_s)[n] : my_negs[n];
    };
    // four consecutive columns of a row, zero past its end
    auto load4 = [&](const float* row, int col, bool whole, float (&v)[4]) __attribute__((always_inline)) {
        if (VW == 4) {
            const bool ok = whole || col < d;
            const float4 x = *reinterpret_cast<const float4*>(row + (ok ? col : 0));
            v[0] = x.x; v[1] = x.y; v[2] = x.z; v[3] = x.w;
        } else if (VW == 2) {
#pragma unroll
            for (int t = 0; t < 4; t += 2) {
                const bool ok = whole || col + t < d;
                const float2 x = *reinterpret_cast<const float2*>(row + (ok ? col + t : 0));
                v[t] = x.x; v[t + 1] = x.y;
            }
        } else {
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const bool ok = whole || col + t < d;
                v[t] = row[ok ? col + t : 0];
            }
        }
    };
    auto mask4 = [&](int col, float (&v)[4]) __attribute__((always_inline)) {
#pragma unroll
        for (int t = 0; t < 4; ++t) v[t] = col + (VW == 4 ? 0 : VW == 2 ? (t & 2) : t) < d ? v[t] : 0.f;
    };

    // A lane's operands of the scores: elements 32 ks + 4 gq .. + 3 and 32 ks + 16 + 4 gq .. + 3 of its row, for either operand.
    float raw[2][KS + (TAIL ? 1 : 0)][8];
    auto raw_load = [&](auto const& rows, int ks) __attribute__((always_inline)) {
#pragma unroll
        for (int nb = 0; nb < 2; ++nb) {
            float v[4];
            load4(rows[nb], 32 * ks + 4 * gq, ks < KS - 1 || TAIL, v);
#pragma unroll
            for (int t = 0; t < 4; ++t) raw[nb][ks][t] = v[t];
            load4(rows[nb], 32 * ks + 16 + 4 * gq, ks < KS - 1 || TAIL, v);
#pragma unroll
            for (int t = 0; t < 4; ++t) raw[nb][ks][4 + t] = v[t];
        }
    };
    auto raw_load_tail = [&](auto const& rows) __attribute__((always_inline)) {
        if constexpr (TAIL) {
#pragma unroll
            for (int nb = 0; nb < 2; ++nb) {
                float v[4];
                load4(rows[nb], 32 * KS, false, v);
#pragma unroll
                for (int t = 0; t < 4; ++t) raw[nb][KS][t] = v[t];
            }
        }
    };
    auto rows_of = [&](int i, int swap, const float* (&rows)[2]) __attribute__((always_inline)) {
#pragma unroll
        for (int nb = 0; nb < 2; ++nb) rows[nb] = En + (int64_t)id_of(neg_at(i, 16 * (nb ^ swap) + l15)) * d;
    };
    // The first tile's loads go out behind those of the positives' rows and are not waited for with them (loads return in order).
    // Its ids are not in LDS yet.
    const int first = !SOFT || !live(w) ? (w & 3) >> 1 : w;
    int first_id[2];
#pragma unroll
    for (int nb = 0; nb < 2; ++nb) first_id[nb] = my_negs[min(neg_at(first, 16 * nb + l15), N - 1)];

    // ---- composed rows: a wave takes rows w, w + 8, ..., its lanes the columns ------------------------------------------
    auto put = [&](int row, int k, float v) __attribute__((always_inline)) {
        const int ch = k >> 2;
        char* p = Qt + ch * (kSRow * 8) + ((row ^ chunk_cross(ch)) * 8) + (k & 3) * 2;
        uint32_t hh, mm, ll;
        split_pair(v, 0.f, hh, mm, ll);
        *reinterpret_cast<uint16_t*>(p) = (uint16_t)hh;
        *reinterpret_cast<uint16_t*>(p + PB) = (uint16_t)mm;
        *reinterpret_cast<uint16_t*>(p + 2 * PB) = (uint16_t)ll;
    };
    // x, y, r at the lane's two columns (ComplEx: the two halves of its component) of the wave's eight rows w, w + 8, ...; all
    // loads of them go out together
    const bool cplx = bp.score == LEGEND_SCORE_COMPLEX, uses_rel = bp.score != LEGEND_SCORE_DOT;
    const int k0 = lane, k1 = cplx ? lane + h : lane + 64;
    const bool ok0 = cplx ? lane < h : lane < d;
    const bool ok1 = cplx ? lane < h : lane + 64 < d;
    const bool two = cplx || d > 64;          // uniform: the second column exists
    struct RowVals { float x0, x1, y0, y1, r0, r1; };
    auto load_rows = [&](int ids, RowVals (&v)[RPW]) __attribute__((always_inline)) {
        const int c0 = ok0 ? k0 : 0, c1 = ok1 ? k1 : 0;
#pragma unroll
        for (int u = 0; u < RPW; ++u) {
            const float* x = Ex + (int64_t)__builtin_amdgcn_readlane(ids, 3 * u + xcol) * d;
            const float* y = Ey + (int64_t)__builtin_amdgcn_readlane(ids, 3 * u + ycol) * d;
            v[u] = RowVals{x[c0], 0.f, y[c0], 0.f, 1.f, 1.f};
            if (two) { v[u].x1 = x[c1]; v[u].y1 = y[c1]; }
            if (uses_rel) {
                const float* r = bp.E_rel + (int64_t)__builtin_amdgcn_readlane(ids, 3 * u + 1) * d;
                v[u].r0 = r[c0];
                if (two) v[u].r1 = r[c1];
            }
        }
    };
    auto compose = [&](const RowVals& v, float& q0, float& q1) __attribute__((always_inline)) {
        if (bp.score == LEGEND_SCORE_DOT) { q0 = v.x0; q1 = v.x1; }
        else if (bp.score == LEGEND_SCORE_DISTMULT) { q0 = v.x0 * v.r0; q1 = v.x1 * v.r1; }
        else if (side == 0) { q0 = v.x0 * v.r0 - v.x1 * v.r1; q1 = v.x0 * v.r1 + v.x1 * v.r0; }
        else                { q0 = v.r0 * v.x0 + v.r1 * v.x1; q1 = v.r0 * v.x1 - v.r1 * v.x0; }
    };
    {
        RowVals v[RPW];
        load_rows(eids, v);
        {
            const float* const rows[2] = {En + (int64_t)first_id[0] * d, En + (int64_t)first_id[1] * d};
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) raw_load(rows, ks);
            raw_load_tail(rows);
        }
        float f[RPW];
#pragma unroll
        for (int u = 0; u < RPW; ++u) {
            const int row = w + kSWaves * u;
            float q0, q1;
            compose(v[u], q0, q1);
            if (!ok0 || row >= nrows) q0 = 0.f;
            if (!ok1 || row >= nrows) q1 = 0.f;
            f[u] = (ok0 && row < nrows ? q0 * v[u].y0 : 0.f) + (ok1 && row < nrows ? q1 * v[u].y1 : 0.f);
            if (cplx) {
                if (ok0) { put(row, k0, q0); put(row, k1, q1); }
                if (d + lane < 16 * NJ) put(row, d + lane, 0.f);
            } else {
                if (k0 < 16 * NJ) put(row, k0, q0);
                if (k1 < 16 * NJ) put(row, k1, q1);
            }
        }
#pragma unroll
        for (int m = 32; m > 0; m >>= 1)
#pragma unroll
            for (int u = 0; u < RPW; ++u) f[u] += wave_shfl_xor(f[u], m);
        if (lane == 0) {
#pragma unroll
            for (int u = 0; u < RPW; ++u) f_s[w + kSWaves * u] = f[u];
        }
    }
    __syncthreads();

    // byte offsets of this lane's chunks in the composed rows: row 16 r + l15, chunk gq of a group of four (r even / odd)
    const int cr = chunk_cross(gq);
    const int qa[2] = {gq * (kSRow * 8) + ((l15 ^ cr) * 8), gq * (kSRow * 8) + (((16 + l15) ^ cr) * 8)};
    auto row_frag = [&](const char* q, int part) __attribute__((always_inline)) {
        Split8 x;
        x.h = join(lds_b64(q), lds_b64(q + 4 * kSRow * 8));
        x.m = join(lds_b64(q + part), lds_b64(q + part + 4 * kSRow * 8));
        x.l = join(lds_b64(q + 2 * part), lds_b64(q + 2 * part + 4 * kSRow * 8));
        return x;
    };
    // Packed tail: the last four elements' six part products side by side in one instruction; lane groups 0 to 2 hold
    // (l h', m m'), (h l', m h'), (h m', h h'), group 3 nothing.  Chunk 8 KS, which is not crossed.
    const int tp1 = gq == 0 ? 2 * PB : 0, tp2 = gq == 2 ? 0 : PB, ta = 8 * KS * (kSRow * 8) + l15 * 8;
    auto cut = [&](int ks, bool minus, Split8 (&B)[2]) __attribute__((always_inline)) {
#pragma unroll
        for (int nb = 0; nb < 2; ++nb) {
            float x[8];
#pragma unroll
            for (int t = 0; t < 8; ++t) x[t] = minus ? -raw[nb][ks][t] : raw[nb][ks][t];
            if (ks == KS - 1 && !TAIL) {
                float lo[4] = {x[0], x[1], x[2], x[3]}, hi[4] = {x[4], x[5], x[6], x[7]};
                mask4(32 * ks + 4 * gq, lo);
                mask4(32 * ks + 16 + 4 * gq, hi);
#pragma unroll
                for (int t = 0; t < 4; ++t) { x[t] = lo[t]; x[4 + t] = hi[t]; }
            }
            B[nb] = split8(x);
        }
    };
    auto cut_tail = [&](uint4 (&B)[2], uint2 (&tail)[3]) __attribute__((always_inline)) {
        if constexpr (TAIL) {
#pragma unroll
            for (int nb = 0; nb < 2; ++nb) {
                float x[4] = {raw[nb][KS][0], raw[nb][KS][1], raw[nb][KS][2], raw[nb][KS][3]};
                mask4(32 * KS, x);
                uint2 hh, mm, ll;
                split_pair(x[0], x[1], hh.x, mm.x, ll.x);
                split_pair(x[2], x[3], hh.y, mm.y, ll.y);
                if (nb == 0) { tail[0] = hh; tail[1] = mm; tail[2] = ll; }
                // (element by element: a choice between structs would go through scratch memory, and its loads wait for the gather)
                auto pick = [&](uint32_t a, uint32_t b, uint32_t c, uint32_t e) __attribute__((always_inline)) {
                    return gq == 0 ? a : gq == 1 ? b : gq == 2 ? c : e;
                };
                B[nb] = make_uint4(pick(hh.x, ll.x, mm.x, 0u), pick(hh.y, ll.y, mm.y, 0u), pick(mm.x, hh.x, hh.x, 0u), pick(mm.y, hh.y, hh.y, 0u));
            }
        }
    };
    // scores of all rows against the tile in `raw`; raw is refilled with tile `next` on the way
    // acc[r][nb]: rows 16 r + 4 gq + v, negative 16 nb + l15
    auto scores_of = [&](auto Up, int next, f32v4 (&acc)[4][2]) __attribute__((always_inline)) {
        constexpr int RP = decltype(Up)::value ? 2 : 1;         // pairs of row blocks
        const float* rows[2];
        rows_of(next, 0, rows);
        f32v4 low[4][2];
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int nb = 0; nb < 2; ++nb) acc[r][nb] = low[r][nb] = f32v4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            Split8 B[2];
            cut(ks, turned(ks), B);
            raw_load(rows, ks);
            if (ks == KS / 2 && turned(0)) {
#pragma unroll
                for (int r = 0; r < 2 * RP; ++r)
#pragma unroll
                    for (int nb = 0; nb < 2; ++nb) acc[r][nb] = -acc[r][nb];
            }
#pragma unroll
            for (int rp = 0; rp < RP; ++rp) {
                Split8 A[2];
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    A[u] = row_frag(Qt + qa[u] + rp * 256 + ks * (8 * kSRow * 8), PB);
                }
#pragma unroll
                for (int p = 0; p < 6; ++p)
#pragma unroll
                    for (int u = 0; u < 2; ++u)
#pragma unroll
                        for (int nb = 0; nb < 2; ++nb) {
                            const uint4 x = p == 1 || p == 4 ? A[u].m : p == 0 ? A[u].l : A[u].h;
                            const uint4 y = p == 1 || p == 3 ? B[nb].m : p == 2 ? B[nb].l : B[nb].h;
                            if (LOW && p < 5) low[2 * rp + u][nb] = mfma_bf16(x, y, low[2 * rp + u][nb]);
                            else acc[2 * rp + u][nb] = mfma_bf16(x, y, acc[2 * rp + u][nb]);
                        }
            }
        }
        if constexpr (TAIL) {
            uint4 B[2];
            uint2 tail[3];
            cut_tail(B, tail);
            raw_load_tail(rows);
#pragma unroll
            for (int r = 0; r < 2 * RP; ++r) {
                const uint4 A = join(lds_b64(Qt + ta + tp1 + r * 128), lds_b64(Qt + ta + tp2 + r * 128));
#pragma unroll
                for (int nb = 0; nb < 2; ++nb) acc[r][nb] = mfma_bf16(A, B[nb], acc[r][nb]);
            }
        }
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int nb = 0; nb < 2; ++nb)
                if (LOW) acc[r][nb] += low[r][nb];
    };
    auto scores = [&](int next, f32v4 (&acc)[4][2]) __attribute__((always_inline)) {
        if (upper) scores_of(std::true_type{}, next, acc);
        else scores_of(std::false_type{}, next, acc);
    };
    auto finite = [](float x) { return fabsf(x) < INFINITY; };

    bool bad = false;                         // a score or a gradient that is not finite: the fp32 kernel takes over
    if (SOFT) {
        // ---- sweep 1: sums of exp(S - reference) 2^-58, the tiles dealt to all eight waves.  The reference of a row is its
        // maximum over the first 64 negatives; a wave that meets a score more than `limit` above it goes on with its own.
        float sum[16];
        float* const myref = Rw + w * kSRow;     // this wave's references
#pragma unroll
        for (int k = 0; k < 16; ++k) sum[k] = 0.f;
        f32v4 acc[4][2];
        auto mask_cols = [&](int i) __attribute__((always_inline)) {
#pragma unroll
            for (int nb = 0; nb < 2; ++nb) {
                const bool ok = neg_at(i, 16 * nb + l15) < N;
#pragma unroll
                for (int r = 0; r < 4; ++r)
#pragma unroll
                    for (int v = 0; v < 4; ++v) acc[r][nb][v] = ok ? acc[r][nb][v] : kSMasked;
            }
        };
        auto row_max = [&](int r, int v) __attribute__((always_inline)) {
            return row16_max(fmaxf(acc[r][0][v], acc[r][1][v]));
        };
        auto next_of = [&](int i) __attribute__((always_inline)) { return live(i + kSWaves) ? i + kSWaves : (w & 3) >> 1; };      // last: the producer's first tile
        for (int i = w;; i += kSWaves) {
            const bool here = live(i);
            if (here) {
                scores(next_of(i), acc);
                mask_cols(i);
            }
            if (i < kSWaves) {                // every wave's first turn
                if (w < 2) {
#pragma unroll
                    for (int r = 0; r < 4; ++r)
#pragma unroll
                        for (int v = 0; v < 4; ++v) {
                            const float m = here ? row_max(r, v) : kSMasked;
                            if (l15 == 0) mx_s[w * kSRow + 16 * r + 4 * gq + v] = m;
                        }
                }
                __syncthreads();
                myref[lane] = lane < nrows ? softmax_ref(fmaxf(mx_s[lane], mx_s[kSRow + lane])) : 1e30f;       // rows past the chunk: sums of 0
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            }
            if (!here) break;
            float over = -1e30f;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float4 rf = lds4(myref + 16 * r + 4 * gq);
                const float ref[4] = {rf.x, rf.y, rf.z, rf.w};
#pragma unroll
                for (int v = 0; v < 4; ++v) over = fmaxf(over, fmaxf(acc[r][0][v], acc[r][1][v]) - ref[v]);
            }
            if (__builtin_expect(__ballot(over > limit) != 0ull, 0)) {
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float4 rf = lds4(myref + 16 * r + 4 * gq);
                    const float ref[4] = {rf.x, rf.y, rf.z, rf.w};
                    float up[4];
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        up[v] = softmax_ref(fmaxf(ref[v], row_max(r, v)));
                        sum[4 * r + v] = times_exp(sum[4 * r + v], ref[v] - up[v]);
                    }
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                    __builtin_amdgcn_wave_barrier();          // every lane has read the old references
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                    if (l15 == 0) *reinterpret_cast<float4*>(myref + 16 * r + 4 * gq) = make_float4(up[0], up[1], up[2], up[3]);
                }
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                if (lane == 0) {
                    flag_s[1] = 1u;
                    if (!rescale_allowed) flag_s[0] = 1u;      // test knob: hand the chunk to the fp32 kernel instead
                }
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float4 rf = lds4(myref + 16 * r + 4 * gq);
                const float ref[4] = {rf.x, rf.y, rf.z, rf.w};
#pragma unroll
                for (int nb = 0; nb < 2; ++nb)
#pragma unroll
                    for (int v = 0; v < 4; ++v) sum[4 * r + v] += exp_lifted(acc[r][nb][v] - ref[v]);
            }
        }
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const float s = row16_sum(sum[4 * r + v]);
                if (l15 == 0) Lw[w * kSRow + 16 * r + 4 * gq + v] = s;
            }
        __syncthreads();
        if (tid < kSRow) {
            float m = Rw[tid];
#pragma unroll
            for (int k = 1; k < kSWaves; ++k) m = fmaxf(m, Rw[k * kSRow + tid]);
            const bool in = tid < nrows;
            const float f = f_s[tid];
            if (bp.softmax_with_pos && in && f - m > limit) {
                m = f;
                flag_s[1] = 1u;
                if (!rescale_allowed) flag_s[0] = 1u;
            }
            float total = 0.f;
#pragma unroll
            for (int k = 0; k < kSWaves; ++k) {
                const float rk = Rw[k * kSRow + tid];
                total += rk == m ? Lw[k * kSRow + tid] : times_exp(Lw[k * kSRow + tid], rk - m);
            }
            const float neg_sum = total;
            if (bp.softmax_with_pos && in) total += exp_lifted(f - m);
            // above a masked column's value no reference exceeds its row's largest term (by more than 2^-13), which contributes at least
            // 2^-58: the sum can only leave this range if a score is not finite.  Where no score lies above that value the
            // reference is the masked columns', which were then counted: left to the fp32 kernel as well.
            if (in && (!(total > 1e-30f && total < 1e36f) || m <= kSMasked)) flag_s[0] = 1u;
            // the log-sum-exp in two floats: weights are exp((S - ref) - low); rows past the chunk: weight 0
            constexpr double lift = 58.0 * 0.693147180559945309;
            const double lse = (double)m + (log((double)total) + lift);
            ref_s[tid] = in ? (float)lse : 1e30f;
            low_s[tid] = in ? (float)(lse - (double)(float)lse) : 0.f;
            // The loss rounded once: the logarithm of a sum that is 2^-58 times too small, and the lift's, are both near 40, and their
            // roundings in fp32 were the larger part of the loss's error (a bias of 3e-8 of a loss of 7).  With the positive
            // score in the sum the loss is softplus(log-sum-exp of the negatives - f): where the positive dominates, lse - f cancels.
            float row_loss = (float)(lse - (double)f);
            if (bp.softmax_with_pos) row_loss = softplusf((float)(((double)m - (double)f) + (log((double)neg_sum) + lift)));
            lse_s[tid] = in ? row_loss : 0.f;
            a_s[tid] = in ? -neg_sum / total : 0.f;
        }
        __syncthreads();
        bad = flag_s[0] != 0u;                // uniform
    } else {
        if (tid < kSRow) a_s[tid] = LOSS == LEGEND_LOSS_LOGISTIC && tid < nrows ? -sigmoidf(-f_s[tid]) : 0.f;
    }

    if (!bad) {
        // ---- sweep 2, in steps of one 64-tile.  Waves 0 to 3 (producers) form scores and weights and bring the weights and the tile
        // of negatives into LDS in parts; waves 4 to 7 (consumers), one step behind, multiply: G_Q += W Neg and
        // G_neg = W^T Q, every one for its own columns, with its part of the composed rows in registers.  Two buffers of
        // each tile: one barrier a step.
        const int p = w & 3;
        if (w < 4) {
            const int rh = p & 1, nh = p >> 1;          // its share of the scores: rows 32 rh .. + 31, negatives 32 nh .. + 31
            Split8 A[KS][2];
            uint4 At[2];
            {
                const char* base = Qt + rh * 256;
#pragma unroll
                for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                    for (int u = 0; u < 2; ++u) {
                        A[ks][u] = row_frag(base + qa[u] + ks * (8 * kSRow * 8), PB);
                        if (turned(ks)) A[ks][u] = minus(A[ks][u]);
                    }
                if constexpr (TAIL) {
#pragma unroll
                    for (int u = 0; u < 2; ++u) At[u] = join(lds_b64(base + ta + tp1 + u * 128), lds_b64(base + ta + tp2 + u * 128));
                }
            }
            float neg_loss = 0.f, cnt[LOSS == LEGEND_LOSS_MARGIN ? 8 : 1];
#pragma unroll
            for (int k = 0; k < (LOSS == LEGEND_LOSS_MARGIN ? 8 : 1); ++k) cnt[k] = 0.f;
            const float wneg = bp.neg_weight;
            bool nan = false;
            float av[2][4], sv[2][4];                    // per row: the log-sum-exp in two parts, or the positive score
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const float4 a = lds4((SOFT ? ref_s : f_s) + 32 * rh + 16 * u + 4 * gq), b = lds4(low_s + 32 * rh + 16 * u + 4 * gq);
                av[u][0] = a.x; av[u][1] = a.y; av[u][2] = a.z; av[u][3] = a.w;
                sv[u][0] = b.x; sv[u][1] = b.y; sv[u][2] = b.z; sv[u][3] = b.w;
            }
            const bool scoring = rh == 0 || upper;
            // a lane's place in a tile of negatives: negative 32 nh + 16 rh + l15 (its half of what it scores), chunk gq
            char* nt = Qt + nh * 256 + qa[rh];
            auto produce = [&](int s) __attribute__((always_inline)) {
                const float* rows[2];
                rows_of(s + 1 < T64 ? 2 * (s + 1) + nh : 0, rh, rows);
                char* to = nt + (s & 1) * Sh::q_bytes;
                f32v4 acc[2][2], low[2][2];
#pragma unroll
                for (int u = 0; u < 2; ++u)
#pragma unroll
                    for (int nb = 0; nb < 2; ++nb) acc[u][nb] = low[u][nb] = f32v4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) {
                    Split8 B[2];
                    cut(ks, false, B);
                    raw_load(rows, ks);
                    if (ks == KS / 2 && turned(0)) {
#pragma unroll
                        for (int u = 0; u < 2; ++u)
#pragma unroll
                            for (int nb = 0; nb < 2; ++nb) acc[u][nb] = -acc[u][nb];
                    }
                    char* t = to + ks * (8 * kSRow * 8);
                    const uint4 parts[3] = {B[0].h, B[0].m, B[0].l};
#pragma unroll
                    for (int k = 0; k < 3; ++k) {
                        *reinterpret_cast<uint2*>(t + k * PB) = make_uint2(parts[k].x, parts[k].y);
                        *reinterpret_cast<uint2*>(t + k * PB + 4 * kSRow * 8) = make_uint2(parts[k].z, parts[k].w);
                    }
                    split_mfma_low(A[ks], B, acc, LOW ? low : acc);
                }
                if constexpr (TAIL) {
                    uint4 B[2];
                    uint2 tail[3];
                    cut_tail(B, tail);
                    raw_load_tail(rows);
                    if (gq == 0) {
#pragma unroll
                        for (int k = 0; k < 3; ++k) *reinterpret_cast<uint2*>(to + k * PB + KS * (8 * kSRow * 8)) = tail[k];
                    }
#pragma unroll
                    for (int u = 0; u < 2; ++u)
#pragma unroll
                        for (int nb = 0; nb < 2; ++nb) acc[u][nb] = mfma_bf16(At[u], B[nb], acc[u][nb]);
                }
                if (!scoring) return;
#pragma unroll
                for (int u = 0; u < 2; ++u)
#pragma unroll
                    for (int nb = 0; nb < 2; ++nb)
                        if (LOW) acc[u][nb] += low[u][nb];
                char* wt = Wt + (s & 1) * kSWTile + (8 * rh) * (kSRow * 8) + nh * 256;
                float step_loss = 0.f;                   // of this step: short sums, and fewer roundings at the size of the long one
#pragma unroll
                for (int nb = 0; nb < 2; ++nb) {
                    const bool in = neg_at(2 * s + nh, 16 * (nb ^ rh) + l15) < N;
                    char* wn = wt + qa[nb ^ rh];
#pragma unroll
                    for (int u = 0; u < 2; ++u) {
                        float x[4];
#pragma unroll
                        for (int v = 0; v < 4; ++v) {
                            const float S = acc[u][nb][v];
                            float wv;
                            if (SOFT) {
                                wv = fast_exp((S - av[u][v]) - sv[u][v]);
                                wv = in ? wv : 0.f;
                            } else {
                                const bool ok = in && 32 * rh + 16 * u + 4 * gq + v < nrows;
                                nan |= !finite(S);
                                if (LOSS == LEGEND_LOSS_MARGIN) {
                                    const float sh = (bp.margin - av[u][v]) + S;
                                    wv = ok && sh > 0.f ? 1.f : 0.f;
                                    step_loss += ok ? fmaxf(sh, 0.f) : 0.f;
                                    cnt[LOSS == LEGEND_LOSS_MARGIN ? 4 * u + v : 0] += wv;
                                } else {
                                    wv = ok ? wneg * sigmoidf(S) : 0.f;
                                    step_loss += ok ? wneg * softplusf(S) : 0.f;
                                }
                            }
                            x[v] = wv;
                        }
                        // chunk of 4 rows 8 rh + 4 u + gq, negative 32 nh + 16 (nb ^ rh) + l15
                        char* at = wn + u * (4 * kSRow * 8);
                        uint2 hh, mm, ll;
                        split_pair(x[0], x[1], hh.x, mm.x, ll.x);
                        split_pair(x[2], x[3], hh.y, mm.y, ll.y);
                        *reinterpret_cast<uint2*>(at) = hh;
                        *reinterpret_cast<uint2*>(at + kSWPart) = mm;
                        *reinterpret_cast<uint2*>(at + 2 * kSWPart) = ll;
                    }
                }
                neg_loss += step_loss;
            };
            if (rh == 1) {                               // the halves of its tile the other way round
#pragma unroll
                for (int ks = 0; ks < KS + (TAIL ? 1 : 0); ++ks)
#pragma unroll
                    for (int t = 0; t < (ks < KS ? 8 : 4); ++t) {
                        const float x = raw[0][ks][t];
                        raw[0][ks][t] = raw[1][ks][t];
                        raw[1][ks][t] = x;
                    }
            }
            __syncthreads();                             // everyone has its part of the composed rows
#pragma unroll 1
            for (int s = 0; s <= T64; ++s) {
                if (s < T64) produce(s);
                __syncthreads();
            }
            if (__ballot(nan) != 0ull && lane == 0) flag_s[0] = 1u;
            if (!SOFT) {
                double sum = (double)neg_loss;
                for (int off = kWave / 2; off > 0; off >>= 1) sum += __shfl_down(sum, off, kWave);
                if (lane == 0) wave_loss[p] = sum;
            }
            if (LOSS == LEGEND_LOSS_MARGIN) {
                // counts of its rows over its half of the negatives
#pragma unroll
                for (int u = 0; u < 2; ++u)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const float k = row16_sum(cnt[LOSS == LEGEND_LOSS_MARGIN ? 4 * u + v : 0]);
                        if (l15 == 0) Lw[nh * kSRow + 32 * rh + 16 * u + 4 * gq + v] = k;
                    }
            }
        } else {
            constexpr int MB = Sh::most, RH = Sh::halves;
            const int q0 = Sh::q0(p), qn = Sh::qn(p), n0 = Sh::n0(p), nn = Sh::nn(p);
            const int half = RH == 2 ? p >> 1 : 0;
            // transposing reads: rows 16 b + 4 gq + l15 / 4, chunk 4 j + l15 % 4 (b even / odd)
            const int ct = chunk_cross(l15 & 3);
            const int trow = 4 * gq + (l15 >> 2);
            const int qt[2] = {(l15 & 3) * (kSRow * 8) + ((trow ^ ct) * 8), (l15 & 3) * (kSRow * 8) + (((16 + trow) ^ ct) * 8)};
            auto col_frag = [&](const char* base, int part) __attribute__((always_inline)) {
                Split8 x;
                x.h = join(lds_tr(base + qt[0]), lds_tr(base + qt[1]));
                x.m = join(lds_tr(base + qt[0] + part), lds_tr(base + qt[1] + part));
                x.l = join(lds_tr(base + qt[0] + 2 * part), lds_tr(base + qt[1] + 2 * part));
                return x;
            };
            Split8 Qr[MB][2];                            // composed rows, transposed: column 16 (n0 + b) + l15, rows of pair q
#pragma unroll
            for (int b = 0; b < MB; ++b)
#pragma unroll
                for (int q = 0; q < 2; ++q) Qr[b][q] = col_frag(Qt + min(n0 + b, NJ - 1) * (4 * kSRow * 8) + q * 256, PB);
            constexpr int RB = 4 / RH;                   // row blocks of G_Q, and blocks of negatives of G_neg, that it has
            f32v4 acc[MB][RB];
#pragma unroll
            for (int b = 0; b < MB; ++b)
#pragma unroll
                for (int r = 0; r < RB; ++r) acc[b][r] = f32v4{0.f, 0.f, 0.f, 0.f};
            bool nan = false;
            // the gradient rows of the chunk's negatives as a buffer
            const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(grad + neg_base * d, 0, N * d * 4, 0x00020000);
            auto n_of = [&](int k, int s) __attribute__((always_inline)) { return k * T64 + s; };
            auto add_rows = [&](auto Up, int s) __attribute__((always_inline)) {         // G_Q
                constexpr int R = RH == 2 ? 2 : decltype(Up)::value ? 4 : 2;
                if (RH == 2 && half == 1 && !decltype(Up)::value) return;
                const char* wt = Wt + (s & 1) * kSWTile + half * (8 * kSRow * 8);
#pragma unroll
                for (int ks = 0; ks < 2; ++ks) {
                    Split8 A[R];
#pragma unroll
                    for (int r = 0; r < R; ++r) A[r] = col_frag(wt + r * (4 * kSRow * 8) + ks * 256, kSWPart);
#pragma unroll
                    for (int b = 0; b < MB; ++b) {
                        if (b < qn) {
                            const Split8 B = col_frag(Qt + (s & 1) * Sh::q_bytes + (q0 + b) * (4 * kSRow * 8) + ks * 256, PB);
                            // the products of these 32 negatives, small ones first, then added up rounded to nearest
#pragma unroll
                            for (int r0 = 0; r0 < R; r0 += 2) {
                                f32v4 t[2] = {f32v4{0.f, 0.f, 0.f, 0.f}, f32v4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
                                for (int pp = 0; pp < 6; ++pp)
#pragma unroll
                                    for (int r = 0; r < 2; ++r) {
                                        const uint4 x = pp == 1 || pp == 4 ? A[r0 + r].m : pp == 0 ? A[r0 + r].l : A[r0 + r].h;
                                        const uint4 y = pp == 1 || pp == 3 ? B.m : pp == 2 ? B.l : B.h;
                                        t[r] = mfma_bf16(x, y, t[r]);
                                    }
#pragma unroll
                                for (int r = 0; r < 2; ++r) {
                                    acc[b][r0 + r] += t[r];
                                    asm volatile("" : "+v"(acc[b][r0 + r]));      // added here: put off, the sums of a step fill the registers
                                }
                            }
                        }
                    }
                }
            };
            auto negative_rows = [&](auto Up, int s, int pair) __attribute__((always_inline)) {      // G_neg, two blocks of negatives
                constexpr int QN = decltype(Up)::value ? 2 : 1;
                const char* wt = Wt + (s & 1) * kSWTile + pair * 256;
                Split8 B[2][QN];
#pragma unroll
                for (int nb = 0; nb < 2; ++nb)
#pragma unroll
                    for (int q = 0; q < QN; ++q) B[nb][q] = row_frag(wt + qa[nb] + q * (8 * kSRow * 8), kSWPart);
#pragma unroll
                for (int b = 0; b < MB; ++b) {
                    if (b < nn) {
                        f32v4 o[2] = {f32v4{0.f, 0.f, 0.f, 0.f}, f32v4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
                        for (int pp = 0; pp < 6; ++pp)           // all small products first
#pragma unroll
                            for (int q = 0; q < QN; ++q)
#pragma unroll
                                for (int nb = 0; nb < 2; ++nb) {
                                    const uint4 x = pp == 1 || pp == 4 ? Qr[b][q].m : pp == 0 ? Qr[b][q].l : Qr[b][q].h;
                                    const uint4 y = pp == 1 || pp == 3 ? B[nb][q].m : pp == 2 ? B[nb][q].l : B[nb][q].h;
                                    o[nb] = mfma_bf16(x, y, o[nb]);
                                }
#pragma unroll
                        for (int nb = 0; nb < 2; ++nb) {
                            const float sum = (o[nb][0] + o[nb][1]) + (o[nb][2] + o[nb][3]);
                            nan |= sum != sum;
                            const int n = n_of(32 * pair + 16 * nb + l15, s), col = 16 * (n0 + b) + 4 * gq;
                            // a store past the end of the chunk's rows does nothing
                            typedef int i32v4 __attribute__((ext_vector_type(4)));
                            typedef int i32v2 __attribute__((ext_vector_type(2)));
#pragma unroll
                            for (int t = 0; t < 4; t += VW) {
                                const int at = n < N && col + t < d ? (n * d + col + t) * 4 : -4096;
                                if (VW == 4) __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(i32v4, o[nb]), rsrc, at, 0, 0);
                                else if (VW == 2) __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(i32v2, f32v2{o[nb][t], o[nb][t + 1]}), rsrc, at, 0, 0);
                                else __builtin_amdgcn_raw_buffer_store_b32(__float_as_int(o[nb][t]), rsrc, at, 0, 0);
                            }
                        }
                    }
                }
            };
            __syncthreads();
            __syncthreads();
#pragma unroll 1
            for (int s = 0; s < T64; ++s) {
                if (upper) {
                    add_rows(std::true_type{}, s);
                    if (RH == 1 || half == 0) negative_rows(std::true_type{}, s, 0);
                    if (RH == 1 || half == 1) negative_rows(std::true_type{}, s, 1);
                } else {
                    add_rows(std::false_type{}, s);
                    if (RH == 1 || half == 0) negative_rows(std::false_type{}, s, 0);
                    if (RH == 1 || half == 1) negative_rows(std::false_type{}, s, 1);
                }
                __syncthreads();
            }
            if (__ballot(nan) != 0ull && lane == 0) flag_s[0] = 1u;
            // G_Q to LDS, over the last tile
            float* Gs = reinterpret_cast<float*>(Qt);
#pragma unroll
            for (int b = 0; b < MB; ++b) {
                if (b < qn) {
#pragma unroll
                    for (int r = 0; r < RB; ++r)
#pragma unroll
                        for (int v = 0; v < 4; ++v) Gs[(32 * half + 16 * r + 4 * gq + v) * Sh::GS + 16 * (q0 + b) + l15] = acc[b][r][v];
                }
            }
        }
        RowVals v[RPW];
        load_rows(eids, v);                   // on their way across the barrier
        __syncthreads();

        // ---- epilogue: G_Q, chain rule, gradient rows of the positives ------------------------------------------------------
        if (LOSS == LEGEND_LOSS_MARGIN && tid < kSRow) {
            float s = 0.f;
            for (int k = 0; k < 2; ++k) s += Lw[k * kSRow + tid];
            a_s[tid] = -s;                    // minus the number of violating negatives
        }
        if (LOSS == LEGEND_LOSS_MARGIN) __syncthreads();
        const float* Gs = reinterpret_cast<const float*>(Qt);
        bool nan = false;
#pragma unroll
        for (int u = 0; u < RPW; ++u) {
            const int row = w + kSWaves * u;
            if (row < nrows) {
                const float a = a_s[row];
                float q0, q1;
                compose(v[u], q0, q1);
                float g0 = ok0 ? Gs[row * Sh::GS + k0] : 0.f, g1 = ok1 ? Gs[row * Sh::GS + k1] : 0.f;
                nan |= g0 != g0 || g1 != g1;
                g0 += a * v[u].y0;
                g1 += a * v[u].y1;
                const int64_t e = e0 + row;
                float* gx = grad + (side_base + (side == 0 ? 0 : g.P) + e) * d;
                float* gy = grad + (side_base + (side == 0 ? g.P : 0) + e) * d;
                float* gr = grad + (side_base + 2 * (int64_t)g.P + e) * d;
                float x0 = g0, x1 = g1, r0 = 0.f, r1 = 0.f;
                if (bp.score == LEGEND_SCORE_DISTMULT) {
                    x0 = v[u].r0 * g0; x1 = v[u].r1 * g1;
                    r0 = v[u].x0 * g0; r1 = v[u].x1 * g1;
                } else if (cplx) {
                    const float xr = v[u].x0, xi = v[u].x1, rr = v[u].r0, ri = v[u].r1;
                    if (side == 0) {
                        x0 = rr * g0 + ri * g1;      x1 = rr * g1 - ri * g0;
                        r0 = xr * g0 + xi * g1;      r1 = xr * g1 - xi * g0;
                    } else {
                        x0 = rr * g0 - ri * g1;      x1 = rr * g1 + ri * g0;
                        r0 = g0 * xr + g1 * xi;      r1 = g0 * xi - g1 * xr;
                    }
                }
                if (ok0) { gx[k0] = x0; gy[k0] = a * q0; }
                if (ok1) { gx[k1] = x1; gy[k1] = a * q1; }
                if (uses_rel) {
                    if (ok0) gr[k0] = r0;
                    if (ok1) gr[k1] = r1;
                }
            }
        }
        if (__ballot(nan) != 0ull && lane == 0) flag_s[0] = 1u;
        if (tid < kSRow) {
            float l = 0.f;
            if (tid < nrows) l = SOFT ? lse_s[tid] : LOSS == LEGEND_LOSS_LOGISTIC ? softplusf(-f_s[tid]) : 0.f;
            rowloss_s[tid] = l;
        }
        __syncthreads();
    }
    if (tid == 0) {
        const bool again = flag_s[0] != 0u;
        redo[blockIdx.x] = again ? 1u : 0u;
        if (SOFT && (again || flag_s[1] != 0u)) atomicAdd(redo_total, 1ull);
        double s = 0.0;
        if (!bad) {
            for (int r = 0; r < kSRow; ++r) s += (double)rowloss_s[r];
            if (!SOFT)
                for (int k = 0; k < 4; ++k) s += wave_loss[k];
        }
        loss_partial[blockIdx.x] = s;
    }
}

template <int NJ, int VW, int LOSS>
static hipError_t launch_split_one(hipStream_t st, const BatchGeom& g, const BucketParams& bp, const Workspace& ws) {
    static PerDeviceFlag configured;
    constexpr size_t lds = SplitShape<NJ>::lds_bytes;
    if (configured.pending()) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_chunk_split<NJ, VW, LOSS>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        configured.set();
    }
    hipLaunchKernelGGL((k_chunk_split<NJ, VW, LOSS>), dim3((unsigned)(g.sides * g.nchunks * g.T)), dim3(kSThreads), lds, st, g, bp,
                       ws.neg_ids, ws.grad, ws.loss_partial, ws.redo, ws.redo_total, ws.fast_limit, ws.fast_no_rescale ? 0 : 1);
    return hipGetLastError();
}

template <int NJ>
hipError_t launch_split_nj(hipStream_t st, const BatchGeom& g, const BucketParams& bp, const Workspace& ws);

#if LEGEND_SPLIT_NJ
template <int NJ, int VW>
static hipError_t launch_split_vw(hipStream_t st, const BatchGeom& g, const BucketParams& bp, const Workspace& ws) {
    if (bp.loss == LEGEND_LOSS_SOFTMAX) return launch_split_one<NJ, VW, LEGEND_LOSS_SOFTMAX>(st, g, bp, ws);
    if (bp.loss == LEGEND_LOSS_LOGISTIC) return launch_split_one<NJ, VW, LEGEND_LOSS_LOGISTIC>(st, g, bp, ws);
    return launch_split_one<NJ, VW, LEGEND_LOSS_MARGIN>(st, g, bp, ws);
}
template <>
hipError_t launch_split_nj<LEGEND_SPLIT_NJ>(hipStream_t st, const BatchGeom& g, const BucketParams& bp, const Workspace& ws) {
    if (bp.dim % 4 == 0) return launch_split_vw<LEGEND_SPLIT_NJ, 4>(st, g, bp, ws);
    if (bp.dim % 2 == 0) return launch_split_vw<LEGEND_SPLIT_NJ, 2>(st, g, bp, ws);
    return launch_split_vw<LEGEND_SPLIT_NJ, 1>(st, g, bp, ws);
}
#else
template <> hipError_t launch_split_nj<2>(hipStream_t, const BatchGeom&, const BucketParams&, const Workspace&);
template <> hipError_t launch_split_nj<4>(hipStream_t, const BatchGeom&, const BucketParams&, const Workspace&);
template <> hipError_t launch_split_nj<6>(hipStream_t, const BatchGeom&, const BucketParams&, const Workspace&);
template <> hipError_t launch_split_nj<7>(hipStream_t, const BatchGeom&, const BucketParams&, const Workspace&);
template <> hipError_t launch_split_nj<8>(hipStream_t, const BatchGeom&, const BucketParams&, const Workspace&);

// Little work per workgroup stays with k_chunk.  Time of a batch with this kernel over that of k_chunk (Dot, one side, chunks of 50; edges:
// loss negatives x dimension ratio), each the smaller of two runs in turn:
// Batches of up to kSmallSortMax gradient rows, whose index sides are made in groups: a batch is its kernels one behind the other, and
// the longest is this one.  500: softmax 30 x 100 0.92, 64 x 100 0.91, 40 x 64 0.96, 60 x 50 0.92, 25 x 128 0.79; logistic 0.86, -, 0.94, 0.92,
// 0.80; margin 0.83, -, 0.87, 0.87, 0.74.  Not at 100 x 32: softmax 1.00, logistic 1.04; 156 x 32 0.91, 0.99.
// Larger batches cost some 25 launches, which bound them up to some 8 000 edges (100 us): the second launch over flagged workgroups
// is then 5 us more, and two workgroups of k_chunk fit a compute unit.  2 500: softmax 100 x 50 1.01, 200 x 50 1.06, 100 x 100 0.97, 400 x 50 0.94,
// 100 x 128 1.04, 200 x 128 0.99; logistic 1.03, 1.03, 1.04, 0.91, 1.03, 1.02.  25 000: softmax 100 x 50 1.02, 64 x 100 1.03, 128 x 100 0.97, 64 x 128
// 1.13, 300 x 100 0.88; logistic 250 x 40 0.99, 64 x 100 1.06, 128 x 100 1.03, 300 x 100 1.00, 64 x 128 1.14, 100 x 128 1.10, 200 x 128 0.97, 333 x
// 128 0.90; margin 64 x 100 0.97, 128 x 100 0.92, 100 x 128 1.06, 200 x 128 0.93.
bool chunk_split_applies(const BatchGeom& g, const BucketParams& bp) {
    if (bp.atomic_mode != 0 || bp.score == LEGEND_SCORE_TRANSE_L1 || bp.dim > kNarrowMaxDim) return false;
    if (g.N > (1 << 20)) return false;        // a chunk's gradient rows are addressed by 32 bits
    const int64_t work = (int64_t)g.N * bp.dim;
    if (g.n_occ <= kSmallSortMax) return work >= (bp.dim > 32 ? 2500 : 5000);
    return work >= (bp.dim <= 100 ? 10000 : 16000);
}

hipError_t launch_chunks_split(hipStream_t st, const BatchGeom& g, const BucketParams& bp, const Workspace& ws) {
    if (bp.dim <= 32) return launch_split_nj<2>(st, g, bp, ws);
    if (bp.dim <= 64) return launch_split_nj<4>(st, g, bp, ws);
    if (bp.dim <= 96) return launch_split_nj<6>(st, g, bp, ws);
    if (bp.dim <= 100) return launch_split_nj<7>(st, g, bp, ws);
    return launch_split_nj<8>(st, g, bp, ws);
}
#endif

}  // namespace legend
