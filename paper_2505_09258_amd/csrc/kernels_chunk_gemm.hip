// Batch computation for wide embeddings (128 < dim <= 512; paper Sec. 2.1
// stage 5, Sec. 6) as a short chain of tiled contractions.  A (row tile of <= 112
// positives) x (all N negatives) score block does not fit on chip next to d-wide operand tiles,
// so the scores go through a device buffer that stays in the L2 / Infinity cache (the paper keeps
// its "Intermediate Result 3" in global memory for the same reason):
//   k_gemm_compose   Q = theta_s (x) theta_r (or conj(theta_r) (x) theta_d), positive scores f
//   k_gemm_scores    S = Q Neg^T, 112 x 128 tiles
//   k_gemm_rowstats  per row: log-sum-exp, loss term, dL/df; S is replaced by the weights W = dL/dS
//   k_gemm_gq        G_Q = W Neg
//   k_gemm_gneg      G_neg = W^T Q, written to the gradient rows of the negatives
//   k_gemm_chain     chain rule: gradient rows of theta_s, theta_r, theta_d of the positives
// The contractions were bound by the fp32 matrix pipe and the LDS reads that feed it (58 to 75 TFLOP/s of 139).  Now every
// operand is cut into three bf16 parts on its way into LDS, as fp32 products of six bf16 instructions (split_bf16.h), and
// read back as the eight contraction elements of a lane, one 128-bit read per part.  All three work on slices of 32
// contraction elements with 128 (small batches: 64) columns or negatives to a tile, the next slice on its way from memory; about 50 KB of
// LDS and at most 168 registers leave three workgroups to a compute unit, which cut and multiply in turn.  An operand whose contraction
// index is the slow one in memory is loaded by one thread per column, eight rows each: whole lines per instruction.
// Measured on batches of 10 000 edges, both sides, 1000 negatives, d = 400 (200 row tiles of 100): G_Q 276 -> 166 us, G_neg 255 ->
// 167 us, an epoch of 49 batches with its read 51.9 -> 36.4 ms.  What bounds them now: vector instructions of the cutting
// and matrix instructions take about a fifth of the time each, the rest waits for slices gathered from the tables.  Below
// d = 128 the chain loses to the two-sweep kernel (d = 50, 50 000 edges a batch: 14.1 against 13.9 ms an epoch), with
// the scores taken in turns that stay in the Infinity cache.
#include "chunk_common.h"
#include "split_bf16.h"

namespace legend {

constexpr int kGRows = 112;              // rows of a tile of positives: seven 16-row blocks
constexpr int kGNeg = 64;                // negatives per tile of the score buffer
constexpr int kGTile = 128;              // negatives or columns per workgroup
constexpr int kGK = 32;                  // contraction elements per slice
constexpr int kGThreads = 256;
// Below this many workgroups (two to a compute unit) the scores and G_neg kernels take tiles of 64 negatives instead of 128:
// a small batch is bound by the latency of its slices, one after the other in every workgroup, and by columns of negatives
// that do not exist.  A batch at d = 400 (start of the work on split products: fp32 tiles of 64), with tiles of 128, with 64, in us:
//   1000 edges, both sides, 100 negatives, 20 tiles of scores    130, 136, 126
//   2000 edges, both sides,  64 negatives, 40 tiles              139, 147, 139
//   5000 edges, 1000 negatives, 800 tiles                        428, 337, 346
// The two cross between 400 and 800 workgroups of either kernel (d = 130 to 512; at 1600 tiles of 64 cost 3 to 8 %).
constexpr int kGFew = 512;

static_assert(kGRows == kWideRowTile, "tile geometry");

// Elements k..k+7 of a row of d; elements past its end are others of the row (loads only: what is done to a loaded value
// at once waits for it).
template <int LW>                            // floats per load: 4 where d is a multiple of four (rows are 16-byte aligned), 2 where it is even, 1
__device__ inline void load8(const float* __restrict__ row, int k, int d, float (&v)[8]) {
    if (LW == 4) {
        const float4 a = *reinterpret_cast<const float4*>(row + (k < d ? k : 0));
        const float4 b = *reinterpret_cast<const float4*>(row + (k + 4 < d ? k + 4 : 0));
        v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
        v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
    } else if (LW == 2) {
#pragma unroll
        for (int t = 0; t < 8; t += 2) {
            const float2 a = *reinterpret_cast<const float2*>(row + (k + t < d ? k + t : 0));
            v[t] = a.x; v[t + 1] = a.y;
        }
    } else {
#pragma unroll
        for (int t = 0; t < 8; ++t) v[t] = row[min(k + t, d - 1)];
    }
}
// zero where element k + t does not exist
__device__ inline void zero_past(float (&v)[8], int k, int n) {
#pragma unroll
    for (int t = 0; t < 8; ++t)
        if (k + t >= n) v[t] = 0.f;
}

__device__ inline bool any_nan(f32v4 x) {
    const float s = (x[0] + x[1]) + (x[2] + x[3]);          // inf - inf as well: a look too many, no harm
    return s != s;
}

// acc[a][b] += A_a B_b^T of one slice for RA blocks of 16 rows (of which two at a time are in registers) and NB blocks
// of 16 columns
template <int RA, int NB, class TA, class TB>
__device__ __forceinline__ void slice_mfma(const char* As, const char* Bs, int col0, int l15, int gq, f32v4 (&acc)[RA][NB]) {
    Split8 B[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) B[b] = TB::load(Bs, col0 + 16 * b + l15, gq);
#pragma unroll
    for (int a = 0; a + 1 < RA; a += 2) {
        Split8 A[2];
        A[0] = TA::load(As, 16 * a + l15, gq);
        A[1] = TA::load(As, 16 * a + 16 + l15, gq);
        f32v4 c[2][NB];
#pragma unroll
        for (int b = 0; b < NB; ++b) { c[0][b] = acc[a][b]; c[1][b] = acc[a + 1][b]; }
        split_mfma(A, B, c);
#pragma unroll
        for (int b = 0; b < NB; ++b) { acc[a][b] = c[0][b]; acc[a + 1][b] = c[1][b]; }
    }
    if constexpr (RA % 2 == 1) {
        Split8 A[1] = {TA::load(As, 16 * (RA - 1) + l15, gq)};
        f32v4 c[1][NB];
#pragma unroll
        for (int b = 0; b < NB; ++b) c[0][b] = acc[RA - 1][b];
        split_mfma(A, B, c);
#pragma unroll
        for (int b = 0; b < NB; ++b) acc[RA - 1][b] = c[0][b];
    }
}

// Workgroup ids are dealt round-robin to the eight XCDs, each with its own L2.  The tiled
// kernels launch a one-dimensional grid of 8 * ceil(total / 8) workgroups and turn the hardware
// id into a virtual id such that consecutive virtual ids (the tiles that share a row tile's
// operands) run on the same XCD.  Returns false for the padding workgroups.
constexpr int kXcds = 8;
__host__ __device__ inline int64_t xcd_grid(int64_t total) { return (total + kXcds - 1) / kXcds * kXcds; }
__device__ inline bool xcd_tile(int64_t total, int nx, int* bx, int64_t* by) {
    const int64_t lin = blockIdx.x;
    const int64_t per = (total + kXcds - 1) / kXcds;
    const int64_t v = (lin % kXcds) * per + lin / kXcds;
    if (v >= total) return false;
    *bx = (int)(v % nx);
    *by = v / nx;
    return true;
}

struct TileCoord {
    int si, side, c, t_row, nrows;
    int64_t e0;          // first edge of the tile inside the batch
    int64_t wgrow;       // (si * nchunks + c) * T + t_row
};

__device__ inline TileCoord tile_coord(const BatchGeom& g, int64_t wgrow) {
    TileCoord tc;
    tc.wgrow = wgrow;
    int64_t q = wgrow;
    tc.t_row = (int)(q % g.T);  q /= g.T;
    tc.c = (int)(q % g.nchunks);
    tc.si = (int)(q / g.nchunks);
    tc.side = g.side_id[tc.si];
    const int chunk_rows = min(g.C, g.P - tc.c * g.C);
    const int row0 = tc.t_row * g.rows_tile;
    tc.nrows = max(0, min(g.rows_tile, chunk_rows - row0));
    tc.e0 = (int64_t)tc.c * g.C + row0;
    return tc;
}

// ---- Q and positive scores --------------------------------------------------------------------
// one workgroup of 128 threads per (side, edge)
template <int SCORE>
__global__ void __launch_bounds__(128)
k_gemm_compose(BatchGeom g, BucketParams bp, float* __restrict__ Q, float* __restrict__ fpos) {
    const int64_t idx = blockIdx.x;
    const int si = (int)(idx / g.P);
    const int64_t e = idx % g.P;
    const int side = g.side_id[si];
    const int d = bp.dim;
    const int32_t* eb = bp.edges + (bp.batch_lo + e) * 3;
    const float* x = (side == 0 ? bp.E_src : bp.E_dst) + (int64_t)eb[side == 0 ? 0 : 2] * d;
    const float* y = (side == 0 ? bp.E_dst : bp.E_src) + (int64_t)eb[side == 0 ? 2 : 0] * d;
    const float* r = SCORE == LEGEND_SCORE_DOT ? x : bp.E_rel + (int64_t)eb[1] * d;
    float* q = Q + idx * d;
    float partial = 0.f;
    if (SCORE == LEGEND_SCORE_COMPLEX) {
        const int h = d >> 1;
        for (int k = threadIdx.x; k < h; k += 128) {
            const float xr = x[k], xi = x[k + h], rr = r[k], ri = r[k + h];
            float qr, qi;
            if (side == 0) { qr = xr * rr - xi * ri; qi = xr * ri + xi * rr; }
            else           { qr = rr * xr + ri * xi; qi = rr * xi - ri * xr; }
            q[k] = qr;
            q[k + h] = qi;
            partial += qr * y[k] + qi * y[k + h];
        }
    } else {
        for (int k = threadIdx.x; k < d; k += 128) {
            const float v = SCORE == LEGEND_SCORE_DOT ? x[k] : x[k] * r[k];
            q[k] = v;
            partial += v * y[k];
        }
    }
    __shared__ float red[128];
    red[threadIdx.x] = partial;
    __syncthreads();
    for (int off = 64; off > 0; off >>= 1) {
        if ((int)threadIdx.x < off) red[threadIdx.x] += red[threadIdx.x + off];
        __syncthreads();
    }
    if (threadIdx.x == 0) fpos[idx] = red[0];
}

// ---- S = Q Neg^T ---------------------------------------------------------------------------------
// grid: (tiles of 64 NB negatives, row tiles).  Four waves; wave w owns the 16 NB negatives from 16 NB w of the tile
// and all row blocks.  S is stored as [row tile][64-negative tile][row][64], so that the tiles the
// later kernels load are contiguous.
// The load width is a template parameter because the compiler made one loop of 32-bit loads of the branches (four times the load
// instructions: 217 us a batch of the shape above, more than the matrix work took before).  An even d that is no multiple of four (150
// of the dimension sweep) has its 64-bit loads: 5 000 edges, 1000 negatives, d = 150 319 -> 255 us a batch, d = 510 614 -> 550.
// NB = 1 is for batches with few workgroups (kGFew): twice as many, and two slices on their way instead of one, since
// nothing else on the compute unit covers their latency.
template <int RB, int LW, int NB>             // row blocks of 16 that the tile geometry needs; floats per load; 64-negative blocks
__global__ void __launch_bounds__(kGThreads, 3)
k_gemm_scores(BatchGeom g, BucketParams bp, const int32_t* __restrict__ neg_ids, const float* __restrict__ Q,
              float* __restrict__ S, int Npad, int nx, int64_t ny) {
    using QTile = SplitTile<16 * RB>;
    using NTile = SplitTile<64 * NB>;
    __shared__ __align__(16) char Qs[QTile::BYTES];
    __shared__ __align__(16) char Ns[NTile::BYTES];
    const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63, l15 = lane & 15, gq = lane >> 4;
    int bx;
    int64_t by;
    if (!xcd_tile((int64_t)nx * ny, nx, &bx, &by)) return;       // uniform
    const TileCoord tc = tile_coord(g, by);
    if (tc.nrows == 0) return;                // uniform: no scores, and nobody reads any
    const int n0 = bx * 64 * NB;
    const int N = g.N, d = bp.dim;
    const float* En = tc.side == 0 ? bp.E_dst : bp.E_src;
    const float* Qrows = Q + ((int64_t)tc.si * g.P + tc.e0) * d;
    const int32_t* my_negs = neg_ids + ((int64_t)tc.si * g.nchunks + tc.c) * N;

    // a thread's share of a slice: elements 8kg..8kg+7 of rows srow, srow + 64 of both operands; rows and negatives that do
    // not exist are replaced by the last one, and their scores are not written
    const int srow = tid >> 2, kg = tid & 3;
    constexpr int QI = (RB + 3) / 4;
    constexpr int AHEAD = NB == 1 ? 2 : 1;    // slices on their way
    const float* qrow[QI];
    const float* nrow[NB];
#pragma unroll
    for (int u = 0; u < QI; ++u) qrow[u] = Qrows + (int64_t)min(srow + 64 * u, tc.nrows - 1) * d;
#pragma unroll
    for (int u = 0; u < NB; ++u) nrow[u] = En + (int64_t)my_negs[min(n0 + srow + 64 * u, N - 1)] * d;
    float qv[AHEAD][QI][8], nv[AHEAD][NB][8];
    auto fetch = [&](int s, int c0) {
#pragma unroll
        for (int u = 0; u < QI; ++u) load8<LW>(qrow[u], c0 + 8 * kg, d, qv[s][u]);
#pragma unroll
        for (int u = 0; u < NB; ++u) load8<LW>(nrow[u], c0 + 8 * kg, d, nv[s][u]);
    };
    f32v4 acc[RB][NB];
#pragma unroll
    for (int r = 0; r < RB; ++r)
#pragma unroll
        for (int b = 0; b < NB; ++b) acc[r][b] = f32v4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < AHEAD; ++s) fetch(s, kGK * s);
    for (int cs = 0; cs < d; cs += kGK * AHEAD) {
#pragma unroll
        for (int s = 0; s < AHEAD; ++s) {
            const int c0 = cs + kGK * s;
            if (c0 >= d) break;               // uniform
            if (c0 + kGK > d) {               // components past the end
#pragma unroll
                for (int u = 0; u < QI; ++u) zero_past(qv[s][u], c0 + 8 * kg, d);
#pragma unroll
                for (int u = 0; u < NB; ++u) zero_past(nv[s][u], c0 + 8 * kg, d);
            }
#pragma unroll
            for (int u = 0; u < QI; ++u)
                if (srow + 64 * u < 16 * RB) QTile::store(Qs, srow + 64 * u, kg, split8(qv[s][u]));
#pragma unroll
            for (int u = 0; u < NB; ++u) NTile::store(Ns, srow + 64 * u, kg, split8(nv[s][u]));
            __syncthreads();
            if (c0 + kGK * AHEAD < d) fetch(s, c0 + kGK * AHEAD);
            slice_mfma<RB, NB, QTile, NTile>(Qs, Ns, 16 * NB * w, l15, gq, acc);
            __syncthreads();
        }
    }
    bool nan = false;                         // an infinity took part, or the score is a NaN
#pragma unroll
    for (int r = 0; r < RB; ++r)
#pragma unroll
        for (int b = 0; b < NB; ++b) nan |= any_nan(acc[r][b]);
    if (__builtin_expect(__any(nan), 0))
        plain_products(d, [&](int r, int k) { return Qrows[(int64_t)min(16 * r + l15, tc.nrows - 1) * d + k]; },
                       [&](int b, int k) { return En[(int64_t)my_negs[min(n0 + 16 * NB * w + 16 * b + l15, N - 1)] * d + k]; }, acc);
    float* Srow = S + (int64_t)tc.wgrow * g.rows_tile * Npad;
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const int n = n0 + 16 * NB * w + 16 * b + l15;
        if (n >= N) continue;
#pragma unroll
        for (int r = 0; r < RB; ++r) {
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int row = 16 * r + 4 * gq + v;
                if (row < tc.nrows) Srow[((int64_t)(n >> 6) * g.rows_tile + row) * kGNeg + (n & 63)] = acc[r][b][v];
            }
        }
    }
}

// ---- row statistics and weights ------------------------------------------------------------
// One workgroup (16 waves) per row tile, one wave per row at a time.  A row of at most 1024 scores
// is read once into registers (16 per lane), reduced, and written back as the weights W = dL/dS:
// exp(S - lse) for the softmax losses, w sigmoid(S) for the logistic loss, the indicator of
// margin - f + S > 0 for the margin loss, 0 in the padding up to Npad; a longer row is read from the cache-resident buffer once per pass instead.
// rowa = dL/df, loss_partial[tile] = sum over the tile's rows.
constexpr int kStatThreads = 1024;
constexpr int kStatRegs = 16;                 // scores of a row per lane on the register path
template <int LOSS>
__global__ void __launch_bounds__(kStatThreads)
k_gemm_rowstats(BatchGeom g, BucketParams bp, float* __restrict__ S, const float* __restrict__ fpos, int Npad,
                float* __restrict__ rowa, double* __restrict__ loss_partial) {
    constexpr int WAVES = kStatThreads / kWave;
    __shared__ double wave_loss[WAVES];
    const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
    const TileCoord tc = tile_coord(g, blockIdx.x);
    const int N = g.N;
    float* Stile = S + (int64_t)tc.wgrow * g.rows_tile * Npad;
    const bool in_regs = Npad <= kStatRegs * kWave;
    double loss = 0.0;
    for (int row = w; row < tc.nrows; row += WAVES) {
        float* s = Stile + (int64_t)row * kGNeg;          // element n of the row sits at s[(n / 64) * tstride + n % 64]
        const int64_t tstride = (int64_t)g.rows_tile * kGNeg;
        auto at = [&](int n) -> float& { return s[(n >> 6) * tstride + (n & 63)]; };
        const int64_t ridx = (int64_t)tc.si * g.P + tc.e0 + row;
        const float f = fpos[ridx];
        float x[kStatRegs];                               // x[j] = score lane + 64 j (register path)
        if (in_regs) {
#pragma unroll
            for (int j = 0; j < kStatRegs; ++j) x[j] = lane + kWave * j < N ? s[j * tstride + lane] : -INFINITY;
        }
        if (LOSS == LEGEND_LOSS_SOFTMAX) {
            float m = -INFINITY;
            if (in_regs) {
#pragma unroll
                for (int j = 0; j < kStatRegs; ++j) m = fmaxf(m, x[j]);
            } else {
                for (int n = lane; n < N; n += kWave) m = fmaxf(m, at(n));
            }
            for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off, kWave));
            if (bp.softmax_with_pos) m = fmaxf(m, f);
            float l = 0.f;
            if (in_regs) {
#pragma unroll
                for (int j = 0; j < kStatRegs; ++j) {     // same order of the lane's terms as the strided loop
                    if (lane + kWave * j < N) { x[j] = fast_exp(x[j] - m); l += x[j]; }
                }
            } else {
                for (int n = lane; n < N; n += kWave) l += fast_exp(at(n) - m);
            }
            for (int off = 32; off > 0; off >>= 1) l += __shfl_xor(l, off, kWave);
            float a = -1.f;
            if (bp.softmax_with_pos) {
                const float pf = expf(f - m);
                a = -l / (l + pf);            // minus the negatives' share of the sum: no cancellation where the positive dominates
                l += pf;
            }
            const float il = 1.f / l;
            if (in_regs) {
#pragma unroll
                for (int j = 0; j < kStatRegs; ++j) {
                    const int n = lane + kWave * j;
                    if (n < Npad) s[j * tstride + lane] = n < N ? x[j] * il : 0.f;
                }
            } else {
                for (int n = lane; n < Npad; n += kWave) at(n) = n < N ? fast_exp(at(n) - m) * il : 0.f;
            }
            if (lane == 0) rowa[ridx] = a;
            loss += (double)(m + logf(l) - f);
        } else if (LOSS == LEGEND_LOSS_MARGIN) {
            // pair (row, negative) pays margin - f + S where that is positive: W is the indicator, dL/df minus their count
            const float base = bp.margin - f;
            float t = 0.f, cnt = 0.f;
            if (in_regs) {
#pragma unroll
                for (int j = 0; j < kStatRegs; ++j) {
                    const int n = lane + kWave * j;
                    const float sh = n < N ? base + x[j] : 0.f;
                    const float wv = sh > 0.f ? 1.f : 0.f;
                    t += fmaxf(sh, 0.f);
                    cnt += wv;
                    if (n < Npad) s[j * tstride + lane] = wv;
                }
            } else {
                for (int n = lane; n < Npad; n += kWave) {
                    const float sh = n < N ? base + at(n) : 0.f;
                    const float wv = sh > 0.f ? 1.f : 0.f;
                    t += fmaxf(sh, 0.f);
                    cnt += wv;
                    at(n) = wv;
                }
            }
            for (int off = 32; off > 0; off >>= 1) { t += __shfl_xor(t, off, kWave); cnt += __shfl_xor(cnt, off, kWave); }
            if (lane == 0) rowa[ridx] = -cnt;
            loss += (double)t;
        } else {
            float t = 0.f;
            if (in_regs) {
#pragma unroll
                for (int j = 0; j < kStatRegs; ++j) {
                    const int n = lane + kWave * j;
                    if (n < N) t += softplusf(x[j]);
                    if (n < Npad) s[j * tstride + lane] = n < N ? bp.neg_weight * sigmoidf(x[j]) : 0.f;
                }
            } else {
                for (int n = lane; n < N; n += kWave) t += softplusf(at(n));
            }
            for (int off = 32; off > 0; off >>= 1) t += __shfl_xor(t, off, kWave);
            if (!in_regs)
                for (int n = lane; n < Npad; n += kWave) at(n) = n < N ? bp.neg_weight * sigmoidf(at(n)) : 0.f;
            if (lane == 0) rowa[ridx] = -sigmoidf(-f);
            loss += (double)(softplusf(-f) + bp.neg_weight * t);
        }
    }
    if (lane == 0) wave_loss[w] = loss;
    __syncthreads();
    if (tid == 0) {
        double t = 0.0;
        for (int k = 0; k < WAVES; ++k) t += wave_loss[k];
        loss_partial[blockIdx.x] = t;
    }
}

// ---- G_Q = W Neg ---------------------------------------------------------------------------------
// grid: (tiles of 128 columns, row tiles).  Wave w owns columns 32w..32w+31 of the tile and all row blocks; the negatives
// are the contraction index, 32 to a slice.
template <int RB>
__global__ void __launch_bounds__(kGThreads, 3)
k_gemm_gq(BatchGeom g, BucketParams bp, const int32_t* __restrict__ neg_ids, const float* __restrict__ W, int Npad,
          float* __restrict__ GQ, int nx, int64_t ny) {
    using WTile = SplitTile<16 * RB>;
    using NTile = SplitTile<kGTile>;
    __shared__ __align__(16) char Ws[WTile::BYTES];
    __shared__ __align__(16) char Ns[NTile::BYTES];
    const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63, l15 = lane & 15, gq = lane >> 4;
    int bx;
    int64_t by;
    if (!xcd_tile((int64_t)nx * ny, nx, &bx, &by)) return;       // uniform
    const TileCoord tc = tile_coord(g, by);
    if (tc.nrows == 0) return;                // uniform: no gradient to write
    const int c0 = bx * kGTile;
    const int N = g.N, d = bp.dim;
    const float* En = tc.side == 0 ? bp.E_dst : bp.E_src;
    const int32_t* my_negs = neg_ids + ((int64_t)tc.si * g.nchunks + tc.c) * N;
    const float* Wtile = W + (int64_t)tc.wgrow * g.rows_tile * Npad;

    // W: eight consecutive negatives of rows srow, srow + 64 (weights past the last negative are zero in the buffer);
    // negatives: eight rows of one column, rows past the last replaced by it
    const int srow = tid >> 2, kg = tid & 3;
    constexpr int WI = (RB + 3) / 4;
    const float* wrow[WI];
#pragma unroll
    for (int u = 0; u < WI; ++u) wrow[u] = Wtile + (int64_t)min(srow + 64 * u, tc.nrows - 1) * kGNeg;
    const int64_t tile_stride = (int64_t)g.rows_tile * kGNeg;
    const int col = c0 + (tid & 127);
    const float* ecol = En + min(col, d - 1);
    const int kgc = __builtin_amdgcn_readfirstlane(tid >> 7);    // column groups kgc and kgc + 2: one per wave
    float wv[WI][8], nv[2][8];
    auto fetch = [&](int n0) {
        const int64_t off = (int64_t)(n0 >> 6) * tile_stride + (n0 & 63) + 8 * kg;
#pragma unroll
        for (int u = 0; u < WI; ++u) load8<4>(wrow[u] + off, 0, 8, wv[u]);
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int t = 0; t < 8; ++t)
                nv[u][t] = ecol[(int64_t)my_negs[min(n0 + 8 * (kgc + 2 * u) + t, N - 1)] * d];
    };
    f32v4 acc[RB][2];
#pragma unroll
    for (int r = 0; r < RB; ++r) acc[r][0] = acc[r][1] = f32v4{0.f, 0.f, 0.f, 0.f};
    const bool live = c0 + 32 * w < d;        // uniform per wave
    fetch(0);
    for (int n0 = 0; n0 < N; n0 += kGK) {
#pragma unroll
        for (int u = 0; u < WI; ++u)
            if (srow + 64 * u < 16 * RB) WTile::store(Ws, srow + 64 * u, kg, split8(wv[u]));
#pragma unroll
        for (int u = 0; u < 2; ++u) NTile::store(Ns, tid & 127, kgc + 2 * u, split8(nv[u]));
        __syncthreads();
        if (n0 + kGK < N) fetch(n0 + kGK);
        if (live) slice_mfma<RB, 2, WTile, NTile>(Ws, Ns, 32 * w, l15, gq, acc);
        __syncthreads();
    }
    bool nan = false;
#pragma unroll
    for (int r = 0; r < RB; ++r)
#pragma unroll
        for (int b = 0; b < 2; ++b) nan |= any_nan(acc[r][b]);
    if (__builtin_expect(__any(nan), 0))
        plain_products(N, [&](int r, int k) { return Wtile[(k >> 6) * tile_stride + min(16 * r + l15, tc.nrows - 1) * kGNeg + (k & 63)]; },
                       [&](int b, int k) { return En[(int64_t)my_negs[k] * d + min(c0 + 32 * w + 16 * b + l15, d - 1)]; }, acc);
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        const int oc = c0 + 32 * w + 16 * b + l15;
        if (oc >= d) continue;
        float* out = GQ + ((int64_t)tc.si * g.P + tc.e0) * d + oc;
#pragma unroll
        for (int r = 0; r < RB; ++r) {
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int row = 16 * r + 4 * gq + v;
                if (row < tc.nrows) out[(int64_t)row * d] = acc[r][b][v];
            }
        }
    }
}

// ---- G_neg = W^T Q -------------------------------------------------------------------------------
// grid: (tiles of 128 columns x tiles of 32 MB negatives, row tiles).  The positives are the contraction index: both operands
// are loaded eight rows of one column (or negative) to a thread.  Wave (wm, wn) owns 16 MB negatives x 64 columns.
// MB = 2 is for batches with few workgroups, as in the scores kernel (kGFew).
template <int MB>
__global__ void __launch_bounds__(kGThreads, 3)
k_gemm_gneg(BatchGeom g, BucketParams bp, const int32_t* __restrict__ neg_ids, const float* __restrict__ W, int Npad,
            const float* __restrict__ Q, float* __restrict__ grad, int ncol, int nx, int64_t ny) {
    constexpr int NEGS = 32 * MB, WU = MB / 2;
    using WTile = SplitTile<NEGS>;
    using QTile = SplitTile<kGTile>;
    __shared__ __align__(16) char Ws[WTile::BYTES];
    __shared__ __align__(16) char Qs[QTile::BYTES];
    const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63, l15 = lane & 15, gq = lane >> 4;
    const int wm = w >> 1, wn = w & 1;
    int bx;
    int64_t by;
    if (!xcd_tile((int64_t)nx * ny, nx, &bx, &by)) return;       // uniform
    const TileCoord tc = tile_coord(g, by);
    const int c0 = bx % ncol * kGTile, n0 = bx / ncol * NEGS;
    const int N = g.N, d = bp.dim, nrows = tc.nrows;
    const int32_t* my_negs = neg_ids + ((int64_t)tc.si * g.nchunks + tc.c) * N;
    const float* Wtile = W + (int64_t)tc.wgrow * g.rows_tile * Npad;
    const float* Qrows = Q + ((int64_t)tc.si * g.P + tc.e0) * d;
    const bool atomic = bp.atomic_mode != 0;
    float* Gn = tc.side == 0 ? bp.G_dst : bp.G_src;
    const int64_t neg_base = (int64_t)tc.si * g.per_side + (int64_t)g.roles * g.P + ((int64_t)tc.c * g.T + tc.t_row) * N;

    const int wcol = min(n0 + tid % NEGS, Npad - 1);
    const float* wp = Wtile + (int64_t)(wcol >> 6) * g.rows_tile * kGNeg + (wcol & 63);
    const float* qp = Qrows + min(c0 + (tid & 127), d - 1);
    const int kgq = __builtin_amdgcn_readfirstlane(tid >> 7), kgw = __builtin_amdgcn_readfirstlane(tid / NEGS);
    constexpr int AHEAD = MB == 2 ? 2 : 1;    // slices on their way
    float wv[AHEAD][WU][8], qv[AHEAD][2][8];
    auto fetch = [&](int s, int r0) {         // rows past the last one are replaced by it and get weight zero below
#pragma unroll
        for (int u = 0; u < WU; ++u)
#pragma unroll
            for (int t = 0; t < 8; ++t) wv[s][u][t] = wp[(int64_t)min(r0 + 8 * (kgw + 2 * u) + t, nrows - 1) * kGNeg];
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int t = 0; t < 8; ++t) qv[s][u][t] = qp[(int64_t)min(r0 + 8 * (kgq + 2 * u) + t, nrows - 1) * d];
    };
    f32v4 acc[MB][4];
#pragma unroll
    for (int a = 0; a < MB; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) acc[a][b] = f32v4{0.f, 0.f, 0.f, 0.f};
    const int live = min(4, (d - c0 - 64 * wn + 15) >> 4);       // column blocks of this wave, uniform
    if (nrows > 0) {
#pragma unroll
        for (int s = 0; s < AHEAD; ++s) fetch(s, kGK * s);
    }
    for (int rs = 0; rs < nrows; rs += kGK * AHEAD) {
#pragma unroll
        for (int s = 0; s < AHEAD; ++s) {
            const int r0 = rs + kGK * s;
            if (r0 >= nrows) break;           // uniform
            if (r0 + kGK > nrows) {
#pragma unroll
                for (int u = 0; u < WU; ++u) zero_past(wv[s][u], r0 + 8 * (kgw + 2 * u), nrows);
            }
#pragma unroll
            for (int u = 0; u < WU; ++u) WTile::store(Ws, tid % NEGS, kgw + 2 * u, split8(wv[s][u]));
#pragma unroll
            for (int u = 0; u < 2; ++u) QTile::store(Qs, tid & 127, kgq + 2 * u, split8(qv[s][u]));
            __syncthreads();
            if (r0 + kGK * AHEAD < nrows) fetch(s, r0 + kGK * AHEAD);
            if (live > 0) {
                Split8 A[MB];
#pragma unroll
                for (int a = 0; a < MB; ++a) A[a] = WTile::load(Ws, 16 * MB * wm + 16 * a + l15, gq);
#pragma unroll
                for (int b = 0; b < 4; ++b) {
                    if (b < live) {
                        Split8 B[1] = {QTile::load(Qs, 64 * wn + 16 * b + l15, gq)};
                        f32v4 c[MB][1];
#pragma unroll
                        for (int a = 0; a < MB; ++a) c[a][0] = acc[a][b];
                        split_mfma(A, B, c);
#pragma unroll
                        for (int a = 0; a < MB; ++a) acc[a][b] = c[a][0];
                    }
                }
            }
            __syncthreads();
        }
    }
    bool nan = false;
#pragma unroll
    for (int a = 0; a < MB; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) nan |= any_nan(acc[a][b]);
    if (__builtin_expect(__any(nan), 0))
        plain_products(nrows,
            [&](int a, int k) {
                const int n = min(n0 + 16 * MB * wm + 16 * a + l15, Npad - 1);
                return Wtile[((n >> 6) * g.rows_tile + k) * kGNeg + (n & 63)];
            },
            [&](int b, int k) { return Qrows[(int64_t)k * d + min(c0 + 64 * wn + 16 * b + l15, d - 1)]; }, acc);
    if (atomic) {
        // all ids first: loaded one at a time between the additions, each of these waited for its own (a batch of 2000 edges, both
        // sides, 64 negatives, d = 130: 22.5 us, 14.2 so)
        int32_t id[MB][4];
#pragma unroll
        for (int a = 0; a < MB; ++a)
#pragma unroll
            for (int v = 0; v < 4; ++v) id[a][v] = my_negs[min(n0 + 16 * MB * wm + 16 * a + 4 * gq + v, N - 1)];
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const int col = c0 + 64 * wn + 16 * b + l15;
            if (col >= d) continue;
#pragma unroll
            for (int a = 0; a < MB; ++a)
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    if (n0 + 16 * MB * wm + 16 * a + 4 * gq + v < N) unsafeAtomicAdd(Gn + (int64_t)id[a][v] * d + col, acc[a][b][v]);
        }
        return;
    }
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        const int col = c0 + 64 * wn + 16 * b + l15;
        if (col >= d) continue;
#pragma unroll
        for (int a = 0; a < MB; ++a)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int n = n0 + 16 * MB * wm + 16 * a + 4 * gq + v;
                if (n < N) row_store(grad + (neg_base + n) * d + col, acc[a][b][v], bp.stream_rows);
            }
    }
}

// ---- chain rule for the positives ---------------------------------------------------------------
template <int SCORE>
__global__ void __launch_bounds__(128)
k_gemm_chain(BatchGeom g, BucketParams bp, const float* __restrict__ Q, const float* __restrict__ GQ,
             const float* __restrict__ rowa, float* __restrict__ grad) {
    const int64_t idx = blockIdx.x;
    const int si = (int)(idx / g.P);
    const int64_t e = idx % g.P;
    const int side = g.side_id[si];
    const int d = bp.dim;
    const int32_t* eb = bp.edges + (bp.batch_lo + e) * 3;
    const int xid = eb[side == 0 ? 0 : 2], yid = eb[side == 0 ? 2 : 0], rid = eb[1];
    const float* x = (side == 0 ? bp.E_src : bp.E_dst) + (int64_t)xid * d;
    const float* y = (side == 0 ? bp.E_dst : bp.E_src) + (int64_t)yid * d;
    const float* r = SCORE == LEGEND_SCORE_DOT ? x : bp.E_rel + (int64_t)rid * d;
    const float* q = Q + idx * d;
    const float* gqr = GQ + idx * d;
    const float a = rowa[idx];
    const bool atomic = bp.atomic_mode != 0;
    const int64_t side_base = (int64_t)si * g.per_side;
    float* gx = grad + (side_base + (side == 0 ? 0 : g.P) + e) * d;
    float* gy = grad + (side_base + (side == 0 ? g.P : 0) + e) * d;
    float* gr = grad + (side_base + 2 * (int64_t)g.P + e) * d;
    if (atomic) {
        gx = (side == 0 ? bp.G_src : bp.G_dst) + (int64_t)xid * d;
        gy = (side == 0 ? bp.G_dst : bp.G_src) + (int64_t)yid * d;
        gr = bp.G_rel + (int64_t)rid * d;
    }
    auto emit = [&](float* p, float v) {
        if (atomic) unsafeAtomicAdd(p, v);
        else *p = v;
    };
    if (SCORE == LEGEND_SCORE_COMPLEX) {
        const int h = d >> 1;
        for (int k = threadIdx.x; k < h; k += 128) {
            const float xr = x[k], xi = x[k + h], rr = r[k], ri = r[k + h];
            const float gre = gqr[k] + a * y[k], gim = gqr[k + h] + a * y[k + h];
            emit(gy + k, a * q[k]);
            emit(gy + k + h, a * q[k + h]);
            if (side == 0) {
                emit(gx + k, rr * gre + ri * gim);      emit(gx + k + h, rr * gim - ri * gre);
                emit(gr + k, xr * gre + xi * gim);      emit(gr + k + h, xr * gim - xi * gre);
            } else {
                emit(gx + k, rr * gre - ri * gim);      emit(gx + k + h, rr * gim + ri * gre);
                emit(gr + k, gre * xr + gim * xi);      emit(gr + k + h, gre * xi - gim * xr);
            }
        }
    } else {
        for (int k = threadIdx.x; k < d; k += 128) {
            const float gv = gqr[k] + a * y[k];
            emit(gy + k, a * q[k]);
            if (SCORE == LEGEND_SCORE_DOT) {
                emit(gx + k, gv);
            } else {
                emit(gx + k, r[k] * gv);
                emit(gr + k, x[k] * gv);
            }
        }
    }
}

int64_t gemm_npad(int N) { return ((int64_t)N + kGNeg - 1) / kGNeg * kGNeg; }

hipError_t launch_chunks_gemm(hipStream_t st, const BatchGeom& g, const BucketParams& bp, const Workspace& ws) {
    if (bp.dim <= kNarrowMaxDim || bp.dim > kWideMaxDim || g.rows_tile > kGRows || !ws.gemm_Q)
        return hipErrorInvalidValue;
    const int64_t tiles = (int64_t)g.sides * g.nchunks * g.T;
    const int64_t rows = (int64_t)g.sides * g.P;
    const int Npad = (int)gemm_npad(g.N);
    const int coltiles = (bp.dim + kGTile - 1) / kGTile;
    const int ntiles128 = (g.N + kGTile - 1) / kGTile, ntiles64 = (g.N + 63) / 64;
    const bool few_scores = tiles * ntiles128 < kGFew;
    const bool few_gneg = tiles * ntiles128 * coltiles < kGFew;
    const int stiles = few_scores ? ntiles64 : ntiles128;
    const int ntiles = few_gneg ? ntiles64 : ntiles128;
    const bool softmax = bp.loss == LEGEND_LOSS_SOFTMAX;
    switch (bp.score) {
        case LEGEND_SCORE_DOT:
            hipLaunchKernelGGL(k_gemm_compose<LEGEND_SCORE_DOT>, dim3((unsigned)rows), dim3(128), 0, st, g, bp, ws.gemm_Q, ws.gemm_f);
            break;
        case LEGEND_SCORE_DISTMULT:
            hipLaunchKernelGGL(k_gemm_compose<LEGEND_SCORE_DISTMULT>, dim3((unsigned)rows), dim3(128), 0, st, g, bp, ws.gemm_Q, ws.gemm_f);
            break;
        default:
            hipLaunchKernelGGL(k_gemm_compose<LEGEND_SCORE_COMPLEX>, dim3((unsigned)rows), dim3(128), 0, st, g, bp, ws.gemm_Q, ws.gemm_f);
            break;
    }
    const int rb = (g.rows_tile + 15) / 16;
#define LEGEND_GEMM_RB(RB)                                                                                             \
    case RB: {                                                                                                         \
        auto scores = bp.dim % 4 == 0   ? (few_scores ? k_gemm_scores<RB, 4, 1> : k_gemm_scores<RB, 4, 2>)              \
                      : bp.dim % 2 == 0 ? (few_scores ? k_gemm_scores<RB, 2, 1> : k_gemm_scores<RB, 2, 2>)              \
                                        : (few_scores ? k_gemm_scores<RB, 1, 1> : k_gemm_scores<RB, 1, 2>);             \
        hipLaunchKernelGGL(scores, dim3((unsigned)xcd_grid(stiles * tiles)), dim3(kGThreads), 0, st, g, bp, ws.neg_ids, \
                           ws.gemm_Q, ws.gemm_S, Npad, stiles, tiles);                                                 \
        break;                                                                                                         \
    }
    switch (rb < 7 ? rb : 7) {
        LEGEND_GEMM_RB(1) LEGEND_GEMM_RB(2) LEGEND_GEMM_RB(3) LEGEND_GEMM_RB(4) LEGEND_GEMM_RB(5) LEGEND_GEMM_RB(6)
        LEGEND_GEMM_RB(7)
    }
#undef LEGEND_GEMM_RB
    if (softmax)
        hipLaunchKernelGGL(k_gemm_rowstats<LEGEND_LOSS_SOFTMAX>, dim3((unsigned)tiles), dim3(kStatThreads), 0, st, g, bp,
                           ws.gemm_S, ws.gemm_f, Npad, ws.gemm_a, ws.loss_partial);
    else if (bp.loss == LEGEND_LOSS_MARGIN)
        hipLaunchKernelGGL(k_gemm_rowstats<LEGEND_LOSS_MARGIN>, dim3((unsigned)tiles), dim3(kStatThreads), 0, st, g, bp,
                           ws.gemm_S, ws.gemm_f, Npad, ws.gemm_a, ws.loss_partial);
    else
        hipLaunchKernelGGL(k_gemm_rowstats<LEGEND_LOSS_LOGISTIC>, dim3((unsigned)tiles), dim3(kStatThreads), 0, st, g, bp,
                           ws.gemm_S, ws.gemm_f, Npad, ws.gemm_a, ws.loss_partial);
#define LEGEND_GEMM_RB(RB)                                                                                             \
    case RB:                                                                                                           \
        hipLaunchKernelGGL(k_gemm_gq<RB>, dim3((unsigned)xcd_grid(coltiles * tiles)), dim3(kGThreads), 0, st, g, bp,   \
                           ws.neg_ids, ws.gemm_S, Npad, ws.gemm_G, coltiles, tiles);                                   \
        break;
    switch (rb < 7 ? rb : 7) {
        LEGEND_GEMM_RB(1) LEGEND_GEMM_RB(2) LEGEND_GEMM_RB(3) LEGEND_GEMM_RB(4) LEGEND_GEMM_RB(5) LEGEND_GEMM_RB(6)
        LEGEND_GEMM_RB(7)
    }
#undef LEGEND_GEMM_RB
    const int negtiles = coltiles * ntiles;
    hipLaunchKernelGGL(few_gneg ? k_gemm_gneg<2> : k_gemm_gneg<4>, dim3((unsigned)xcd_grid(negtiles * tiles)), dim3(kGThreads), 0, st, g, bp, ws.neg_ids,
                       ws.gemm_S, Npad, ws.gemm_Q, ws.grad, coltiles, negtiles, tiles);
    switch (bp.score) {
        case LEGEND_SCORE_DOT:
            hipLaunchKernelGGL(k_gemm_chain<LEGEND_SCORE_DOT>, dim3((unsigned)rows), dim3(128), 0, st, g, bp, ws.gemm_Q, ws.gemm_G, ws.gemm_a, ws.grad);
            break;
        case LEGEND_SCORE_DISTMULT:
            hipLaunchKernelGGL(k_gemm_chain<LEGEND_SCORE_DISTMULT>, dim3((unsigned)rows), dim3(128), 0, st, g, bp, ws.gemm_Q, ws.gemm_G, ws.gemm_a, ws.grad);
            break;
        default:
            hipLaunchKernelGGL(k_gemm_chain<LEGEND_SCORE_COMPLEX>, dim3((unsigned)rows), dim3(128), 0, st, g, bp, ws.gemm_Q, ws.gemm_G, ws.gemm_a, ws.grad);
            break;
    }
    return hipGetLastError();
}

}  // namespace legend
