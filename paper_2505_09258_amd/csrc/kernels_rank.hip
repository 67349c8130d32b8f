// Link-prediction ranks (Sec. 7 "Metrics": MRR and Hits@k are functions of these ranks).
//
// A test triple's corrupted endpoint is replaced by every candidate node; with the score in the
// form (theta_s (x) theta_r) (+) theta_d of Sec. 6 the scores of all replacements are one real
// matrix product: rows q_e = theta_s (x) theta_r (destination side) or conj(theta_r) (x) theta_d
// (source side) against the candidates' embedding rows.  The product runs on the matrix pipe,
// every float cut into three bf16 parts, and is never stored: each block of scores is compared with the triples' own scores and
// only the counts (strictly greater / equal) leave the kernel.
#include <hip/hip_runtime.h>

#include "legend_internal.h"
#include "device_utils.h"
#include "split_bf16.h"

namespace legend {

namespace {

constexpr int kRankRows = 64;       // the scratch buffers hold whole tiles of this many triples
constexpr int kRankGroups = 2048;   // workgroups of the counting kernel to aim at

__host__ __device__ inline int rank_dpad(int d) { return (d + 15) & ~15; }
__host__ __device__ inline int rank_stride(int d) { return rank_dpad(d) + 4; }

// ---- q_e, f_e and the true endpoint of every triple: one wavefront per triple ----------------
__global__ void __launch_bounds__(256)
k_rank_compose(const int64_t* __restrict__ src, const int32_t* __restrict__ rel, const int64_t* __restrict__ dst,
               int64_t m, int64_t m_pad, int32_t side, float* const* __restrict__ part_emb, int32_t rows_pp,
               int64_t num_nodes, const float* __restrict__ E_rel, int32_t num_rel, int32_t d, int32_t score,
               float* __restrict__ Q, float* __restrict__ f, int32_t* __restrict__ true_id,
               uint32_t* __restrict__ err_flag) {
    const int lane = lane_id();
    const int64_t e = (int64_t)blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave;
    if (e >= m_pad) return;
    const int dp = rank_dpad(d);
    float* q = Q + e * dp;
    const float* sp = nullptr;
    const float* tp = nullptr;
    int32_t r = 0;
    int64_t s = 0, t = 0;
    bool ok = e < m;
    if (ok) {
        s = src[e]; t = dst[e];
        r = rel ? rel[e] : 0;
        bool bad = s < 0 || s >= num_nodes || t < 0 || t >= num_nodes;
        if (score != LEGEND_SCORE_DOT) bad |= r < 0 || r >= num_rel;
        if (bad) { if (lane == 0) atomicOr(err_flag, 1u); ok = false; }
    }
    if (ok) {
        sp = part_emb[s / rows_pp];
        tp = part_emb[t / rows_pp];
        if (!sp || !tp) { if (lane == 0) atomicOr(err_flag, 2u); ok = false; }
    }
    if (!ok) {
        for (int k = lane; k < dp; k += kWave) q[k] = 0.f;
        if (lane == 0) { f[e] = 0.f; true_id[e] = -1; }
        return;
    }
    sp += (s % rows_pp) * d;
    tp += (t % rows_pp) * d;
    const float* rp = E_rel + (int64_t)r * d;
    // a = the endpoint that stays, b = the endpoint that is replaced
    const float* a = side == LEGEND_CORRUPT_SRC ? tp : sp;
    const float* b = side == LEGEND_CORRUPT_SRC ? sp : tp;
    // the triple's own score decides every comparison of its row: summed in 64 bits, rounded once
    double acc = 0.0;
    if (score == LEGEND_SCORE_COMPLEX) {
        const int h = d >> 1;
        for (int k = lane; k < h; k += kWave) {
            float qr, qi;
            if (side == LEGEND_CORRUPT_SRC) {   // conj(r) * d
                qr = rp[k] * a[k] + rp[k + h] * a[k + h];
                qi = rp[k] * a[k + h] - rp[k + h] * a[k];
            } else {                            // s * r
                qr = a[k] * rp[k] - a[k + h] * rp[k + h];
                qi = a[k] * rp[k + h] + a[k + h] * rp[k];
            }
            q[k] = qr; q[k + h] = qi;
            acc += (double)qr * b[k] + (double)qi * b[k + h];
        }
    } else if (score == LEGEND_SCORE_TRANSE_L1) {
        for (int k = lane; k < d; k += kWave) {       // s + r meets d; d - r meets s
            const float v = side == LEGEND_CORRUPT_SRC ? a[k] - rp[k] : a[k] + rp[k];
            q[k] = v;
            acc -= fabsf(v - b[k]);
        }
    } else {
        for (int k = lane; k < d; k += kWave) {
            const float v = score == LEGEND_SCORE_DISTMULT ? a[k] * rp[k] : a[k];
            q[k] = v;
            acc += (double)v * b[k];
        }
    }
    for (int k = d + lane; k < dp; k += kWave) q[k] = 0.f;
    for (int off = kWave / 2; off > 0; off >>= 1) acc += __shfl_down(acc, off, kWave);
    if (lane == 0) { f[e] = (float)acc; true_id[e] = (int32_t)(side == LEGEND_CORRUPT_SRC ? s : t); }
}

// Four consecutive components k..k+3 of a candidate row (zeros past the row's end).
template <bool ALIGNED>
__device__ inline float4 cand_load4(const float* __restrict__ row, int k, int d) {
    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
    if (!row) return v;
    if (ALIGNED) {
        if (k < d) v = *reinterpret_cast<const float4*>(row + k);
    } else {
        if (k < d) v.x = row[k];
        if (k + 1 < d) v.y = row[k + 1];
        if (k + 2 < d) v.z = row[k + 2];
        if (k + 3 < d) v.w = row[k + 3];
    }
    return v;
}

// Workgroup (x, y): 128 triples (tile x) against the y-th share of the candidates, 128 of them at a time; four waves,
// wave (wm, wn) owns 64 candidates x 64 triples as 4 x 4 blocks of 16 x 16.  The scores are one contraction and used to be
// bound by the fp32 matrix pipe; here both operands are cut into three bf16 parts on their way into LDS and multiplied by
// six bf16 instructions (split_bf16.h).  An operand element meets 128 others, which pays for cutting both sides anew
// for every tile: an operand cut beforehand would need 6 bytes an element of scratch memory, which the call on static
// scratch does not have.  Slices of 32 components, the next one on its way from memory while this one is multiplied;
// 49 KB of LDS and at most 256 registers leave two workgroups on a compute unit, whose cutting and multiplying overlap.
// Measured, whole calls: 10 000 triples against 15 000 candidates of 400 components 1.46 -> 0.89 ms, against a list of 50 000 of
// 100 components 1.24 -> 1.00 ms (fp32 matrix instructions, q rows in LDS, candidates straight from memory).  Loading and
// masking in one step had the multiplication wait for memory: 0.97 and 1.13 ms.
// Candidates are the A operand: a lane then holds four triples (columns l15) and sixteen candidates, and counts in
// eight registers.  A candidate that does not count (past the share's end, out of range) is a row of NaN: every
// comparison with its scores is false.
constexpr int kRankTile = 128;
constexpr int kRankK = 32;
constexpr int kRankThreads = 256;

template <bool ALIGNED>
__global__ void __launch_bounds__(kRankThreads, 2)
k_rank(const float* __restrict__ Q, const float* __restrict__ f, const int32_t* __restrict__ true_id, int64_t m, int64_t m_pad,
       const int64_t* __restrict__ cand, int64_t n_cand, int64_t cand_per_wg, float* const* __restrict__ part_emb,
       int32_t rows_pp, int64_t num_nodes, int32_t d, int32_t* __restrict__ greater, int32_t* __restrict__ equal,
       uint32_t* __restrict__ err_flag) {
    using Tile = SplitTile<kRankTile>;
    __shared__ __align__(16) char cs[Tile::BYTES];
    __shared__ __align__(16) char qs[Tile::BYTES];
    __shared__ __align__(16) int32_t id_s[2][kRankTile];         // candidate ids of this and the next tile, -1 = does not count
    __shared__ int32_t cnt_s[kRankTile][2];

    const int dp = rank_dpad(d);
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int li = lane & 15, g = lane >> 4;
    const int wm = w >> 1, wn = w & 1;
    const int64_t row0 = (int64_t)blockIdx.x * kRankTile;
    const int64_t c_lo = (int64_t)blockIdx.y * cand_per_wg;
    const int64_t c_hi = c_lo + cand_per_wg < n_cand ? c_lo + cand_per_wg : n_cand;
    const int nk = (dp + kRankK - 1) / kRankK;

    // a thread's share of a slice: elements 8kg..8kg+7 of rows srow and srow + 64 of either operand
    const int srow = tid >> 2, kg = tid & 3;
    const float* crow[2];
    bool dead[2];
    auto open_tile = [&](int64_t cb, int buf) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int64_t j = cb + srow + 64 * u;
            int32_t cid = -1;
            crow[u] = Q;                               // some row: what is loaded is replaced by NaN
            if (j < c_hi) {
                const int64_t id = cand ? cand[j] : j;
                if (id < 0 || id >= num_nodes) {
                    if (kg == 0) atomicOr(err_flag, 1u);
                } else {
                    const uint32_t part = (uint32_t)id / (uint32_t)rows_pp;      // num_nodes < 2^31
                    const float* base = part_emb[part];
                    if (!base) { if (kg == 0) atomicOr(err_flag, 2u); }
                    else {
                        cid = (int32_t)id;
                        crow[u] = base + (int64_t)((uint32_t)id - part * (uint32_t)rows_pp) * d;
                    }
                }
            }
            if (kg == 0) id_s[buf][srow + 64 * u] = cid;
            dead[u] = cid < 0;
        }
    };
    // Loads only: anything done to a loaded value here would wait for it in front of the multiplication.  Components past
    // the row's end are replaced by others of the row, which meet zeros of Q.
    const float* qrow[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int64_t r = row0 + srow + 64 * u;
        qrow[u] = Q + (r < m_pad ? r : m_pad - 1) * dp;          // a row past the last one is never counted
    }
    float cv[2][8], qv[2][8];
    auto fetch = [&](int ks) {
        const int k = kRankK * ks + 8 * kg;
        const int kq = k < dp ? k : 0;                 // dp is a multiple of 16: both halves or none
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            if (ALIGNED) {
                const float4 x = *reinterpret_cast<const float4*>(crow[u] + (k < d ? k : 0));
                const float4 y = *reinterpret_cast<const float4*>(crow[u] + (k + 4 < d ? k + 4 : 0));
                cv[u][0] = x.x; cv[u][1] = x.y; cv[u][2] = x.z; cv[u][3] = x.w;
                cv[u][4] = y.x; cv[u][5] = y.y; cv[u][6] = y.z; cv[u][7] = y.w;
            } else {
#pragma unroll
                for (int t = 0; t < 8; ++t) cv[u][t] = crow[u][k + t < d ? k + t : d - 1];
            }
            const float4 x = *reinterpret_cast<const float4*>(qrow[u] + kq);
            const float4 y = *reinterpret_cast<const float4*>(qrow[u] + kq + 4);
            qv[u][0] = x.x; qv[u][1] = x.y; qv[u][2] = x.z; qv[u][3] = x.w;
            qv[u][4] = y.x; qv[u][5] = y.y; qv[u][6] = y.z; qv[u][7] = y.w;
        }
    };
    // the slice of the last fetch into LDS
    auto commit = [&](int ks) {
        if (ks == 0) {                                 // one NaN factor makes the whole score a NaN
#pragma unroll
            for (int u = 0; u < 2; ++u)
                if (dead[u]) cv[u][0] = __builtin_nanf("");
        }
        if (kRankK * (ks + 1) > dp && kg >= 2) {
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int t = 0; t < 8; ++t) qv[u][t] = 0.f;
        }
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            Tile::store(cs, srow + 64 * u, kg, split8(cv[u]));
            Tile::store(qs, srow + 64 * u, kg, split8(qv[u]));
        }
    };

    // this lane's triples: columns 64wn + 16b + li
    float fv[4];
    int32_t tv[4];
    int gt[4], eq[4];
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        const int64_t r = row0 + 64 * wn + 16 * b + li;
        fv[b] = r < m_pad ? f[r] : 0.f;
        tv[b] = r < m_pad ? true_id[r] : -1;
        gt[b] = eq[b] = 0;
    }
    if (tid < kRankTile) cnt_s[tid][0] = cnt_s[tid][1] = 0;

    int buf = 0;
    open_tile(c_lo, 0);
    fetch(0);
    for (int64_t cb = c_lo; cb < c_hi; cb += kRankTile, buf ^= 1) {
        f32v4 acc[4][4];
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int b = 0; b < 4; ++b) acc[a][b] = f32v4{0.f, 0.f, 0.f, 0.f};
        for (int ks = 0; ks < nk; ++ks) {
            commit(ks);
            __syncthreads();
            if (ks + 1 < nk) {
                fetch(ks + 1);
            } else if (cb + kRankTile < c_hi) {
                open_tile(cb + kRankTile, buf ^ 1);
                fetch(0);
            }
            Split8 A[4], B[4];
#pragma unroll
            for (int b = 0; b < 4; ++b) B[b] = Tile::load(qs, 64 * wn + 16 * b + li, g);
#pragma unroll
            for (int a = 0; a < 4; ++a) A[a] = Tile::load(cs, 64 * wm + 16 * a + li, g);
            split_mfma(A, B, acc);
            __syncthreads();
        }
        // acc[a][b][v] = score of candidate 64wm + 16a + 4g + v against triple 64wn + 16b + li
#pragma unroll
        for (int a = 0; a < 4; ++a) {
            const int4 c4 = *reinterpret_cast<const int4*>(&id_s[buf][64 * wm + 16 * a + 4 * g]);
            const int32_t cid[4] = {c4.x, c4.y, c4.z, c4.w};
            float sum = 0.f;
#pragma unroll
            for (int b = 0; b < 4; ++b)
#pragma unroll
                for (int v = 0; v < 4; ++v) sum += acc[a][b][v];
            if (__builtin_expect(sum != sum, 0)) {
                // An infinity took part, or a score is a NaN: the plain sums of the candidates that count say which.  A sum ends
                // at its first NaN: a diverged table's rows are NaN from the first component on (3000 triples, 6000
                // candidates, d = 256: 0.11 ms finite, 0.15 ms all NaN, 11 ms when every sum was carried to its end).
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    if (cid[v] < 0) continue;
                    const uint32_t part = (uint32_t)cid[v] / (uint32_t)rows_pp;
                    const float* x = part_emb[part] + (int64_t)((uint32_t)cid[v] - part * (uint32_t)rows_pp) * d;
#pragma unroll
                    for (int b = 0; b < 4; ++b) {
                        if (acc[a][b][v] == acc[a][b][v]) continue;
                        const int64_t r = row0 + 64 * wn + 16 * b + li;
                        const float* q = Q + (r < m_pad ? r : m_pad - 1) * dp;
                        float s = 0.f;
                        for (int k = 0; k < d && s == s; ++k) s = fmaf(q[k], x[k], s);
                        acc[a][b][v] = s;
                    }
                }
            }
#pragma unroll
            for (int b = 0; b < 4; ++b)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const float s = acc[a][b][v];
                    const bool counted = cid[v] != tv[b];
                    gt[b] += (counted && s > fv[b]) ? 1 : 0;
                    eq[b] += (counted && s == fv[b]) ? 1 : 0;
                }
        }
    }
    // the four lane groups and the two candidate halves hold different candidates of the same triples
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        int x = gt[b], e = eq[b];
        x += __shfl_xor(x, 16, kWave); e += __shfl_xor(e, 16, kWave);
        x += __shfl_xor(x, 32, kWave); e += __shfl_xor(e, 32, kWave);
        if (g == 0) {
            if (x) atomicAdd(&cnt_s[64 * wn + 16 * b + li][0], x);
            if (e) atomicAdd(&cnt_s[64 * wn + 16 * b + li][1], e);
        }
    }
    __syncthreads();
    if (tid < kRankTile && row0 + tid < m) {
        if (cnt_s[tid][0]) atomicAdd(&greater[row0 + tid], cnt_s[tid][0]);
        if (cnt_s[tid][1]) atomicAdd(&equal[row0 + tid], cnt_s[tid][1]);
    }
}

// The same counts for the translational score -|q - c|_1: no matrix product.  A lane keeps one
// candidate row in registers (dim <= 128) and meets the 64 q rows of the tile one after the other
// (LDS broadcast reads); the comparisons of a row against 64 candidates are counted by ballot.
constexpr int kRankTransWaves = 4;
constexpr int kRankTransMaxD4 = 32;

template <bool ALIGNED>
__global__ void __launch_bounds__(kRankTransWaves* kWave)
k_rank_trans(const float* __restrict__ Q, const float* __restrict__ f, const int32_t* __restrict__ true_id, int64_t m,
             const int64_t* __restrict__ cand, int64_t n_cand, int64_t cand_per_wg, float* const* __restrict__ part_emb,
             int32_t rows_pp, int64_t num_nodes, int32_t d, int32_t* __restrict__ greater, int32_t* __restrict__ equal,
             uint32_t* __restrict__ err_flag) {
    extern __shared__ __align__(16) float lds[];
    const int dp = rank_dpad(d);
    const int stride = rank_stride(d);
    float* q_s = lds;
    float* f_s = q_s + kRankRows * stride;
    int32_t* t_s = reinterpret_cast<int32_t*>(f_s + kRankRows);
    int32_t* cnt_s = t_s + kRankRows;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int64_t row0 = (int64_t)blockIdx.x * kRankRows;
    for (int idx = tid; idx < kRankRows * (dp / 4); idx += kRankTransWaves * kWave) {
        const int r = idx / (dp / 4), k4 = idx % (dp / 4);
        *reinterpret_cast<float4*>(q_s + r * stride + 4 * k4) =
            *reinterpret_cast<const float4*>(Q + (row0 + r) * dp + 4 * k4);
    }
    if (tid < kRankRows) {
        f_s[tid] = f[row0 + tid];
        t_s[tid] = true_id[row0 + tid];
        cnt_s[2 * tid] = 0;
        cnt_s[2 * tid + 1] = 0;
    }
    __syncthreads();
    const int64_t c_lo = (int64_t)blockIdx.y * cand_per_wg;
    const int64_t c_hi = c_lo + cand_per_wg < n_cand ? c_lo + cand_per_wg : n_cand;
    const int d4 = (d + 3) >> 2;
    const int nrows = (int)(m - row0 < kRankRows ? m - row0 : kRankRows);
    for (int64_t cb = c_lo + kWave * w; cb < c_hi; cb += kWave * kRankTransWaves) {
        const int64_t j = cb + lane;
        int64_t cid = -1;
        const float* row = nullptr;
        if (j < c_hi) {
            cid = cand ? cand[j] : j;
            if (cid < 0 || cid >= num_nodes) {
                atomicOr(err_flag, 1u);
                cid = -1;
            } else {
                const float* base = part_emb[cid / rows_pp];
                if (!base) { atomicOr(err_flag, 2u); cid = -1; }
                else row = base + (cid % rows_pp) * d;
            }
        }
        float4 cr[kRankTransMaxD4];
#pragma unroll
        for (int j4 = 0; j4 < kRankTransMaxD4; ++j4)
            cr[j4] = j4 < d4 ? cand_load4<ALIGNED>(row, 4 * j4, d) : make_float4(0.f, 0.f, 0.f, 0.f);
        const int32_t cid32 = (int32_t)cid;
        for (int r = 0; r < nrows; ++r) {
            const float* qr = q_s + r * stride;
            float s = 0.f;
#pragma unroll
            for (int j4 = 0; j4 < kRankTransMaxD4; ++j4) {
                if (j4 < d4) {
                    const float4 q4 = *reinterpret_cast<const float4*>(qr + 4 * j4);
                    s += (fabsf(q4.x - cr[j4].x) + fabsf(q4.y - cr[j4].y)) + (fabsf(q4.z - cr[j4].z) + fabsf(q4.w - cr[j4].w));
                }
            }
            const float S = -s, fv = f_s[r];
            const bool counted = cid >= 0 && cid32 != t_s[r];
            const unsigned long long gtm = __ballot(counted && S > fv), eqm = __ballot(counted && S == fv);
            if (lane == 0) {
                if (gtm) atomicAdd(&cnt_s[2 * r], __popcll(gtm));
                if (eqm) atomicAdd(&cnt_s[2 * r + 1], __popcll(eqm));
            }
        }
    }
    __syncthreads();
    if (tid < kRankRows && row0 + tid < m) {
        if (cnt_s[2 * tid]) atomicAdd(&greater[row0 + tid], cnt_s[2 * tid]);
        if (cnt_s[2 * tid + 1]) atomicAdd(&equal[row0 + tid], cnt_s[2 * tid + 1]);
    }
}

// rank = 1 + greater + equal / 2;  sums of 1/rank and of the hit indicators in a fixed order
__global__ void __launch_bounds__(256)
k_rank_metrics(const int32_t* __restrict__ greater, const int32_t* __restrict__ equal, int64_t m,
               double* __restrict__ out /* [4]: mrr, hits@1, hits@3, hits@10 */) {
    __shared__ double part[4][256];
    double s[4] = {0.0, 0.0, 0.0, 0.0};
    for (int64_t e = threadIdx.x; e < m; e += 256) {
        const double rank = 1.0 + (double)greater[e] + 0.5 * (double)equal[e];
        s[0] += 1.0 / rank;
        s[1] += rank <= 1.0 ? 1.0 : 0.0;
        s[2] += rank <= 3.0 ? 1.0 : 0.0;
        s[3] += rank <= 10.0 ? 1.0 : 0.0;
    }
    for (int k = 0; k < 4; ++k) part[k][threadIdx.x] = s[k];
    __syncthreads();
    for (int off = 128; off > 0; off >>= 1) {
        if ((int)threadIdx.x < off)
            for (int k = 0; k < 4; ++k) part[k][threadIdx.x] += part[k][threadIdx.x + off];
        __syncthreads();
    }
    if (threadIdx.x < 4) out[threadIdx.x] = m > 0 ? part[threadIdx.x][0] / (double)m : 0.0;
}

}  // namespace

int64_t rank_rows_padded(int64_t m) { return (m + kRankRows - 1) / kRankRows * kRankRows; }
int rank_dim_padded(int d) { return rank_dpad(d); }

hipError_t launch_rank(hipStream_t st, const int64_t* src, const int32_t* rel, const int64_t* dst, int64_t m,
                       int32_t side, const int64_t* cand, int64_t n_cand, float* const* part_emb,
                       int32_t rows_per_partition, int64_t num_nodes, const float* E_rel, int32_t num_relations,
                       int32_t dim, int32_t score, float* Q, float* f, int32_t* true_id, int32_t* greater,
                       int32_t* equal, double* metrics, uint32_t* err_flag) {
    if (m <= 0) return hipSuccess;
    const int64_t m_pad = rank_rows_padded(m);
    hipLaunchKernelGGL(k_rank_compose, dim3((unsigned)((m_pad + 3) / 4)), dim3(256), 0, st, src, rel, dst, m, m_pad, side,
                       part_emb, rows_per_partition, num_nodes, E_rel, num_relations, dim, score, Q, f, true_id, err_flag);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (n_cand > 0) {
        const int64_t tiles = m_pad / kRankRows;
        const bool aligned = dim % 4 == 0;
        const size_t lds = sizeof(float) * ((size_t)kRankRows * rank_stride(dim) + kRankRows) + sizeof(int32_t) * 3 * kRankRows;
        if (score == LEGEND_SCORE_TRANSE_L1) {
            if (dim > 4 * kRankTransMaxD4) return hipErrorInvalidValue;
            const int64_t step = kWave * kRankTransWaves;
            int64_t shares = (4096 + tiles - 1) / tiles;
            const int64_t max_shares = (n_cand + step - 1) / step;
            if (shares > max_shares) shares = max_shares;
            if (shares < 1) shares = 1;
            if (shares > 65535) shares = 65535;
            int64_t per = (n_cand + shares - 1) / shares;
            per = (per + step - 1) / step * step;
            shares = (n_cand + per - 1) / per;
            const void* fn = aligned ? reinterpret_cast<const void*>(&k_rank_trans<true>) : reinterpret_cast<const void*>(&k_rank_trans<false>);
            e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
            if (e != hipSuccess) return e;
            dim3 grid((unsigned)tiles, (unsigned)shares), block(kRankTransWaves * kWave);
            if (aligned)
                hipLaunchKernelGGL(k_rank_trans<true>, grid, block, lds, st, Q, f, true_id, m, cand, n_cand, per, part_emb,
                                   rows_per_partition, num_nodes, dim, greater, equal, err_flag);
            else
                hipLaunchKernelGGL(k_rank_trans<false>, grid, block, lds, st, Q, f, true_id, m, cand, n_cand, per, part_emb,
                                   rows_per_partition, num_nodes, dim, greater, equal, err_flag);
            e = hipGetLastError();
            if (e != hipSuccess) return e;
            hipLaunchKernelGGL(k_rank_metrics, dim3(1), dim3(256), 0, st, greater, equal, m, metrics);
            return hipGetLastError();
        }
        // workgroups to fill the chip (two on a compute unit) a few times over, each with at least two tiles of candidates
        const int64_t row_tiles = (m_pad + kRankTile - 1) / kRankTile;
        int64_t shares = (kRankGroups + row_tiles - 1) / row_tiles;
        const int64_t max_shares = (n_cand + 2 * kRankTile - 1) / (2 * kRankTile);
        if (shares > max_shares) shares = max_shares;
        if (shares < 1) shares = 1;
        if (shares > 65535) shares = 65535;
        int64_t per = (n_cand + shares - 1) / shares;
        per = (per + kRankTile - 1) / kRankTile * kRankTile;
        shares = (n_cand + per - 1) / per;
        dim3 grid((unsigned)row_tiles, (unsigned)shares), block(kRankThreads);
        if (aligned)
            hipLaunchKernelGGL(k_rank<true>, grid, block, 0, st, Q, f, true_id, m, m_pad, cand, n_cand, per, part_emb,
                               rows_per_partition, num_nodes, dim, greater, equal, err_flag);
        else
            hipLaunchKernelGGL(k_rank<false>, grid, block, 0, st, Q, f, true_id, m, m_pad, cand, n_cand, per, part_emb,
                               rows_per_partition, num_nodes, dim, greater, equal, err_flag);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(k_rank_metrics, dim3(1), dim3(256), 0, st, greater, equal, m, metrics);
    return hipGetLastError();
}

}  // namespace legend
