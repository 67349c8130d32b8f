// Small device/host helpers: the negative-sampling counter hash and wavefront utilities.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace legend {

// splitmix64 output function; the hash of a tuple absorbs one field at a time:
// h <- mix64(h + golden + field).
__host__ __device__ inline uint64_t hash_mix64(uint64_t z) {
    z ^= z >> 30;
    z *= 0xBF58476D1CE4E5B9ull;
    z ^= z >> 27;
    z *= 0x94D049BB133111EBull;
    z ^= z >> 31;
    return z;
}

__host__ __device__ inline uint64_t hash_fold(uint64_t h, uint64_t field) {
    return hash_mix64(h + 0x9E3779B97F4A7C15ull + field);
}

constexpr int kWave = 64;

__device__ inline int lane_id() { return threadIdx.x & (kWave - 1); }

__device__ inline float wave_shfl_xor(float v, int mask) { return __shfl_xor(v, mask, kWave); }

// Gradient rows are written once and read once, by the next kernel.  Where they and the tables do not fit the caches together
// (BucketParams::stream_rows), their loads and stores are marked as streaming, so that they displace less of the tables.
typedef float nt_f4 __attribute__((ext_vector_type(4)));
typedef float nt_f2 __attribute__((ext_vector_type(2)));
template <bool STREAM>
__device__ inline float4 row_load4(const float* p) {
    if (!STREAM) return *reinterpret_cast<const float4*>(p);
    const nt_f4 v = __builtin_nontemporal_load(reinterpret_cast<const nt_f4*>(p));
    return make_float4(v.x, v.y, v.z, v.w);
}
template <bool STREAM>
__device__ inline float2 row_load2(const float* p) {
    if (!STREAM) return *reinterpret_cast<const float2*>(p);
    const nt_f2 v = __builtin_nontemporal_load(reinterpret_cast<const nt_f2*>(p));
    return make_float2(v.x, v.y);
}
// (The empty statements around a marked store keep the compiler from making one unmarked store of the two branches.)
__device__ inline void row_store4(float* p, float4 v, int stream) {
    const nt_f4 x = {v.x, v.y, v.z, v.w};
    if (stream) {
        asm volatile("");
        __builtin_nontemporal_store(x, reinterpret_cast<nt_f4*>(p));
        asm volatile("");
    } else {
        *reinterpret_cast<nt_f4*>(p) = x;
    }
}
__device__ inline void row_store2(float* p, float2 v, int stream) {
    const nt_f2 x = {v.x, v.y};
    if (stream) {
        asm volatile("");
        __builtin_nontemporal_store(x, reinterpret_cast<nt_f2*>(p));
        asm volatile("");
    } else {
        *reinterpret_cast<nt_f2*>(p) = x;
    }
}
__device__ inline void row_store(float* p, float v, int stream) {
    if (stream) {
        asm volatile("");
        __builtin_nontemporal_store(v, p);
        asm volatile("");
    } else {
        *p = v;
    }
}

}  // namespace legend
