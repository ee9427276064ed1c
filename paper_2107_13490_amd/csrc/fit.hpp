// Pieces of the "fitting" requantization that several kernels share: an exact accumulator tensor is stored in
// WL bits with the smallest right shift that makes its largest magnitude fit (the gradient tensors of the
// chained step; Sec. 3.3 "Dealing with Fixed-Points Limited Range" makes their common scale irrelevant).
#pragma once
#include "common.hpp"

namespace adapt {

struct FitArgs {
    const void *acc;
    void *q;
    const uint64_t *part;
    int nparts;
    uint64_t n;
    int wl, mode;
    uint64_t seed, stream;
    int32_t *shift_out;
    unsigned long long *sumsq;
    // exponent of the codes: *e_out = (e_in ? *e_in : 0) + e_add - shift (device memory; e_out may be null)
    const long long *e_in;
    long long e_add;
    long long *e_out;
};

__device__ __forceinline__ uint64_t magnitude(long long v) { return v < 0 ? 0ull - (uint64_t)v : (uint64_t)v; }

__device__ __forceinline__ uint64_t wave_max_u64(uint64_t v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        const uint64_t o = __shfl_xor((unsigned long long)v, off, 64);
        v = o > v ? o : v;
    }
    return v;
}

// The requantize rule for a shift that was fitted to the tensor: |acc| >> shift is below 2^(wl-1)
// <= 2^15, so after one 64-bit shift everything is 32-bit arithmetic.  floor((acc + r') / 2^s) is
// taken as (acc >> s) + carry of the dropped bits plus r', which cannot overflow.
__device__ __forceinline__ int fit_one(long long acc, int shift, uint32_t r16, int qlo, int qhi)
{
    int q;
    if (shift == 0) {
        q = (int)acc;
    } else if (shift <= 16) {
        const uint32_t low = (uint32_t)acc & ((1u << shift) - 1u);
        q = (int)(acc >> shift) + (int)((low + (r16 >> (16 - shift))) >> shift);
    } else {
        const int t = (int)(acc >> (shift - 16));            // |t| < 2^(wl-1+16) <= 2^31
        q = (t >> 16) + (int)((((uint32_t)t & 0xffffu) + r16) >> 16);
    }
    return min(max(q, qlo), qhi);
}

// fit_one on sums of 32 bits, and on 256 u + low (0 <= low < 256, u in 32 bits): the same values, since the shift is one after which
// they fit 16 bits
__device__ __forceinline__ int fit_one32(int v, int shift, uint32_t r16)
{
    if (shift == 0) return v;
    if (shift <= 16) return (v >> shift) + (int)((((uint32_t)v & ((1u << shift) - 1u)) + (r16 >> (16 - shift))) >> shift);
    const int t = v >> (shift - 16);
    return (t >> 16) + (int)((((uint32_t)t & 0xffffu) + r16) >> 16);
}
__device__ __forceinline__ int fit_pair(int u, int low, int shift, uint32_t r16)
{
    if (shift < 8) return (int)((uint32_t)u << (8 - shift)) + ((low + (int)(r16 >> (16 - shift))) >> shift);
    if (shift <= 16) return (u + ((low + (int)(r16 >> (16 - shift))) >> 8)) >> (shift - 8);
    const int t = shift >= 24 ? u >> (shift - 24) : (int)((uint32_t)u << (24 - shift)) | (low >> (shift - 16));
    return (t >> 16) + (int)((((uint32_t)t & 0xffffu) + r16) >> 16);
}

// shift = max(0, bit_length(m) - (wl - 1)) for the largest magnitude m
__device__ __forceinline__ int fit_shift_of(uint64_t m, int wl)
{
    const int bits = m ? 64 - __clzll((long long)m) : 0;
    return max(0, bits - (wl - 1));
}

// a thread's share of the maximum over part[0..nparts), nparts >= 1: a fitting pass starts with it in every block, up to
// 8192 values behind nothing but the latency of their loads, so eight are in flight (one at a time: 32 latencies for 256
// threads; with the 1024-thread form of the pass that sums squares, AlexNet step 1134 -> 1123 us, ResNet-18 4734 -> 4705)
template <int THREADS>
__device__ __forceinline__ uint64_t max_of_parts(const uint64_t *__restrict__ part, const int nparts)
{
    uint64_t m = 0;
    for (int i = threadIdx.x; i < nparts; i += 8 * THREADS) {
        uint64_t t[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) t[u] = part[min(i + u * THREADS, nparts - 1)];      // repeats the last value past the end
#pragma unroll
        for (int u = 0; u < 8; ++u) m = t[u] > m ? t[u] : m;
    }
    return m;
}

// block-wide maximum of per-thread values (all threads get it); sm: one word per wavefront
__device__ __forceinline__ uint64_t block_max_u64(uint64_t m, uint64_t *sm, int nwaves)
{
    m = wave_max_u64(m);
    if ((threadIdx.x & (kWave - 1)) == 0) sm[threadIdx.x / kWave] = m;
    __syncthreads();
    m = sm[0];
    for (int i = 1; i < nwaves; ++i) m = sm[i] > m ? sm[i] : m;
    __syncthreads();
    return m;
}

}  // namespace adapt
