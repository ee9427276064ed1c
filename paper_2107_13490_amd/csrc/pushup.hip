// PushUp (Sec. 3.3 "The PushUp Operation", "Dealing with Fixed-Points Limited Range",
// "Strategy, Resolution and Lookback") for gfx950.
//
// Device part: the gradient-diversity equation over a lookback window of gradient tensors held
// as fixed-point codes.  One pass over the window: every thread owns 8 consecutive elements (16 in windows of
// int32 codes), reads them from each tensor in turn, keeps the running element-wise sum of the aligned codes in
// registers and the per-tensor sums of squares in LDS counters.  All sums are integers (exact, order-independent); a one-block
// follow-up kernel adds the block partials and forms the norms and the ratio in fp64.
//
// Host part: the scalar rules that turn the diversity into a new <WL,FL>, lookback,
// resolution and strategy.  They are plain functions and need no device.
#include <algorithm>
#include <cmath>

#include "common.hpp"
#include "context.hpp"
#include "grad_window.hpp"
#include "ticket.hpp"
#include "wide.hpp"

namespace adapt {

constexpr int kGdThreads = 256;
constexpr int kGdPerThread = 16;          // elements per thread
constexpr int kGdFinalThreads = 1024;

typedef unsigned gd_v4u __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint64_t wave_sum_u64(uint64_t v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor((unsigned long long)v, off, 64);
    return v;
}

__device__ __forceinline__ void unpack16(const gd_v4u (&raw)[2], int es, int (&c)[16])
{
    if (es == 1) {
#pragma unroll
        for (int j = 0; j < 16; ++j) c[j] = (int)(int8_t)(raw[0][j >> 2] >> (8 * (j & 3)));
    } else {
#pragma unroll
        for (int j = 0; j < 16; ++j) c[j] = (int)(int16_t)(raw[j >> 3][(j >> 1) & 3] >> (16 * (j & 1)));
    }
}

// ---- windows of int8 / int16 codes ---------------------------------------------------------------------------
// What bounds it: HBM for large layers, the latency of a window's loads for small ones.  A thread owns eight consecutive
// elements of a chunk and has the loads of 16 tensors in flight (one 8- or 16-byte load each), so a window of 25 costs two
// memory latencies; the squares of a tensor go to a lane's own LDS counter (one conflict-free addition per tensor and
// wavefront), so that the reduction over lanes happens once per block and not once per tensor.  Measured on ResNet-18's
// layers, windows of 25: 36,864 elements 20 -> 9 us, 0.6 M int16 elements 22.8 -> 12.2, 2.4 M int16 elements (118 MB)
// 31.6 -> 30.4 us (was: 16 elements per thread, eight tensors in flight, a 64-bit wavefront reduction per tensor; that form
// is still up to 0.4 us faster for one tensor below 0.6 M elements, and 0.9 us for five at 2.4 M).
constexpr int kGdChunk = kGdThreads * 8;      // elements of a block's chunk
constexpr uint32_t kGdMaxBlocks = 1024;       // four blocks per CU; more elements than that: several chunks per block


// Short windows of large tensors have too few loads in flight with one chunk at a time, so a block has four chunks' (and takes
// at least four): 8.4 M int8 elements, one tensor 13.8 -> 8.9 us, four 17.2 -> 12.0; 50 M 52 -> 22 and 68 -> 39.  Below
// 1024 chunks that would leave CUs without a block; more than four tensors or six bytes per element fill the queue by
// themselves, and the registers of four chunks (two wavefronts per SIMD instead of four) cost more than they give (8.4 M,
// five int8 tensors 19.3 -> 22.9; 16.8 M, three int16 tensors 26.4 -> 25.5, four 29.3 -> 32.3).
constexpr int kGdShort = 4;
constexpr int kGdShortChunks = 4;
static bool gd_short(uint64_t n, int count, int element_bytes) { return count <= kGdShort && element_bytes <= 6 && n > (uint64_t)1023 * kGdChunk; }

// Few blocks: the last one to finish adds the sums, no second launch.  Its ticket costs every block about 20 ns behind the
// others', a second launch and its reduction 0.8 us plus 40 ns per tensor (device time; and 2.5 us of the host's).  Two launches
// -> one, in a captured graph: 25 tensors of 36,864 elements 11.3 -> 9.1 us, of 147,456 (72 blocks) 11.7 -> 9.8; 8 of 73,728
// 7.4 -> 7.1; one of 147,456 6.3 -> 7.0 (not taken: 72 blocks).  One tensor of 1,728 elements is taken for the host's sake: its
// graph takes 5.1 -> 5.4 us, calls one behind the other 9.9 -> 5.8.
static bool gd_one_launch(int blocks, int count) { return blocks <= 32 + 2 * count; }

// Blocks of a tensor, each with at least `each` chunks (1, or 2 where the workspace does not hold one block's sums per chunk).  As
// many as are resident together (four per CU), also where some then take one chunk more than others: 1152 chunks on 576 blocks of
// two leave a quarter of the CUs with half as much to read again as the rest (2.4 M elements, 25 tensors, int8 21.5 -> 20.3 us with 1024 blocks,
// int16 29.5 -> 28.4).
static uint32_t gd_blocks(uint64_t n, bool brief, uint64_t each)
{
    const uint64_t chunks = std::max<uint64_t>(1, (n + kGdChunk - 1) / kGdChunk);
    if (!brief && each == 1) return (uint32_t)std::min<uint64_t>(chunks, kGdMaxBlocks);
    if (brief) each = kGdShortChunks;
    each = std::max(each, (chunks + kGdMaxBlocks - 1) / kGdMaxBlocks);
    return (uint32_t)((chunks + each - 1) / each);
}

// The window's table as every wavefront holds it: lane k has tensor k's entry (one load for the whole table), and
// readlane hands it out as a scalar.
struct GdTable { uint32_t ptr_lo, ptr_hi, es, shift; };

// ES: element bytes of every tensor of the window, or 0 when they differ (16 bytes are loaded for eight codes of either size);
// U: tensors, and V: chunks whose loads are in flight together; DOT: every alignment is at most 6 bits (int8) or 14 (int16), so that
// 2^shift fits a code and the aligned code joins its sum in one dot product with (.., 2^shift, ..) (a small tensor's time is the
// chain of a wavefront's instructions: 25 int8 tensors of 1,728 elements spent 9,000 of 18,400 clocks in this loop)
template <int ES, int U, int V, bool DOT>
__device__ __forceinline__ void gd_chunks(const GdTable &tab, const int count, const uint32_t n, unsigned long long *slots,
                                          const uint32_t blk, const uint32_t nblk)
{
    constexpr int NW = ES == 1 ? 2 : 4;       // 32-bit words per tensor and thread
    typedef unsigned gd_v2u __attribute__((ext_vector_type(2)));
    typedef short gd_v2s __attribute__((ext_vector_type(2)));
    const int lane = threadIdx.x & (kWave - 1);
    const uint32_t nchunks = (n + kGdChunk - 1) / kGdChunk;
    for (uint32_t ch = blk; ch < nchunks; ch += V * nblk) {
        // chunk v of the round starts at element c0(v); past the last chunk (below 2^30 + 2^23) every load reads as 0
        auto c0 = [&](int v) { return (ch + (uint32_t)v * nblk) * kGdChunk; };
        // One element size: the descriptor returns zeros from the first whole word past the tensor on, so codes past n (other than
        // zeros) are in the one word that n divides, if it does; its mask is the same for all tensors.
        const bool ragged = ES != 0 && (n * (uint32_t)ES & 3u) != 0;
        uint32_t keep[V][NW];
        if (ragged) {
            constexpr int epd = ES == 1 ? 4 : 2;      // codes per word
#pragma unroll
            for (int v = 0; v < V; ++v)
#pragma unroll
                for (int i = 0; i < NW; ++i) {
                    const uint32_t e = c0(v) + threadIdx.x * 8 + i * epd;
                    keep[v][i] = e < n && n - e < (uint32_t)epd ? (1u << (8 * ES * (n - e))) - 1u : 0xffffffffu;
                }
        }
        int S[V][8];
#pragma unroll
        for (int v = 0; v < V; ++v)
#pragma unroll
            for (int j = 0; j < 8; ++j) S[v][j] = 0;
        for (int k0 = 0; k0 < count; k0 += U) {
            uint32_t raw[U][V][NW];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                // The descriptor covers the tensor rounded up to whole 32-bit words (16-byte aligned, so mapped); words past
                // it, and whole tensors past the window, read as 0 without memory traffic.
                const uint32_t es = ES ? (uint32_t)ES : (uint32_t)__builtin_amdgcn_readlane((int)tab.es, k0 + u);
                const uint64_t ptr = (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)tab.ptr_hi, k0 + u) << 32 |
                                     (uint32_t)__builtin_amdgcn_readlane((int)tab.ptr_lo, k0 + u);
                const uint32_t bytes = k0 + u < count ? (n * es + 3u) & ~3u : 0u;
                const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void *>(ptr), 0, (int)bytes, 0x00020000);
#pragma unroll
                for (int v = 0; v < V; ++v) {
                    const uint32_t off = (c0(v) + threadIdx.x * 8) * es;
                    if constexpr (NW == 2) {
                        const gd_v2u x = __builtin_amdgcn_raw_buffer_load_b64(rsrc, off, 0, 0);
                        raw[u][v][0] = x[0]; raw[u][v][1] = x[1];
                    } else {
                        const gd_v4u x = __builtin_amdgcn_raw_buffer_load_b128(rsrc, off, 0, 0);
#pragma unroll
                        for (int i = 0; i < NW; ++i) raw[u][v][i] = x[i];
                    }
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (k0 + u < count) {
                    const int es = ES ? ES : __builtin_amdgcn_readlane((int)tab.es, k0 + u);
                    const int sh = __builtin_amdgcn_readlane((int)tab.shift, k0 + u);
#pragma unroll
                    for (int v = 0; v < V; ++v) {
                        if (ES) {
                            if (ragged)
#pragma unroll
                                for (int i = 0; i < NW; ++i) raw[u][v][i] &= keep[v][i];
                        } else if (n - c0(v) < (uint32_t)kGdChunk) {         // the last chunk: clear the codes past n
                            const int epd = es == 1 ? 4 : 2;      // codes per word
#pragma unroll
                            for (int i = 0; i < NW; ++i) {
                                const int left = (int)n - (int)(c0(v) + threadIdx.x * 8 + i * epd);
                                raw[u][v][i] = left >= epd ? raw[u][v][i] : left <= 0 ? 0u : raw[u][v][i] & ((1u << (8 * es * left)) - 1u);
                            }
                        }
                    }
                    unsigned long long *slot = slots + (k0 + u) * kWave + lane;
                    if (es == 1) {
                        int d = 0;                // at most 8 * 2^14 per chunk, a counter at most 2^28 (512 chunks per block)
#pragma unroll
                        for (int v = 0; v < V; ++v) {
#pragma unroll
                            for (int j = 0; j < 8; ++j) {
                                if (DOT) S[v][j] = __builtin_amdgcn_sdot4((int)raw[u][v][j >> 2], (int)(1u << (8 * (j & 3) + sh)), S[v][j], false);
                                else S[v][j] += (int)((unsigned)(int)(int8_t)(raw[u][v][j >> 2] >> (8 * (j & 3))) << sh);
                            }
                            d = __builtin_amdgcn_sdot4((int)raw[u][v][0], (int)raw[u][v][0], d, false);
                            d = __builtin_amdgcn_sdot4((int)raw[u][v][1], (int)raw[u][v][1], d, false);
                        }
                        atomicAdd(reinterpret_cast<uint32_t *>(slot), (uint32_t)d);
                    } else {
                        unsigned long long t = 0;
#pragma unroll
                        for (int v = 0; v < V; ++v) {
#pragma unroll
                            for (int j = 0; j < 8; ++j) {
                                const uint32_t x = raw[u][v][(j >> 1) % NW];
                                if (DOT) S[v][j] = __builtin_amdgcn_sdot2(__builtin_bit_cast(gd_v2s, x), __builtin_bit_cast(gd_v2s, 1u << (16 * (j & 1) + sh)), S[v][j], false);
                                else S[v][j] += (int)((unsigned)(int)(int16_t)(x >> (16 * (j & 1))) << sh);
                            }
#pragma unroll
                            for (int i = 0; i < NW; ++i) {
                                const gd_v2s x = __builtin_bit_cast(gd_v2s, raw[u][v][i]);
                                t += (uint32_t)__builtin_amdgcn_sdot2(x, x, 0, false);      // <= 2^31
                            }
                        }
                        atomicAdd(slot, t);
                    }
                }
            }
        }
        unsigned long long lo = 0, hi = 0;    // halves of the squared sums: neither can overflow
#pragma unroll
        for (int v = 0; v < V; ++v)
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const uint64_t q = (uint64_t)((long long)S[v][j] * (long long)S[v][j]);
                lo += q & 0xffffffffull;
                hi += q >> 32;
            }
        atomicAdd(slots + count * kWave + lane, lo);
        atomicAdd(slots + (count + 1) * kWave + lane, hi);
    }
}

__host__ __device__ inline size_t gd_lds_bytes(int count) { return (size_t)(count + 2) * kWave * sizeof(unsigned long long); }

// partial[col][block] (SHARED: [block][col]): col k < count: sum of squares of tensor k; col count / count+1: sums of the
// low / high 32-bit halves of (aligned element sum)^2
// blk of nblk: this block's place among the blocks of the tensor (a chained step runs all layers in one launch)
// FORM: GD_LONG / GD_SHORT, or by the window and the tensor (a chained step's layers differ)
enum { GD_LONG, GD_SHORT, GD_EITHER };
template <int FORM, bool SHARED = false>
__device__ __forceinline__ void gd_partial_body(const GradWindow &w, uint32_t n, uint64_t *partial, const uint32_t blk, const uint32_t nblk)
{
    extern __shared__ unsigned long long gd_slots[];
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    const int count = __builtin_amdgcn_readfirstlane(w.count);
    const uint64_t ptr = (uint64_t)w.g[lane];           // entries past the window hold nothing that is used
    const GdTable tab = {(uint32_t)ptr, (uint32_t)(ptr >> 32), w.es[lane], w.shift[lane]};
    for (int i = threadIdx.x; i < (count + 2) * kWave; i += kGdThreads) gd_slots[i] = 0;
    // one element size for the whole window (a window is emptied when its layer changes format)?
    const int es0 = __builtin_amdgcn_readfirstlane((int)tab.es);
    const bool mixed = __ballot(lane < count && (int)tab.es != es0) != 0;
    const bool dot = __ballot(lane < count && tab.shift > (es0 == 1 ? 6u : 14u)) == 0;
    __syncthreads();
    const bool brief = FORM == GD_SHORT || (FORM == GD_EITHER && count <= kGdShort && n > nblk * (uint32_t)kGdChunk);
    if (FORM != GD_LONG && brief) {
        constexpr int V = kGdShortChunks;
        if (mixed) gd_chunks<0, kGdShort, V, false>(tab, count, n, gd_slots, blk, nblk);
        else if (es0 == 1) dot ? gd_chunks<1, kGdShort, V, true>(tab, count, n, gd_slots, blk, nblk) : gd_chunks<1, kGdShort, V, false>(tab, count, n, gd_slots, blk, nblk);
        else dot ? gd_chunks<2, kGdShort, V, true>(tab, count, n, gd_slots, blk, nblk) : gd_chunks<2, kGdShort, V, false>(tab, count, n, gd_slots, blk, nblk);
    } else if (FORM != GD_SHORT) {
        if (mixed) gd_chunks<0, 16, 1, false>(tab, count, n, gd_slots, blk, nblk);
        else if (es0 == 1) dot ? gd_chunks<1, 16, 1, true>(tab, count, n, gd_slots, blk, nblk) : gd_chunks<1, 16, 1, false>(tab, count, n, gd_slots, blk, nblk);
        else dot ? gd_chunks<2, 16, 1, true>(tab, count, n, gd_slots, blk, nblk) : gd_chunks<2, 16, 1, false>(tab, count, n, gd_slots, blk, nblk);
    }
    __syncthreads();
    // The 64 lane counters of a column are added by eight threads (eight words each, rotated so that neighbouring columns meet
    // different banks), so that all columns of a window of up to 30 are one round of three lane exchanges.
    const int part = threadIdx.x & 7;
    for (int col = threadIdx.x >> 3; col < (count + 2 + 7) / 8 * 8; col += kGdThreads / 8) {
        uint64_t v = 0;
        if (col < count + 2) {
#pragma unroll
            for (int i = 0; i < 8; ++i) v += gd_slots[col * kWave + 8 * ((i + col) & 7) + part];
        }
#pragma unroll
        for (int off = 4; off > 0; off >>= 1) v += __shfl_xor((unsigned long long)v, off, 64);
        // the first word of a column's counters, which only the column's own eight threads (one wavefront) have read
        if (part == 0 && col < count + 2) gd_slots[col * kWave] = v;
    }
    __syncthreads();
    if (threadIdx.x < kWave)
        for (int col = lane; col < count + 2; col += kWave) {
            const uint64_t v = gd_slots[col * kWave];
            if (SHARED) store_partial(partial + (size_t)blk * (count + 2) + col, v);
            else partial[(size_t)col * nblk + blk] = v;
        }
}

// The norms and the ratio from the column sums; every thread of the block calls it.
__device__ __forceinline__ void gd_ratio(const GradWindow &w, const uint64_t *col_sum, double *out)
{
    // the norms side by side (a square root and a scaling in fp64 take longer than the sums), added in window order
    __shared__ double norm[kGdMaxTensors];
    if ((int)threadIdx.x < w.count) norm[threadIdx.x] = ldexp(sqrt((double)col_sum[threadIdx.x]), -(int)w.fl[threadIdx.x]);
    __syncthreads();
    if (threadIdx.x != 0) return;
    double num = 0.0;
    for (int k = 0; k < w.count; ++k) num += norm[k];
    const double sq = (double)col_sum[w.count + 1] * 4294967296.0 + (double)col_sum[w.count];
    const double den = ldexp(sqrt(sq), -w.fl_max);
    const double ds = den > 0.0 ? num / den : (num > 0.0 ? (double)INFINITY : (double)NAN);
    out[0] = ds;
    out[1] = (ds > 0.0 && ds < (double)INFINITY) ? log(ds) : 1.0;
}

// One block: column sums of [col][block] (one wavefront per column at a time), then the norms and the ratio.
__device__ __forceinline__ void gd_final_body(const GradWindow &w, const uint64_t *__restrict__ partial, int nblocks, uint64_t *sums_out,
                                              double *out)
{
    __shared__ uint64_t col_sum[kGdMaxTensors + 2];
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    for (int col = wave; col < w.count + 2; col += kGdFinalThreads / kWave) {
        const uint64_t *p = partial + (size_t)col * nblocks;
        uint64_t v = 0;
        int b0 = 0;
        // Eight rows per lane in flight, the last one repeated past the end (one behind the other beyond whole rounds of 512 rows:
        // 589,824 elements, 25 tensors, 15.3 instead of 13.5 us); up to three rounds of one are as fast.
        for (; b0 + 3 * kWave < nblocks; b0 += 8 * kWave) {
            uint64_t t[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) t[u] = p[min(b0 + u * kWave + lane, nblocks - 1)];
#pragma unroll
            for (int u = 0; u < 8; ++u) v += b0 + u * kWave + lane < nblocks ? t[u] : 0ull;
        }
        for (; b0 + lane < nblocks; b0 += kWave) v += p[b0 + lane];
        v = wave_sum_u64(v);
        if (lane == 0) {
            col_sum[col] = v;
            if (sums_out) sums_out[col] = v;
        }
    }
    __syncthreads();
    gd_ratio(w, col_sum, out);
}

// The same in the block that finishes last, from rows [block][count + 2] written in this launch: a thread adds one column of
// every (kGdThreads / columns)-th row with all its loads in flight, neighbouring threads read neighbouring words.
constexpr int kGdRows = 10;
__device__ __forceinline__ void gd_last_block(const GradWindow &w, const uint64_t *partial, int nblocks, uint64_t *sums_out, double *out)
{
    __shared__ uint64_t wave_part[kGdThreads / kWave][kGdMaxTensors + 2];
    __shared__ uint64_t col_sum[kGdMaxTensors + 2];
    const int cols = w.count + 2, lp = 32 - __builtin_clz(cols - 1);      // cols <= 2^lp; cols >= 3
    const int col = threadIdx.x & ((1 << lp) - 1), groups = kGdThreads >> lp;
    uint64_t v = 0;
    if (col < cols)
        for (int b = threadIdx.x >> lp; b < nblocks; b += kGdRows * groups) {
            uint64_t t[kGdRows];
#pragma unroll
            for (int u = 0; u < kGdRows; ++u) {      // the last row repeated past the end
                const uint64_t *p = partial + (size_t)min(b + u * groups, nblocks - 1) * cols + col;
                t[u] = load_partial(p);
            }
#pragma unroll
            for (int u = 0; u < kGdRows; ++u) v += b + u * groups < nblocks ? t[u] : 0ull;
        }
    // the threads of a wavefront that hold the same column, then the wavefronts that do (all, up to 64 columns; else each second)
    for (int off = 1 << lp; off < kWave; off <<= 1) v += __shfl_xor((unsigned long long)v, off, 64);
    const int wave = threadIdx.x / kWave;
    if ((lp >= 6 || (int)(threadIdx.x & (kWave - 1)) < (1 << lp)) && col < cols) wave_part[wave][col] = v;
    __syncthreads();
    if ((int)threadIdx.x < cols) {
        const int first = (int)threadIdx.x >= kWave ? 1 : 0, step = lp > 6 ? 2 : 1;
        v = 0;
#pragma unroll
        for (int i = 0; i < kGdThreads / kWave; ++i)
            if (first + i * step < kGdThreads / kWave) v += wave_part[first + i * step][threadIdx.x];
        col_sum[threadIdx.x] = v;
        if (sums_out) sums_out[threadIdx.x] = v;
    }
    __syncthreads();
    gd_ratio(w, col_sum, out);
}

template <int FORM>
__global__ void __launch_bounds__(kGdThreads)
gd_partial_kernel(const GradWindow w, uint32_t n, uint64_t *partial)
{
    gd_partial_body<FORM>(w, n, partial, blockIdx.x, gridDim.x);
}

__global__ void __launch_bounds__(kGdFinalThreads)
gd_final_kernel(const GradWindow w, const uint64_t *__restrict__ partial, int nblocks, uint64_t *sums_out, double *out)
{
    gd_final_body(w, partial, nblocks, sums_out, out);
}

// both phases in one launch: the block that finishes last adds the rows
__global__ void __launch_bounds__(kGdThreads)
gd_small_kernel(const GradWindow w, uint32_t n, uint64_t *partial, uint32_t *ticket, uint64_t *sums_out, double *out)
{
    gd_partial_body<GD_LONG, true>(w, n, partial, blockIdx.x, gridDim.x);
    if (finished_last(ticket)) gd_last_block(w, partial, (int)gridDim.x, sums_out, out);
}

// ---- windows that hold int32 codes (word lengths 17..32) --------------------------------------------------------
// The aligned element sum is kept in 64 bits (its bound is below 2^48), every sum of squares in 128 bits.
// partial[col][block] as two words, low first: col k < count: sum of squares of tensor k; col count: sum of the
// squared aligned element sums.
__device__ __forceinline__ void load16_any(const void *g, int es, uint32_t n, uint32_t e0, int (&c)[16])
{
    if (e0 + 16 <= n) {
        if (es == 4) {
            const int4 *p = reinterpret_cast<const int4 *>(static_cast<const int32_t *>(g) + e0);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int4 v = p[i];
                c[4 * i] = v.x; c[4 * i + 1] = v.y; c[4 * i + 2] = v.z; c[4 * i + 3] = v.w;
            }
        } else {
            gd_v4u raw[2];
            const gd_v4u *p = reinterpret_cast<const gd_v4u *>(static_cast<const char *>(g) + (size_t)e0 * es);
            raw[0] = p[0];
            raw[1] = es == 2 ? p[1] : gd_v4u{0, 0, 0, 0};
            unpack16(raw, es, c);
        }
    } else {
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            int v = 0;
            if (e0 + j < n) v = es == 4 ? static_cast<const int32_t *>(g)[e0 + j] : es == 2 ? (int)static_cast<const int16_t *>(g)[e0 + j]
                                                                                          : (int)static_cast<const int8_t *>(g)[e0 + j];
            c[j] = v;
        }
    }
}

__device__ __forceinline__ void gd_partial_wide_body(const GradWindow &w, uint32_t n, uint64_t *partial, const uint32_t blk,
                                                     const uint32_t nblk)
{
    __shared__ unsigned long long wave_part[kGdThreads / kWave][kGdMaxTensors + 1][2];
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    const uint32_t e0 = (blk * kGdThreads + threadIdx.x) * kGdPerThread;
    long long S[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) S[j] = 0;
    for (int k = 0; k < w.count; ++k) {
        int c[16];
        if (e0 < n) {
            load16_any(w.g[k], w.es[k], n, e0, c);
        } else {
#pragma unroll
            for (int j = 0; j < 16; ++j) c[j] = 0;
        }
        const int sh = w.shift[k];
        u128 sq = 0;
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            S[j] += (long long)((unsigned long long)(long long)c[j] << sh);
            sq += (u128)(unsigned long long)((long long)c[j] * (long long)c[j]);
        }
        sq = wave_sum_u128(sq);
        if (lane == 0) { wave_part[wave][k][0] = (unsigned long long)sq; wave_part[wave][k][1] = (unsigned long long)(sq >> 64); }
    }
    u128 t = 0;
#pragma unroll
    for (int j = 0; j < 16; ++j) t += (u128)((i128)S[j] * (i128)S[j]);
    t = wave_sum_u128(t);
    if (lane == 0) { wave_part[wave][w.count][0] = (unsigned long long)t; wave_part[wave][w.count][1] = (unsigned long long)(t >> 64); }
    __syncthreads();
    for (int col = threadIdx.x; col < w.count + 1; col += kGdThreads) {
        u128 v = 0;
#pragma unroll
        for (int i = 0; i < kGdThreads / kWave; ++i) v += ((u128)wave_part[i][col][1] << 64) | wave_part[i][col][0];
        uint64_t *dst = partial + 2 * ((size_t)col * nblk + blk);
        dst[0] = (uint64_t)v;
        dst[1] = (uint64_t)(v >> 64);
    }
}

template <bool BYPTR>
__global__ void __launch_bounds__(kGdThreads)
gd_partial_wide_kernel(const GradWindow wv, const GradWindow *__restrict__ wp, uint32_t n, uint64_t *partial)
{
    gd_partial_wide_body(BYPTR ? *wp : wv, n, partial, blockIdx.x, gridDim.x);
}

__device__ __forceinline__ void gd_final_wide_body(const GradWindow &w, const uint64_t *__restrict__ partial, int nblocks,
                                                   uint64_t *sums_out, double *out)
{
    __shared__ unsigned long long col_sum[kGdMaxTensors + 1][2];
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    for (int col = wave; col < w.count + 1; col += kGdFinalThreads / kWave) {
        const uint64_t *p = partial + 2 * (size_t)col * nblocks;
        u128 v = 0;
        for (int b = lane; b < nblocks; b += kWave) v += ((u128)p[2 * b + 1] << 64) | p[2 * b];
        v = wave_sum_u128(v);
        if (lane == 0) {
            col_sum[col][0] = (unsigned long long)v;
            col_sum[col][1] = (unsigned long long)(v >> 64);
            if (sums_out) { sums_out[2 * col] = (uint64_t)v; sums_out[2 * col + 1] = (uint64_t)(v >> 64); }
        }
    }
    __syncthreads();
    if (threadIdx.x != 0) return;
    double num = 0.0;
    for (int k = 0; k < w.count; ++k) num += ldexp(sqrt(u128_to_double(col_sum[k][0], col_sum[k][1])), -(int)w.fl[k]);
    const double den = ldexp(sqrt(u128_to_double(col_sum[w.count][0], col_sum[w.count][1])), -w.fl_max);
    const double ds = den > 0.0 ? num / den : (num > 0.0 ? (double)INFINITY : (double)NAN);
    out[0] = ds;
    out[1] = (ds > 0.0 && ds < (double)INFINITY) ? log(ds) : 1.0;
}

template <bool BYPTR>
__global__ void __launch_bounds__(kGdFinalThreads)
gd_final_wide_kernel(const GradWindow wv, const GradWindow *__restrict__ wp, const uint64_t *__restrict__ partial, int nblocks,
                     uint64_t *sums_out, double *out)
{
    gd_final_wide_body(BYPTR ? *wp : wv, partial, nblocks, sums_out, out);
}

size_t ws_need_gradient_diversity(uint64_t n, int count);

// All layers of a chained step in one launch per phase: the blocks of layer l are [first[l], first[l + 1]), its
// partial sums start part_off[l] words into the scratch.
struct ChainGeo {
    uint32_t first[kGdMaxLayers + 1];
    uint32_t n[kGdMaxLayers];
    uint64_t part_off[kGdMaxLayers];
    uint8_t wide[kGdMaxLayers];
    int nlayers;
};

__global__ void __launch_bounds__(kGdThreads)
gd_partial_chain_kernel(const ChainGeo geo, const GradWindow *__restrict__ win, uint64_t *partial)
{
    // The layer this block belongs to: every lane holds one entry of the tables and compares, the wavefront votes, and
    // readlane hands out the layer's entries.  (Indexed scalar loads of tables with different element sizes made the
    // compiler split the addresses into parts that are not multiples of four, which scalar loads round down.)
    const int lane = threadIdx.x & (kWave - 1), e = min(lane, geo.nlayers - 1);
    const uint32_t first = lane < geo.nlayers ? geo.first[lane] : 0xffffffffu;
    const int l = __popcll(__ballot(blockIdx.x >= first)) - 1;
    auto entry = [&](uint32_t v) { return (uint32_t)__builtin_amdgcn_readlane((int)v, l); };
    const uint32_t first_l = entry(geo.first[e]), nblk = entry(geo.first[e + 1]) - first_l, n = entry(geo.n[e]);
    uint64_t *part = partial + ((uint64_t)entry((uint32_t)(geo.part_off[e] >> 32)) << 32 | entry((uint32_t)geo.part_off[e]));
    if (entry(geo.wide[e])) gd_partial_wide_body(win[l], n, part, blockIdx.x - first_l, nblk);
    else gd_partial_body<GD_EITHER>(win[l], n, part, blockIdx.x - first_l, nblk);
}

__global__ void __launch_bounds__(kGdFinalThreads)
gd_final_chain_kernel(const ChainGeo geo, const GradWindow *__restrict__ win, const uint64_t *__restrict__ partial, ChainLayerOut *out)
{
    const int l = blockIdx.x;
    const int nblk = (int)(geo.first[l + 1] - geo.first[l]);
    if (geo.wide[l]) gd_final_wide_body(win[l], partial + geo.part_off[l], nblk, nullptr, &out[l].ds);
    else gd_final_body(win[l], partial + geo.part_off[l], nblk, nullptr, &out[l].ds);
}

// One thread per layer of a chained step: the exponent of this batch's gradient lies in device memory (the fitting
// pass of the backward pass wrote it), so the window can be laid out without the host reading it first.  The aligned
// element sum of the diversity kernel is a 32-bit integer (a 64-bit one with the bound 2^48 when the window holds codes
// above 16 bits): when the scales of the window lie too far apart for that, the oldest entries are left out until the
// rest fits (at least the newest entry stays).
__global__ void chain_prep_kernel(const ChainLayerIn *__restrict__ in, int nlayers, const long long *__restrict__ e_g, size_t e_stride,
                                  GradWindow *__restrict__ win, ChainLayerOut *__restrict__ out)
{
    const int l = blockIdx.x * blockDim.x + threadIdx.x;
    if (l >= nlayers) return;
    const ChainLayerIn &c = in[l];
    const int count = c.count;
    const long long e_new = e_g[(size_t)l * e_stride];
    auto exp_of = [&](int k) { return k == count - 1 ? e_new : c.exp[k]; };
    bool wide = false;                              // codes above 16 bits: 64-bit element sums, bound 2^48
    for (int k = 0; k < count; ++k) wide = wide || c.wl[k] > 16;
    const int cap = wide ? 48 : 31;
    int first = 0;
    long long e_min = 0, e_max = 0;
    for (;; ++first) {
        e_min = e_max = exp_of(first);
        for (int k = first + 1; k < count; ++k) {
            const long long e = exp_of(k);
            e_min = e < e_min ? e : e_min;
            e_max = e > e_max ? e : e_max;
        }
        unsigned long long bound = 0;               // sum of 2^(wl - 1 + e_max - e_k), capped
        for (int k = first; k < count; ++k) {
            const long long b = (long long)c.wl[k] - 1 + e_max - exp_of(k);
            bound += b >= cap ? (1ull << cap) : (1ull << b);
        }
        if (bound < (1ull << cap) || first == count - 1) break;
    }
    GradWindow &w = win[l];
    const int used = count - first;
    for (int i = 0; i < used; ++i) {
        const int k = first + i;
        w.g[i] = c.g[k];
        w.es[i] = (uint8_t)(c.wl[k] <= 8 ? 1 : c.wl[k] <= 16 ? 2 : 4);
        w.shift[i] = (uint8_t)(e_max - exp_of(k));
        w.fl[i] = (int8_t)(exp_of(k) - e_min);
    }
    w.count = used;
    w.fl_max = (int)(e_max - e_min);
    out[l].exp_new = e_new;
    out[l].used = used;
}

int gradient_diversity_chain(adapt_ctx *ctx, const ChainLayerIn *in, int nlayers, const size_t *n, const long long *e_g, size_t e_stride,
                             GradWindow *win, ChainLayerOut *out)
{
    if (nlayers < 1) return ADAPT_EINVAL;
    if (nlayers > kGdMaxLayers) return ADAPT_EUNSUPPORTED;
    const size_t per_block = (size_t)kGdThreads * kGdPerThread;
    ChainGeo geo = {};
    geo.nlayers = nlayers;
    int most = 1;
    bool brief[kGdMaxLayers];
    for (int l = 0; l < nlayers; ++l) {
        if (in[l].count < 1 || in[l].count > kGdMaxTensors || n[l] > ((size_t)1 << 30)) return ADAPT_EUNSUPPORTED;
        int bytes = 0;
        for (int k = 0; k < in[l].count; ++k) {
            geo.wide[l] = geo.wide[l] || in[l].wl[k] > 16;
            bytes += in[l].wl[k] <= 8 ? 1 : 2;
        }
        brief[l] = gd_short(n[l], in[l].count, bytes);
        most = std::max(most, in[l].count);
        geo.n[l] = (uint32_t)n[l];
    }
    uint64_t blocks = 0;
    size_t words = 0;
    for (uint64_t each = 1; each <= 2; ++each) {                 // one chunk per block, or two when the workspace is too small for that
        blocks = words = 0;
        for (int l = 0; l < nlayers; ++l) {
            const uint64_t grid = geo.wide[l] ? std::max<size_t>(1, (n[l] + per_block - 1) / per_block) : gd_blocks(n[l], brief[l], each);
            geo.first[l] = (uint32_t)blocks;
            geo.part_off[l] = words;
            blocks += grid;
            words += grid * (size_t)(geo.wide[l] ? 2 * (in[l].count + 1) : in[l].count + 2);
        }
        if (words * sizeof(uint64_t) <= scratch_bytes(ctx)) break;
    }
    geo.first[nlayers] = (uint32_t)blocks;
    if (blocks >= ((uint64_t)1 << 31)) return ADAPT_EUNSUPPORTED;
    if (words * sizeof(uint64_t) > scratch_bytes(ctx)) return ADAPT_EWORKSPACE;
    uint64_t *partial = reinterpret_cast<uint64_t *>(scratch(ctx));
    hipLaunchKernelGGL(chain_prep_kernel, dim3(1), dim3(64), 0, ctx->stream, in, nlayers, e_g, e_stride, win, out);
    hipLaunchKernelGGL(gd_partial_chain_kernel, dim3((unsigned)blocks), dim3(kGdThreads), gd_lds_bytes(most), ctx->stream, geo, win, partial);
    hipLaunchKernelGGL(gd_final_chain_kernel, dim3(nlayers), dim3(kGdFinalThreads), 0, ctx->stream, geo, win, partial, out);
    return hip_status(ctx, hipGetLastError());
}

size_t ws_need_gradient_diversity(uint64_t n, int count)
{
    const size_t per_block = (size_t)kGdThreads * kGdPerThread;
    // (count + 2) words per block, or (count + 1) pairs of words for windows with int32 codes
    return std::max(std::max<size_t>(1, (n + per_block - 1) / per_block) * (size_t)(count + 1) * 2,
                    (size_t)gd_blocks(n, false, 1) * (size_t)(count + 2)) * sizeof(uint64_t);
}

}  // namespace adapt

using namespace adapt;

extern "C" int adapt_gradient_diversity(adapt_ctx *ctx, const adapt_grad_item *items, int count, size_t n,
                                        uint64_t *sums, double *out)
{
    if (!ctx || !items || !out || count < 1) return ADAPT_EINVAL;
    if (count > kGdMaxTensors) return ADAPT_EUNSUPPORTED;
    if (((uintptr_t)out & 7) || (sums && ((uintptr_t)sums & 7))) return ADAPT_EINVAL;
    if (n > ((size_t)1 << 30)) return ADAPT_EUNSUPPORTED;      // 32-bit byte offsets, with room for the last block's overhang
    GradWindow w;
    w.count = count;
    w.fl_max = 0;
    int wl_max = 0;
    for (int k = 0; k < count; ++k) {
        const adapt_fmt f = adapt_fmt{items[k].wl, items[k].fl};
        if (!fmt_ok_wide(f)) return ADAPT_EINVAL;
        if (n > 0 && (!items[k].g || !aligned16(items[k].g))) return ADAPT_EINVAL;
        w.fl_max = std::max(w.fl_max, f.fl);
        wl_max = std::max(wl_max, f.wl);
    }
    // the aligned element sum is kept in int32: count * 2^(wl-1) * 2^(fl_max - fl) must stay below 2^31
    double bound = 0.0;
    for (int k = 0; k < count; ++k) {
        w.g[k] = items[k].g;
        w.es[k] = (uint8_t)(items[k].wl <= 8 ? 1 : items[k].wl <= 16 ? 2 : 4);
        w.shift[k] = (uint8_t)(w.fl_max - items[k].fl);
        w.fl[k] = (int8_t)items[k].fl;
        bound += std::ldexp(1.0, items[k].wl - 1 + w.fl_max - items[k].fl);
    }
    const size_t per_block = (size_t)kGdThreads * kGdPerThread;
    const int grid = (int)std::max<size_t>(1, (n + per_block - 1) / per_block);
    if (wl_max > 16) {           // int32 codes in the window: 64-bit element sums (bound 2^48), 128-bit sums of squares
        if (bound >= 281474976710656.0) return ADAPT_EUNSUPPORTED;
        if ((size_t)grid * (count + 1) * 2 * sizeof(uint64_t) > scratch_bytes(ctx)) return ADAPT_EWORKSPACE;
        uint64_t *part = reinterpret_cast<uint64_t *>(scratch(ctx));
        hipLaunchKernelGGL(gd_partial_wide_kernel<false>, dim3(grid), dim3(kGdThreads), 0, ctx->stream, w, nullptr, (uint32_t)n, part);
        hipLaunchKernelGGL(gd_final_wide_kernel<false>, dim3(1), dim3(kGdFinalThreads), 0, ctx->stream, w, nullptr, part, grid, sums, out);
        return hip_status(ctx, hipGetLastError());
    }
    if (bound >= 2147483648.0) return ADAPT_EUNSUPPORTED;
    int bytes = 0;
    for (int k = 0; k < count; ++k) bytes += w.es[k];
    const bool brief = gd_short(n, count, bytes);
    auto fits = [&](uint32_t b) { return (size_t)b * (count + 2) * sizeof(uint64_t) <= scratch_bytes(ctx); };
    const int blocks = (int)gd_blocks(n, brief, fits(gd_blocks(n, brief, 1)) ? 1 : 2);
    if (!fits((uint32_t)blocks)) return ADAPT_EWORKSPACE;
    uint64_t *partial = reinterpret_cast<uint64_t *>(scratch(ctx));
    if (gd_one_launch(blocks, count)) {
        hipLaunchKernelGGL(gd_small_kernel, dim3(blocks), dim3(kGdThreads), gd_lds_bytes(count), ctx->stream, w, (uint32_t)n, partial, ticket(ctx, 0), sums, out);
        return hip_status(ctx, hipGetLastError());
    }
    hipLaunchKernelGGL(brief ? gd_partial_kernel<GD_SHORT> : gd_partial_kernel<GD_LONG>, dim3(blocks), dim3(kGdThreads), gd_lds_bytes(count), ctx->stream,
                       w, (uint32_t)n, partial);
    hipLaunchKernelGGL(gd_final_kernel, dim3(1), dim3(kGdFinalThreads), 0, ctx->stream, w, partial, blocks, sums, out);
    return hip_status(ctx, hipGetLastError());
}

// ---- host-side scalar rules ------------------------------------------------------------------

static bool usable(double ds) { return ds > 0.0 && ds < (double)INFINITY; }

extern "C" int adapt_pushup_suggest(double ds, int wl_min, int fl_min, int strategy, int buff, int wl_cap,
                                    adapt_pushup_result *res)
{
    if (!res || wl_cap < 2 || wl_cap > 32 || buff < 0 || buff > wl_cap || wl_min < 1 || fl_min < 0) return ADAPT_EINVAL;
    if (strategy != ADAPT_ST_MIN && strategy != ADAPT_ST_MEAN && strategy != ADAPT_ST_MAX) return ADAPT_EINVAL;
    const double L = usable(ds) ? std::log(ds) : 1.0;
    int s1 = 1, s2 = 1, s = 1;
    if (L > 0.0) {
        s1 = L == 1.0 ? wl_cap : (int)std::min<double>(std::max(std::ceil(1.0 / (L - 1.0)), 1.0), (double)wl_cap);
        const double s2f = std::max(std::min(32.0 * L * L - 1.0, 32.0) - (double)fl_min, 1.0);
        s2 = (int)std::min<double>(std::ceil(s2f), (double)wl_cap);
        if (strategy == ADAPT_ST_MIN) s = std::min(s1, s2);
        else if (strategy == ADAPT_ST_MEAN) s = (int)std::ceil(0.5 * (s1 + s2));
        else s = std::max(s1, s2);
    }
    int fl = std::min(fl_min + s, wl_cap);
    int wl = std::min(std::max(wl_min, fl_min) + 1, wl_cap);
    fl = std::min(fl, wl_cap - buff);
    wl = std::max(std::min(fl + buff, wl_cap), wl);
    res->wl = wl; res->fl = fl; res->s1 = s1; res->s2 = s2; res->s = s;
    return ADAPT_OK;
}

extern "C" int adapt_strategy_next(int strategy, double loss_avg, double loss_now)
{
    if (std::fabs(loss_avg) > std::fabs(loss_now)) return ADAPT_ST_MIN;
    return strategy == ADAPT_ST_MIN ? ADAPT_ST_MEAN : ADAPT_ST_MAX;
}

extern "C" int adapt_lookback_next(int lb, double ds, int lb_lwr, int lb_upr, double gamma)
{
    double lb_new = (double)lb_upr;
    if (usable(ds)) lb_new = std::min(std::max(std::ceil((double)lb_upr / ds), (double)lb_lwr), (double)lb_upr);
    return (int)std::ceil(lb_new * gamma + (1.0 - gamma) * (double)lb);
}

extern "C" int adapt_resolution_next(int r, int lb, int lb_lwr, int lb_upr, int r_lwr, int r_upr)
{
    if (lb == lb_upr) return std::min(std::max(r + 1, r_lwr), r_upr);
    if (lb == lb_lwr) return std::min(std::max(r - 1, r_lwr), r_upr);
    return r;
}
