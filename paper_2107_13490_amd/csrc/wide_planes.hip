// Forward convolutions with word lengths 17..32 in one contraction kernel.
//
// Both operands are first rewritten as P planes of signed bytes (P = 3 up to 24 bits, 4 above), a = sum_i 2^(8 i) a_i, with
// their channels padded to a multiple of 16; the kernel then multiplies every plane of one operand with every plane of
// the other on the int8 matrix cores, adds the products of equal weight i + j in one int32 accumulator set (2 P - 1 sets),
// and recombines them once in its epilogue, where the requantizing rule (or the exact 128-bit sum) is applied.
//   balanced digits (word lengths up to 8 P - 1): every digit in [-128, 127], nothing to correct;
//   offset digits (word length 8 P, where the balanced top digit would reach +128): the lower P - 1 digits are the
//     unsigned bytes less 128, so a = A + O with O = 128 (2^(8 (P - 1)) - 1) / 255, and with both sums taken over every
//     multiplied index, sum a b = sum A B + O_b sum A + O_a sum B + O_a O_b K.  Padding must then be the code 0 and not the
//     byte 0: every plane ends in 16 bytes of its digit of 0, and invalid chunks are fetched from there.
//
// What bounds it: P^2 products of 2 M N K operations at about a third of what the matrix cores reach alone (at P = 3 a sub-step
// of a 64 x 32 wavefront tile is 18 products behind 9 fragment reads), then the 64- or 128-bit epilogue and the splitting pass.
// 128 x 16 x 16 x 64 -> 192, 3x3, <24,21>: 327 us as four two-limb contractions with 128-bit accumulation passes between them,
// 47.4 us with this kernel and its splitting pass.  Grids of few tiles with a long reduction, and narrow operands beside wide
// ones, stay with the composition (wide_fwd_composed_faster below).
#include <algorithm>
#include <cmath>

#include "contract_dma.hpp"
#include "wide.hpp"

namespace adapt {

constexpr int kPlaneChunk = 16;                     // codes per thread of the splitting pass, bytes of a plane's zero chunk
constexpr int kWidePlanesMaxK = 32704;              // int32 accumulators: at most 4 products of 2^14 per index; whole stages of 64

static size_t a256w(size_t v) { return (v + 255) & ~(size_t)255; }
static inline int pad16(int c) { return (c + 15) & ~15; }

static inline size_t plane_stride(uint64_t rows, int cp) { return a256w(rows * (uint64_t)cp + kPlaneChunk); }
static inline int planes_for(adapt_fmt a, adapt_fmt b) { return std::max(a.wl, b.wl) <= 24 ? 3 : 4; }

// codes [rows][c] -> P planes [rows][cp] (channels c..cp-1: the code 0), each followed by one chunk of the code 0
struct PlaneSplit {
    const void *src;
    int8_t *dst;
    uint64_t rows;
    size_t stride;                  // bytes between planes
    int c, cp, es, offset;
};

// blk of nblk: this block's place among the operand's blocks
template <typename T, int P>
__device__ __forceinline__ void split_planes(const PlaneSplit &o, const uint32_t blk, const uint32_t nblk)
{
    const T *__restrict__ src = static_cast<const T *>(o.src);
    int8_t *__restrict__ dst = o.dst;
    const int c = o.c, cp = o.cp, offset = o.offset;
    const uint64_t rows = o.rows;
    const size_t stride = o.stride;
    const int cpr = cp / kPlaneChunk;
    const uint64_t chunks = rows * (uint64_t)cpr;
    for (uint64_t i = (uint64_t)blk * 256 + threadIdx.x; i <= chunks; i += (uint64_t)nblk * 256) {
        int v[kPlaneChunk];
        const uint64_t r = i / (uint32_t)cpr;
        const int c0 = (int)(i - r * cpr) * kPlaneChunk;
        if (i == chunks) {
#pragma unroll
            for (int e = 0; e < kPlaneChunk; ++e) v[e] = 0;
        } else if (c == cp) {
            constexpr int W = kPlaneChunk * (int)sizeof(T) / 16;
            uint4 raw[W];
            const uint4 *p = reinterpret_cast<const uint4 *>(src + r * (uint64_t)c + c0);
#pragma unroll
            for (int q = 0; q < W; ++q) raw[q] = p[q];
#pragma unroll
            for (int e = 0; e < kPlaneChunk; ++e) v[e] = (int)reinterpret_cast<const T *>(raw)[e];
        } else {
#pragma unroll
            for (int e = 0; e < kPlaneChunk; ++e) v[e] = c0 + e < c ? (int)src[r * (uint64_t)c + c0 + e] : 0;
        }
#pragma unroll
        for (int p = 0; p < P; ++p) {
            uint32_t w[4] = {0, 0, 0, 0};
#pragma unroll
            for (int e = 0; e < kPlaneChunk; ++e) {
                const int digit = p == P - 1 ? v[e] : offset ? (v[e] & 255) - 128 : (int)(int8_t)(v[e] & 255);
                w[e >> 2] |= (uint32_t)(digit & 255) << (8 * (e & 3));
                // next digit: the balanced one carries (v - digit overflows int32 only at P = 4 with 32-bit codes, which
                // take the offset form)
                v[e] = offset ? v[e] >> 8 : (v[e] - digit) >> 8;
            }
            *reinterpret_cast<uint4 *>(dst + p * stride + i * kPlaneChunk) = make_uint4(w[0], w[1], w[2], w[3]);
        }
    }
}

// Both operands in one launch: the filter's blocks come first and are done while the activations' run (two launches: 49.2
// instead of 47.4 us for 128 x 16 x 16 x 64 -> 192, 3x3, <24,21>, contraction included).
template <int P>
__global__ void __launch_bounds__(256) split_planes_kernel(const PlaneSplit act, const PlaneSplit wgt, const uint32_t wgt_blocks)
{
    const bool is_wgt = blockIdx.x < wgt_blocks;
    const PlaneSplit &o = is_wgt ? wgt : act;
    const uint32_t blk = is_wgt ? blockIdx.x : blockIdx.x - wgt_blocks, nblk = is_wgt ? wgt_blocks : gridDim.x - wgt_blocks;
    if (o.es == 4) split_planes<int32_t, P>(o, blk, nblk);
    else if (o.es == 2) split_planes<int16_t, P>(o, blk, nblk);
    else split_planes<int8_t, P>(o, blk, nblk);
}

struct WidePlanesArgs {
    ContractArgs a;                 // geometry of the padded contraction; act / wgt: first planes
    uint32_t act_stride, wgt_stride, act_zero, wgt_zero;      // bytes between planes; byte offset of a plane's zero chunk
    long long off_a, off_b;         // O_a, O_b (0: balanced digits)
    int raw, wl_o;                  // output: exact 128-bit sums, or codes of wl_o bits
};

template <int P> struct WideSum { typedef __int128 type; };
template <> struct WideSum<3> { typedef long long type; };      // 24 + 24 - 2 + 15 bits

// the contraction epilogue's rule; the sums leave room for the rounding bits
template <typename S>
__device__ __forceinline__ int requantize_sum(S acc, int shift, long long qlo, long long qhi, uint32_t r16)
{
    S q;
    if (shift <= 0) {
        const S lim = (S)1 << 31;               // saturates whatever the shift (at most 31: fractional bits go up to 31)
        const S c = acc > lim ? lim : acc < -lim ? -lim : acc;
        q = c * ((S)1 << -shift);
    } else if (shift <= 16) {
        q = (acc + (S)(r16 >> (16 - shift))) >> shift;
    } else {
        q = ((acc >> (shift - 16)) + (S)r16) >> 16;
    }
    return (int)(q > (S)qhi ? (S)qhi : q < (S)qlo ? (S)qlo : q);
}

template <int P, bool SUMS, int BM, int BN>
__global__ void __launch_bounds__(kThreads, 2)
wide_fwd_kernel(const WidePlanesArgs w)
{
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const ContractArgs &a = w.a;
    constexpr int BKT = 64, KS = BKT / 32, G = 2 * P - 1;
    constexpr int WM = BM / 2, WN = BN / 2, MB = WM / 32;
    static_assert(WN == 32, "a wavefront takes one 32-column block");
    typedef DmaK<true, BM> LA;
    typedef DmaK<false, BN> LB;
    constexpr int STAGE = P * (LA::TILE_BYTES + LB::TILE_BYTES);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wm = wave >> 1, wn = wave & 1, l32 = lane & 31, g = lane >> 5;
    const int nperm = 16 * ((l32 >> 2) & 1) + 4 * (l32 >> 3) + (l32 & 3);
    const unsigned nwg = gridDim.x, per_xcd = nwg / kXcds, extra = nwg % kXcds, xcd = blockIdx.x % kXcds;
    const unsigned tile = xcd * per_xcd + min(xcd, extra) + blockIdx.x / kXcds;
    const int tiles_n = (a.N + BN - 1) / BN;
    const int m0 = (int)(tile / tiles_n) * BM, n0 = (int)(tile % tiles_n) * BN;
    const int ksteps = (a.K + BKT - 1) / BKT;

    LA la;
    LB lb;
    la.init(a, m0);
    lb.init(a, n0);
    const __amdgpu_buffer_rsrc_t ra = make_rsrc(a.act, P * w.act_stride), rb = make_rsrc(a.wgt, P * w.wgt_stride);
    const uint32_t lds0 = lds_address(smem);
    // every plane of the stage that starts at reduction index k0; nothing is out of range, invalid chunks are the zero chunk
    auto fetch = [&](int k0, uint32_t buf) {
        const uint32_t dst = buf + wave * 1024;
        uint32_t tap, koff;
        if (a.uniform_tap) k_major_tap<OP_FWD>(a, (uint32_t)__builtin_amdgcn_readfirstlane(k0), k0, tap, koff);
        else k_major_tap<OP_FWD>(a, (uint32_t)(k0 + la.col), k0, tap, koff);
        const bool kin = k0 + la.col < a.K;
#pragma unroll
        for (int u = 0; u < LA::UNITS; ++u) {
            const bool ok = kin && ((la.tapmask[u] >> (tap & 31u)) & 1u);
            const uint32_t off = ok ? la.base[u] + koff : w.act_zero;
#pragma unroll
            for (int p = 0; p < P; ++p)
                load_to_lds(ra, dst + p * LA::TILE_BYTES + u * 4096, off, p * w.act_stride);
        }
#pragma unroll
        for (int u = 0; u < LB::UNITS; ++u) {
            const bool ok = k0 + lb.col < a.K && lb.tapmask[u] != 0;
            const uint32_t off = ok ? lb.base[u] + k0 : w.wgt_zero;
#pragma unroll
            for (int p = 0; p < P; ++p)
                load_to_lds(rb, dst + P * LA::TILE_BYTES + p * LB::TILE_BYTES + u * 4096, off, p * w.wgt_stride);
        }
    };
    fetch(0, lds0);

    uint32_t ad_a[KS], ad_w[KS];
    LA::addresses(0, wm * WM, l32, g, ad_a);
    LB::addresses(P * LA::TILE_BYTES, wn * WN, nperm, g, ad_w);
    v16i acc[G][MB];
#pragma unroll
    for (int s = 0; s < G; ++s)
#pragma unroll
        for (int j = 0; j < MB; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[s][j][r] = 0;
    int sum_m[MB][P], sum_n[P];
#pragma unroll
    for (int p = 0; p < P; ++p) {
#pragma unroll
        for (int j = 0; j < MB; ++j) sum_m[j][p] = 0;
        sum_n[p] = 0;
    }

    uint32_t cur = lds0, nxt = lds0 + STAGE;
    for (int kt = 0; kt < ksteps; ++kt) {
        wait_loads<0>();
        __builtin_amdgcn_s_barrier();
        if (kt + 1 < ksteps) fetch((kt + 1) * BKT, nxt);
        auto sub_step = [&](auto ksc) {
            constexpr int ks = decltype(ksc)::value;
            v4i fa[MB][P], fw[P];
            read_planes<P, MB, LA::TILE_BYTES, 32 * LA::ROW_BYTES, LB::TILE_BYTES>(fa, fw, cur + ad_a[ks], cur + ad_w[ks]);
#pragma unroll
            for (int pa = 0; pa < P; ++pa)
#pragma unroll
                for (int pb = 0; pb < P; ++pb)
#pragma unroll
                    for (int j = 0; j < MB; ++j)
                        acc[pa + pb][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fw[pb], fa[j][pa], acc[pa + pb][j], 0, 0, 0);
            if (SUMS) {
#pragma unroll
                for (int p = 0; p < P; ++p)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
#pragma unroll
                        for (int j = 0; j < MB; ++j) sum_m[j][p] = __builtin_amdgcn_sdot4(fa[j][p][e], 0x01010101, sum_m[j][p], false);
                        sum_n[p] = __builtin_amdgcn_sdot4(fw[p][e], 0x01010101, sum_n[p], false);
                    }
            }
        };
        sub_step(std::integral_constant<int, 0>{});
        sub_step(std::integral_constant<int, 1>{});
        const uint32_t t = cur;
        cur = nxt;
        nxt = t;
    }

    // ---- epilogue: a lane holds 16 consecutive outputs n of one row m per 32 x 32 block
    typedef typename WideSum<P>::type S;
    long long corr_m[MB];
    long long *sn = reinterpret_cast<long long *>(smem);      // [4 waves][32]
    if (SUMS) {
        __syncthreads();
        auto total = [&](const int (&s)[P]) {
            long long t = 0;
#pragma unroll
            for (int p = P - 1; p >= 0; --p) t = (t << 8) + (long long)(s[p] + __shfl_xor(s[p], 32, 64));
            return t;
        };
#pragma unroll
        for (int j = 0; j < MB; ++j) corr_m[j] = total(sum_m[j]);
        const long long t = total(sum_n);
        if (g == 0) sn[wave * 32 + nperm] = t;
        __syncthreads();
    }
    const long long qhi = (1ll << (w.wl_o - 1)) - 1, qlo = a.relu ? 0 : -(1ll << (w.wl_o - 1));
    const S both = SUMS ? (S)w.off_a * (S)w.off_b * (S)((long long)ksteps * BKT) : (S)0;
#pragma unroll
    for (int j = 0; j < MB; ++j) {
        const int m = m0 + wm * WM + j * 32 + l32, nb0 = n0 + wn * WN + 16 * g;
        if (m >= a.M || nb0 >= a.N) continue;
        const int cnt = min(16, a.N - nb0);
        const uint64_t idx0 = (uint64_t)m * (uint64_t)a.N + (uint64_t)nb0;
        uint32_t rw[8];
        if (!w.raw) {
            if (a.rmode != ADAPT_SR) {
#pragma unroll
                for (int e = 0; e < 8; ++e) rw[e] = 0x80008000u;
            } else if ((a.N & 7) == 0) {
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const u32x4 b = rounding_block(a.seed, a.stream, (idx0 >> 3) + h);
                    rw[4 * h] = b.x; rw[4 * h + 1] = b.y; rw[4 * h + 2] = b.z; rw[4 * h + 3] = b.w;
                }
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    rw[e] = rounding_bits_of(a.seed, a.stream, idx0 + 2 * e, a.rmode) |
                            rounding_bits_of(a.seed, a.stream, idx0 + 2 * e + 1, a.rmode) << 16;
            }
        }
        int q[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            S v = (S)acc[G - 1][j][r];
#pragma unroll
            for (int s = G - 2; s >= 0; --s) v = v * 256 + (S)acc[s][j][r];
            if (SUMS) v += (S)w.off_b * (S)corr_m[j] + (S)w.off_a * (S)sn[wave * 32 + 16 * g + r] + both;
            if (w.raw) {
                if (r < cnt) {
                    const __int128 x = (__int128)v;
                    reinterpret_cast<longlong2 *>(a.out)[idx0 + r] = make_longlong2((long long)x, (long long)(x >> 64));
                }
            } else {
                q[r] = requantize_sum<S>(v, a.shift, qlo, qhi, (rw[r >> 1] >> (16 * (r & 1))) & 0xffffu);
            }
        }
        if (w.raw) continue;
        const bool whole = cnt == 16 && (a.N & 15) == 0;
        if (w.wl_o > 16) {
            int32_t *o = static_cast<int32_t *>(a.out) + idx0;
            if (whole) {
#pragma unroll
                for (int e = 0; e < 4; ++e) reinterpret_cast<int4 *>(o)[e] = make_int4(q[4 * e], q[4 * e + 1], q[4 * e + 2], q[4 * e + 3]);
            } else {
#pragma unroll
                for (int e = 0; e < 16; ++e)
                    if (e < cnt) o[e] = q[e];
            }
        } else if (w.wl_o > 8) {
            int16_t *o = static_cast<int16_t *>(a.out) + idx0;
#pragma unroll
            for (int e = 0; e < 16; ++e)
                if (e < cnt) o[e] = (int16_t)q[e];
        } else {
            int8_t *o = static_cast<int8_t *>(a.out) + idx0;
#pragma unroll
            for (int e = 0; e < 16; ++e)
                if (e < cnt) o[e] = (int8_t)q[e];
        }
    }
}

template <int P, int BM, int BN>
static hipError_t launch_wide_fwd(adapt_ctx *ctx, const WidePlanesArgs &w)
{
    const size_t lds = (size_t)2 * P * (BM + BN) * 64;
    const unsigned tiles = (unsigned)(((w.a.M + BM - 1) / BM) * ((w.a.N + BN - 1) / BN));
    auto kern = (w.off_a || w.off_b) ? wide_fwd_kernel<P, true, BM, BN> : wide_fwd_kernel<P, false, BM, BN>;
    if (hipError_t e = allow_big_lds(ctx, reinterpret_cast<const void *>(kern), lds); e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3(tiles), dim3(kThreads), lds, ctx->stream, w);
    return hipGetLastError();
}

template <int P>
static void launch_split_planes(adapt_ctx *ctx, const PlaneSplit &act, const PlaneSplit &wgt)
{
    auto blocks = [&](const PlaneSplit &o) {
        const uint64_t chunks = o.rows * (uint64_t)(o.cp / kPlaneChunk) + 1;
        return (unsigned)std::min<uint64_t>((chunks + 255) / 256, (uint64_t)ctx->num_cu * 16);
    };
    const unsigned nw = blocks(wgt);
    hipLaunchKernelGGL(split_planes_kernel<P>, dim3(nw + blocks(act)), dim3(256), 0, ctx->stream, act, wgt, nw);
}

// Whether the kernel takes this convolution: filter taps and reduction length within its bounds, planes within 32-bit offsets
static bool planes_fit(const adapt_conv_desc &d, int P)
{
    const int cp = pad16(d.c);
    return d.r * d.s <= 32 && (long long)d.r * d.s * cp <= kWidePlanesMaxK &&
           (uint64_t)P * plane_stride((uint64_t)d.n * d.h * d.w, cp) < ((uint64_t)1 << 32) &&
           (uint64_t)P * plane_stride((uint64_t)d.k * d.r * d.s, cp) < ((uint64_t)1 << 32);
}

size_t ws_need_wide_fwd(const adapt_conv_desc &d, adapt_fmt fx, adapt_fmt fw)
{
    const int P = planes_for(fx, fw), cp = pad16(d.c);
    if (!planes_fit(d, P)) return 0;
    return (size_t)P * (plane_stride((uint64_t)d.n * d.h * d.w, cp) + plane_stride((uint64_t)d.k * d.r * d.s, cp));
}

// The planes take P^2 products for every pair of operands, on one block per 128 x 64 (64 x 64) outputs that walks the whole
// reduction; the composition multiplies a narrow operand as it is and splits a long reduction over blocks, but launches
// several kernels and takes its exact partial results through memory.  So neither is the faster one everywhere (us,
// composition / planes): 128 x 16 x 16 x 64 -> 192 3x3 <24,24> bits 217 / 55, <8,24> 93 / 48; 128 x 4096 -> 4096 <24,24>
// 148 / 103, <8,24> 78 / 103; 128 x 4096 -> 10 <24,24> 53 / 93, <8,24> 26 / 93; 32 x 4 x 4 x 512 -> 512 3x3 <24,24> 113 / 101,
// <24,8> 54 / 102.  The line is drawn by two sums over what each does, fitted to 667 calls of 1 to 256 images of 1 x 1 to
// 32 x 32, 3 to 4096 channels, 8 to 32 bits a side on 256 CUs: with it a call takes 0.3 % more than the faster form on
// average, at most 22 % (always the planes: 19 %, up to 5.4 times; always the composition: 2.1 times), and 300 calls that
// it was not fitted to 0.4 % (at most 27 %).
static double planes_us(int num_cu, const adapt_conv_desc &d, adapt_fmt fx, adapt_fmt fw, double m, double n)
{
    const int P = planes_for(fx, fw), cp = pad16(d.c), bm = P == 3 ? 128 : 64;
    const double stages = (d.r * d.s * cp + 63) / 64, tiles = std::ceil(m / bm) * std::ceil(n / 64);
    const double rounds = std::max(1.0, tiles / num_cu), xr = (double)d.n * d.h * d.w, wr = (double)d.k * d.r * d.s;
    const double stage = fx.wl == 8 * P || fw.wl == 8 * P ? 1.17 : 0.93;                 // with / without the sums of offset digits
    const double bytes = (xr * storage_bytes(fx) + wr * storage_bytes(fw)) * d.c + (xr + wr) * cp * P;      // of the splitting pass
    return 11.0 + (d.k % 8 ? 4.5 * rounds : 0.0) + stage * stages * rounds + 1.7e-6 * m * n + 0.15e-6 * bytes;
}

static double composed_us(int num_cu, const adapt_conv_desc &d, adapt_fmt fx, adapt_fmt fw, double m, double n)
{
    adapt_fmt pa[3], pb[3];
    int step;
    const int na = wide_parts(fx, pa, &step), nb = wide_parts(fw, pb, &step);
    const double k = (double)d.r * d.s * pad16(d.c), tiles = std::ceil(m / 64) * std::ceil(n / 64);
    double launches = 1, chain = 0, bytes = 0;
    for (int i = 0; i < na; ++i)
        for (int j = 0; j < nb; ++j) {
            const int la = pa[i].wl > 8 ? 2 : 1, lb = pb[j].wl > 8 ? 2 : 1, bkt = la * lb == 1 ? 128 : 64;
            double splits = 1;                                   // as plan_contraction splits
            if (tiles < num_cu && k >= 8 * bkt) splits = std::max(1.0, std::min(std::ceil(2 * num_cu / tiles), std::floor(k / (4 * bkt))));
            const double acc = adapt_acc_bits((int64_t)d.r * d.s * d.c, pa[i], pb[j]) == 32 ? 4 : 8;
            launches += (splits > 1 ? 2 : 1) + (d.c % 16 ? 1 : 0);      // the slab sum, the padded copies
            chain += k / 64 / splits * std::max(1.0, tiles * splits / (2 * num_cu)) * la * lb;
            bytes += 2 * m * n * acc * (1 + (splits > 1 ? splits : 0));      // partial results and slabs, written and read
        }
    double split = 0;
    if (fx.wl > 16) { launches += 1; split += (double)d.n * d.h * d.w * d.c * (4 + 2 * na); }
    if (fw.wl > 16) { launches += 1; split += (double)d.k * d.r * d.s * d.c * (4 + 2 * nb); }
    return 3.6 * launches + 0.19 * chain + 0.35e-6 * bytes + 0.14e-6 * split;
}

bool wide_fwd_composed_faster(int num_cu, const adapt_conv_desc &d, adapt_fmt fx, adapt_fmt fw)
{
    const double m = (double)d.n * ((d.h + 2 * d.pad - d.r) / d.stride + 1) * ((d.w + 2 * d.pad - d.s) / d.stride + 1), n = d.k;
    return planes_us(num_cu, d, fx, fw, m, n) >= 1.05 * composed_us(num_cu, d, fx, fw, m, n);
}

// The forward convolution by planes, or ADAPT_EWORKSPACE / ADAPT_EUNSUPPORTED when the composed path takes it (nothing
// has been launched then): where the planes do not apply, or where the composition is faster and the workspace holds its
// faster form
int wide_fwd_planes(adapt_ctx *ctx, const adapt_conv_desc &d, const void *x, adapt_fmt fx, const void *wt, adapt_fmt fw, void *y, adapt_epilogue ep)
{
    if (!fmt_ok_wide(fx) || !fmt_ok_wide(fw)) return ADAPT_EINVAL;
    if (!ep.raw && (!fmt_ok_wide(ep.fmt) || (ep.rng.mode != ADAPT_SR && ep.rng.mode != ADAPT_RN_HALF_UP))) return ADAPT_EINVAL;
    const int P = planes_for(fx, fw), cp = pad16(d.c);
    if (fx.wl <= 16 && fw.wl <= 16) return ADAPT_EUNSUPPORTED;      // only the output is wide
    const size_t need = ws_need_wide_fwd(d, fx, fw);
    if (need == 0) return ADAPT_EUNSUPPORTED;
    if (need > scratch_bytes(ctx)) return ADAPT_EWORKSPACE;
    const uint64_t xrows = (uint64_t)d.n * d.h * d.w, wrows = (uint64_t)d.k * d.r * d.s;
    const uint64_t outputs = (uint64_t)d.n * ((d.h + 2 * d.pad - d.r) / d.stride + 1) * ((d.w + 2 * d.pad - d.s) / d.stride + 1) * d.k;
    const size_t inner = d.c % 16 ? (size_t)(xrows + wrows) * cp * 2 + 1024 : 0;      // the part contractions' padded copies
    if (wide_fwd_composed_faster(ctx->num_cu, d, fx, fw) &&
        ws_need_wide_all_pairs(fx, xrows * d.c, fw, wrows * d.c, outputs) + std::max((size_t)1 << 20, inner) <= scratch_bytes(ctx))
        return ADAPT_EUNSUPPORTED;
    const size_t xs = plane_stride(xrows, cp), wsd = plane_stride(wrows, cp);
    int8_t *xp = reinterpret_cast<int8_t *>(scratch(ctx)), *wp = xp + (size_t)P * xs;
    WidePlanesArgs w = {};
    adapt_conv_desc d2 = d;
    d2.c = cp;
    if (int s = fill_fwd(w.a, d2, xp, adapt_fmt{8, 0}, wp, adapt_fmt{8, 0}, y)) return s;
    w.act_stride = (uint32_t)xs;
    w.wgt_stride = (uint32_t)wsd;
    w.act_zero = (uint32_t)(xrows * cp);
    w.wgt_zero = (uint32_t)(wrows * cp);
    const long long off = P == 3 ? 128ll * 257 : 128ll * 65793;
    w.off_a = fx.wl == 8 * P ? off : 0;
    w.off_b = fw.wl == 8 * P ? off : 0;
    w.raw = ep.raw != 0;
    w.wl_o = ep.raw ? 32 : ep.fmt.wl;
    w.a.shift = ep.raw ? 0 : fx.fl + fw.fl - ep.fmt.fl;
    w.a.relu = !ep.raw && ep.relu != 0;
    w.a.rmode = ep.rng.mode;
    w.a.seed = ep.rng.seed;
    w.a.stream = ep.rng.stream;
    const PlaneSplit act = {x, xp, xrows, xs, d.c, cp, storage_bytes(fx), fx.wl == 8 * P};
    const PlaneSplit wgt = {wt, wp, wrows, wsd, d.c, cp, storage_bytes(fw), fw.wl == 8 * P};
    if (P == 3) launch_split_planes<3>(ctx, act, wgt);
    else launch_split_planes<4>(ctx, act, wgt);
    hipError_t e = hipGetLastError();
    // seven accumulator sets of a 64 x 32 wavefront tile do not leave room for two blocks per CU
    if (e == hipSuccess) e = P == 3 ? launch_wide_fwd<3, 128, 64>(ctx, w) : launch_wide_fwd<4, 64, 64>(ctx, w);
    return hip_status(ctx, e);
}

}  // namespace adapt
