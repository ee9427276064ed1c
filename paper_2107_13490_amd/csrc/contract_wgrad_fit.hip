// Weight gradients of layers with a short reduction and one filter tap (fully connected layers at training batch sizes), fitted to a
// word length without the exact sums ever being stored: the contraction runs twice, first for the largest magnitude alone, then, the
// shift known, for the codes.
//
// A block owns 64 output channels (rows) and walks over tiles of 64 input channels (columns).  dy's codes of its rows, all of the
// reduction, stay in LDS, split into limbs; x's come in stages of 128 reduction indices of a tile through a double buffer, the loads of
// the stage after the next in flight.  A wavefront holds one block of 32 x 32 sums.  (4096 x 4096 at batch 128, 16 bits, traced: the
// contraction with its 134 MB of sums 61 us and the fitting pass 31; here 26 and 38, vector instructions for the most part: the sums in
// 64 bits, as the other kernels have them, 31 and 45; one LDS buffer and three blocks per CU 28 and 38; the kernels with 128 x 128 tiles
// of contract_kernel.hpp, one tile per block, 47 and 67.)
#include "contract_kernel.hpp"
#include "fit.hpp"

namespace adapt {

constexpr int kShortSlots = 128;       // reduction indices of a stage
constexpr int kShortTile = 64;         // rows of a block, columns of a tile
constexpr int kShortPitch = 96;        // bytes of an LDS line: an odd multiple of 32, so that the lines of a transposing read meet different banks
constexpr int kShortMaxK = 256;        // sums as 256 u + (0..255) with u in 32 bits; with at most one int16 operand they fit 32 bits themselves

struct ShortArgs {
    ContractArgs a;                    // M, N, K, operands, out, out_mode, wl_o, rounding
    int tiles, per_block, chunks;      // column tiles, of a block; stages of a tile
    FitTarget t;
    int nparts;                        // second pass: maxima at t.part
};

constexpr size_t short_lds(int la, int lb, int chunks) { return (size_t)kShortSlots * kShortPitch * (la * chunks + 2 * lb); }

// first: of lanes 0..31 their own a, of lanes 32..63 their partner's b; second: the partner's a, the own b
__device__ __forceinline__ void exchange(uint32_t a, uint32_t b, uint32_t &first, uint32_t &second)
{
    typedef unsigned v2u __attribute__((ext_vector_type(2)));
    const v2u r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
    first = r[0];
    second = r[1];
}

template <int AES, int WES, bool FIT>
__global__ void __launch_bounds__(kThreads, 2)
short_kernel(const ShortArgs h)
{
    extern __shared__ __attribute__((aligned(16))) char smem[];
    __shared__ unsigned long long red[4];
    __shared__ __attribute__((aligned(16))) int col_sum[4][32];      // offset split: a wavefront's column sums
    const ContractArgs &a = h.a;
    constexpr int LAL = limbs_of(AES), LBL = limbs_of(WES), EA = es_of(AES), EB = es_of(WES), LP = kShortPitch, KP = kShortSlots;
    constexpr bool BOTH2 = LAL == 2 && LBL == 2, OFFS = AES == 2 || WES == 2;
    constexpr int PA = 16 / EA, PX = 16 / EB, CLA = kShortTile / PA, CLX = kShortTile / PX;      // codes of a 16-byte chunk, chunks of a line
    constexpr int UA = KP * CLA / kThreads, UX = KP * CLX / kThreads;                            // chunks of a stage per thread
    constexpr int A_STAGE = LAL * KP * LP, A_LO = KP * LP, X_STAGE = LBL * KP * LP, X_LO = KP * LP;
    constexpr uint32_t NOWHERE = 0xfffffff0u;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l32 = lane & 31, g = lane >> 5, wm = wave >> 1, wn = wave & 1;
    const int m0 = blockIdx.x * kShortTile, first = blockIdx.y * h.per_block, last = min(first + h.per_block, h.tiles);
    const int stages = (last - first) * h.chunks;
    const __amdgpu_buffer_rsrc_t ra = make_rsrc(a.act, a.act_bytes), rx = make_rsrc(a.wgt, a.wgt_bytes);
    char *const xbuf = smem + h.chunks * A_STAGE;

    uint64_t part_max = 0;             // the thread's share of the maximum
    if (FIT) part_max = max_of_parts<kThreads>(reinterpret_cast<const uint64_t *>(h.t.part), h.nparts);

    const int x_slot = threadIdx.x / CLX, x_col = threadIdx.x % CLX * PX;      // chunk i of a stage of x: slot x_slot + i * kThreads / CLX
    v4u xv[UX];
    auto load_x = [&](int st) {
        const int tile = first + st / h.chunks, k0 = st % h.chunks * KP, col = tile * kShortTile + x_col;
#pragma unroll
        for (int i = 0; i < UX; ++i) {
            const int k = k0 + x_slot + i * (kThreads / CLX);
            const bool ok = st < stages && k < a.K && col < a.N;
            xv[i] = __builtin_amdgcn_raw_buffer_load_b128(rx, ok ? ((uint32_t)k * (uint32_t)a.N + (uint32_t)col) * EB : NOWHERE, 0, 0);
        }
    };
    auto store_x = [&](int st) {
        char *const buf = xbuf + (st & 1) * X_STAGE;
#pragma unroll
        for (int i = 0; i < UX; ++i) store_limbs<WES>(xv[i], buf + (x_slot + i * (kThreads / CLX)) * LP + x_col, X_LO);
    };
    load_x(0);
    for (int c = 0; c < h.chunks; ++c) {
        v4u av[UA];
        const int slot = threadIdx.x / CLA, col = threadIdx.x % CLA * PA;
#pragma unroll
        for (int i = 0; i < UA; ++i) {
            const int k = c * KP + slot + i * (kThreads / CLA);
            const bool ok = k < a.K && m0 + col < a.M;
            av[i] = __builtin_amdgcn_raw_buffer_load_b128(ra, ok ? ((uint32_t)k * (uint32_t)a.k + (uint32_t)(m0 + col)) * EA : NOWHERE, 0, 0);
        }
#pragma unroll
        for (int i = 0; i < UA; ++i) store_limbs<AES>(av[i], smem + c * A_STAGE + (slot + i * (kThreads / CLA)) * LP + col, A_LO);
    }
    int shift = 0;
    if (FIT) {
        part_max = wave_max_u64(part_max);
        if (lane == 0) red[wave] = part_max;
    }
    store_x(0);
    load_x(1);
    __syncthreads();
    if (FIT) {
        uint64_t most = red[0];
#pragma unroll
        for (int i = 1; i < 4; ++i) most = red[i] > most ? red[i] : most;
        shift = fit_shift_of(most, a.wl_o);
        if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) {
            if (h.t.shift != nullptr) *h.t.shift = shift;
            if (h.t.e_out != nullptr) *h.t.e_out = (h.t.e_in != nullptr ? *h.t.e_in : 0) + h.t.e_add - shift;
        }
    }

    // fragments as LoaderR::frag
    typedef v2i __attribute__((address_space(3))) * lds_v2i;
    const int grp = lane >> 4, f0 = (16 * (grp >> 1) + ((lane & 15) >> 1)) * LP + 16 * (grp & 1) + 8 * (lane & 1);
    auto frag = [&](const char *p) {
        const v2i u = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_v2i)(p)), v = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_v2i)(p + 8 * LP));
        v4i f;
        f[0] = u[0]; f[1] = u[1]; f[2] = v[0]; f[3] = v[1];
        return f;
    };
    v16i hh, xx, ll;
    auto clear = [&]() {
#pragma unroll
        for (int e = 0; e < 16; ++e) { hh[e] = 0; xx[e] = 0; ll[e] = 0; }
    };
    clear();
    int sum_m = 0, sum_n = 0;          // offset split: as in contract_body
    unsigned long long total = 0;      // the largest magnitude, or the sum of the squared codes
    int chunk = 0, tile = first;
    for (int st = 0; st < stages; ++st) {
        if (st + 1 < stages) store_x(st + 1);
        load_x(st + 2);
        const char *const ab = smem + chunk * A_STAGE + f0 + wm * 32, *const xb = xbuf + (st & 1) * X_STAGE + f0 + wn * 32;
#pragma unroll
        for (int ks = 0; ks < KP / 32; ++ks) {
            const v4i ah = frag(ab + ks * 32 * LP), xh = frag(xb + ks * 32 * LP);
            v4i al, xl;
            if (LAL == 2) al = frag(ab + A_LO + ks * 32 * LP);
            if (LBL == 2) xl = frag(xb + X_LO + ks * 32 * LP);
            hh = __builtin_amdgcn_mfma_i32_32x32x32_i8(xh, ah, hh, 0, 0, 0);
            if (LAL == 2) xx = __builtin_amdgcn_mfma_i32_32x32x32_i8(xh, al, xx, 0, 0, 0);
            if (BOTH2) ll = __builtin_amdgcn_mfma_i32_32x32x32_i8(xl, al, ll, 0, 0, 0);
            if (LBL == 2) xx = __builtin_amdgcn_mfma_i32_32x32x32_i8(xl, ah, xx, 0, 0, 0);
            if (OFFS && LBL == 2 && tile == first) {      // the rows' sums are those of every tile
#pragma unroll
                for (int e = 0; e < 4; ++e) sum_m += LAL == 2 ? 256 * dot4_ones((uint32_t)ah[e]) + dot4_ones((uint32_t)al[e]) : dot4_ones((uint32_t)ah[e]);
            }
            if (OFFS && LAL == 2) {
#pragma unroll
                for (int e = 0; e < 4; ++e) sum_n += LBL == 2 ? 256 * dot4_ones((uint32_t)xh[e]) + dot4_ones((uint32_t)xl[e]) : dot4_ones((uint32_t)xh[e]);
            }
        }
        if (++chunk == h.chunks) {     // the tile is done
            chunk = 0;
            // the exact sums: BOTH2, 256 u + low with 0 <= low < 256; else u
            int u[16], low[16];
            const int corr_m = OFFS && LBL == 2 ? sum_m + __shfl_xor(sum_m, 32, 64) : 0;
            if (OFFS && LAL == 2) {
                const int n_sum = sum_n + __shfl_xor(sum_n, 32, 64);
                if (g == 0) col_sum[wave][l32] = n_sum;
                __builtin_amdgcn_wave_barrier();
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                v4i s_n = {0, 0, 0, 0};
                if (OFFS && LAL == 2) s_n = *reinterpret_cast<const v4i *>(&col_sum[wave][8 * k + 4 * g]);
#pragma unroll
                for (int b = 0; b < 4; ++b) {
                    const int e = 4 * k + b;             // column 8 k + 4 g + b of the wavefront's 32
                    if (BOTH2) {
                        // 128 c = 256 (c >> 1) + 128 (c & 1), the correction of contract_epilogue
                        const int c = corr_m + s_n[b], l = OFFS ? ll[e] + ((c & 1) << 7) : ll[e];
                        u[e] = (hh[e] << 8) + xx[e] + (l >> 8);
                        if (OFFS) u[e] += (c >> 1) + 64 * h.chunks * KP;
                        low[e] = l & 255;
                    } else {
                        u[e] = LAL == 2 || LBL == 2 ? (hh[e] << 8) + xx[e] : hh[e];
                        if (OFFS) u[e] += 128 * (LBL == 2 ? corr_m : s_n[b]);
                        low[e] = 0;
                    }
                }
            }
            const int m = m0 + wm * 32 + l32, n0 = tile * kShortTile + wn * 32;
            if (!FIT) {
                // columns and rows beyond the output are sums of zeros
                uint32_t most = 0;
#pragma unroll
                for (int e = 0; e < 16; ++e) most = max(most, (uint32_t)abs(u[e]));
                unsigned long long mag = most;
                if (BOTH2) {
                    // What counts is the bit length.  |256 u + low| has that of 256 |u| unless |u| is a power of two (or 0).
                    mag = (unsigned long long)most << 8;
                    if (__any((most & (most - 1)) == 0)) {
                        mag = 0;
#pragma unroll
                        for (int e = 0; e < 16; ++e) {
                            const unsigned long long v = magnitude((long long)u[e] * 256 + low[e]);
                            mag = v > mag ? v : mag;
                        }
                    }
                }
                total = mag > total ? mag : total;
            } else {
                // Rounding bits: a Philox block covers 8 outputs, of which the lane and its partner of the other half hold four each; each
                // draws two of their four blocks and they exchange halves.
                uint32_t rw[8];
                if (a.rmode == ADAPT_SR) {
                    const uint64_t blk = ((uint64_t)m * (uint64_t)a.N + (uint64_t)n0) / 8 + 2 * g;
                    const u32x4 p = rounding_block(a.seed, a.stream, blk), r = rounding_block(a.seed, a.stream, blk + 1);
                    exchange(p.x, p.z, rw[0], rw[4]);
                    exchange(p.y, p.w, rw[1], rw[5]);
                    exchange(r.x, r.z, rw[2], rw[6]);
                    exchange(r.y, r.w, rw[3], rw[7]);
                } else {
#pragma unroll
                    for (int k = 0; k < 8; ++k) rw[k] = 0x80008000u;
                }
                const int qhi = (1 << (a.wl_o - 1)) - 1, qlo = -(1 << (a.wl_o - 1));
                int q[16];
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const uint32_t r16 = (rw[2 * (e >> 2) + ((e & 3) >> 1)] >> (16 * (e & 1))) & 0xffffu;
                    q[e] = BOTH2 ? fit_pair(u[e], low[e], shift, r16) : fit_one32(u[e], shift, r16);
                    q[e] = min(max(q[e], qlo), qhi);
                }
                if (m < a.M && n0 + 32 <= a.N) {
#pragma unroll
                    for (int e = 0; e < 16; ++e) total += (uint32_t)(q[e] * q[e]);
                } else if (m < a.M) {
#pragma unroll
                    for (int e = 0; e < 16; ++e)
                        if (n0 + 8 * (e >> 2) < a.N) total += (uint32_t)(q[e] * q[e]);      // (N is a multiple of 16)
                }
                // to 16 consecutive columns per lane: columns 16 g .. 16 g + 15
                const bool in = m < a.M && n0 + 16 * g < a.N;
                const size_t at = (size_t)m * (size_t)a.N + (size_t)(n0 + 16 * g);
                if (a.out_mode == OUT_Q8) {
                    uint32_t w[4], x[4];
#pragma unroll
                    for (int k = 0; k < 4; ++k) w[k] = pack4_i8(q[4 * k], q[4 * k + 1], q[4 * k + 2], q[4 * k + 3]);
                    exchange(w[0], w[2], x[0], x[1]);
                    exchange(w[1], w[3], x[2], x[3]);
                    if (in) store16(static_cast<int8_t *>(a.out) + at, x[0], x[1], x[2], x[3]);
                } else {
                    uint32_t w[8], x[8];
#pragma unroll
                    for (int k = 0; k < 8; ++k) w[k] = (uint32_t)(q[2 * k] & 0xffff) | ((uint32_t)q[2 * k + 1] << 16);
                    exchange(w[0], w[4], x[0], x[2]);
                    exchange(w[1], w[5], x[1], x[3]);
                    exchange(w[2], w[6], x[4], x[6]);
                    exchange(w[3], w[7], x[5], x[7]);
                    if (in) {
                        store16(static_cast<int16_t *>(a.out) + at, x[0], x[1], x[2], x[3]);
                        store16(static_cast<int16_t *>(a.out) + at + 8, x[4], x[5], x[6], x[7]);
                    }
                }
            }
            ++tile;
            clear();
            sum_n = 0;
        }
        __syncthreads();
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        const unsigned long long o = __shfl_xor(total, off, 64);
        if (FIT) total += o;
        else total = o > total ? o : total;
    }
    if (lane == 0) red[wave] = total;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long r = red[0];
#pragma unroll
        for (int i = 1; i < 4; ++i) {
            if (FIT) r += red[i];
            else r = red[i] > r ? red[i] : r;
        }
        if (FIT) {
            if (r) atomicAdd(h.t.sumsq, r);
        } else {
            h.t.part[blockIdx.y * gridDim.x + blockIdx.x] = r;
            if (blockIdx.x == 0 && blockIdx.y == 0) *h.t.sumsq = 0;
        }
    }
}

template <int AES, int WES>
static hipError_t launch_short(adapt_ctx *ctx, const ShortArgs &h)
{
    const size_t lds = short_lds(limbs_of(AES), limbs_of(WES), h.chunks);
    const size_t most = short_lds(limbs_of(AES), limbs_of(WES), kShortMaxK / kShortSlots);
    const dim3 grid((h.a.M + kShortTile - 1) / kShortTile, (h.tiles + h.per_block - 1) / h.per_block);
    void (*const passes[2])(const ShortArgs) = {short_kernel<AES, WES, false>, short_kernel<AES, WES, true>};
    for (auto kern : passes) {
        if (hipError_t e = allow_big_lds(ctx, reinterpret_cast<const void *>(kern), most); e != hipSuccess) return e;
        hipLaunchKernelGGL(kern, grid, dim3(kThreads), lds, ctx->stream, h);
        if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
    }
    return hipSuccess;
}

int wgrad_fit(adapt_ctx *ctx, const adapt_conv_desc &d, const void *dy, adapt_fmt fdy, const void *x, adapt_fmt fx, const FitTarget &t)
{
    if (!conv_ok(d) || !fmt_ok(fdy) || !fmt_ok(fx) || t.wl < 2 || t.wl > 16 || !check_ptrs(dy, x, t.q)) return ADAPT_EUNSUPPORTED;
    if (d.r != 1 || d.s != 1 || d.stride != 1 || d.pad != 0) return ADAPT_EUNSUPPORTED;
    ShortArgs h = {};
    ContractArgs &a = h.a;
    if (fill_wgrad(a, d, dy, fdy, x, fx, t.q) != ADAPT_OK) return ADAPT_EUNSUPPORTED;
    // Where the second contraction costs less than the sums' way through memory: us, backward pass of a c -> k layer and a small one behind
    // it, before -> here.  One limb: 128 x 4096 -> 4096 68.0 -> 51.9, 256 images 73.0 -> 61.7, 1024 -> 1024 32.5 -> 30.7; below 2^20 weights 768 -> 768
    // 29.3 -> 29.4 for 8 images and 30.4 -> 29.5 for 128, an int8 layer on int16 inputs 31.1 -> 31.7 and 33.1 -> 33.0, 512 -> 512 29.6 -> 30.7.  Two: 16 bits
    // 108.8 -> 82.0, 12 bits 83.8 -> 67.4, 9216 -> 4096 at 16 bits 264 -> 132; 256 images (two stages per tile) 120.5 -> 146.7; 2048 -> 2048 50.7 ->
    // 50.6 with two tiles per block (8 images, 12 bits 44.5 -> 45.1, 16 x 8 bits 52.7 -> 46.7), 1024 -> 1024 35.0 -> 40.4 with one.  90 layers and word lengths at
    // 8 to 256 images: none slower where the rule takes it.
    const bool one_limb = a.act_es == 1 && a.wgt_es == 1;
    if (a.act_load != LOAD_ROWS || a.wgt_load != LOAD_ROWS || a.K < 1 || a.K > (one_limb ? kShortMaxK : kShortSlots)) return ADAPT_EUNSUPPORTED;
    if ((long long)a.M * a.N < 1 << 20) return ADAPT_EUNSUPPORTED;
    a.out_mode = t.wl <= 8 ? OUT_Q8 : OUT_Q16;
    a.wl_o = t.wl;
    a.rmode = t.rng.mode;
    a.seed = t.rng.seed;
    a.stream = t.rng.stream;
    a.balanced = fdy.wl <= 15 && fx.wl <= 15;
    h.t = t;
    h.chunks = (a.K + kShortSlots - 1) / kShortSlots;
    h.tiles = (a.N + kShortTile - 1) / kShortTile;
    const int rows = (a.M + kShortTile - 1) / kShortTile;
    // two blocks per CU
    const int want = std::max(1, 2 * ctx->num_cu / rows);
    h.per_block = (h.tiles + want - 1) / want;
    h.nparts = rows * ((h.tiles + h.per_block - 1) / h.per_block);
    if ((!one_limb && h.per_block < 4) || h.nparts > t.parts) return ADAPT_EUNSUPPORTED;
    hipError_t e;
    if (one_limb) e = launch_short<1, 1>(ctx, h);
    else if (a.act_es == 2 && a.wgt_es == 2) e = a.balanced ? launch_short<3, 3>(ctx, h) : launch_short<2, 2>(ctx, h);
    else if (a.act_es == 2) e = a.balanced ? launch_short<3, 1>(ctx, h) : launch_short<2, 1>(ctx, h);
    else e = a.balanced ? launch_short<1, 3>(ctx, h) : launch_short<1, 2>(ctx, h);
    return hip_status(ctx, e);
}

}  // namespace adapt
