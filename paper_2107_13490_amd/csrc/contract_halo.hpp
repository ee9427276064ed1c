// Stride-1 convolutions (forward and data gradient) on input patches held in LDS.
//
// The implicit GEMM of contract_kernel.hpp fetches an input pixel once per filter tap and splits it into limbs every time.  Here
// a block keeps the patch of input pixels that its output rows see (with its halo of zeros) in LDS, 64 channels at a time,
// already split: every pixel is fetched and split once per block, the taps read it from LDS at shifted places, and only the
// filters stream through a double buffer.  A stage is one tap of one 64-channel chunk: while it is multiplied, the filters of the
// next stage and a share of the next chunk's patch are fetched into registers, and they are written to the other buffers between
// the stage's two sub-steps; one barrier per stage.
//
//   op      rows m       input image          offset of tap (r, s)      filters
//   fwd     (n,p,q)      x, h x w x c         (r - pad, s - pad)        w[kout][r][s][c], reduction index c
//   dgrad   (n,h,w)      dy, p x q x k        the same with pad' = R-1-pad and S-1-pad and the taps in reverse order;
//                                             reduction index kout
//
// LDS rows are an odd number of 16-byte units apart (64 codes per limb and 16 bytes), so that the 16-byte fragment reads of
// neighbouring pixels meet different banks.
#pragma once
#include "contract_kernel.hpp"

namespace adapt {

struct HaloArgs {
    ContractArgs a;              // M, N, K, pointers, extents, epilogue
    int ih, iw, ch;              // input image and its channels (the reduction runs over taps x ch)
    int oh, ow;                  // output image
    int pr, pc;                  // input pixel of output pixel (y, x) and tap (r, s): (y - pr + r, x - pc + s)
    int pw;                      // columns of a patch: ow + s - 1
    int pix;                     // most pixels a block's patch has (its LDS buffer)
    int patches;                 // LDS buffers for patches: two, one where the channels are one chunk
    FastDiv div_ow, div_oh, div_pw, div_ir;      // output columns, output rows, patch columns, patch rows of a whole image (oh + r - 1)
};

template <int OP, int LIMBS, int AES, int WES, int BM, int BN, int WGM, int WGN, bool AMAX>
__global__ void __launch_bounds__(64 * WGM * WGN, 2)
halo_kernel(const HaloArgs h)
{
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const ContractArgs &a = h.a;
    constexpr int NT = 64 * WGM * WGN;
    constexpr int LAL = limbs_of(AES), LBL = limbs_of(WES), EA = es_of(AES), EB = es_of(WES);
    constexpr bool BOTH2 = LAL == 2 && LBL == 2, OFFS = AES == 2 || WES == 2, W_R = OP == OP_DGRAD;
    constexpr int WM = BM / WGM, WN = BN / WGN, MB = WM / 32, NB = WN / 32;
    constexpr int PS = halo_row_bytes(LAL), BB = halo_b_bytes(OP, LBL, BN);
    constexpr int BRS = W_R ? BN + 16 : halo_row_bytes(LBL);      // bytes of a filter row (forward) or line (data gradient)
    constexpr int B_LO = W_R ? kHaloK * BRS : kHaloK;             // from a filter's high limb to its low limb
    constexpr int BT = BN * (kHaloK / 16), BU = BT / NT;          // 16-code filter units of a stage, and of a thread
    static_assert(BT % NT == 0, "every thread has the same number of filter units");
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l32 = lane & 31, g = lane >> 5;
    const int wm = wave / WGN, wn = wave % WGN;
    const int nperm = 16 * ((l32 >> 2) & 1) + 4 * (l32 >> 3) + (l32 & 3);

    // neighbouring blocks (same rows, other columns) on one XCD, as in contract_body
    const unsigned lin = blockIdx.x, nwg = gridDim.x, per_xcd = nwg / kXcds, extra = nwg % kXcds, xcd = lin % kXcds;
    const unsigned tile = xcd * per_xcd + min(xcd, extra) + lin / kXcds;
    const int tiles_n = (a.N + BN - 1) / BN;
    const int m0 = (int)(tile / tiles_n) * BM, n0 = (int)(tile % tiles_n) * BN;

    // the block's output rows: image rows g0 .. g1 (counted over all images)
    const uint32_t g0 = fdiv(m0, h.div_ow), g1 = fdiv(min(m0 + BM, a.M) - 1, h.div_ow);
    const uint32_t img0 = fdiv(g0, h.div_oh), y0 = g0 - img0 * h.oh, img1 = fdiv(g1, h.div_oh);
    const int halo_r = a.r - 1;
    const int rows0 = (int)min((uint32_t)h.oh - y0, g1 - g0 + 1) + halo_r;                      // patch rows of the first image
    const int prows = (int)(g1 - g0 + 1) + (int)(img1 - img0 + 1) * halo_r;
    const int punits = prows * h.pw * (kHaloK / 16);

    // LDS addresses of the lane's output rows in the patch, tap (0, 0)
    int abase[MB];
#pragma unroll
    for (int j = 0; j < MB; ++j) {
        const uint32_t m = min(m0 + wm * WM + j * 32 + l32, a.M - 1);
        const uint32_t gr = fdiv(m, h.div_ow), x = m - gr * h.ow, im = fdiv(gr, h.div_oh);
        abase[j] = (((int)(gr - g0) + (int)(im - img0) * halo_r) * h.pw + (int)x) * PS + 16 * g;
    }

    const __amdgpu_buffer_rsrc_t ra = make_rsrc(a.act, a.act_bytes), rb = make_rsrc(a.wgt, a.wgt_bytes);
    char *const patch = smem, *const bbuf = smem + h.patches * h.pix * PS;      // one or two patches, two filter stages
    const int taps = a.r * a.s, chunks = h.ch / kHaloK, stages = chunks * taps;

    // unit u of the patch: 16 channels of one pixel.  Beyond the image (and beyond the patch) it loads zeros.
    auto patch_load = [&](int u, int chunk, uint32_t (&r0)[4], uint32_t (&r1)[4]) {
        const uint32_t px = (uint32_t)u >> 2, prow = fdiv(px, h.div_pw), pcol = px - prow * h.pw;
        uint32_t im = img0;
        int iy = (int)(y0 + prow) - h.pr;
        if ((int)prow >= rows0) {
            const uint32_t t = prow - rows0, i = fdiv(t, h.div_ir);
            im += 1 + i;
            iy = (int)(t - i * (uint32_t)(h.oh + halo_r)) - h.pr;
        }
        const int ix = (int)pcol - h.pc;
        const bool ok = u < punits && (unsigned)iy < (unsigned)h.ih && (unsigned)ix < (unsigned)h.iw && chunk < chunks;
        load_unit<EA>(ra, ((im * (uint32_t)h.ih + (uint32_t)iy) * (uint32_t)h.iw + (uint32_t)ix) * (uint32_t)h.ch + chunk * kHaloK + (u & 3) * 16, ok, r0, r1);
    };
    auto patch_store = [&](int u, char *dst, const uint32_t (&r0)[4], const uint32_t (&r1)[4]) {
        if (u >= punits) return;
        uint32_t hi[4], lo[4];
        split_unit<EA, bal_of(AES)>(r0, r1, hi, lo);
        char *p = dst + (u >> 2) * PS + (u & 3) * 16;
        *reinterpret_cast<uint4 *>(p) = make_uint4(hi[0], hi[1], hi[2], hi[3]);
        if (LAL == 2) *reinterpret_cast<uint4 *>(p + kHaloK) = make_uint4(lo[0], lo[1], lo[2], lo[3]);
    };
    // the thread's filter units: forward, 16 codes of a filter row; data gradient, 16 columns of one line
    uint32_t boff[BU];
    bool bok[BU];
    int bdst[BU];
#pragma unroll
    for (int i = 0; i < BU; ++i) {
        const int id = threadIdx.x + i * NT;
        if (W_R) {
            const int line = id / (BN / 16), col = id % (BN / 16) * 16;
            boff[i] = (uint32_t)line * (uint32_t)(taps * a.c) + (uint32_t)(n0 + col);
            bok[i] = n0 + col < a.N;
            bdst[i] = line * BRS + col;
        } else {
            const int row = id >> 2, col = (id & 3) * 16;
            boff[i] = (uint32_t)(n0 + row) * (uint32_t)a.K + (uint32_t)col;
            bok[i] = n0 + row < a.N;
            bdst[i] = row * BRS + col;
        }
    }
    auto b_load = [&](int i, int chunk, int tap, bool on, uint32_t (&r0)[4], uint32_t (&r1)[4]) {
        const uint32_t at = W_R ? (uint32_t)(chunk * kHaloK * taps + (taps - 1 - tap)) * (uint32_t)a.c : (uint32_t)(tap * h.ch + chunk * kHaloK);
        load_unit<EB>(rb, boff[i] + at, bok[i] && on, r0, r1);
    };
    auto b_store = [&](int i, char *dst, const uint32_t (&r0)[4], const uint32_t (&r1)[4]) {
        uint32_t hi[4], lo[4];
        split_unit<EB, bal_of(WES)>(r0, r1, hi, lo);
        *reinterpret_cast<uint4 *>(dst + bdst[i]) = make_uint4(hi[0], hi[1], hi[2], hi[3]);
        if (LBL == 2) *reinterpret_cast<uint4 *>(dst + bdst[i] + B_LO) = make_uint4(lo[0], lo[1], lo[2], lo[3]);
    };

    v16i acc_hh[NB][MB], acc_x[NB][MB], acc_ll[NB][MB];
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int j = 0; j < MB; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) { acc_hh[i][j][r] = 0; acc_x[i][j][r] = 0; acc_ll[i][j][r] = 0; }
    int sum_m[MB], sum_n[NB];
#pragma unroll
    for (int j = 0; j < MB; ++j) sum_m[j] = 0;
#pragma unroll
    for (int i = 0; i < NB; ++i) sum_n[i] = 0;

    // the first chunk's patch and the first stage's filters
    {
        uint32_t b0[BU][4], b1[BU][4];
#pragma unroll
        for (int i = 0; i < BU; ++i) b_load(i, 0, 0, true, b0[i], b1[i]);
        for (int u0 = threadIdx.x; u0 < punits; u0 += 4 * NT) {
            uint32_t r0[4][4], r1[4][4];
#pragma unroll
            for (int v = 0; v < 4; ++v) patch_load(u0 + v * NT, 0, r0[v], r1[v]);
#pragma unroll
            for (int v = 0; v < 4; ++v) patch_store(u0 + v * NT, patch, r0[v], r1[v]);
        }
#pragma unroll
        for (int i = 0; i < BU; ++i) b_store(i, bbuf, b0[i], b1[i]);
    }
    __syncthreads();

    // Eight wavefronts, two per SIMD, in two groups half a sub-step apart: while one group reads its fragments of a sub-step (and
    // writes the next stage's operands), the other multiplies.  Every sub-step is a reading and a multiplying phase with a barrier
    // after each; the second group passes one barrier more before the loop, the first one more after it.
    constexpr bool PP = NT == 512 && BOTH2;
    auto phase_end = [&]() {
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };
    const bool second = PP && __builtin_amdgcn_readfirstlane(wave) >= 4;
    if (second) phase_end();

    int tap = 0, tr = 0, ts = 0, chunk = 0;
    uint32_t b0[BU][4], b1[BU][4], p0[4], p1[4];
    for (int st = 0; st < stages; ++st) {
        const char *const pcur = patch + (chunk & 1) * h.pix * PS;
        char *const pnext = patch + ((chunk + 1) & 1) * h.pix * PS;
        const char *const bcur = bbuf + (st & 1) * BB;
        char *const bnext = bbuf + ((st + 1) & 1) * BB;
        const int toff = (tr * h.pw + ts) * PS;
        const int ntap = tap + 1 == taps ? 0 : tap + 1, nchunk = tap + 1 == taps ? chunk + 1 : chunk;
        // share t of the next chunk's patch is loaded in the second sub-step of tap t and written in the first one of tap t + 1
        const bool pload = tap * NT < punits && chunk + 1 < chunks, pwrite = tap > 0 && (tap - 1) * NT < punits && chunk + 1 < chunks;
#pragma unroll
        for (int ks = 0; ks < kHaloK / 32; ++ks) {
            // the operands of later stages first, so that their registers are free again when the fragments arrive
            if (ks == 0) {
                if (pwrite) patch_store((tap - 1) * NT + (int)threadIdx.x, pnext, p0, p1);
#pragma unroll
                for (int i = 0; i < BU; ++i) b_load(i, nchunk, ntap, st + 1 < stages, b0[i], b1[i]);
            } else {
#pragma unroll
                for (int i = 0; i < BU; ++i) b_store(i, bnext, b0[i], b1[i]);
                if (pload) patch_load(tap * NT + (int)threadIdx.x, chunk + 1, p0, p1);
            }
            __builtin_amdgcn_sched_barrier(0);
            v4i fa_h[MB], fa_l[MB], fb_h, fb_l;
            auto read_b = [&](int i, bool low) {
                const int at = low ? B_LO : 0;
                if constexpr (W_R) {
                    typedef LoaderR<OP_DGRAD, false, BN, LBL, kHaloK, EB, bal_of(WES)> LB;
                    return LB::frag(bcur + at, wn * WN + i * 32, ks, lane);
                } else {
                    return *reinterpret_cast<const v4i *>(bcur + at + (wn * WN + i * 32 + nperm) * BRS + ks * 32 + 16 * g);
                }
            };
#pragma unroll
            for (int j = 0; j < MB; ++j) {
                fa_h[j] = *reinterpret_cast<const v4i *>(pcur + abase[j] + toff + ks * 32);
                if (LAL == 2) fa_l[j] = *reinterpret_cast<const v4i *>(pcur + abase[j] + toff + ks * 32 + kHaloK);
            }
            if (LBL == 2) fb_l = read_b(0, true);
            fb_h = read_b(0, false);
            if (PP) {
                phase_end();
                __builtin_amdgcn_s_setprio(1);
            }
            // The filters' fragments of a 32-column block take the registers of the block before, limb by limb (a second set would
            // not fit beside the accumulators): one limb's products cover the read of the other.
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                // row sums for the offset split, as in contract_body
                if (OFFS && LAL == 2) {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        sum_n[i] += LBL == 2 ? 256 * dot4_ones((uint32_t)fb_h[e]) + dot4_ones((uint32_t)fb_l[e]) : dot4_ones((uint32_t)fb_h[e]);
                }
                if (LBL == 2) {
#pragma unroll
                    for (int j = 0; j < MB; ++j) {
                        acc_x[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fb_l, fa_h[j], acc_x[i][j], 0, 0, 0);
                        if (BOTH2) acc_ll[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fb_l, fa_l[j], acc_ll[i][j], 0, 0, 0);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                    if (i + 1 < NB) fb_l = read_b(i + 1, true);
                    __builtin_amdgcn_sched_barrier(0);
                }
#pragma unroll
                for (int j = 0; j < MB; ++j) {
                    acc_hh[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fb_h, fa_h[j], acc_hh[i][j], 0, 0, 0);
                    if (LAL == 2) acc_x[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fb_h, fa_l[j], acc_x[i][j], 0, 0, 0);
                }
                __builtin_amdgcn_sched_barrier(0);
                if (i + 1 < NB) fb_h = read_b(i + 1, false);
                __builtin_amdgcn_sched_barrier(0);
                if (OFFS && LBL == 2 && i == 0) {
#pragma unroll
                    for (int j = 0; j < MB; ++j)
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            sum_m[j] += LAL == 2 ? 256 * dot4_ones((uint32_t)fa_h[j][e]) + dot4_ones((uint32_t)fa_l[j][e]) : dot4_ones((uint32_t)fa_h[j][e]);
                }
            }
            if (PP) {
                __builtin_amdgcn_s_setprio(0);
                phase_end();
            }
        }
        if (!PP) __syncthreads();
        tap = ntap;
        chunk = nchunk;
        ts = ts + 1 == a.s ? 0 : ts + 1;
        tr = ts != 0 ? tr : tr + 1 == a.r ? 0 : tr + 1;
    }
    if (PP && !second) phase_end();

    int rows[MB];
#pragma unroll
    for (int j = 0; j < MB; ++j) rows[j] = m0 + wm * WM + j * 32 + l32;
    contract_epilogue<LIMBS, LAL, LBL, OFFS, W_R, MB, NB, WGM * WGN, AMAX>(a, acc_hh, acc_x, acc_ll, sum_m, sum_n, smem, rows, n0 + wn * WN,
                                                                          (long long)stages * kHaloK, a.out, lin);
}

template <int OP, int AES, int WES, int TILE, int WGM, int WGN, bool AMAX>
static hipError_t launch_halo_as(adapt_ctx *ctx, const HaloArgs &h)
{
    constexpr int BM = kHaloShape[TILE][0], BN = kHaloShape[TILE][1];
    static_assert(kHaloShape[TILE][2] == 64 * WGM * WGN, "threads of the tile");
    void (*kern)(const HaloArgs) = halo_kernel<OP, AES == 1 && WES == 1 ? 1 : 2, AES, WES, BM, BN, WGM, WGN, AMAX>;
    const size_t lds = halo_lds<OP>(h.a, TILE, h.patches);
    // a launch's LDS depends on the layer: the most that any layer takes is requested
    if (hipError_t e = allow_big_lds(ctx, reinterpret_cast<const void *>(kern), kHaloMaxLds[TILE]); e != hipSuccess) return e;
    const unsigned tiles = (unsigned)((h.a.M + BM - 1) / BM) * (unsigned)((h.a.N + BN - 1) / BN);
    hipLaunchKernelGGL(kern, dim3(tiles), dim3(64 * WGM * WGN), lds, ctx->stream, h);
    note_amax_blocks(ctx, h.a, tiles);
    return hipGetLastError();
}

template <int OP, int AES, int WES, int TILE, int WGM, int WGN>
static hipError_t launch_halo_tile(adapt_ctx *ctx, const HaloArgs &h)
{
    if constexpr (OP == OP_DGRAD)
        if (h.a.amax_part != nullptr) return launch_halo_as<OP, AES, WES, TILE, WGM, WGN, true>(ctx, h);
    return launch_halo_as<OP, AES, WES, TILE, WGM, WGN, false>(ctx, h);
}

template <int OP, int AES, int WES>
static hipError_t launch_halo_modes(adapt_ctx *ctx, const ContractPlan &p)
{
    const ContractArgs &a = p.kern;
    HaloArgs h = {};
    h.a = a;
    if (OP == OP_FWD) {
        h.ih = a.h; h.iw = a.w; h.ch = a.c; h.oh = a.p; h.ow = a.q; h.pr = h.pc = a.pad;
    } else {
        h.ih = a.p; h.iw = a.q; h.ch = a.k; h.oh = a.h; h.ow = a.w; h.pr = a.r - 1 - a.pad; h.pc = a.s - 1 - a.pad;
    }
    h.pw = h.ow + a.s - 1;
    h.pix = halo_pixels(kHaloShape[p.halo][0], h.oh, h.ow, a.r, a.s);
    h.patches = halo_patches<OP>(a);
    h.div_ow = make_fastdiv(h.ow); h.div_oh = make_fastdiv(h.oh); h.div_pw = make_fastdiv(h.pw); h.div_ir = make_fastdiv(h.oh + a.r - 1);
    if constexpr (!(AES == 2 && WES == 2))      // not planned: spills
        if (p.halo == HALO_256x128) return launch_halo_tile<OP, AES, WES, HALO_256x128, 4, 2>(ctx, h);
    return launch_halo_tile<OP, AES, WES, HALO_128x64, 2, 2>(ctx, h);
}

// limb modes of the operands, as launch_variant takes them (two limbs at least in one)
template <int OP>
static hipError_t launch_halo(adapt_ctx *ctx, const ContractPlan &p)
{
    const ContractArgs &a = p.kern;
    if (a.act_es == 2 && a.wgt_es == 2) return a.balanced ? launch_halo_modes<OP, 3, 3>(ctx, p) : launch_halo_modes<OP, 2, 2>(ctx, p);
    if (a.act_es == 2) return a.balanced ? launch_halo_modes<OP, 3, 1>(ctx, p) : launch_halo_modes<OP, 2, 1>(ctx, p);
    return a.balanced ? launch_halo_modes<OP, 1, 3>(ctx, p) : launch_halo_modes<OP, 1, 2>(ctx, p);
}

}  // namespace adapt
