// Weight gradients of stride-1 convolutions with filters three taps wide, on image rows held in LDS.
//
//   dw[kout][r][t][c] = sum over pixels (n, p, q) of dy[n,p,q,kout] * x[n, p + r - pad, q + t - pad, c],   t = 0, 1, 2
//
// The implicit GEMM of contract_kernel.hpp fetches an input pixel once per filter tap, and splits it into limbs every time.  Here a
// block owns one filter row r, 64 output channels and 64 input channels.  A stage is as many whole output rows as fit 128 reduction
// slots: dy's pixels in one LDS buffer and the input rows they meet (with two more columns) in another, split into limbs once; the
// three taps read the same lines, shifted by one.  Slots beyond the stage's pixels hold zeros of dy, so what x they meet does not
// matter.
//
// A wavefront multiplies 32 output channels by 32 input channels for all three taps: nine accumulator sets at two limbs, two
// wavefronts per SIMD.  The eight wavefronts are two groups that take half of a stage's slots each, half a sub-step apart: one group
// reads its fragments while the other multiplies.  The groups are added up at the end, through LDS, each finishing half of the columns.
//
// What it took (256 x 16 x 16 x 128 -> 128, <12,9>, clocks per stage, of which the products alone are 1540): all wavefronts in step 4200;
// in two groups 3200; chunks fetched by neighbouring lanes, advanced offsets instead of divisions 2800; splitting, LDS stores and loads one
// behind each product, where they stand in the matrix unit's shadow (behind every third they do not: 3600), 2640.
#pragma once
#include "contract_kernel.hpp"

namespace adapt {

struct RowsArgs {
    ContractArgs a;              // M, N, pointers, extents, epilogue
    RowsGeometry g;
    int stages_per_split, tiles_c;
    FastDiv div_pw;
};

// RUN8: output rows are whole groups of 8 pixels, so that 8 slots are 8 neighbouring lines: the middle tap's fragment is made of
// the other two's bytes and not read
// SLAB: partial sums to slabs; else the output itself.
template <int AES, int WES, bool RUN8, bool SLAB, bool AMAX>
__global__ void __launch_bounds__(512, 2)
rows_kernel(const RowsArgs h)
{
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const ContractArgs &a = h.a;
    constexpr int NT = 512, BM = kRowsChannels, BC = kRowsChannels, KP = kRowsSlots;
    constexpr int WGM = BM / 32, WGN = BC / 32, WGK = 2, KS = KP / 32 / WGK, TAPS = kRowsTaps;
    constexpr int LAL = limbs_of(AES), LBL = limbs_of(WES), EA = es_of(AES), EB = es_of(WES);
    constexpr bool BOTH2 = LAL == 2 && LBL == 2, OFFS = AES == 2 || WES == 2;
    // bytes of a line, per limb: an odd multiple of 32, so that the eight lines of a transposing read meet different banks
    constexpr int ARB = BM + 32, XRB = BC + 32;
    // Operands are fetched in chunks of 16 bytes, neighbouring lanes neighbouring chunks: 16 clocks of the address unit per load (a lane
    // that takes 32 bytes with two loads makes it 32)
    constexpr int PA = 16 / EA, PX = 16 / EB, CLA = BM / PA, CLX = BC / PX;      // codes of a chunk, chunks of a line
    constexpr int UA = KP * CLA / NT, UX = (kRowsLines * CLX + NT - 1) / NT, U = UX + UA;      // chunks of a stage per thread
    constexpr int LINES = UX * NT / CLX;                                         // lines of x that have room
    static_assert(WGM * WGN * WGK == 8 && UA * NT == KP * CLA && LINES >= kRowsLines && KS == 2, "chunks are dealt evenly");
    constexpr int A_LO = KP * ARB, X_HI = LAL * KP * ARB, X_LO = LINES * XRB, STAGE = X_HI + LBL * LINES * XRB;
    static_assert(2 * STAGE <= (int)rows_lds(LAL, LBL), "two stages");
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l32 = lane & 31, g = lane >> 5;
    const int wk = wave / (WGM * WGN), wm = wave / WGN % WGM, wn = wave % WGN;

    // as in contract_body: a contiguous range of (split, tile) per XCD
    const unsigned lin = blockIdx.y * gridDim.x + blockIdx.x, nwg = gridDim.x * gridDim.y;
    const unsigned per_xcd = nwg / kXcds, extra = nwg % kXcds, xcd = lin % kXcds;
    const unsigned vid = xcd * per_xcd + min(xcd, extra) + lin / kXcds;
    const int split = vid / gridDim.x, tile = vid % gridDim.x;
    const int tm = tile / (h.tiles_c * a.r), r = tile / h.tiles_c % a.r, tc = tile % h.tiles_c;
    const int m0 = tm * BM, c0 = tc * BC;
    const int first = split * h.stages_per_split, last = min(first + h.stages_per_split, h.g.stages);

    const __amdgpu_buffer_rsrc_t ra = make_rsrc(a.act, a.act_bytes), rx = make_rsrc(a.wgt, a.wgt_bytes);
    const int a_slot = threadIdx.x / CLA, a_col = m0 + threadIdx.x % CLA * PA;       // chunk i of dy: slot a_slot + i * NT / CLA
    const int x_line = threadIdx.x / CLX, x_ch = c0 + threadIdx.x % CLX * PX;        // chunk i of x: line x_line + i * NT / CLX
    const int wave_line = __builtin_amdgcn_readfirstlane(x_line);
    // Byte offsets of the chunks, advanced from stage to stage: the loads stand between the products, where every instruction counts.
    // dy: the descriptor's extent ends the reduction.  x: the chunk's row of the image moves on by step_p, over into the next image
    // where it passes the last output row.
    uint32_t a_off[UA], x_off[UX];
    int x_p[UX];                                            // output row of the chunk's line in its image; lines that are never read: none
    const uint32_t a_step = (uint32_t)h.g.slots * (uint32_t)a.k * EA;
    const int step_p = h.g.rps % a.p;
    const uint32_t row_bytes = (uint32_t)a.w * (uint32_t)a.c * EB;
    const uint32_t x_step = ((uint32_t)(h.g.rps / a.p) * (uint32_t)a.h + (uint32_t)step_p) * row_bytes, x_wrap = (uint32_t)(a.h - a.p) * row_bytes;
    constexpr uint32_t NOWHERE = 0xfffffff0u;
    bool a_ok[UA];
#pragma unroll
    for (int i = 0; i < UA; ++i) {
        const int slot = a_slot + i * (NT / CLA);
        a_ok[i] = slot < h.g.slots && a_col < a.M;
        a_off[i] = ((uint32_t)(first * h.g.slots + slot) * (uint32_t)a.k + (uint32_t)a_col) * EA;
    }
#pragma unroll
    for (int i = 0; i < UX; ++i) {
        const int line = x_line + i * (NT / CLX), lrow = (int)fdiv(line, h.div_pw), col = line - lrow * h.g.pw - a.pad;
        const int row = first * h.g.rps + lrow, im = (int)fdiv(row, a.div_p), p = row - im * a.p;
        const bool ok = line < h.g.lines && (unsigned)col < (unsigned)a.w && x_ch < a.c;
        x_p[i] = ok ? p : INT_MIN / 2;                      // far below any image: it grows by less than the rows of all images
        x_off[i] = (((uint32_t)(im * a.h + p + r - a.pad) * (uint32_t)a.w + (uint32_t)col) * (uint32_t)a.c + (uint32_t)x_ch) * EB;
    }
    v4u av[UA], xv[UX];                                     // one stage in flight, as it lies in memory
    // loads are called for consecutive stages; no lane and no wavefront leaves one out, so that the waits count exactly
    auto load_a = [&](int i) {
        av[i] = __builtin_amdgcn_raw_buffer_load_b128(ra, a_ok[i] ? a_off[i] : NOWHERE, 0, 0);
        a_off[i] += a_step;
    };
    auto load_x = [&](int i) {
        const bool ok = (unsigned)(x_p[i] + r - a.pad) < (unsigned)a.h;
        xv[i] = __builtin_amdgcn_raw_buffer_load_b128(rx, ok ? x_off[i] : NOWHERE, 0, 0);
        const int p = x_p[i] + step_p;
        const bool over = p >= a.p;
        x_p[i] = p - (over ? a.p : 0);
        x_off[i] += x_step + (over ? x_wrap : 0u);
    };
    auto store_a = [&](char *buf, int i) {
        store_limbs<AES>(av[i], buf + (a_slot + i * (NT / CLA)) * ARB + threadIdx.x % CLA * PA, A_LO);
    };
    auto store_x = [&](char *buf, int i) {
        if (wave_line + i * (NT / CLX) < h.g.lines)
            store_limbs<WES>(xv[i], buf + X_HI + (x_line + i * (NT / CLX)) * XRB + threadIdx.x % CLX * PX, X_LO);
    };
    auto load = [&](int i) { if (i < UX) load_x(i); else load_a(i - UX); };
    auto store = [&](char *buf, int i) { if (i < UX) store_x(buf, i); else store_a(buf, i - UX); };

    // Fragments: as LoaderR::frag; lane 2j + b of a group of 16 points at 8 channels of slot j, twice (slots 0..7 and 8..15)
    const int grp = lane >> 4, fk = wk * KS * 32 + 16 * (grp >> 1) + ((lane & 15) >> 1), fc = 16 * (grp & 1) + 8 * (lane & 1);
    const int fa = fk * ARB + wm * 32 + fc;
    int fx[KS][2];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const int slot = min(fk + ks * 32 + e * 8, h.g.slots - 1);
            const int row = (int)fdiv(slot, a.div_q);
            fx[ks][e] = X_HI + (row * h.g.pw + slot - row * a.q) * XRB + wn * 32 + fc;
        }
    typedef v2i __attribute__((address_space(3))) * lds_v2i;
    auto tr8 = [&](const char *p) { return __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_v2i)p); };

    v16i acc_hh[TAPS][1], acc_x[TAPS][1], acc_ll[TAPS][1];
#pragma unroll
    for (int t = 0; t < TAPS; ++t)
#pragma unroll
        for (int e = 0; e < 16; ++e) { acc_hh[t][0][e] = 0; acc_x[t][0][e] = 0; acc_ll[t][0][e] = 0; }
    int sum_m[1] = {0}, sum_n[TAPS] = {0, 0, 0};

    auto barrier = [&]() {       // LDS only: the loads in flight are not waited for
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };
#pragma unroll
    for (int i = 0; i < UX + UA; ++i) load(i);
#pragma unroll
    for (int i = 0; i < UX + UA; ++i) store(smem, i);
#pragma unroll
    for (int i = 0; i < UX + UA; ++i) load(i);
    barrier();
    // Two groups of four wavefronts, one per SIMD each, half a sub-step apart (as in contract_halo.hpp): while one group reads its
    // fragments and writes its share of the next stage, the other multiplies; a barrier after each phase.
    const bool second = __builtin_amdgcn_readfirstlane(wave) >= 4;
    if (second) barrier();
    for (int st = first; st < last; ++st) {
        const char *const cur = smem + ((st - first) & 1) * STAGE;
        char *const next = smem + ((st - first + 1) & 1) * STAGE;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            v4i ah, al, xh[TAPS], xl[TAPS];
            auto read_a = [&](int lo, v4i &f) {
                const v2i u = tr8(cur + lo + fa + ks * 32 * ARB), v = tr8(cur + lo + fa + (ks * 32 + 8) * ARB);
                f[0] = u[0]; f[1] = u[1]; f[2] = v[0]; f[3] = v[1];
            };
            auto read_x = [&](int lo, v4i (&f)[TAPS]) {
#pragma unroll
                for (int e = 0; e < 2; ++e)
#pragma unroll
                    for (int t = 0; t < TAPS; ++t) {
                        if (RUN8 && t == 1) continue;
                        const v2i u = tr8(cur + lo + fx[ks][e] + t * XRB);
                        f[t][2 * e] = u[0]; f[t][2 * e + 1] = u[1];
                    }
            };
            // lines 1..8 out of lines 0..7 and 2..9
            auto middle = [&](v4i (&f)[TAPS]) {
                if (!RUN8) return;
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    f[1][2 * e] = (int)__builtin_amdgcn_alignbyte((uint32_t)f[0][2 * e + 1], (uint32_t)f[0][2 * e], 1);
                    f[1][2 * e + 1] = (int)__builtin_amdgcn_perm((uint32_t)f[2][2 * e + 1], (uint32_t)f[0][2 * e + 1], 0x06030201u);
                }
            };
            read_a(0, ah);
            read_x(0, xh);
            if (LAL == 2) read_a(A_LO, al);
            if (LBL == 2) read_x(X_LO, xl);
            barrier();
            __builtin_amdgcn_s_setprio(1);
            // The multiplying phase.  Behind each product, in the matrix unit's shadow, one of: a chunk of the next stage is split and
            // written (all in the first sub-step: the other group reads them a phase after its second), then the loads for the registers
            // that this has freed are issued, one each; they have a whole stage's time.
            constexpr int PRODUCTS = TAPS * (BOTH2 ? 4 : 2);
            static_assert(U <= PRODUCTS && 2 * U <= KS * PRODUCTS, "a product for each");
            auto behind = [&](int n) {
                n += ks * PRODUCTS;
                __builtin_amdgcn_sched_barrier(0);
                if (n < U) store(next, n);
                else if (n < 2 * U) load(n - U);
                __builtin_amdgcn_sched_barrier(0);
            };
            // row sums for the offset split, as in contract_body
            auto sums_n = [&](int t) {
                if (OFFS && LAL == 2) {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        sum_n[t] += LBL == 2 ? 256 * dot4_ones((uint32_t)xh[t][e]) + dot4_ones((uint32_t)xl[t][e]) : dot4_ones((uint32_t)xh[t][e]);
                }
            };
            auto sums_m = [&]() {
                if (OFFS && LBL == 2) {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        sum_m[0] += LAL == 2 ? 256 * dot4_ones((uint32_t)ah[e]) + dot4_ones((uint32_t)al[e]) : dot4_ones((uint32_t)ah[e]);
                }
            };
            constexpr int order[TAPS] = {0, 2, 1};      // the middle tap last, its fragment is still to be made
#pragma unroll
            for (int k = 0; k < TAPS; ++k) {
                const int t = order[k];
                acc_hh[t][0] = __builtin_amdgcn_mfma_i32_32x32x32_i8(xh[t], ah, acc_hh[t][0], 0, 0, 0);
                if (k == 0) middle(xh);
                if (k == 1) sums_m();
                behind(k);
            }
            if (LAL == 2) {
#pragma unroll
                for (int k = 0; k < TAPS; ++k) {
                    const int t = order[k];
                    acc_x[t][0] = __builtin_amdgcn_mfma_i32_32x32x32_i8(xh[t], al, acc_x[t][0], 0, 0, 0);
                    if (k == 0 && LBL == 2) middle(xl);
                    if (LBL == 1) sums_n(t);
                    behind(TAPS + k);
                }
            }
            if (LBL == 2) {
                if (LAL == 1) middle(xl);
#pragma unroll
                for (int k = 0; k < TAPS; ++k) {
                    const int t = order[k];
                    acc_x[t][0] = __builtin_amdgcn_mfma_i32_32x32x32_i8(xl[t], ah, acc_x[t][0], 0, 0, 0);
                    behind(TAPS * (LAL == 2 ? 2 : 1) + k);
                }
                if (LAL == 2) {
#pragma unroll
                    for (int k = 0; k < TAPS; ++k) {
                        const int t = order[k];
                        acc_ll[t][0] = __builtin_amdgcn_mfma_i32_32x32x32_i8(xl[t], al, acc_ll[t][0], 0, 0, 0);
                        sums_n(t);
                        behind(TAPS * 3 + k);
                    }
                }
            }
            __builtin_amdgcn_s_setprio(0);
            barrier();
        }
    }
    if (!second) barrier();

    constexpr int SETS = BOTH2 ? 3 : LAL == 2 || LBL == 2 ? 2 : 1;
    // element e of accumulator set k of tap t
    auto acc = [&](int t, int k, int e) -> int { return k == 0 ? acc_hh[t][0][e] : k == 1 ? acc_x[t][0][e] : acc_ll[t][0][e]; };
    auto add = [&](int t, int k, int e, int v) {
        if (k == 0) acc_hh[t][0][e] += v;
        else if (k == 1) acc_x[t][0][e] += v;
        else acc_ll[t][0][e] += v;
    };
    // The first group finishes elements 0..7 of each set (columns 0..15 of a 32-column block), the second 8..15; the others travel.
    // (The output itself: all to the first group.)
    int *const x = reinterpret_cast<int *>(smem) + threadIdx.x, *const y = reinterpret_cast<int *>(smem) + (threadIdx.x ^ 256);
    if (SLAB) {
#pragma unroll
        for (int t = 0; t < TAPS; ++t) {
#pragma unroll
            for (int k = 0; k < SETS; ++k)
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const int v0 = acc(t, k, e), v1 = acc(t, k, 8 + e);      // (loads in the arms of a conditional would keep the sets in memory)
                    x[((t * SETS + k) * 8 + e) * NT] = wk == 0 ? v1 : v0;
                }
            if (OFFS) x[(TAPS * SETS * 8 + t) * NT] = sum_n[t];
        }
        if (OFFS) x[(TAPS * SETS * 8 + TAPS) * NT] = sum_m[0];
        __syncthreads();
        // slab layout: [32 output channels][column][output channel of the 32], so that a wavefront's stores are whole lines
        const size_t block = (size_t)((m0 + wm * 32) / 32) * (size_t)a.N * 32;
        const int ncol = r * TAPS * a.c + c0 + wn * 32;
        char *const slab = static_cast<char *>(a.out) + (long long)split * a.slab_bytes;
        const bool in = m0 + wm * 32 < a.M && c0 + wn * 32 + 16 * wk < a.c;
        long long corr_m = 0;
        if (OFFS) {
            const int m = sum_m[0] + y[(TAPS * SETS * 8 + TAPS) * NT];
            corr_m = m + __shfl_xor(m, 32, 64);
        }
#pragma unroll
        for (int t = 0; t < TAPS; ++t) {
            int n_sum = 0;                                // of column l32
            if (OFFS) {
                n_sum = sum_n[t] + y[(TAPS * SETS * 8 + t) * NT];
                n_sum += __shfl_xor(n_sum, 32, 64);
            }
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                int u[SETS];
#pragma unroll
                for (int k = 0; k < SETS; ++k) {
                    const int v0 = acc(t, k, e), v1 = acc(t, k, 8 + e);
                    u[k] = (wk == 0 ? v0 : v1) + y[((t * SETS + k) * 8 + e) * NT];
                }
                const int nl = 16 * wk + 8 * (e >> 2) + 4 * g + (e & 3);
                long long v = u[0];
                if (BOTH2) v = (v << 16) + ((long long)u[1] << 8) + (long long)u[SETS - 1];
                else if (SETS == 2) v = (v << 8) + (long long)u[1];
                if (OFFS) {
                    // as in contract_epilogue
                    const long long s_n = LAL == 2 ? __shfl(n_sum, nl, 64) : 0;
                    v += BOTH2 ? 128 * (corr_m + s_n) + 16384ll * (last - first) * KP : 128 * (LBL == 2 ? corr_m : s_n);
                }
                const size_t at = block + (size_t)(ncol + t * a.c + nl) * 32 + l32;
                if (in) {
                    if (a.out_mode == OUT_RAW32) reinterpret_cast<int32_t *>(slab)[at] = (int32_t)v;
                    else reinterpret_cast<long long *>(slab)[at] = v;
                }
            }
        }
    } else {
        if (wk == 1) {
#pragma unroll
            for (int t = 0; t < TAPS; ++t) {
#pragma unroll
                for (int k = 0; k < SETS; ++k)
#pragma unroll
                    for (int e = 0; e < 16; ++e) y[((t * SETS + k) * 16 + e) * 256] = acc(t, k, e);
                if (OFFS) y[(TAPS * SETS * 16 + t) * 256] = sum_n[t];
            }
            if (OFFS) y[(TAPS * SETS * 16 + TAPS) * 256] = sum_m[0];
        }
        __syncthreads();
        if (wk == 0) {
#pragma unroll
            for (int t = 0; t < TAPS; ++t) {
#pragma unroll
                for (int k = 0; k < SETS; ++k)
#pragma unroll
                    for (int e = 0; e < 16; ++e) add(t, k, e, x[((t * SETS + k) * 16 + e) * 256]);
                if (OFFS) sum_n[t] += x[(TAPS * SETS * 16 + t) * 256];
            }
            if (OFFS) sum_m[0] += x[(TAPS * SETS * 16 + TAPS) * 256];
        }
        __syncthreads();
        const bool in = wk == 0 && c0 + wn * 32 + 16 * g < a.c;      // the lane's run of 16 columns
        const int lane_rows[1] = {in ? m0 + wm * 32 + l32 : a.M};
        contract_epilogue<LAL == 2 || LBL == 2 ? 2 : 1, LAL, LBL, OFFS, true, 1, TAPS, 8, AMAX>(
            a, acc_hh, acc_x, acc_ll, sum_m, sum_n, smem, lane_rows, r * TAPS * a.c + c0 + wn * 32, (long long)(last - first) * KP, a.out, lin, a.c);
    }
}

template <int AES, int WES, bool RUN8, bool SLAB, bool AMAX>
static hipError_t launch_rows_as(adapt_ctx *ctx, const RowsArgs &h, unsigned tiles, unsigned splits)
{
    void (*kern)(const RowsArgs) = rows_kernel<AES, WES, RUN8, SLAB, AMAX>;
    const size_t lds = rows_lds(limbs_of(AES), limbs_of(WES));
    if (hipError_t e = allow_big_lds(ctx, reinterpret_cast<const void *>(kern), lds); e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3(tiles, splits), dim3(512), lds, ctx->stream, h);
    note_amax_blocks(ctx, h.a, (long long)tiles * splits);
    return hipGetLastError();
}

template <int AES, int WES>
static hipError_t launch_rows_modes(adapt_ctx *ctx, const ContractPlan &p)
{
    RowsArgs h = {};
    h.a = p.kern;
    h.g = rows_geometry(h.a);
    h.stages_per_split = h.a.k_per_split;
    h.tiles_c = (h.a.c + kRowsChannels - 1) / kRowsChannels;
    h.div_pw = make_fastdiv(h.g.pw);
    const unsigned tiles = (unsigned)rows_tiles(h.a), splits = (unsigned)p.splits;
    const bool run8 = h.a.q % 8 == 0;
    if (h.a.slab_rows) return run8 ? launch_rows_as<AES, WES, true, true, false>(ctx, h, tiles, splits) : launch_rows_as<AES, WES, false, true, false>(ctx, h, tiles, splits);
    if (h.a.amax_part != nullptr) return run8 ? launch_rows_as<AES, WES, true, false, true>(ctx, h, tiles, splits) : launch_rows_as<AES, WES, false, false, true>(ctx, h, tiles, splits);
    return run8 ? launch_rows_as<AES, WES, true, false, false>(ctx, h, tiles, splits) : launch_rows_as<AES, WES, false, false, false>(ctx, h, tiles, splits);
}

}  // namespace adapt
