// Host program (no GPU): plans contractions of random geometries, formats and workspace sizes and checks that what the planned
// kernels may read lies inside the tensor or the copy that they read.
//   vector loads     read through a buffer descriptor: its extent has to end inside the operand
//   gathered codes   are read by address: the largest offset that the gather forms has to lie inside the operand
// Prints one line per violation; the exit status says whether there was one.
#include <stdio.h>

#include <random>

#include "contract_kernel.hpp"

using namespace adapt;

namespace {

constexpr size_t kFar = (size_t)1 << 40;      // distance of the made-up operand addresses
char *const kA = reinterpret_cast<char *>(kFar), *const kB = reinterpret_cast<char *>(2 * kFar), *const kC = reinterpret_cast<char *>(3 * kFar),
           *const kWorkspace = reinterpret_cast<char *>(5 * kFar);
struct Operand { const void *at; uint64_t bytes; };
int failures = 0, gathers = 0, copies = 0, rows = 0, rows_slabs = 0;

uint64_t bytes_at(const void *p, const Operand *ops, int count, const PadJobs &pads)
{
    for (int i = 0; i < pads.count; ++i)
        if (pads.job[i].dst == p) return (uint64_t)pads.job[i].chunks * 16;
    for (int i = 0; i < count; ++i)
        if (ops[i].at == p) return ops[i].bytes;
    return 0;
}

// codes up to the last one that the element-wise gather of `OP` reads: act_offset / wgt_offset at their largest arguments
template <int OP> uint64_t act_end(const ContractArgs &a)
{
    if (OP == OP_GEMM) return (uint64_t)(a.M - 1) * a.act_rs + (uint64_t)(a.K - 1) * a.act_ks + 1;
    if (OP == OP_FWD) return (uint64_t)a.n * a.h * a.w * a.c;
    if (OP == OP_DGRAD) return (uint64_t)a.n * a.p * a.q * a.k;
    return (uint64_t)(a.K - 1) * a.k + a.M;
}
template <int OP> uint64_t wgt_end(const ContractArgs &a)
{
    if (OP == OP_GEMM) return (uint64_t)(a.N - 1) * a.wgt_rs + (uint64_t)(a.K - 1) * a.wgt_ks + 1;
    if (OP == OP_FWD) return (uint64_t)a.N * a.K;
    if (OP == OP_DGRAD) return ((uint64_t)a.k * a.r * a.s - 1) * a.c + a.N;
    return (uint64_t)a.n * a.h * a.w * a.c;
}

void fail(const char *what, const char *why, uint64_t reads, uint64_t has)
{
    ++failures;
    printf("%s: %s %llu of %llu bytes\n", what, why, (unsigned long long)reads, (unsigned long long)has);
}

// the copies: source rows inside their tensor, copies inside the workspace
void check_copies(const Operand *ops, int count, const PadJobs &pads, size_t limit, const char *what)
{
    for (int i = 0; i < pads.count; ++i) {
        const PadJob &j = pads.job[i];
        const uint64_t reads = (j.chunks / j.cpr - 1) * j.stride + j.row_bytes, has = bytes_at(j.src, ops, count, PadJobs{});
        if (reads > has || j.row_bytes > j.cpr * 16) fail(what, "copy reads", reads, has);
        const uint64_t end = (uint64_t)(static_cast<char *>(j.dst) - (kWorkspace + kCtlBytes)) + (uint64_t)j.chunks * 16;
        if (end > limit) fail(what, "copy ends at", end, limit);
    }
    copies += pads.count;
}

template <int OP> void check(const ContractPlan &p, const Operand *ops, int count, const PadJobs &pads, size_t limit, const char *what)
{
    if (p.empty) return;
    const ContractArgs &a = p.kern;
    // as launch_modes chooses
    const bool gather_act = OP == OP_DGRAD ? a.act_load == LOAD_SCALAR : a.act_load == LOAD_SCALAR || a.wgt_load == LOAD_SCALAR;
    const bool gather_wgt = a.act_load == LOAD_SCALAR || a.wgt_load == LOAD_SCALAR;
    const uint64_t act = gather_act ? act_end<OP>(a) * a.act_es : a.act_bytes, act_has = bytes_at(a.act, ops, count, pads);
    const uint64_t wgt = gather_wgt ? wgt_end<OP>(a) * a.wgt_es : a.wgt_bytes, wgt_has = bytes_at(a.wgt, ops, count, pads);
    gathers += gather_act || gather_wgt;
    if (act > act_has) fail(what, "left operand", act, act_has);
    if (wgt > wgt_has) fail(what, "right operand", wgt, wgt_has);
    if (p.acc == nullptr) return;
    const char *slabs_end = p.acc + (uint64_t)a.slab_bytes * p.splits;
    if (slabs_end > kWorkspace + kCtlBytes + limit) fail(what, "slabs end at", (uint64_t)(slabs_end - kWorkspace) - kCtlBytes, limit);
    for (int i = 0; i < pads.count; ++i)
        if (p.acc < static_cast<char *>(pads.job[i].dst) + (uint64_t)pads.job[i].chunks * 16) fail(what, "slabs over a copy", 0, 0);
}

}  // namespace

int main()
{
    adapt_ctx ctx = {};
    ctx.num_cu = 256;
    ctx.ws = kWorkspace;
    std::mt19937 rng(1);
    auto pick = [&](int lo, int hi) { return lo + (int)(rng() % (unsigned)(hi - lo + 1)); };
    const adapt_epilogue exact = {1, {8, 0}, {ADAPT_RN_HALF_UP, 0, 0}, 0}, requant = {0, {8, 4}, {ADAPT_SR, 1, 2}, 0};
    char what[256];
    for (int t = 0; t < 40000; ++t) {
        const size_t limit = (size_t)1 << pick(8, t % 16 == 2 ? 32 : 28);
        const adapt_fmt f[3] = {{pick(2, 16), 4}, {pick(2, 16), 4}, {pick(2, 16), 4}};
        const adapt_epilogue ep = pick(0, 1) ? exact : requant;
        PadJobs pads;
        ContractPlan p = {}, pw = {};
        if (t % 4 == 0) {
            const int ta = pick(0, 1), tb = pick(0, 1), m = pick(1, 300), n = pick(1, 300), k = pick(1, 300);
            const int lda = (ta ? m : k) + pick(0, 1) * pick(0, 20), ldb = (tb ? k : n) + pick(0, 1) * pick(0, 20);
            const Operand ops[2] = {{kA, ((uint64_t)((ta ? k : m) - 1) * lda + (ta ? m : k)) * storage_bytes(f[0])},
                                    {kB, ((uint64_t)((tb ? n : k) - 1) * ldb + (tb ? k : n)) * storage_bytes(f[1])}};
            if (plan_gemm(&ctx, ta, tb, m, n, k, kA, f[0], lda, kB, f[1], ldb, kC, n, ep, limit, pads, p) != ADAPT_OK) continue;
            snprintf(what, sizeof what, "gemm %d%d %dx%dx%d ld %d %d, %d and %d bits, scratch %zu", ta, tb, m, n, k, lda, ldb, f[0].wl, f[1].wl, limit);
            check_copies(ops, 2, pads, limit, what);
            check<OP_GEMM>(p, ops, 2, pads, limit, what);
            continue;
        }
        adapt_conv_desc d = {};
        d.n = pick(1, 40); d.h = pick(1, 20); d.w = pick(1, 20); d.c = pick(1, 130); d.k = pick(1, 130);
        if (pick(0, 2) == 0) d.c = (d.c + 15) / 16 * 16;
        if (pick(0, 2) == 0) d.k = (d.k + 15) / 16 * 16;
        d.r = pick(1, 7); d.s = pick(1, 7); d.stride = pick(1, 3); d.pad = pick(0, 3);
        if (t % 16 == 2) {      // weight gradients on image rows: fuller tiles, longer reductions
            const int wide = pick(0, 2) == 0 ? 350 : 0;      // enough tiles for one split each
            d.n *= wide ? 1 : pick(1, 60);
            d.w = pick(4, 40); d.c = d.c % 8 * 16 + pick(32, 80) + wide; d.k = d.k % 8 * 16 + pick(32, 80) + wide;
            d.r = pick(0, 1) ? 3 : pick(1, 5); d.s = 3; d.stride = 1; d.pad = pick(0, 2);
        }
        if (!conv_ok(d)) continue;
        const uint64_t dy = (uint64_t)d.n * ((d.h + 2 * d.pad - d.r) / d.stride + 1) * ((d.w + 2 * d.pad - d.s) / d.stride + 1) * d.k;
        const uint64_t x = (uint64_t)d.n * d.h * d.w * d.c, w = (uint64_t)d.k * d.r * d.s * d.c;
        snprintf(what, sizeof what, "%dx%dx%dx%d->%d %dx%d stride %d pad %d, %d, %d and %d bits, scratch %zu, call %d", d.n, d.h, d.w, d.c, d.k, d.r, d.s,
                 d.stride, d.pad, f[0].wl, f[1].wl, f[2].wl, limit, t % 4);
        if (t % 4 == 1) {
            const Operand ops[2] = {{kA, x * storage_bytes(f[0])}, {kB, w * storage_bytes(f[1])}};
            if (plan_fwd(&ctx, d, kA, f[0], kB, f[1], kC, ep, limit, pads, p) != ADAPT_OK) continue;
            check_copies(ops, 2, pads, limit, what);
            check<OP_FWD>(p, ops, 2, pads, limit, what);
            continue;
        }
        const int which = pick(GRAD_DX, GRAD_DX | GRAD_DW);
        const Operand ops[3] = {{kA, dy * storage_bytes(f[0])}, {kB, w * storage_bytes(f[1])}, {kC, x * storage_bytes(f[2])}};
        if (plan_gradients(&ctx, which, d, kA, f[0], kB, f[1], kC, f[2], kC + kFar / 2, ep, kC + kFar / 4, ep, limit, pads, p, pw) != ADAPT_OK) continue;
        check_copies(ops, 3, pads, limit, what);
        if (which & GRAD_DX) check<OP_DGRAD>(p, ops, 3, pads, limit, what);
        if (which & GRAD_DW) check<OP_WGRAD>(pw, ops, 3, pads, limit, what);
        if (which & GRAD_DW && pw.halo) {
            ++rows;
            rows_slabs += pw.acc != nullptr;
        }
    }
    printf("%d failures, %d plans with gathered operands, %d copies, %d on image rows, %d of them with slabs\n", failures, gathers, copies, rows, rows_slabs);
    return failures != 0 || gathers == 0 || copies == 0 || rows_slabs < 100 || rows == rows_slabs;
}
