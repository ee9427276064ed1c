// C entry point of the gemm contraction (the kernel template lives in contract_kernel.hpp), and the copies of all contractions'
// operands whose rows are not whole 16-byte groups
#include "contract_kernel.hpp"

using namespace adapt;

namespace adapt {

// One launch for all copies of a call.  A chunk's 16 source bytes start at any byte: five aligned words around them are loaded
// (only words that hold a byte of the row) and shifted.
__global__ void __launch_bounds__(256) pad_rows_kernel(const PadJobs jobs)
{
    const PadJob &j = jobs.job[(int)(jobs.count > 1 && blockIdx.x >= jobs.job[1].first) + (int)(jobs.count > 2 && blockIdx.x >= jobs.job[2].first)];
    const uint32_t i = (blockIdx.x - j.first) * kPadChunksPerBlock + threadIdx.x;
    if (i >= j.chunks) return;
    const uint32_t r = fdiv(i, j.div_cpr), at = (i - r * j.cpr) * 16;
    const int valid = min(16, (int)j.row_bytes - (int)at);      // bytes of the row in this chunk (none: 0 or less)
    const uint64_t addr = (uint64_t)j.src + (uint64_t)r * j.stride + at;
    const uint32_t *p = reinterpret_cast<const uint32_t *>(addr & ~3ull);
    const int sh = (int)(addr & 3);
    uint32_t w[5], o[4];
#pragma unroll
    for (int k = 0; k < 5; ++k) w[k] = 4 * k - sh < valid ? p[k] : 0u;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int left = valid - 4 * k;
        const uint32_t v = __builtin_amdgcn_alignbyte(w[k + 1], w[k], (uint32_t)sh);
        o[k] = left >= 4 ? v : left <= 0 ? 0u : v & ((1u << (8 * left)) - 1u);
    }
    reinterpret_cast<uint4 *>(j.dst)[i] = make_uint4(o[0], o[1], o[2], o[3]);
}

hipError_t launch_pads(adapt_ctx *ctx, const PadJobs &jobs)
{
    if (jobs.blocks == 0) return hipSuccess;
    hipLaunchKernelGGL(pad_rows_kernel, dim3(jobs.blocks), dim3(256), 0, ctx->stream, jobs);
    return hipGetLastError();
}

}  // namespace adapt

extern "C" int adapt_fxp_gemm(adapt_ctx *ctx, int transA, int transB, int M, int N, int K, const void *A, adapt_fmt fa,
                              int lda, const void *B, adapt_fmt fb, int ldb, void *C, int ldc, adapt_epilogue ep)
{
    if (ctx && wants_wide(fa, fb, ep)) {
        if (M < 0 || N < 0 || K < 0) return ADAPT_EINVAL;
        if (M == 0 || N == 0) return ADAPT_OK;
        if (!C || !aligned16(C) || (K > 0 && (!A || !B || !aligned16(A) || !aligned16(B)))) return ADAPT_EINVAL;
        if (lda < (transA ? M : K) || ldb < (transB ? K : N)) return ADAPT_EINVAL;
        if (ldc != N || K == 0) return ADAPT_EUNSUPPORTED;
        const SubContraction sub = [&](const void *pa, adapt_fmt fpa, const void *pb, adapt_fmt fpb, void *c, adapt_epilogue ex) {
            return adapt_fxp_gemm(ctx, transA, transB, M, N, K, pa, fpa, lda, pb, fpb, ldb, c, N, ex);
        };
        return wide_contraction(ctx, A, fa, (uint64_t)(transA ? K : M) * lda, B, fb, (uint64_t)(transB ? N : K) * ldb, (uint64_t)M * N, K, C,
                                ep, sub);
    }
    if (!ctx || !fmt_ok(fa) || !fmt_ok(fb) || M < 0 || N < 0 || K < 0) return ADAPT_EINVAL;
    if (M == 0 || N == 0) return ADAPT_OK;
    if (!C || !aligned16(C) || ldc < N) return ADAPT_EINVAL;
    if (K > 0 && (!A || !B || !aligned16(A) || !aligned16(B))) return ADAPT_EINVAL;
    if (lda < (transA ? M : K) || ldb < (transB ? K : N)) return ADAPT_EINVAL;
    // the kernels index every tensor with 32-bit element offsets
    if ((long long)(transA ? K : M) * lda * storage_bytes(fa) >= (1ll << 32) || (long long)(transB ? N : K) * ldb * storage_bytes(fb) >= (1ll << 32))
        return ADAPT_EUNSUPPORTED;
    PadJobs pads;
    ContractPlan p;
    if (int s = plan_gemm(ctx, transA, transB, M, N, K, A, fa, lda, B, fb, ldb, C, ldc, ep, scratch_bytes(ctx), pads, p)) return s;
    hipError_t e = launch_pads(ctx, pads);
    if (e == hipSuccess) e = launch_and_finish(ctx, p, launch_planned<OP_GEMM>);
    return hip_status(ctx, e);
}
