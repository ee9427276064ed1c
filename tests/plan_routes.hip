// Host program (no GPU): reads calls, a line of numbers each (n h w c k r s stride pad, word lengths of dy, w and x), and prints for
// each which kernels a context with enough workspace would take for its weight gradient, alone and together with the data gradient:
//   rows splits positions threads   rows splits positions threads
// rows: on image rows in LDS; positions of the slab sum and the threads that share one, 0 0 where there is none.
#include <stdio.h>

#include "contract_kernel.hpp"

using namespace adapt;

int main()
{
    char *const base = reinterpret_cast<char *>((size_t)1 << 40);
    adapt_ctx ctx = {};
    ctx.num_cu = 256;
    ctx.ws = 5 * ((size_t)1 << 40) + (char *)nullptr;
    const adapt_epilogue ep = {1, {8, 0}, {ADAPT_RN_HALF_UP, 0, 0}, 0};
    adapt_conv_desc d;
    adapt_fmt dy = {0, 4}, w = {0, 4}, x = {0, 4};
    while (scanf("%d %d %d %d %d %d %d %d %d %d %d %d", &d.n, &d.h, &d.w, &d.c, &d.k, &d.r, &d.s, &d.stride, &d.pad, &dy.wl, &w.wl, &x.wl) == 12) {
        for (int which : {(int)GRAD_DW, GRAD_DX | GRAD_DW}) {
            PadJobs pads;
            ContractPlan pd = {}, pw = {};
            if (plan_gradients(&ctx, which, d, base, dy, base, w, base, x, base, ep, base, ep, (size_t)1 << 36, pads, pd, pw) != ADAPT_OK) return 1;
            printf("%d %d %llu %d ", pw.halo, pw.splits, (unsigned long long)(pw.acc ? slab_sum_positions(pw) : 0), pw.acc ? slab_sum_share(pw) : 0);
        }
        printf("\n");
    }
    return 0;
}
