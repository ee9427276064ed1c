// Operand tiles that go from memory straight to LDS (wide_planes.hip).
//
// A stage is 64 reduction indices of an operand as they lie in memory.  It is fetched with 16-byte loads whose
// destination is LDS: no staging registers, no LDS stores.  Such a load writes 64 x 16 consecutive bytes per wavefront, so
// tiles have no padding; bank conflicts are avoided by permuting which 16-byte chunk a lane fetches: chunk c of row r
// lies at position c ^ swizzle(r).
//
// LDS fragment reads are written in assembly, the wait for them in the same statement: the compiler would otherwise wait
// for every outstanding load to LDS before each of them.
//
// (A main loop of this kind for the two-limb kernels, which fetched int16 codes and split them into limbs between LDS and the
// matrix units, measured within 15 % of the kernels of contract_kernel.hpp either way: there a wavefront's splitting, LDS
// reads and products follow one another, and splitting in every wavefront that reads a fragment doubles that work.  Two limbs
// split beforehand, as the byte planes here are, have not been measured.)
#pragma once
#include "contract_kernel.hpp"

namespace adapt {

typedef __attribute__((address_space(3))) char lds_char;
__device__ __forceinline__ uint32_t lds_address(const char *p) { return (uint32_t)(uintptr_t)(const lds_char *)p; }

// 64 lanes x 16 bytes from per-lane offsets of the buffer (plus a uniform one) to consecutive LDS bytes starting at lds (uniform)
__device__ __forceinline__ void load_to_lds(__amdgpu_buffer_rsrc_t rsrc, uint32_t lds, uint32_t byte_off, uint32_t uniform_off)
{
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, reinterpret_cast<__attribute__((address_space(3))) void *>(lds), 16, byte_off, uniform_off, 0, 0);
}
template <int N>
__device__ __forceinline__ void wait_loads() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }

// ---- ROWS rows of 64 one-byte reduction indices of a forward contraction's operand (ACT: activations, else filters); thread
//      t fetches chunk position t % 4 of rows (u * 4 + wave) * 16 + (t % 64) / 4
template <bool ACT, int ROWS>
struct DmaK {
    static constexpr int ROW_BYTES = 64, CH = ROW_BYTES / 16, RPI = 64 / CH;
    static constexpr int UNITS = ROWS * CH / kThreads;
    static constexpr int TILE_BYTES = ROWS * ROW_BYTES;
    static __device__ __forceinline__ int swizzle(int row) { return (row >> 1) & 3; }
    uint32_t base[UNITS];        // element offset of the row's part of the address, plus the thread's column
    uint32_t tapmask[UNITS];     // as in LoaderK
    int col;                     // reduction index of the thread's chunk inside a stage

    __device__ __forceinline__ void init(const ContractArgs &a, int row0)
    {
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
        col = ((lane % CH) ^ swizzle(lane / CH)) * 16;
#pragma unroll
        for (int u = 0; u < UNITS; ++u) {
            const int row = row0 + (u * 4 + wave) * RPI + lane / CH;
            tapmask[u] = k_major_row<OP_FWD, ACT>(a, row, base[u]);
            base[u] += col;
        }
    }

    // LDS addresses of a lane's fragments, one per 32 indices, of the 32 rows starting at row32 (lane / 32 = g takes reduction
    // indices [32 ks + 16 g, +16)); row: the row of the 32 that the lane takes
    __device__ __forceinline__ static void addresses(uint32_t tile, int row32, int row, int g, uint32_t (&ad)[2])
    {
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) ad[ks] = tile + (row32 + row) * ROW_BYTES + (((ks * 2 + g) ^ swizzle(row)) * 16);
    }
};

// LDS reads of every plane's fragments of one sub-step: one (MB = 1) or two 32-row blocks of the activations, TA bytes
// between planes, RA between the blocks, and one block of the weights, TB bytes between planes.  The results are written at
// different times, so none of them may share a register with an address (early clobber).
template <int P, int MB, int TA, int RA, int TB>
__device__ __forceinline__ void read_planes(v4i (&fa)[MB][P], v4i (&fw)[P], uint32_t xa, uint32_t xw)
{
    static_assert((P == 3 && MB == 2) || (P == 4 && MB == 1), "the forms that wide_planes.hip launches");
    if constexpr (P == 3)
        asm volatile("ds_read_b128 %0, %9 offset:%11\n\tds_read_b128 %1, %9 offset:%12\n\tds_read_b128 %2, %10 offset:%17\n\t"
                     "ds_read_b128 %3, %9 offset:%13\n\tds_read_b128 %4, %9 offset:%14\n\tds_read_b128 %5, %10 offset:%18\n\t"
                     "ds_read_b128 %6, %9 offset:%15\n\tds_read_b128 %7, %9 offset:%16\n\tds_read_b128 %8, %10 offset:%19\n\t"
                     "s_waitcnt lgkmcnt(0)"
                     : "=&v"(fa[0][0]), "=&v"(fa[MB - 1][0]), "=&v"(fw[0]), "=&v"(fa[0][1]), "=&v"(fa[MB - 1][1]), "=&v"(fw[1]),
                       "=&v"(fa[0][2]), "=&v"(fa[MB - 1][2]), "=&v"(fw[2])
                     : "v"(xa), "v"(xw), "n"(0), "n"(RA), "n"(TA), "n"(TA + RA), "n"(2 * TA), "n"(2 * TA + RA), "n"(0), "n"(TB), "n"(2 * TB)
                     : "memory");
    else
        asm volatile("ds_read_b128 %0, %8 offset:%10\n\tds_read_b128 %1, %9 offset:%14\n\t"
                     "ds_read_b128 %2, %8 offset:%11\n\tds_read_b128 %3, %9 offset:%15\n\t"
                     "ds_read_b128 %4, %8 offset:%12\n\tds_read_b128 %5, %9 offset:%16\n\t"
                     "ds_read_b128 %6, %8 offset:%13\n\tds_read_b128 %7, %9 offset:%17\n\t"
                     "s_waitcnt lgkmcnt(0)"
                     : "=&v"(fa[0][0]), "=&v"(fw[0]), "=&v"(fa[0][1]), "=&v"(fw[1]), "=&v"(fa[0][2]), "=&v"(fw[2]), "=&v"(fa[0][P - 1]),
                       "=&v"(fw[P - 1])
                     : "v"(xa), "v"(xw), "n"(0), "n"(TA), "n"(2 * TA), "n"(3 * TA), "n"(0), "n"(TB), "n"(2 * TB), "n"(3 * TB)
                     : "memory");
}

}  // namespace adapt
