// Operand tiles that go from memory straight to LDS (wide_planes.hip).
//
// A stage is BKT reduction indices of an operand as they lie in memory.  It is fetched with 16-byte loads whose
// destination is LDS: no staging registers, no LDS stores.  Such a load writes 64 x 16 consecutive bytes per wavefront, so
// tiles have no padding; bank conflicts are avoided by permuting which 16-byte chunk a lane fetches: chunk c of row r
// lies at position c ^ swizzle(r).
//
// LDS fragment reads are written in assembly with explicit waits: the compiler would otherwise wait for every
// outstanding load to LDS before each of them.
//
// (As the main loop of the two-limb kernels, with the limb split between LDS and the matrix units, this measured within
// 15 % of the kernels of contract_kernel.hpp either way: there a wavefront's splitting, LDS reads and products follow one
// another, and splitting in every wavefront that reads a fragment doubles that work.)
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

// ---- K-major: thread t fetches chunk position t % CH of rows (u * 4 + wave) * RPI + (t % 64) / CH
template <int OP, bool ACT, int ROWS, int ES, int BKT>
struct DmaK {
    static constexpr int ROW_BYTES = BKT * ES, CH = ROW_BYTES / 16, RPI = 64 / CH;
    static constexpr int UNITS = ROWS * CH / kThreads;
    static constexpr int TILE_BYTES = ROWS * ROW_BYTES;
    static_assert(CH == 4 || CH == 8, "a row is 64 or 128 bytes");
    static __device__ __forceinline__ int swizzle(int row) { return CH == 8 ? (row & 7) : ((row >> 1) & 3); }
    uint32_t base[UNITS];        // element offset of the row's part of the address, plus the thread's column
    uint32_t tapmask[UNITS];     // as in LoaderK
    int col;                     // reduction index of the thread's chunk inside a stage

    __device__ __forceinline__ void init(const ContractArgs &a, int row0)
    {
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
        col = ((lane % CH) ^ swizzle(lane / CH)) * (16 / ES);
#pragma unroll
        for (int u = 0; u < UNITS; ++u) {
            const int row = row0 + (u * 4 + wave) * RPI + lane / CH;
            tapmask[u] = k_major_row<OP, ACT>(a, row, base[u]);
            base[u] += col;
        }
    }

    // LDS addresses of a lane's fragment of the 32 rows starting at row32 (lane / 32 = g takes reduction indices
    // [32 ks + 16 g, +16)); row: the row of the 32 that the lane takes
    static constexpr int ADDR = ES * (BKT / 32);      // distinct addresses: chunk within the row
    __device__ __forceinline__ static void addresses(uint32_t tile, int row32, int row, int g, uint32_t (&ad)[ADDR])
    {
#pragma unroll
        for (int i = 0; i < ADDR; ++i) {
            const int ks = i / ES, e = i % ES;
            ad[i] = tile + (row32 + row) * ROW_BYTES + (((ks * 2 * ES + ES * g + e) ^ swizzle(row)) * 16);
        }
    }
};

// LDS read at addr + off (a constant), completion by the reader's own wait
#define ADAPT_LDS_READ(instr, dst, addr, off) asm volatile(instr " %0, %1 offset:%2" : "=v"(dst) : "v"(addr), "n"(off))

}  // namespace adapt
