// Device helpers shared by the kernels that take whole chunks, forwards (gla_onepass.hip) and backwards (gla_onepass_bwd.hip).
#pragma once
#include "gla_mfma_util.h"

namespace gla {
namespace {

// Head classes: DT groups of four tail channels behind the 32 of a contraction step, NX tiles of 16 value columns, of which
// NV columns exist.
struct HeadsXL {
    static constexpr int DT = 1, NX = 5, NV = 72;
};
struct HeadsS {
    static constexpr int DT = 0, NX = 4, NV = 64;
};

// what the totals of a chunk's tiles become: 2^(b_C), 2^(b_m), 2^(b_C - b_m), b_C
enum { kDecay, kToAnchor, kFromAnchor, kLogDecay };

// 16 bytes a lane from the view to LDS, lane i's at `lds` + 16 i
__device__ inline void load_to_lds(Rsrc r, void *lds, uint32_t at) {
    typedef __attribute__((address_space(3))) void *lds_ptr;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_ptr)lds, 16, (int)at, 0, 0, 0);
}

// Identity that the optimiser cannot see through, of a value that the whole wave shares
template <typename V>
__device__ inline V afresh(V x) {
    asm volatile("" : "+s"(x));
    return x;
}
// The kernel's arguments (`args`), loaded where they are used: all of them at once do not fit the scalar registers.
#define ARG afresh(args)

// This lane, afresh in every stage: what is derived from it is not carried from one to the next in registers.
#define LANE [[maybe_unused]] const int lane = recompute_per_chunk(threadIdx.x) & 63, lm = lane & 15, g = lane >> 4

}  // namespace
}  // namespace gla
