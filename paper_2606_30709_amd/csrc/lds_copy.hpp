// Copies from global memory straight into LDS (buffer loads with the LDS
// destination), and the waits they need.  They are inline assembly because
// the compiler's own tracking of LDS-destination loads would wait for every
// copy in flight before any LDS read; every user waits with an explicit
// count (loads complete in issue order).
#pragma once

#include "hga_device.hpp"

namespace hga {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

constexpr uint32_t kAbsent = 0xffff0000u;  // an offset past every buffer: reads zeros

// Descriptor words of a raw buffer [base, base + bytes) for the copies below
// (base address, no stride, num_records = bytes); the operands are uniform.
__device__ __forceinline__ u32x4 rsrc_words(const void* base, uint32_t bytes) {
    const uint64_t a = reinterpret_cast<uint64_t>(base);
    u32x4 r;
    r.x = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(a));
    r.y = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(a >> 32) & 0xffffu);
    r.z = __builtin_amdgcn_readfirstlane(bytes);
    r.w = 0x00020000u;
    return r;
}

// Copy 16 bytes per lane from buffer offset voff to LDS byte lds + 16*lane.
__device__ __forceinline__ void copy16_to_lds(const u32x4& rs, uint32_t voff, uint32_t lds) {
    asm volatile("s_mov_b32 m0, %2\n\tbuffer_load_dwordx4 %0, %1, 0 offen lds"
                 :
                 : "v"(voff), "s"(rs), "s"(lds)
                 : "memory");
}

// Copy 4 bytes per lane from buffer offset voff to LDS byte lds + 4*lane.
__device__ __forceinline__ void copy4_to_lds(const u32x4& rs, uint32_t voff, uint32_t lds) {
    asm volatile("s_mov_b32 m0, %2\n\tbuffer_load_dword %0, %1, 0 offen lds"
                 :
                 : "v"(voff), "s"(rs), "s"(lds)
                 : "memory");
}

// Wait until at most N vector-memory loads of this wavefront are in flight;
// the compiler moves no memory access across it.
template <int N>
__device__ __forceinline__ void wait_copies() {
    static_assert(N >= 0 && N < 64, "vmcnt range");
    asm volatile("s_waitcnt vmcnt(%0)" : : "n"(N) : "memory");
}

// Every LDS read of this wavefront has returned (its source may be
// overwritten).
__device__ __forceinline__ void lds_reads_done() {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
}

// Row-major staging of bf16 rows of D dimensions: 16-byte chunk j of row r is stored at j ^ swz_rows(r).  The 16-byte
// fragment reads of 16 consecutive rows then fall in distinct banks, and so
// do the transpose reads (32 bytes of rows 0..7, or of rows 0..3 and 8..11, or
// 64 bytes of rows 0..3 of a 16-row block in one cycle).
template <int D>
__device__ __forceinline__ int swz_rows(int r) {
    if constexpr (D == 64)  // two rows span the banks: r >> 1 counts
        return (((r >> 1) & 1) << 2) | ((((r >> 2) ^ (r >> 3)) & 1) << 1) | ((r >> 3) & 1);
    else
        return ((r & 1) << 3) | (((r >> 1) & 1) << 2) | ((((r >> 2) ^ (r >> 3)) & 1) << 1) |
               ((r >> 3) & 1);
}

}  // namespace hga
