// Device helpers shared by the tile GEMM kernels: LDS-DMA loads and the
// XCD-aware tile order.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace p4q {
namespace {

typedef int v4i __attribute__((ext_vector_type(4)));

constexpr int kXcds = 8;
constexpr int kGroupM = 8;

typedef __attribute__((address_space(3))) void *lds_ptr_t;

// Buffer descriptor of a raw byte range (stride 0, range-checked: loads past
// `bytes` return zeros).
__device__ __forceinline__ v4i buffer_desc(const void *base, uint32_t bytes) {
    const uint64_t b = reinterpret_cast<uint64_t>(base);
    return v4i{(int)(uint32_t)b, (int)((b >> 32) & 0xFFFFu), (int)bytes, 0x00020000};
}

// 16 (or 4) bytes per lane from a buffer straight into LDS at lds + 16 *
// lane (4 * lane).  Issued as inline asm so the compiler does not add its
// conservative vmcnt(0) before every LDS read (it cannot tell the ring slots
// apart); the kernel waits with explicit vmcnt counts instead.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void dma16(v4i desc, uint32_t voffset, uint32_t lds_addr) {
    asm volatile("s_mov_b32 m0, %2\n\tbuffer_load_dwordx4 %0, %1, 0 offen lds"
                 :
                 : "v"(voffset), "s"(desc), "s"(lds_addr)
                 : "memory", "m0");
}
__device__ __forceinline__ void dma4(v4i desc, uint32_t voffset, uint32_t lds_addr) {
    asm volatile("s_mov_b32 m0, %2\n\tbuffer_load_dword %0, %1, 0 offen lds"
                 :
                 : "v"(voffset), "s"(desc), "s"(lds_addr)
                 : "memory", "m0");
}
#pragma clang diagnostic pop

__device__ __forceinline__ uint32_t lds_addr(const void *p) {
    return (uint32_t)(size_t)(lds_ptr_t)p;
}

// Work-group id -> logical index such that the ids of one XCD (dealt
// round-robin) form a contiguous range of [0, total).
__device__ __forceinline__ int xcd_logical(int wg, int total) {
    const int q = total / kXcds, r = total % kXcds;
    const int x = wg % kXcds, i = wg / kXcds;
    return (x < r) ? x * (q + 1) + i : r * (q + 1) + (x - r) * q + i;
}

// logical index -> tile, walking groups of kGroupM tile rows column by column
__device__ __forceinline__ void grouped_tile(int logical, int tiles_m, int tiles_n, int &tm,
                                             int &tn) {
    const int per_group = kGroupM * tiles_n;
    const int g = logical / per_group;
    const int first_m = g * kGroupM;
    const int gsize = min(tiles_m - first_m, kGroupM);
    const int in_g = logical - g * per_group;
    tm = first_m + in_g % gsize;
    tn = in_g / gsize;
}

}  // namespace
}  // namespace p4q
