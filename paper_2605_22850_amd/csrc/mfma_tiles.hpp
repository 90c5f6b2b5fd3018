// Device building blocks shared by the matrix kernels: LDS tile layouts whose
// operand reads are free of bank conflicts, global -> LDS copies, and the
// waits and barriers that order them.
#pragma once

#include <mutex>

#include "common.hpp"

namespace oc {

constexpr int kMaxDevices = 64;   // devices a process may launch on

// Let `Kernel` use `bytes` of dynamic LDS, above the default limit; set once
// per device (any thread may make the first launch on a device).
template <auto Kernel>
inline hipError_t allow_dynamic_lds(int bytes) {
    int dev = 0;
    const hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    static std::once_flag once[kMaxDevices];
    static hipError_t status[kMaxDevices];
    std::call_once(once[dev], [dev, bytes] {
        status[dev] = hipFuncSetAttribute(reinterpret_cast<const void *>(Kernel),
                                          hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    });
    return status[dev];
}

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// Workgroup barrier that waits only for this wavefront's LDS operations.
// (__syncthreads() would also wait for every outstanding global -> LDS copy, and
// so for the tiles that are being fetched ahead.)
__device__ inline void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// LDS element offset of 16-byte column c of K tile row r (D/8 columns per row)
template <int D>
__device__ inline int k_lds(int r, int c) {
    constexpr int NS = D / 8;
    return r * D + ((c ^ (r & (NS - 1))) << 3);
}

// XOR applied to the 16-byte column index of V tile row r.  The transposing
// reads of the PV operand take 4 dims x 4 keys per 16-lane group, from rows
// that differ in their low key bits; this spreads those rows over all banks.
template <int D>
__device__ inline int v_swz(int r) {
    if constexpr (D == 128) return 4 * (r & 3);
    else return 4 * ((r >> 1) & 1);
}

typedef __attribute__((address_space(3))) void *lds_ptr_t;
typedef __attribute__((address_space(3))) bf16x4 lds_bf16x4;

// one 16-byte global -> LDS copy per lane from `base` (wave-uniform) plus the
// lane's byte offset; the wavefront's 64 lanes fill 1 KiB of LDS starting at
// `lds_chunk`, lane i at byte 16*i.  Issued as inline
// assembly on purpose: the compiler treats every outstanding global->LDS copy
// as a possible writer of any LDS address, and would make each operand read
// of the current tile wait (vmcnt(0)) for the copies of the blocks still in
// flight, which serialises the prefetch.  The kernels order these copies
// themselves:
//  - a tile that the whole workgroup reads (256-row attention, GEMM): every
//    wavefront waits for its own copies (wait_vmcnt), then a barrier makes the
//    tile readable; it is refilled only after a barrier that follows its last
//    read;
//  - a ring of one wavefront's own (attention tiles of 32 and 64 rows): that
//    wavefront's wait_vmcnt before it reads, and s_waitcnt lgkmcnt(0) after its
//    last read, before it refills.  No barrier stands in for either.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"   // m0 is written here and read by nothing else in these kernels
__device__ inline void dma16(const void *base, uint32_t lane_off, uint16_t *lds_chunk) {
    const uint32_t m0 = (uint32_t)(uintptr_t)(lds_ptr_t)lds_chunk;   // LDS byte address, wave-uniform
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
                 :
                 : "v"(lane_off), "s"(base), "s"(m0)
                 : "memory", "m0");
}
#pragma clang diagnostic pop

// wait until at most N of this wavefront's vector memory operations are
// outstanding (they complete in order)
template <int N>
__device__ inline void wait_vmcnt() {
    static_assert(N >= 0 && N < 64, "vmcnt holds 6 bits");
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// V^T fragment n of a PV pass (n = 8-key group * D/32 + dim tile): eight
// consecutive keys of one dimension per lane, from two transposing LDS reads
// of the token-major tile; voff[et] = vt_offset<D>(lane, et).
template <int D>
__device__ __forceinline__ bf16x8 load_vt(const uint16_t *V, const int (&voff)[D / 32], int n) {
    constexpr int NET = D / 32;
    const int et = n % NET, g4 = n / NET;     // g4 = 2*half + key group
    const uint16_t *vp = V + voff[et] + ((g4 >> 1) * 32 + (g4 & 1) * 16) * D;
    const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4 *)vp);
    const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4 *)(vp + 4 * D));
    return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
}

// Transposing V reads: in each 16-lane group, source lane 4j+q names the
// four dims [4q, 4q+4) of key row j; output lane i then holds dim i of
// the four rows.  Group k covers dims 16*(k%2) + [0,16) and keys
// 8*(k/2) + [0,4) of the 16-key slice (the second read adds 4 rows).
template <int D>
__device__ __forceinline__ int vt_offset(int lane, int et) {
    const int k16 = lane >> 4, j = (lane >> 2) & 3, q4 = lane & 3;
    const int key = 8 * (k16 >> 1) + j;
    const int dim = et * 32 + 16 * (k16 & 1) + 4 * q4;
    return key * D + (((dim >> 3) ^ v_swz<D>(key)) << 3) + (dim & 7);
}

}  // namespace oc
