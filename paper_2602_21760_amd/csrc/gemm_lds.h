// Copies of operand slabs to LDS that the MFMA GEMM kernels share.
#pragma once
#include "common.h"

typedef void __attribute__((address_space(3)))* lptr_t;

// XOR swizzle of the eight 16-byte slots of a 128-byte row of a slab.
__device__ __forceinline__ int swz(int r) { return (r ^ (r >> 3)) & 7; }

// 16 bytes per lane from a raw buffer (base address, size in bytes) straight into LDS: lane i's bytes land at
// lds + 16 i; the address is base + voffset (per lane) + soffset (scalar).  Not a template: the descriptor type
// only exists in the device pass.
__device__ __forceinline__ void buffer_load_lds16(const void* base, unsigned bytes, void* lds, int voffset, int soffset) {
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, (int)bytes, 0x00020000);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lptr_t)lds, 16, voffset, soffset, 0, 0);
}
