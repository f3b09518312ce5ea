// Direct-to-LDS loads and the waits around them, as the operand rings of the
// products and of the attention use them.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace kvr {

typedef __attribute__((address_space(3))) void lds_void;
constexpr int BUF_WORD3 = 0x00020000;  // gfx9 buffer descriptor: 32-bit data format

// s_waitcnt with only the vector-memory / only the LDS counter constrained
#define KVR_WAIT_VMCNT(n) \
  __builtin_amdgcn_s_waitcnt(((n) & 0xF) | (((n) >> 4) << 14) | (0x7 << 4) | (0xF << 8))
#define KVR_WAIT_LGKM0() __builtin_amdgcn_s_waitcnt(0xF | (0x3 << 14) | (0x7 << 4))

// LDS layout of a product's operands: 1 KB blocks of 8 rows of 128 bytes; row r
// (of 16) holds its 16-byte k-unit u at slot u ^ swz(r).  A direct-to-LDS load
// writes 64 lanes x 16 B contiguously, so one instruction fills one block with
// whole 128-byte rows.  The LDS serves a b128 read 16 lanes at a time, lanes 0-3,
// 12-15 and 20-27 in one pass: with rows 0-15 at unit u in lanes 0-15 and at
// unit u+1 in lanes 16-31 this swizzle puts each pass on 64 distinct banks
// (r ^ (r >> 3) took two passes for every one).
__device__ __forceinline__ int swz(int r) { return (r >> 1) & 7; }

// One direct-to-LDS load: 16 bytes per lane from base + voff + soff to 1 KB at dst
__device__ __forceinline__ void load_lds(const void* base, int bytes, char* dst, int voff, int soff) {
  const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, bytes, BUF_WORD3);
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_void*)dst, 16, voff, soff, 0, 0);
}

}  // namespace kvr
