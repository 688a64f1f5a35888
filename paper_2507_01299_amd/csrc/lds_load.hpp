// Loads from global memory straight into LDS (no destination registers), counted by hand.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace larosa {

typedef __attribute__((address_space(3))) char lds_char;

// A 16-byte piece whose offset lies at or beyond the buffer's size arrives as zeros: what must not count gets this
// offset.  Buffers are smaller than 2 GiB, so it stays outside when an offset below that is added to it.
constexpr uint32_t kOutside = 0x80000000u;

// Raw buffer over `bytes` bytes at p (both uniform over the wave).
__device__ __forceinline__ uint32_t __attribute__((ext_vector_type(4))) raw_buffer(const void* p, uint32_t bytes) {
  typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
  const uint64_t base = reinterpret_cast<uint64_t>(p);
  return u32x4_t{static_cast<uint32_t>(base), static_cast<uint32_t>(base >> 32) & 0xFFFFu, bytes, 0x00027000u};
}

// 16 bytes per lane from buffer offset `off`: lane l's piece lands at LDS byte lds_byte + 16 l.  Written as an
// instruction because the compiler would wait for every outstanding load of this kind before each LDS read; the callers
// count them themselves (s_waitcnt vmcnt).  m0 is declared as
// overwritten; what a load writes to LDS is ordered by those waits, which are memory barriers to the compiler.
__device__ __forceinline__ void load_to_lds(uint32_t __attribute__((ext_vector_type(4))) buf, uint32_t lds_byte, uint32_t off) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" ::"s"(lds_byte), "v"(off), "s"(buf) : "m0");
}

// The same for data that is read once (non-temporal).
__device__ __forceinline__ void load_to_lds_stream(uint32_t __attribute__((ext_vector_type(4))) buf, uint32_t lds_byte, uint32_t off) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen nt lds" ::"s"(lds_byte), "v"(off), "s"(buf) : "m0");
}

}  // namespace larosa
