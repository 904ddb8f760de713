// Loads from global memory straight into LDS, and the waits that go with them.  Written as inline assembly so that the only
// waits on these loads are the explicit ones (the compiler would otherwise drain all of them before any LDS read).
#pragma once

#include <cstdint>
#include <hip/hip_runtime.h>

#pragma clang diagnostic ignored "-Winline-asm"

typedef int hdet_rsrc __attribute__((ext_vector_type(4)));

// 64 lanes x 16 bytes from the buffer `rsrc` at byte offsets `voff` (out of range: zeros) to the
// LDS bytes [lds_addr, lds_addr + 1024), lane l at lds_addr + 16 l.  Completion is counted by vmcnt.
__device__ __forceinline__ void lds_load16(hdet_rsrc rsrc, uint32_t lds_addr, uint32_t voff) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" ::"s"(lds_addr), "v"(voff), "s"(rsrc)
               : "memory", "m0");
}
// 64 lanes x 4 bytes, lane l at lds_addr + 4 l
__device__ __forceinline__ void lds_load4(hdet_rsrc rsrc, uint32_t lds_addr, uint32_t voff) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dword %1, %2, 0 offen lds" ::"s"(lds_addr), "v"(voff), "s"(rsrc)
               : "memory", "m0");
}
// raw buffer descriptor: base, stride 0, extent in bytes, 32-bit untyped data
__device__ __forceinline__ hdet_rsrc make_rsrc(const void* p, uint32_t bytes) {
  const uint64_t a = (uint64_t)p;
  const hdet_rsrc r = {(int)(uint32_t)a, (int)(uint32_t)(a >> 32), (int)bytes, 0x00020000};
  return r;
}
__device__ __forceinline__ uint32_t lds_addr_of(const uint16_t* p) {
  return (uint32_t)(size_t)((__attribute__((address_space(3))) const uint16_t*)p);
}
// own LDS-direct loads older than the newest N have landed and own LDS reads are complete; then
// the block meets
template <int N> __device__ __forceinline__ void wait_and_barrier() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}
