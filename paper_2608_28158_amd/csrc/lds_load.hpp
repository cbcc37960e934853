// Loads from global memory straight into LDS (gfx950, 16 bytes a lane): no
// registers hold the data on its way and no LDS write instructions are issued.
// The 64 lanes of a wave fill 1,024 consecutive bytes of LDS from dst, lane l
// the 16 bytes at 16 l; each lane chooses where it reads, so a tile's layout
// is chosen by the lanes' addresses.  dst has to lie in the first 64 KB of
// the workgroup's LDS (16 bits of M0) and is the same for the whole wave.
//
// Written as asm because the compiler lets every LDS read wait for a load of
// this kind.  M0 is declared as overwritten, so that an M0 of the compiler's
// own would be set again after it (there is none in the kernels now); it warns
// that the register is one of its reserved ones.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"

namespace harts {

template <typename T>
__device__ inline uint32_t lds_base(const T* dst) {
  typedef __attribute__((address_space(3))) const T lds_T;
  return __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(reinterpret_cast<uintptr_t>((lds_T*)dst)));
}

// from base (the same for the whole wave) + off bytes
template <typename T>
__device__ inline void lds_load16(const void* base, uint32_t off, const T* dst) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
               :
               : "s"(lds_base(dst)), "v"(off), "s"(base)
               : "m0", "memory");
}

// from each lane's own address
template <typename T>
__device__ inline void lds_load16(const void* p, const T* dst) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off"
               :
               : "s"(lds_base(dst)), "v"(p)
               : "m0", "memory");
}

// Every load of this wave has landed (vmcnt 0; the builtin also tells the
// compiler that no load of its own is out, or it would wait inside a loop for
// registers loaded before it, and with them for the next loads into LDS);
// then the workgroup meets, and all of its loads have.
__device__ inline void lds_landed() {
  __builtin_amdgcn_s_waitcnt(0x0f70);
  __syncthreads();
}

}  // namespace harts

#pragma clang diagnostic pop
