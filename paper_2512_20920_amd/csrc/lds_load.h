// Loads straight from memory into LDS (buffer_load ... lds) through raw buffer descriptors.
//
// A wave-load brings 64 lanes x 16 bytes (4): the LDS address is wave-uniform, lane l's part lands 16 l (4 l) bytes after
// it.  The byte offset is per lane; one at or past the descriptor's size reads as zeros without traffic, so "outside the
// problem" needs no branch.
#pragma once
#include "kernels.h"

typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;

#define OOB 0x80000000u              // an offset out of range of every descriptor of make_desc (2 GiB)

__device__ __forceinline__ u32x4 make_desc(const void* p) {
  // (operand bases are the same for every lane; saying so keeps the descriptor in scalar registers whatever the
  // compiler can prove about how the base was picked)
  const unsigned long long a = (unsigned long long)p;
  u32x4 d = {(unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)a),
             (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(a >> 32)), OOB, 0x00020000u};
  return d;
}
__device__ __forceinline__ unsigned lds_address(const void* p) { return (unsigned)(unsigned long long)(const __attribute__((address_space(3))) unsigned char*)p; }

template <class D> __device__ __forceinline__ void load_lds_b128(D desc, unsigned lds_addr, unsigned voff) {
  asm volatile("s_mov_b32 m0, %0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
               :: "s"(lds_addr), "v"(voff), "s"(desc) : "memory", "m0");
}
// the same for data that is used once: it does not push other lines out of the caches
template <class D> __device__ __forceinline__ void load_lds_b128_once(D desc, unsigned lds_addr, unsigned voff) {
  asm volatile("s_mov_b32 m0, %0\n\tbuffer_load_dwordx4 %1, %2, 0 offen nt lds"
               :: "s"(lds_addr), "v"(voff), "s"(desc) : "memory", "m0");
}
// the same with a wave-uniform byte offset added
__device__ __forceinline__ void load_lds_b128_s(u32x4 desc, unsigned lds_addr, unsigned voff, unsigned soff) {
  soff = __builtin_amdgcn_readfirstlane(soff);
  asm("" : "+s"(soff));                             // (a literal is no offset operand)
  asm volatile("s_mov_b32 m0, %0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
               :: "s"(lds_addr), "v"(voff), "s"(desc), "s"(soff) : "memory", "m0");
}
template <class D> __device__ __forceinline__ void load_lds_b32(D desc, unsigned lds_addr, unsigned voff) {
  asm volatile("s_mov_b32 m0, %0\n\tbuffer_load_dword %1, %2, 0 offen lds"
               :: "s"(lds_addr), "v"(voff), "s"(desc) : "memory", "m0");
}
template <int N> __device__ __forceinline__ void wait_vmcnt() { asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory"); }
