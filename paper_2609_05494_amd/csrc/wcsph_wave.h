// wcsph_wave.h -- device helpers shared by the forward kernels and the reverse
// sweep of libwcsph.so (internal).
#pragma once

#include "wcsph_dev.h"

// Spread consecutive blocks over the 8 XCDs in contiguous chunks: hardware
// dispatches block b to XCD b % 8, so logical chunk x (one L2) is served by
// the blocks with b % 8 == x.
__device__ __forceinline__ int xcd_block(int bid, int nblk) {
  const int q = nblk >> 3, r = nblk & 7, x = bid & 7;
  return x * q + min(x, r) + (bid >> 3);
}

// (The parameter blocks do not change while a kernel runs: read through the
// constant address space, a block that is the same on every lane comes
// through the scalar cache wherever it is read.)
typedef const __attribute__((address_space(4))) InstParams ConstParams;
// A copy of a block that no one writes meanwhile, read through the constant
// address space. (When it is inlined only the fields that are used are read;
// the kernel itself must not write those either, since the compiler may load
// them again at any place.)
template <class T>
__device__ __forceinline__ T scalar_copy(const T* p) {
  static_assert(sizeof(T) % 8 == 0, "whole words");
  typedef const __attribute__((address_space(4))) unsigned long long Word;
  unsigned long long w[sizeof(T) / 8];
#pragma unroll
  for (int k = 0; k < (int)(sizeof(T) / 8); ++k) w[k] = ((Word*)p)[k];
  T t;
  __builtin_memcpy(&t, w, sizeof t);
  return t;
}

// Order the wave's LDS accesses: stores before this point are seen by every
// lane's loads after it (accesses of one wave are performed in order; the
// fences keep the compiler from moving them across).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
