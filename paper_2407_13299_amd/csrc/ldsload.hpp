// Loads from global memory straight into LDS (gfx950) and the waits and
// barrier that go with them; shared by the slice GEMM and the residue GEMM.
#pragma once

#include "common.hpp"

namespace dmp {

typedef int v1i __attribute__((ext_vector_type(1)));
typedef int v2i __attribute__((ext_vector_type(2)));
typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef _Float16 v8h __attribute__((ext_vector_type(8)));

// Workgroup barrier without the memory fence __syncthreads() implies (that
// fence would also wait for the prefetch loads in flight); the signal fences
// keep the compiler from moving memory accesses across it.  Before each
// barrier the kernel waits for its own operand loads and LDS reads itself
// (ops_wait).
__device__ inline void bare_barrier() {
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __builtin_amdgcn_s_barrier();
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
}

// Fourth word of a raw buffer descriptor on gfx950 (32-bit data format,
// no swizzle, no index stride).
constexpr int kBufferWord3 = 0x00020000;

typedef __attribute__((address_space(3))) uint8_t lds_u8;

// Byte offset of a shared-memory address inside the workgroup's LDS.
__device__ inline uint32_t lds_offset(const void* p) {
    return static_cast<uint32_t>(reinterpret_cast<size_t>((const lds_u8*)(p)));
}

// A raw buffer descriptor (base, no stride, ``bytes`` records) as four
// wave-uniform words, for the inline assembly below, which takes it in
// scalar registers.
__device__ inline v4i sgpr_desc(const void* base, int bytes) {
    const uint64_t b = reinterpret_cast<uint64_t>(base);
    v4i d;
    d[0] = __builtin_amdgcn_readfirstlane(int(uint32_t(b)));
    d[1] = __builtin_amdgcn_readfirstlane(int(uint32_t(b >> 32) & 0xffffu));
    d[2] = __builtin_amdgcn_readfirstlane(bytes);
    d[3] = kBufferWord3;
    return d;
}

// One 1 KiB fragment block from global memory straight into LDS (a buffer
// load with the LDS flag): lane l's 16 bytes at buffer offset voff + soff
// land at LDS byte lds + 16 l, which is exactly the fragment layout, so no
// register staging and no LDS store instruction is needed.  It is written
// as inline assembly so that the compiler's wait counting, which would
// otherwise wait for every such load before any LDS read, leaves it alone;
// the kernel waits for these loads itself (ops_wait) before the barrier
// that publishes them.  The load has no register destination; m0 holds the
// LDS address and is set right before it.  m0 is a register the compiler
// reserves; nothing else in these kernels reads it (gfx950 LDS instructions
// do not use it), which tests/test_isa_m0.py checks on the compiled code.
__device__ inline void frag_to_lds(v4i r, uint32_t lds, int voff, int soff) {
    // the operands are wave-uniform; reading them from the first lane makes
    // them scalar registers at this point even where register pressure has
    // moved them to vector registers in between
    v4i rs;
#pragma unroll
    for (int q = 0; q < 4; ++q) rs[q] = __builtin_amdgcn_readfirstlane(r[q]);
    const uint32_t ls = __builtin_amdgcn_readfirstlane(lds);
    const int ss = __builtin_amdgcn_readfirstlane(soff);
    asm volatile("s_mov_b32 m0, %0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                 :: "s"(ls), "v"(voff), "s"(rs), "s"(ss) : "memory", "m0");
}

// s_waitcnt vmcnt(N) lgkmcnt(0): at most N vector-memory operations of the
// wavefront still in flight, and every LDS read returned.
// vm_wait: the vector-memory part alone.
template <int N>
__device__ inline void vm_wait() {
    asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory");
}
template <int N>
__device__ inline void ops_wait() {
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" :: "n"(N) : "memory");
}

}  // namespace dmp
