// The few things the tile engines need from the device tool chain that have no meaning on a CPU, in one place:
// the address of a shared-memory pointer inside LDS, the global -> LDS loads written in assembly, the LDS transpose
// read.  The device build gets the HIP runtime header and these inline functions.  A host build for checking memory
// accesses (TT_HOST_EMULATION: one thread of one workgroup at a time on the CPU, every global and LDS access a real,
// bounds-checked host access; see tests/emu/) gets stand-ins with the same names from its own emu_device.h.
#pragma once
#ifdef TT_HOST_EMULATION
#include "emu_device.h"
#else
#include <hip/hip_runtime.h>
#include <cstdint>

namespace tt {
namespace dev {

typedef short s16x4 __attribute__((ext_vector_type(4)));

// byte address inside the workgroup's LDS of a pointer into its shared memory
__device__ __forceinline__ uint32_t lds_addr(char *p)
{
    return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)p;
}

// global -> LDS, 16 bytes per lane: lane i's chunk lands at lds_wave_addr + 16 i (M0 holds the wave-uniform LDS
// address).  Assembly on purpose: for the builtin form the compiler's wait-count pass assumes that any later LDS read may
// alias the incoming data and puts s_waitcnt vmcnt(0) in front of the next fragment read; here the waits are the explicit
// s_waitcnt + barrier pairs of the main loops.
//
// Wait states: where a vector instruction (v_readfirstlane) writes a scalar register, the ISA asks for five wait states
// before a vector-memory instruction reads it, and the compiler, which puts them in front of its own instructions, does not
// look into assembly (a kernel whose base was read two instructions after it was written loaded from a stale address and
// faulted).  A scalar instruction may read such a register at once, and what a scalar instruction writes a vector-memory
// instruction may read at once, M0 after one wait state.  So every block first copies its scalar operands with scalar
// instructions, and its load reads nothing but those copies, wherever the compiler got the operands from.  (s_nop 4 in front
// of every load is as safe, but idles a wave for 32 cycles per K tile of 64: a step of four 8192 x 8192 layers at batch 2048
// takes 2823 us with it and 2800 us so.)
// ... every lane supplies a full global address
__device__ __forceinline__ void lds_dma16(const void *g, uint32_t lds_wave_addr)
{
    uint32_t m0;
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, off" : "=&{m0}"(m0) : "s"(lds_wave_addr), "v"(g) : "memory");
}
// ... a wave-uniform base (scalar registers) plus a 32-bit offset per lane; the move of the base is the wait state after M0's
__device__ __forceinline__ void lds_dma16(uint32_t lane_offset, uint64_t uniform_base, uint32_t lds_wave_addr)
{
    uint32_t m0;
    uint64_t base;
    asm volatile("s_mov_b32 m0, %4\n\ts_mov_b64 %1, %3\n\tglobal_load_lds_dwordx4 %2, %1"
                 : "=&{m0}"(m0), "=&s"(base) : "v"(lane_offset), "s"(uniform_base), "s"(lds_wave_addr) : "memory");
}

// 16-byte global store.  A named function because kernels that leave stores in flight over a wait count them
// (s_waitcnt vmcnt(n) counts a wave's loads and stores alike, in issue order), and the host emulation counts them here.
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
template <bool NON_TEMPORAL> __device__ __forceinline__ void store16(void *p, u32x4_t v)
{
    if constexpr (NON_TEMPORAL) __builtin_nontemporal_store(v, reinterpret_cast<u32x4_t *>(p));
    else *reinterpret_cast<u32x4_t *>(p) = v;
}

// LDS transpose read: 8 bytes per lane at a, handed out transposed over each group of 16 lanes (four bf16 per lane)
__device__ __forceinline__ s16x4 lds_read_tr16_b64(const char *a)
{
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)a);
}

} // namespace dev
} // namespace tt
#endif
