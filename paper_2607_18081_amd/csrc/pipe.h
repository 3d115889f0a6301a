// Building blocks of the pipelined MFMA GEMMs: loads straight into LDS, counted waits and a
// bare barrier.
//
// A K step's operands go from memory to LDS without passing through registers (buffer loads
// with an LDS destination: lane l's 16 bytes land at base + 16 l, a lane whose offset is out
// of the buffer's range writes zeros). Such loads are counted like any vector memory load, in
// issue order, so "the stage's loads have landed" is a wait for the count of the loads issued
// after them. __syncthreads() would wait for all of them; wg_barrier() waits for none, and its
// caller first waits for what the barrier is to publish.
#pragma once

#include "common.h"

namespace si {

typedef __attribute__((address_space(3))) void lds_void;

// 16 bytes per lane from r at voff + soff to lds + 16 * lane (lds wave-uniform)
// (POL: the cache policy, kNonTemporal or 0)
template <int POL = 0>
__device__ __forceinline__ void load_lds16(__amdgpu_buffer_rsrc_t r, char* lds, int voff, int soff);
template <>
__device__ __forceinline__ void load_lds16<0>(__amdgpu_buffer_rsrc_t r, char* lds, int voff,
                                              int soff) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void*)lds, 16, voff, soff, 0, 0);
}
template <>
__device__ __forceinline__ void load_lds16<kNonTemporal>(__amdgpu_buffer_rsrc_t r, char* lds,
                                                         int voff, int soff) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void*)lds, 16, voff, soff, 0, kNonTemporal);
}

// Waits until at most N of this wave's vector memory loads are outstanding and none of its LDS
// accesses. (Specialised: the builtin takes a literal. Immediate: vmcnt in bits 3:0 and 15:14,
// expcnt 6:4 left at its maximum, lgkmcnt 11:8.)
template <int N>
__device__ __forceinline__ void wait_vm_lds();
#define SI_WAIT_VM(n)                                                             \
    template <>                                                                   \
    __device__ __forceinline__ void wait_vm_lds<n>() {                            \
        __builtin_amdgcn_s_waitcnt(((n) & 15) | 0x70 | (((n) >> 4) << 14));       \
    }
SI_WAIT_VM(0) SI_WAIT_VM(1) SI_WAIT_VM(2) SI_WAIT_VM(3) SI_WAIT_VM(4) SI_WAIT_VM(5)
SI_WAIT_VM(6) SI_WAIT_VM(7) SI_WAIT_VM(8) SI_WAIT_VM(9) SI_WAIT_VM(10) SI_WAIT_VM(11)
SI_WAIT_VM(12) SI_WAIT_VM(13) SI_WAIT_VM(14) SI_WAIT_VM(15) SI_WAIT_VM(16) SI_WAIT_VM(17)
SI_WAIT_VM(18) SI_WAIT_VM(19) SI_WAIT_VM(20) SI_WAIT_VM(21) SI_WAIT_VM(22) SI_WAIT_VM(23)
SI_WAIT_VM(24) SI_WAIT_VM(25) SI_WAIT_VM(26) SI_WAIT_VM(27) SI_WAIT_VM(28) SI_WAIT_VM(29)
SI_WAIT_VM(30) SI_WAIT_VM(31) SI_WAIT_VM(32) SI_WAIT_VM(33) SI_WAIT_VM(34) SI_WAIT_VM(35)
SI_WAIT_VM(36) SI_WAIT_VM(37) SI_WAIT_VM(38) SI_WAIT_VM(39) SI_WAIT_VM(40) SI_WAIT_VM(41)
SI_WAIT_VM(42) SI_WAIT_VM(43) SI_WAIT_VM(44) SI_WAIT_VM(45) SI_WAIT_VM(46) SI_WAIT_VM(47)
SI_WAIT_VM(48) SI_WAIT_VM(49) SI_WAIT_VM(50) SI_WAIT_VM(51) SI_WAIT_VM(52) SI_WAIT_VM(53)
SI_WAIT_VM(54) SI_WAIT_VM(55) SI_WAIT_VM(56) SI_WAIT_VM(57) SI_WAIT_VM(58) SI_WAIT_VM(59)
SI_WAIT_VM(60) SI_WAIT_VM(61) SI_WAIT_VM(62) SI_WAIT_VM(63)
#undef SI_WAIT_VM

// Barrier of the work-group's waves; memory operations do not move across it at compile time.
__device__ __forceinline__ void wg_barrier() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// Tile (tm, st) of an ntm x nst grid for work-group id, both wave-uniform; false: no tile. The
// hardware deals work-groups to the 8 XCDs in turn (id % 8), and an XCD's share is one run of
// the order that takes up to 8 row tiles tm of a column tile st, then the next column tile, so
// the 32 or so tiles an XCD works on at a time share few operand slices in its L2.
__device__ __forceinline__ bool xcd_tile(int id, int ntm, int nst, int& tm, int& st) {
    const unsigned nt = (unsigned)ntm * (unsigned)nst;
    const unsigned per = (nt + 7) >> 3;
    const unsigned q = (unsigned)(id & 7) * per + (unsigned)(id >> 3);
    if ((unsigned)(id >> 3) >= per || q >= nt) return false;
    const unsigned band = 8u * (unsigned)nst;
    const unsigned b = q / band;
    const unsigned r = q - b * band;
    const unsigned rows = (unsigned)ntm - 8u * b < 8u ? (unsigned)ntm - 8u * b : 8u;
    const unsigned s = r / rows;
    // scalar again: the compiler divides in vector registers
    st = __builtin_amdgcn_readfirstlane((int)s);
    tm = __builtin_amdgcn_readfirstlane((int)(8u * b + r - s * rows));
    return true;
}

}  // namespace si
