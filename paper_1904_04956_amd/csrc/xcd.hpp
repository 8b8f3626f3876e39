// Workgroups that exchange data and sit on one XCD share its L2: what one of them stores there by an ordinary (write-back) store the others
// find by loads past their L1, in half of the time that a write-through store takes to come back from the memory side.  Measured between two
// workgroups, a round trip: write-through 1074 ns on one XCD and 1293 across, ordinary 558 ns on one XCD and never across.
//
// Ids are dealt round-robin to the eight XCDs, and the kernels place whole groups by that, but nothing guarantees it.  So every workgroup
// of a group writes down which XCD it is on, each wavefront reads what its whole group wrote, and only a group found on one XCD
// uses ordinary stores; all its members come to the same answer.  The words are marked "not written" (all ones) with the exchange
// copies they lie between, and written write-through.  Costs a launch half a microsecond to one and a half, behind the loads of the weights.
//
// Not everywhere the better one: what is written back late is written at the launch's end or in the way of other traffic.  A whole step of
// four layers (21 frames), us, write-through / through the L2: 128 sequences of 512 cells 804 / 836, 173 967 / 988, 256 of 320 824 / 847, but 500 of
// 128 675 / 652, 700 of 256 1515 / 1452 and (the forward kernel alone, several tiles a workgroup) 300 of 512 1642 / 1594, 2048 of 512, two layers, 3829 / 3748.
// So each kernel says where it asks.
#pragma once
#include <hip/hip_runtime.h>

namespace blstm {

constexpr size_t XCD_TABLE_BYTES = 8192;                 // of a launch: a word per workgroup, by group and slice
constexpr int XCD_GROUP_MAX = 64;                        // slices of a group that are looked at (a lane each)

__device__ __forceinline__ unsigned xcd_id() { return (unsigned)__builtin_amdgcn_s_getreg(20 | 3 << 11); }   // hwreg(HW_REG_XCC_ID, 0, 4)
// table: the group's words, or null (no answer wanted); me: this workgroup's slice.
__device__ __forceinline__ void tell_xcd(unsigned* table, int me) {
    if (table && threadIdx.x == 0) __hip_atomic_store(table + me, xcd_id(), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Whether all n workgroups of the group are on this one's XCD.  *gave_up: the wait for their words was abandoned.
__device__ __forceinline__ bool one_xcd(const unsigned* table, int n, unsigned* abort_word, unsigned long long limit, bool* gave_up) {
    *gave_up = false;
    if (!table || n > XCD_GROUP_MAX) return false;
    const int lane = threadIdx.x & 63;
    const unsigned own = xcd_id();
    const unsigned long long t0 = wall_clock64();
    for (unsigned it = 1;; ++it) {
        const unsigned v = lane < n ? __hip_atomic_load(table + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : own;
        if (__all(v != 0xFFFFFFFFu)) return __all(v == own) != 0;
        if ((it & 31u) == 0) {
            if (__hip_atomic_load(abort_word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) { *gave_up = true; return false; }
            if (wall_clock64() - t0 > limit) {
                __hip_atomic_store(abort_word, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                *gave_up = true;
                return false;
            }
        }
    }
}

}  // namespace blstm
