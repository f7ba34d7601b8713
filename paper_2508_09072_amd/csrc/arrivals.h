// Workgroups of one launch that wait for each other, so that what needs the results or the progress of others does not
// have to be a launch of its own.
//
// Every workgroup has a 64-bit mark in the workspace and sets it to the launch's token when it has got somewhere.  A token
// is used once per process (the host counts them up from a random start), so whatever the marks held before is no arrival and
// nothing has to be cleared.  A captured graph would use its token again with every replay: while a stream is being captured
// the launches stay apart.
//
// Marks, and what they vouch for, pass the XCDs' caches: stores are written through, marks are looked at past them (agent
// scope), and a wavefront waits for its own stores (vmcnt 0) before the mark is set, and for the mark before it looks at another's.
// No cache is written back or invalidated (an invalidation by every wavefront took 17 us).  What workgroups of one XCD have
// written (their marks say where they run) is in the L2 that all its compute units share, and plain loads find it there, of
// lines that this compute unit has not read before in the launch.  Plain stores would be there sooner too, but the launch would end with that much more to write
// back (one prompt of 4 K tokens in 15 shares: 11.7 instead of 12.5 us until the last row is merged, but 19.0 instead of 17.0
// for the step).
//
// Who waits for whom, and what happens to the work of those who leave: handshake.h.
#pragma once

#include <hip/hip_runtime.h>

#include "handshake.h"
#include "internal.h"
#include "tree_attn_common.h"

namespace reader {

constexpr int kMaxMarks = kMaxAttnWorkgroups * 4 / 8;   // the workspace header holds so many

__device__ __forceinline__ mark_t agent_load(const mark_t *m) { return __hip_atomic_load(m, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void agent_store(mark_t *m, mark_t v) { __hip_atomic_store(m, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ float agent_load(const float *m) { return __hip_atomic_load(m, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void agent_store(float *m, float v) { __hip_atomic_store(m, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

__device__ __forceinline__ mark_t my_xcc() {
    unsigned id;
    asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID, 0, 4)" : "=s"(id));
    return (mark_t)id << kXccShift;
}

// One look of a wavefront at n <= kMaxMarks marks: are they all there?
__device__ __forceinline__ bool all_here(const mark_t *marks, int n, mark_t token, int lane) {
    bool here = true;
#pragma unroll 1
    for (int base = 0; base < n; base += 512) {
        mark_t v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = agent_load(marks + min(base + i * 64 + lane, n - 1));   // (asked for together)
#pragma unroll
        for (int i = 0; i < 8; ++i) here &= (v[i] & ~kMarkBits) == token;
    }
    return __all(here);
}

// A wavefront's way to the marks (handshake.h): one lane stores, all of them load.
struct AgentMarks {
    int lane;
    __device__ __forceinline__ void set(mark_t *m, mark_t v) const {
        if (lane == 0) agent_store(m, v);
    }
    __device__ __forceinline__ mark_t get(const mark_t *m) const { return agent_load(m); }
    __device__ __forceinline__ void settle() const { wait_vmcnt<0>(); }
    __device__ __forceinline__ bool swap(mark_t *m, mark_t from, mark_t to) const {
        int done = 0;
        if (lane == 0)
            done = __hip_atomic_compare_exchange_strong(m, &from, to, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ? 1 : 0;
        return __builtin_amdgcn_readfirstlane(done) != 0;
    }
    template <typename F>
    __device__ __forceinline__ bool wait_until(F &&seen, unsigned long long ticks) const {   // of the 100 MHz counter
        const unsigned long long start = __builtin_amdgcn_s_memrealtime();
        for (;;) {
            if (seen()) return true;
            if (__builtin_amdgcn_s_memrealtime() - start >= ticks) return false;
        }
    }
};

// 16 bytes written through to where every XCD sees them.  (The wait states: the registers may be written again behind it.)
typedef unsigned int u32x4_agent __attribute__((ext_vector_type(4)));
__device__ __forceinline__ void agent_store16(void *dst, u32x4_agent v) {
    asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 1" :: "v"(dst), "v"(v) : "memory");
}
__device__ __forceinline__ uint4 agent_load16(const void *src) {
    const mark_t a = agent_load(static_cast<const mark_t *>(src)), b = agent_load(static_cast<const mark_t *>(src) + 1);
    return make_uint4((unsigned)a, (unsigned)(a >> 32), (unsigned)b, (unsigned)(b >> 32));
}

}  // namespace reader
