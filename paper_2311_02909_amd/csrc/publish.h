// What a call leaves for the host, by a kernel of its own or by the workgroup of the call's last kernel that is done last.
#pragma once
#include "bms_device.h"
#include "bms_internal.h"

namespace bms {

// A store past the die's cache.  Where all of a launch's stores are such, the launch is visible everywhere as soon as they have left
// the compute units, and its last workgroup may tell the host: releasing ordinary stores instead writes a cache back per workgroup,
// which took as long as the launch that it saved.
template <class T>
__device__ inline void store_through(T *p, T v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Everything that was there before this launch, by one workgroup of NT threads: the call's scalars but for `later`, a slot that this
// launch writes, and kRaised, which it may raise (the host clears that one), and the offsets but for the last hop's entries.
constexpr int kRaisedSlot = 60;
template <int NT>
__device__ inline void publish_before(const PublishArgs &a, const int64_t *later)
{
    const int tid = threadIdx.x;
    if (tid < 64 && a.scalars + tid != later) {
        const int64_t v = a.scalars[tid];
        if (tid != kRaisedSlot || v != 0)
            store_through(a.host + tid, v);
    }
    if (a.off)
        for (int32_t x = tid; x < a.L * (a.k + 1); x += NT) {
            const int32_t h = x / (a.k + 1), i = x - h * (a.k + 1);
            int64_t *to = a.off + (int64_t)h * 3 * (a.k + 1) + i;
            const int64_t r = a.rowoff[h][i];
            store_through(to, r);
            if (h + 1 < a.L)
                store_through(to + a.k + 1, a.rowptr[h][r]);
            store_through(to + 2 * (a.k + 1), a.coloff[h][i]);
        }
}

// Called by all threads of each of a launch's `parts` workgroups when the workgroup has written everything, with store_through:
// the one that comes here last says that the call is done.
__device__ inline void announce_through(const PublishArgs &a, uint32_t parts)
{
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); // every wave's
    __syncthreads();
    if (threadIdx.x == 0 && __hip_atomic_fetch_add(a.done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == parts - 1u) {
        __hip_atomic_store(a.done, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); // a call that the host makes now, on another stream, counts from zero
        store_through(a.arrived, a.arrival);
    }
}

} // namespace bms
