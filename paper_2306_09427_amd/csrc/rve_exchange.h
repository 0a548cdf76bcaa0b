// Exchange of words between the workgroups of a team (rve_spread.hip and the
// spread tangent of rve_tangent.hip).
//
// Every word carries its own tag, one relaxed 64-bit store of (tag << 32 |
// value) at device scope, and a reader polls the word until the tag is the one
// it waits for: no fence, no atomic counter, and no ordering between words.
// Two halves of an area alternate: a member writes tag n + 2 over tag n only
// after it has read every member's word of tag n + 1, which they publish after
// reading tag n.  Polls are bounded.
//
// Workgroups take slots from one counter, k consecutive slots for each task in
// the order of the list, so all tasks before the newest are complete teams of
// running workgroups, whatever k each has, and the newest is completed by the
// workgroups that finish theirs.  Task t uses area t % n_areas once the task
// before it there is over, which the area's first word says: (number of tasks
// done << 32 | last tag).
#pragma once

#include <hip/hip_runtime.h>

#include "rve_internal.h"
#include "rve_relax.h"

namespace rve {

namespace {

typedef unsigned long long u64;

__device__ __forceinline__ void put_word(u64* p, unsigned tag, unsigned v)
{
    __hip_atomic_store(p, (u64)tag << 32 | v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ u64 get_word(const u64* p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ bool tagged(u64 w, unsigned tag) { return (unsigned)(w >> 32) == tag; }

struct TeamSlot {
    int ticket, bad;
    unsigned tag;
};

// The workgroup's place in a team.
struct Team {
    int task, rank, k;
    u64* area;      // [1 + 2 halves]
    int gen;
    unsigned tag;   // of the last exchange; every member counts alike
};

// Next slot; false when none is left or the area did not come free in time.
template <typename Q>
__device__ __forceinline__ bool team_take(Q& A, TeamSlot& red, Team& tm)
{
    __syncthreads();
    if (threadIdx.x == 0) red.ticket = atomicAdd(A.queue, 1);
    __syncthreads();
    const int s = uniform32(red.ticket);
    int lo = 0, hi = A.n_tasks;   // task_first[lo] <= s < task_first[hi]
    if (s >= uniform32(A.task_first[hi])) return false;
    while (hi - lo > 1) {
        const int m = (lo + hi) >> 1;
        if (uniform32(A.task_first[m]) <= s)
            lo = m;
        else
            hi = m;
    }
    tm.task = lo;
    const int first = uniform32(A.task_first[lo]);
    tm.rank = s - first;
    tm.k = uniform32(A.task_first[lo + 1]) - first;
    tm.gen = lo / A.n_areas;
    tm.area = A.xchg + (int64_t)(lo - tm.gen * A.n_areas) * A.area_words;
    if (threadIdx.x == 0) {
        u64 v = get_word(tm.area);
        for (int polls = 1; (int)(v >> 32) != tm.gen && polls < A.spin_limit; ++polls) v = get_word(tm.area);
        if ((int)(v >> 32) != tm.gen) red.bad = 1;
        red.tag = (unsigned)v;
    }
    __syncthreads();
    tm.tag = (unsigned)uniform32((int)red.tag);
    return uniform32(red.bad) == 0;
}

// A member says that it is done; the first one waits for all (their last reads
// of the area are then over) and hands the area on.  `words`: the members'
// words of the half of the tag.  For the first member: whether all are done.
template <typename Q>
__device__ __forceinline__ bool team_done(Q& A, TeamSlot& red, Team& tm, u64* words)
{
    __syncthreads();
    const int t = threadIdx.x;
    if (t == 0) put_word(words + tm.rank, tm.tag, 0u);
    if (tm.rank != 0) return true;
    if (t < tm.k) {
        int polls = 1;
        u64 v = get_word(words + t);
        while (!tagged(v, tm.tag) && polls++ < A.spin_limit) v = get_word(words + t);
        if (!tagged(v, tm.tag)) red.bad = 1;
    }
    __syncthreads();
    const bool all = uniform32(red.bad) == 0;
    if (t == 0 && all)
        __hip_atomic_store(tm.area, (u64)(tm.gen + 1) << 32 | tm.tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return all;
}

}  // namespace

}  // namespace rve
