// team.h -- a team of workgroups on one XCD with its own barrier, for work in
// many short dependent phases (the small levels of a cycle, the rounds of a
// matching), where a kernel boundary per phase costs more than the phase.
//
// A launch has 8 W workgroups; those with blockIdx % 8 == pick are candidates
// (the chip hands workgroups to its 8 XCDs in turn, so they land on one XCD),
// the rest leave at once.  The candidates that are running when the first of
// them closes the enrolment, and that run on its XCD by the hardware's own
// XCC_ID, are the team: every member is resident, so every barrier ends
// whatever else the device runs, and a candidate that starts late just leaves.
// At least one workgroup is in the team, and its size n only decides how the
// rows are shared out: no result may depend on it.
//
// The CUs of an XCD share one L2, to which stores are written through.  So a
// barrier needs the stores' acknowledgements (vmcnt 0) and a flag per member,
// and what other members wrote is read past the L1 (team_ld, a load of device
// scope): 0.28 us a barrier of 32 workgroups, against 2.0 us with an
// invalidation of the caches in it and 4.5-6 us for a kernel of its own.  A
// device-wide release would write back the whole L2.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace llg {

constexpr int TEAM_W = 32;  // candidates (an XCD has 32 CUs)
constexpr int TEAM_T = 1024;  // threads of a member
constexpr int TEAM_POLLS = 64;

// One per stream that launches teams; zero before the first launch and after
// every launch.  When all candidates are members, the last to leave clears it.
// Otherwise the last one may run on another XCD, and its zeros would wait in
// that one's L2 while the members' flags are in that of theirs, their order of
// arrival in memory open: then the last member clears the flags, and the last
// candidate the rest, past its L2.
struct TeamState {
  unsigned long long enrol;  // candidates arrived, 7 bits per XCD; bit 63: closed
  unsigned pad0[30];
  unsigned closed;  // (leader's XCD + 1) << 8 | members, once closed
  unsigned pad1[31];
  unsigned left;  // candidates that have left
  unsigned pad2[30];
  unsigned done;  // members that have left a team of fewer; of the team's XCD, as the flags
  unsigned flag[TEAM_W];  // barriers each member has reached
  // totals the members publish for a scan, by slot (written again only after
  // two barriers; not cleared)
  int32_t sum[4][TEAM_W];
};

#if defined(__HIPCC__)
__device__ inline unsigned team_xcc() { return __builtin_amdgcn_s_getreg(20 | (3 << 11)) & 7; }  // HW_REG_XCC_ID

// a value that another member may have written since the launch
template <typename X>
__device__ inline X team_ld(const X* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

struct Team {
  TeamState* s;
  unsigned rank, n, epoch;

  // All threads of the workgroup; false: not a member, and nothing is left to do.
  // polls: how long the first waits for the others, about 0.3 us each.
  __device__ bool join(TeamState* st, unsigned pick, int polls = TEAM_POLLS) {
    __shared__ unsigned sh[3];
    s = st;
    epoch = 0;
    if (blockIdx.x % 8 != pick) return false;
    if (threadIdx.x == 0) {
      const unsigned x = team_xcc();
      const unsigned long long old =
          __hip_atomic_fetch_add(&s->enrol, 1ull << (7 * x), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      unsigned ok = 0, r = (unsigned)(old >> (7 * x)) & 127u, cnt = 0;
      if (!(old >> 63)) {
        if (old == 0) {  // the first: closes when all are here, or after that time
          for (int k = 0; k < polls; ++k)
            if (((team_ld(&s->enrol) >> (7 * x)) & 127u) >= TEAM_W) break;
          const unsigned long long v =
              __hip_atomic_fetch_or(&s->enrol, 1ull << 63, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          cnt = (unsigned)(v >> (7 * x)) & 127u;
          __hip_atomic_store(&s->closed, (x + 1) << 8 | cnt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          ok = 1;
        } else {  // the first is running: it closes the enrolment
          unsigned c;
          do c = team_ld(&s->closed);
          while (c == 0);
          ok = (c >> 8) == x + 1;
          cnt = c & 255u;
        }
      }
      sh[0] = ok;
      sh[1] = r;
      sh[2] = cnt;
    }
    __syncthreads();
    rank = __builtin_amdgcn_readfirstlane(sh[1]);
    n = __builtin_amdgcn_readfirstlane(sh[2]);
    if (sh[0]) return true;
    depart<false>();
    return false;
  }

  // Every thread of every member: a team_ld after it sees the stores before it.
  __device__ void barrier() {
    ++epoch;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x < 64) {
      // a store of workgroup scope goes to the XCD's L2 and no further
      if (threadIdx.x == 0)
        __hip_atomic_store(&s->flag[rank], epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      const unsigned l = threadIdx.x < n ? threadIdx.x : 0;
      while (!__all(team_ld(&s->flag[l]) >= epoch)) {
      }
    }
    __syncthreads();
  }

  // Every member, once, when it needs the state no more.
  __device__ void leave() { depart<true>(); }

  template <bool MEMBER>
  __device__ void depart() {
    __syncthreads();
    if (threadIdx.x == 0) {
      const bool whole = MEMBER && n == TEAM_W;
      if (MEMBER && !whole) {
        // the leader's store of `closed` comes before its count
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        if (__hip_atomic_fetch_add(&s->done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) + 1 == n) {
          s->done = 0;
          for (int i = 0; i < TEAM_W; ++i) s->flag[i] = 0;
        }
      }
      const unsigned k = __hip_atomic_fetch_add(&s->left, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (k + 1 < TEAM_W) return;
      if (whole) {
        s->enrol = 0;
        s->closed = 0;
        s->left = 0;
        for (int i = 0; i < TEAM_W; ++i) s->flag[i] = 0;
      } else {
        __hip_atomic_store(&s->enrol, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&s->closed, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&s->left, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
    }
  }
};
#endif

}  // namespace llg
