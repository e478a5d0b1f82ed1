// Device primitives of the kernels whose waves wait for each other (flags,
// bounded polling, completion of stores) and the team of workgroups that runs
// several phases of one launch (k_fg_rest).
#pragma once
#include <hip/hip_runtime.h>

#include "kernels.h"

namespace kktlu {

namespace {

constexpr int WAVE = 64;

__device__ __forceinline__ int ld_flag(const int* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_flag(int* p, int v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// 2^20 polling rounds (each a device-scope load plus a short sleep, about a
// microsecond): far longer than any legitimate wait of one factorization or
// solve, short enough that a broken schedule drains in about a second
constexpr int SPIN_LIMIT = 1 << 20;

// Broadcast of a lane-0 value through a scalar register.  Unlike a shuffle,
// the result is provably wave-uniform, so loops whose exit depends on it stay
// uniform loops (a shuffle-broadcast exit condition lets the compiler treat
// the loop as divergent and split lane 0's flag store out of it).
__device__ __forceinline__ unsigned int bcast0(unsigned int v) {
  return (unsigned int)__builtin_amdgcn_readfirstlane((int)v);
}

// One more round of waiting allowed?  False once the limit is hit here (the
// wave raises *stall) or anywhere else (another wave raised it).
// The stall flag is polled every 64th round only; between rounds the wave
// pauses 64 cycles.  (A pause growing with the wait, meant to keep far-ahead
// waves off the memory system, measured slower: it delays the waves at the
// dependency front by up to the pause length.)
// stall[1] (DevStats::spin_limit) > 0 is a host-set debug limit on a wave's
// polls, read on its second poll and with every stall-flag check.
__device__ __forceinline__ bool keep_waiting(int* spins, int* stall) {
  if ((*spins & 63) == 63 || *spins == 1) {
    if ((*spins & 63) == 63 && ld_flag(stall)) return false;
    const int lim = stall[1];
    if (lim > 0 && *spins >= lim) {
      st_flag(stall, 1);
      return false;
    }
  }
  if (++*spins > SPIN_LIMIT) {
    st_flag(stall, 1);
    return false;
  }
  __builtin_amdgcn_s_sleep(1);
  return true;
}

// Every outstanding memory operation of this wave is complete (stores have
// reached the level their scope asks for)
__device__ __forceinline__ void stores_done() {
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
  __builtin_amdgcn_s_waitcnt(0);
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
}

// A team of the workgroups of one launch (k_fg_rest)
struct FgTeam {
  unsigned int* t;  // joined, size, barrier root, group counts, group release words
  unsigned int rank, size, gen;
  int* stall;
};
// The first workgroup's wait for the others, in polls of about a microsecond:
// long enough for another stream's launch to let go of the chip.  A team of the
// few workgroups that fit beside one goes through every phase that way: two
// iterations at 10k buses beside three refactorizations of 128 x 2k buses (8 ms)
// took 16-87 ms with 512 polls, 3.8 with 8192.  Alone, the whole grid joins
// within a few microseconds.
constexpr int FG_TEAM_POLLS = 8192;

__device__ __forceinline__ unsigned int ld_u32(const unsigned int* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_u32(unsigned int* p, unsigned int v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// false: the team was closed before this workgroup came
__device__ __forceinline__ bool fg_team_join(FgTeam& tm) {
  constexpr unsigned int CLOSED = 0x80000000u;
  __shared__ unsigned int s_rank, s_size;
  if (threadIdx.x < WAVE) {
    unsigned int* t = tm.t;
    const unsigned int m = bcast0(atomicAdd(t, threadIdx.x == 0 ? 1u : 0u));
    unsigned int size = 0;
    if (m == 0) {
      for (int k = 0; k < FG_TEAM_POLLS && bcast0(ld_u32(t)) < gridDim.x; k++)
        __builtin_amdgcn_s_sleep(1);
      size = bcast0(atomicOr(t, threadIdx.x == 0 ? CLOSED : 0u)) & ~CLOSED;
      st_u32(t + FG_TICK_STRIDE, size);
    } else if (!(m & CLOSED)) {
      int spins = 0;
      for (;;) {
        size = bcast0(ld_u32(t + FG_TICK_STRIDE));
        if (size != 0 || bcast0(keep_waiting(&spins, tm.stall) ? 1u : 0u) == 0u) break;
      }
    }
    s_rank = m;  // every lane writes the same value
    s_size = size;
  }
  __syncthreads();
  tm.rank = (unsigned int)__builtin_amdgcn_readfirstlane((int)s_rank);
  tm.size = (unsigned int)__builtin_amdgcn_readfirstlane((int)s_size);
  tm.gen = 0;
  return tm.size != 0;
}

// Barrier over the team; the workgroup that arrives last runs fin before any
// leaves.  False after a stall.  Every wave waits for its own stores first (a
// workgroup barrier does not, and thread 0's wait covers its own wave's stores
// only).  What passes from phase to phase is written and read device-coherent,
// so no caches are written back or invalidated, but for
//   FIN: fin reads and writes with plain accesses; the workgroup that runs it
//        invalidates its caches before and writes them back behind it;
//   ACQ: the phase behind the barrier reads with plain loads (what device-
//        coherent stores wrote); each workgroup invalidates its caches.
// (With a write-back and an invalidation by every workgroup at every barrier,
// six iterations took 2.86 ms at 10k buses and 4.53 at 30k.)  Each arrival group
// polls a release word of its own.
template <bool FIN, bool ACQ, class F>
__device__ __forceinline__ bool fg_team_barrier(FgTeam& tm, F fin) {
  __shared__ int s_last, s_ok;
  const unsigned int G = (unsigned int)FG_TICK_GROUPS;
  unsigned int* root = tm.t + 2 * FG_TICK_STRIDE;
  const unsigned int g = tm.rank % G, ng = (tm.size - g + G - 1) / G;
  const unsigned int ngr = tm.size < G ? tm.size : G;
  unsigned int* cnt = tm.t + (3 + g) * FG_TICK_STRIDE;
  unsigned int* go = tm.t + (3 + G) * FG_TICK_STRIDE;  // a word per group
  const unsigned int gen = ++tm.gen;
  stores_done();
  __syncthreads();
  if (threadIdx.x == 0) {
    int last = 0;
    if (__hip_atomic_fetch_add(cnt, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1u ==
        ng * gen)
      last = __hip_atomic_fetch_add(root, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1u ==
             ngr * gen;
    if (FIN && last) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    s_last = last;
    s_ok = 1;
  }
  __syncthreads();
  if (s_last) {
    if (FIN) {
      fin();
      stores_done();
      __syncthreads();
    }
    if (threadIdx.x < WAVE) {
      if (FIN) __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
      if (threadIdx.x < ngr) st_u32(go + threadIdx.x * FG_TICK_STRIDE, gen);
      if (ACQ) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    }
  } else if (threadIdx.x < WAVE) {
    int spins = 0;
    while (bcast0(ld_u32(go + g * FG_TICK_STRIDE)) < gen)
      if (bcast0(keep_waiting(&spins, tm.stall) ? 1u : 0u) == 0u) {
        s_ok = 0;  // every lane writes the same value
        break;
      }
    if (ACQ) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
  }
  __syncthreads();
  const bool ok = s_ok != 0;
  __syncthreads();  // s_last and s_ok are read before the next barrier sets them
  return ok;
}
template <bool ACQ = false>
__device__ __forceinline__ bool fg_team_sync(FgTeam& tm) {
  return fg_team_barrier<false, ACQ>(tm, [] {});
}
template <class F>
__device__ __forceinline__ bool fg_team_sync(FgTeam& tm, F fin) {
  return fg_team_barrier<true, false>(tm, fin);
}

}  // namespace

}  // namespace kktlu
