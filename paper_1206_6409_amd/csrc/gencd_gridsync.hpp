// Resident grids: workgroups of one launch that meet at barriers
// (gencd_grid.hip says how memory and residency are handled).
#pragma once

#include "gencd_common.hpp"
#include "gencd_kernels.hpp"

namespace gencd {

template <typename T>
__device__ __forceinline__ T agent_load(const T *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ void agent_store(T *p, T v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

constexpr int kGridPolls = 1 << 22;      // about 2 s; a barrier takes about a microsecond
constexpr int kEnrollPolls = 4096;       // about 2 ms for the whole grid to start
constexpr int32_t kClosed = 1 << 20;     // above any number of workgroups

// Members of the grid of up to `want` workgroups: this workgroup's index (-1:
// not one of them).
__device__ __forceinline__ int grid_enroll(GridCtl *c, int want, int *sm, int &members) {
  if (threadIdx.x == 0) {
    int idx = atomicAdd(&c->count, 1), m = 0;
    if (idx == 0) {
      for (int p = 0; p < kEnrollPolls && agent_load(&c->count) < want; ++p)
        __builtin_amdgcn_s_sleep(2);
      m = atomicAdd(&c->count, kClosed);
      agent_store(&c->members, m);
    } else if (idx < kClosed) {
      for (int p = 0; p < kGridPolls && (m = agent_load(&c->members)) == 0; ++p)
        __builtin_amdgcn_s_sleep(1);
    }
    sm[0] = idx < m ? idx : -1;
    sm[1] = m;
  }
  __syncthreads();
  members = sm[1];
  return sm[0];
}

// Every member has arrived at `round`, and its accesses before have been
// performed.  The flags are packed, so that the first wave reads all of them
// with one or two loads; one hop, no counter that the arrivals queue on.
__device__ __forceinline__ bool grid_barrier(GridCtl *c, unsigned long long *bad, int me, int members,
                                             int round, int *sm) {
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
  __syncthreads();
  if (threadIdx.x < kWave) {
    if (threadIdx.x == 0) agent_store(&c->flag[me], round);
    int p = 0;
    bool ok;
    do {
      ok = true;
      for (int i = int(threadIdx.x); i < members; i += kWave)
        ok = ok && agent_load(&c->flag[i]) >= round;
    } while (!__all(ok) && ++p < kGridPolls);
    if (threadIdx.x == 0) {
      sm[0] = p < kGridPolls;
      if (p >= kGridPolls) atomicOr(bad, 16ull);
    }
  }
  __syncthreads();
  return sm[0] != 0;
}

typedef int int4v __attribute__((ext_vector_type(4)));

// The packed rows as a buffer: 16-byte loads with the agent-scope policy.
struct Rows {
  __amdgpu_buffer_rsrc_t r;
};
__device__ __forceinline__ float4 row_load(const Rows &z, int32_t i) {
  const int4v v = __builtin_amdgcn_raw_buffer_load_b128(z.r, i * 16, 0, 16);
  return make_float4(__int_as_float(v.x), __int_as_float(v.y), __int_as_float(v.z), 0.0f);
}

}  // namespace gencd
