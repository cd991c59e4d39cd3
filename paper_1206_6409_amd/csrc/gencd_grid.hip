// Whole epochs of a mid-size problem on a grid of resident workgroups.
//
// A window of a few thousand columns is a few tens of thousands of entries:
// about two microseconds of dependent loads and atomics, but two launches
// with a drained device between them (11 us an iteration on MI355X, of which
// the two kernels' own chains of loads are most).  Here one launch runs all
// windows of an epoch.  Its workgroups meet at a barrier where the two-launch
// form has a kernel boundary, and a wave loads the descriptors, entries and
// weights of its share of the next windows while it works on the current one,
// so what is left between two barriers is the row gather, the reduction and
// the step, or the atomics.
//
// What bounds it: the two barriers (about 1.2 us each) and the chains between
// them.  Per window, two launches -> this: 2k entries 7.3 -> 4.6 us, 15k 9.9
// -> 7.0, 61k (|J| = 4096 of the text-like matrix) 11.0 -> 10.0, 122k 12.7 ->
// 15.0.  Coloring, 560 windows of 10k entries: 7.4 -> 5.2 us.
//
// Memory between workgroups.  The eight XCDs have an L2 each, so everything
// one workgroup writes and another reads inside the launch goes through
// agent-scope accesses: the rows are read with the agent-scope cache policy
// and changed by atomics (Coloring: by agent-scope stores), partial sums and
// barrier flags are agent-scope atomics.  A wave waits for its own accesses
// before its workgroup raises its flag.  What the launch only reads (matrix,
// order, curvature) takes the ordinary path, and a column's weight is read
// and written by the waves of that column alone, once per epoch.
//
// Residency.  The workgroups that meet are those that enrolled before the
// first of them closed the list; a workgroup that starts later leaves at
// once, so a device busy with other work gives a smaller grid, never a wait
// for a workgroup that is not running.  Every wait is bounded; a wait that
// runs out raises an error flag that the host reads with the next check.
//
// Beside other work an epoch waits for room once, the separate launches 2 T
// times, but a workgroup of 1024 threads needs more room than theirs of 256.
// Two launches -> this, ms a solve: beside a stream of 8192^3 bf16 products
// |J| = 5000 of 10 entries 480 -> 31, |J| = 200 1615 -> 29; beside FP64
// elementwise work 21.6 -> 26 and 53 -> 18; beside long-running workgroups that
// leave 7 waves free on every CU (sums of 1600 long rows) 10.5 -> 50 and
// 28.6 -> 15.5.  A lower bound on the members with a way back to the launches
// gains up to a factor of two in the last kind of case only (17 -> 11 beside
// 1400 rows) and would lose an order of magnitude in the first.
#include <algorithm>

#include "gencd_gridsync.hpp"

namespace gencd {

// Compensated update of a row that this lane owns in the window (columns of a
// colour class have disjoint rows), from its values at the window's start.
__device__ __forceinline__ void row_store(float4 *zs, int32_t i, float hi, float lo, float d,
                                          float v) {
  const float p = d * v;
  const float pe = fmaf(d, v, -p);
  const float h = hi + p, l = lo + (twosum_err(hi, p) + pe);
  const unsigned long long b = (static_cast<unsigned long long>(__float_as_uint(l)) << 32) |
                               static_cast<unsigned long long>(__float_as_uint(h));
  agent_store(reinterpret_cast<unsigned long long *>(zs + i), b);
}

// One wave's work unit of a window: 64 / GS short columns, or one piece of a
// long column; kUnroll entries per lane either way.
struct Unit {
  int4 d;         // the group's descriptor (length 0: nothing to do)
  int32_t pf, pe; // split column: its pieces [pf, pe)
  float w, c;
  int32_t ri[kUnroll];
  float vv[kUnroll];
};

// 16 waves with one unit each beat 8 waves with two and 4 with three by 2 to
// 10% (the units of a wave follow each other through its instructions).
constexpr int kGridThreads = 1024;
constexpr int kUnits = 1;  // units a wave holds in registers; more are taken from memory

struct WindowPos {
  int32_t P0, P1, q0, q1;  // positions and long pieces
};

template <int GS>
struct GridWave {
  const IterArgs &a;
  int wave, nw, lane;

  // Bounds of the windows from `base` on, one per lane, read back by
  // readlane: a load per window would have to be waited for at its first use.
  int32_t base, wb, wo;
  __device__ __forceinline__ void bounds(int32_t t, int32_t T) {
    base = t;
    const int32_t i = t + lane < T ? t + lane : T;
    wb = a.wbl[i];
    wo = a.win_off ? a.win_off[i] : 0;
  }
  __device__ __forceinline__ WindowPos window(int32_t t, int32_t T) {
    WindowPos w{0, 0, 0, 0};
    if (t >= T) return w;
    if (t - base > kWave - 2) bounds(t, T);
    if (a.win_off) {
      w.P0 = __builtin_amdgcn_readlane(wo, t - base);
      w.P1 = __builtin_amdgcn_readlane(wo, t - base + 1);
    } else {
      w.P0 = t * a.S;
      w.P1 = a.k_live - w.P0 < a.S ? a.k_live : w.P0 + a.S;
    }
    w.q0 = __builtin_amdgcn_readlane(wb, t - base);
    w.q1 = __builtin_amdgcn_readlane(wb, t - base + 1);
    return w;
  }
  __device__ __forceinline__ int32_t units(const WindowPos &w) const {
    return w.q1 - w.q0 + (w.P1 - w.P0 + kWave / GS - 1) / (kWave / GS);
  }
  // long unit: one piece per wave
  __device__ __forceinline__ bool is_long(const WindowPos &w, int32_t u) const {
    return u < w.q1 - w.q0;
  }
  __device__ __forceinline__ int4 desc(const WindowPos &w, int32_t u) const {
    if (is_long(w, u)) return a.desc_l[w.q0 + u];
    const int32_t p = w.P0 + (u - (w.q1 - w.q0)) * (kWave / GS) + lane / GS;
    return p < w.P1 ? a.desc_s[p] : make_int4(0, 0, 0, 0);
  }
  // entries (first kUnroll of a lane), weight, curvature of a unit
  __device__ __forceinline__ void fill(bool lng, Unit &x) const {
    const int32_t len = x.d.w & 0x7FFFFFFF;
    const uint32_t beg = uint32_t(x.d.x);
    const int32_t g = lng ? kWave : GS, l = lng ? lane : (lane & (GS - 1));
    x.w = a.w[x.d.y];
    x.c = a.c[x.d.y];
    // nothing here may use a loaded value: the loads stay in flight
    if (lng) {  // (only split columns read these)
      x.pf = a.loff[x.d.z];
      x.pe = a.loff[x.d.z + 1];
    }
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      const int32_t e = u * g + l;
      const int64_t at = int64_t(beg) + (e < len ? e : 0);
      x.ri[u] = a.row_idx[at];
      x.vv[u] = a.val[at];
    }
  }
  // whether entry u of this lane exists (past the end ri, vv repeat the first)
  __device__ __forceinline__ bool has(bool lng, const Unit &x, int u) const {
    return u * (lng ? kWave : GS) + (lng ? lane : (lane & (GS - 1))) < (x.d.w & 0x7FFFFFFF);
  }
};

// Sum of the four row sums of a wave, in every lane.
__device__ __forceinline__ float rows_sum(float x) {
  const int b = __float_as_int(x);
  return (__int_as_float(__builtin_amdgcn_readlane(b, 0)) +
          __int_as_float(__builtin_amdgcn_readlane(b, 16))) +
         (__int_as_float(__builtin_amdgcn_readlane(b, 32)) +
          __int_as_float(__builtin_amdgcn_readlane(b, 48)));
}

// Sum of a unit's lanes in every lane: GS lanes of a short column, or the wave.
template <int GS>
__device__ __forceinline__ float unit_sum(bool lng, float s) {
  if constexpr (GS <= 16) {
    s = row_group_sum<GS>(s);
    if (!lng) return s;  // uniform over the wave
    if constexpr (GS < 16) {
      if constexpr (GS < 8) s += dpp_move<0x141>(s);
      s += dpp_move<0x140>(s);
    }
    return rows_sum(s);
  } else {
    return lng ? group_sum<kWave>(s) : group_sum<GS>(s);
  }
}

// Partial sums of a split column, in piece order (every piece's wave gets
// the same value).
__device__ __forceinline__ float split_total(const float *part, int32_t pf, int32_t np, int lane) {
  float t = 0.0f;
  for (int32_t u0 = 0; u0 < np; u0 += kWave * kUnroll) {
    float v[kUnroll];
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      const int32_t i = u0 + u * kWave + lane;
      v[u] = i < np ? agent_load(&part[pf + i]) : 0.0f;
    }
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) t += v[u];
  }
  return rows_sum(row_group_sum<16>(t));
}

// Windows [t0, T) of an epoch.  MODE 0: Jacobi windows, atomic scatter.  MODE 1: Coloring (rows of a window
// disjoint): compensated stores.
template <int GS, int MODE>
__global__ __launch_bounds__(kGridThreads) void k_epoch_grid(IterArgs a, GridCtl *ctl,
                                                             unsigned long long *bad, int32_t t0,
                                                             int32_t T) {
  __shared__ int sm[2];
  int members;
  const int me = __builtin_amdgcn_readfirstlane(grid_enroll(ctl, int(gridDim.x), sm, members));
  members = __builtin_amdgcn_readfirstlane(members);
  if (me < 0) return;
  // waves numbered slot-major: consecutive units go to different workgroups
  const int lane = int(threadIdx.x) & (kWave - 1);
  const int slot = __builtin_amdgcn_readfirstlane(int(threadIdx.x) / kWave);
  GridWave<GS> gw{a, slot * members + me, members * (kGridThreads / kWave), lane, 0, 0, 0};
  gw.bounds(t0, T);
  const Rows z{__builtin_amdgcn_make_buffer_rsrc(a.zs, 0, int(a.nrows * 16), 0x00027000)};
  Unit cur[kUnits], nxt[kUnits];
  WindowPos wp = gw.window(t0, T), wn = gw.window(t0 + 1, T);
#pragma unroll
  for (int k = 0; k < kUnits; ++k) {
    const int32_t u = gw.wave + k * gw.nw;
    cur[k].d = u < gw.units(wp) ? gw.desc(wp, u) : make_int4(0, 0, 0, 0);
    nxt[k].d = u < gw.units(wn) ? gw.desc(wn, u) : make_int4(0, 0, 0, 0);
  }
#pragma unroll
  for (int k = 0; k < kUnits; ++k) gw.fill(gw.is_long(wp, gw.wave + k * gw.nw), cur[k]);
  int round = 0;
  for (int32_t t = t0; t < T; ++t) {
    const WindowPos w2 = gw.window(t + 2, T);
    const int32_t nu = gw.units(wp);
    if (nu == 0) {  // an empty colour class: the same decision in every workgroup
      wp = wn;
      wn = w2;
#pragma unroll
      for (int k = 0; k < kUnits; ++k) {
        const int32_t u = gw.wave + k * gw.nw;
        cur[k].d = nxt[k].d;
        if (u < gw.units(wp)) gw.fill(gw.is_long(wp, u), cur[k]);
        nxt[k].d = u < gw.units(wn) ? gw.desc(wn, u) : make_int4(0, 0, 0, 0);
      }
      continue;
    }
    // rows of the units in registers
    float zh[kUnits][kUnroll], zl[kUnits][kUnroll], yy[kUnits][kUnroll];
#pragma unroll
    for (int k = 0; k < kUnits; ++k) {
      if (gw.wave + k * gw.nw >= nu) break;  // uniform over the wave
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) {
        const float4 r = row_load(z, cur[k].ri[u]);
        zh[k][u] = r.x;
        zl[k][u] = r.y;
        yy[k][u] = r.z;
      }
    }
    // the next window's entries, and the descriptors of the one after
    int4 dd[kUnits];
#pragma unroll
    for (int k = 0; k < kUnits; ++k) {
      const int32_t u = gw.wave + k * gw.nw;
      if (u < gw.units(wn)) gw.fill(gw.is_long(wn, u), nxt[k]);
      dd[k] = u < gw.units(w2) ? gw.desc(w2, u) : make_int4(0, 0, 0, 0);
    }
    // Propose
    float d[kUnits];
#pragma unroll
    for (int k = 0; k < kUnits; ++k) {
      d[k] = 0.0f;
      const int32_t u = gw.wave + k * gw.nw;
      if (u >= nu) break;
      const bool lng = gw.is_long(wp, u);
      float s = 0.0f;
#pragma unroll
      for (int v = 0; v < kUnroll; ++v)
        if (gw.has(lng, cur[k], v)) s += cur[k].vv[v] * dloss_f32(a.loss, yy[k][v], zh[k][v] + zl[k][v]);
      s = unit_sum<GS>(lng, s);
      if (lng && cur[k].d.w >= 0) {
        if (lane == 0) agent_store(&a.gacc[wp.q0 + u], s);
      } else {
        float ph;
        propose_f32(s / a.n_f, cur[k].c, cur[k].w, a.lam, d[k], ph);
      }
    }
    // units beyond the registers: increments of short and one-piece columns
    // to delta (read back by the same lanes), partial sums to gacc
    for (int32_t u = gw.wave + kUnits * gw.nw; u < nu; u += gw.nw) {
      Unit x;
      const bool lng = gw.is_long(wp, u);
      x.d = gw.desc(wp, u);
      gw.fill(lng, x);
      float s = 0.0f;
#pragma unroll
      for (int v = 0; v < kUnroll; ++v) {
        const float4 r = row_load(z, x.ri[v]);
        if (gw.has(lng, x, v)) s += x.vv[v] * dloss_f32(a.loss, r.z, r.x + r.y);
      }
      s = unit_sum<GS>(lng, s);
      if (lng && x.d.w >= 0) {
        if (lane == 0) {
          agent_store(&a.gacc[wp.q0 + u], s);
          // the weight before any wave of the column updates it
          agent_store(&a.wsnap[x.d.z - wp.P0], x.w);
        }
      } else {
        float de, ph;
        propose_f32(s / a.n_f, x.c, x.w, a.lam, de, ph);
        if ((x.d.w & 0x7FFFFFFF) > 0) a.delta[x.d.z - wp.P0] = de;
      }
    }
    if (!grid_barrier(ctl, bad, me, members, ++round, sm)) return;
    // Update
#pragma unroll
    for (int k = 0; k < kUnits; ++k) {
      const int32_t u = gw.wave + k * gw.nw;
      if (u >= nu) break;
      const bool lng = gw.is_long(wp, u);
      const bool split = lng && cur[k].d.w >= 0;
      if (split) {
        float ph;
        const float g = split_total(a.gacc, cur[k].pf, cur[k].pe - cur[k].pf, lane) / a.n_f;
        propose_f32(g, cur[k].c, cur[k].w, a.lam, d[k], ph);
      }
      if (d[k] == 0.0f || (cur[k].d.w & 0x7FFFFFFF) == 0) continue;
      const bool owner = lng ? lane == 0 && (!split || wp.q0 + u == cur[k].pf)
                             : (lane & (GS - 1)) == 0;
      if (owner) a.w[cur[k].d.y] = cur[k].w + d[k];
#pragma unroll
      for (int v = 0; v < kUnroll; ++v) {
        const int32_t i = cur[k].ri[v];
        if (!gw.has(lng, cur[k], v)) continue;
        if (MODE == 0)
          atomicAdd(&a.zs[i].y, d[k] * cur[k].vv[v]);
        else
          row_store(a.zs, i, zh[k][v], zl[k][v], d[k], cur[k].vv[v]);
      }
    }
    for (int32_t u = gw.wave + kUnits * gw.nw; u < nu; u += gw.nw) {
      Unit x;
      const bool lng = gw.is_long(wp, u);
      x.d = gw.desc(wp, u);
      gw.fill(lng, x);
      const bool split = lng && x.d.w >= 0;
      float de, ph;
      if (split) {
        const float g = split_total(a.gacc, x.pf, x.pe - x.pf, lane) / a.n_f;
        x.w = agent_load(&a.wsnap[x.d.z - wp.P0]);
        propose_f32(g, x.c, x.w, a.lam, de, ph);
      } else {
        de = (x.d.w & 0x7FFFFFFF) > 0 ? a.delta[x.d.z - wp.P0] : 0.0f;
      }
      if (de == 0.0f) continue;
      const bool owner = lng ? lane == 0 && (!split || wp.q0 + u == x.pf)
                             : (lane & (GS - 1)) == 0;
      if (owner) a.w[x.d.y] = x.w + de;
#pragma unroll
      for (int v = 0; v < kUnroll; ++v) {
        const int32_t i = x.ri[v];
        if (!gw.has(lng, x, v)) continue;
        if (MODE == 0) {
          atomicAdd(&a.zs[i].y, de * x.vv[v]);
        } else {
          const float4 r = row_load(z, i);
          row_store(a.zs, i, r.x, r.y, de, x.vv[v]);
        }
      }
    }
    if (!grid_barrier(ctl, bad, me, members, ++round, sm)) return;
    wp = wn;
    wn = w2;
#pragma unroll
    for (int k = 0; k < kUnits; ++k) {
      cur[k] = nxt[k];
      nxt[k].d = dd[k];
    }
  }
}

// A barrier at which a workgroup can leave a 16-bit mark for the others: the
// flag is round << 16 | mark of its last marked window.  A member that is
// already past this barrier shows the same mark until it passes the next
// barrier, for which it needs this workgroup.  *seen: some member's mark is
// `mark`.
__device__ __forceinline__ bool grid_barrier_marked(GridCtl *c, unsigned long long *bad, int me,
                                                    int members, uint32_t round, uint32_t own,
                                                    uint32_t mark, int *sm, bool *seen) {
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
  __syncthreads();
  if (threadIdx.x < kWave) {
    if (threadIdx.x == 0) agent_store(&c->flag[me], int32_t(round << 16 | own));
    int p = 0;
    bool ok, hit;
    do {
      ok = true;
      hit = false;
      for (int i = int(threadIdx.x); i < members; i += kWave) {
        const uint32_t f = uint32_t(agent_load(&c->flag[i]));
        ok = ok && (f >> 16) >= round;
        hit = hit || (f & 0xFFFFu) == mark;
      }
    } while (!__all(ok) && ++p < kGridPolls);
    const bool any = __any(hit);
    if (threadIdx.x == 0) {
      sm[0] = p < kGridPolls;
      sm[1] = any;
      if (p >= kGridPolls) atomicOr(bad, 16ull);
    }
  }
  __syncthreads();
  *seen = sm[1] != 0;
  return sm[0] != 0;
}

// Thread-Greedy (section 2.3): in each block of B window positions the first
// one with the smallest phi is accepted.  Per window: Propose (increments and
// proxies of short and one-piece columns, partial sums of split ones, as
// agent-scope words) | barrier | one wave per block finishes the block's split
// columns, finds the winner and scatters it | barrier.  A winner of more than
// kDirect entries is published instead and scattered by all waves, piece by
// chunk, before a third barrier that only such windows have (with a text-like
// matrix most have one).  Bound by the three or two barriers and the chains
// between them.  Per window of |J| = 1024, B = 64, 14k entries: three launches
// 17 us, this 12.
constexpr int32_t kDirect = kWave * kUnroll;

// One window position as its block's accept sees it.
struct AcceptPos {
  int4 ds;          // short descriptor (length 0: long column)
  int32_t pf, pe;   // pieces of a long column
  float c, w;
};
constexpr int kSplits = 4;

template <int GS>
__global__ __launch_bounds__(kGridThreads) void k_greedy_grid(IterArgs a, GridCtl *ctl,
                                                              unsigned long long *bad, int32_t t0,
                                                              int32_t T, int32_t B) {
  __shared__ int sm[2];
  __shared__ int smb[2];
  int members;
  const int me = __builtin_amdgcn_readfirstlane(grid_enroll(ctl, int(gridDim.x), sm, members));
  members = __builtin_amdgcn_readfirstlane(members);
  if (me < 0) return;
  const int lane = int(threadIdx.x) & (kWave - 1);
  const int slot = __builtin_amdgcn_readfirstlane(int(threadIdx.x) / kWave);
  GridWave<GS> gw{a, slot * members + me, members * (kGridThreads / kWave), lane, 0, 0, 0};
  gw.bounds(t0, T);
  const Rows z{__builtin_amdgcn_make_buffer_rsrc(a.zs, 0, int(a.nrows * 16), 0x00027000)};
  // {phi, delta} of a window slot in one word (delta and phi are adjacent
  // arrays of k); the published winners {first entry, length}, {0, delta} in the
  // count scratch (two words a block of at least two positions)
  unsigned long long *const prop = reinterpret_cast<unsigned long long *>(a.delta);
  unsigned long long *const win = reinterpret_cast<unsigned long long *>(a.bw_pos);
  auto word = [](uint32_t hi, float d) {
    return static_cast<unsigned long long>(hi) << 32 | __float_as_uint(d);
  };
  WindowPos wp = gw.window(t0, T), wn = gw.window(t0 + 1, T);
  Unit cur, nxt;
  cur.d = gw.wave < gw.units(wp) ? gw.desc(wp, gw.wave) : make_int4(0, 0, 0, 0);
  nxt.d = gw.wave < gw.units(wn) ? gw.desc(wn, gw.wave) : make_int4(0, 0, 0, 0);
  gw.fill(gw.is_long(wp, gw.wave), cur);
  unsigned long long acc_nnz = 0, acc_cnt = 0;  // this wave's accepted columns (lane 0)
  uint32_t round = 0, own = 0;
  __shared__ uint32_t published;  // this workgroup's last window with a published winner
  if (threadIdx.x == 0) published = 0;
  __syncthreads();
  auto propose = [&](const Unit &x, int32_t u, const float4 (&r)[kUnroll]) {
    const bool lng = gw.is_long(wp, u);
    float s = 0.0f;
#pragma unroll
    for (int v = 0; v < kUnroll; ++v)
      if (gw.has(lng, x, v)) s += x.vv[v] * dloss_f32(a.loss, r[v].z, r[v].x + r[v].y);
    s = unit_sum<GS>(lng, s);
    if (lng && x.d.w >= 0) {
      if (lane == 0) agent_store(&a.gacc[wp.q0 + u], s);
    } else if ((x.d.w & 0x7FFFFFFF) > 0) {
      float d, ph;
      propose_f32(s / a.n_f, x.c, x.w, a.lam, d, ph);
      if ((lng ? lane : (lane & (GS - 1))) == 0)
        agent_store(&prop[x.d.z - wp.P0], word(__float_as_uint(ph), d));
    }
  };
  // what an accept reads of a position that no wave writes, in two stages
  auto accept_desc = [&](int32_t q, AcceptPos &x) {
    x.ds = a.desc_s[q];
    x.pf = a.loff[q];
    x.pe = a.loff[q + 1];
  };
  auto accept_scalars = [&](AcceptPos &x) {
    x.c = a.c[x.ds.y];
    x.w = a.w[x.ds.y];
  };
  // position of this lane in the wave's first block of a window
  auto accept_pos = [&](const WindowPos &w) {
    const int32_t lo = w.P0 + gw.wave * B, p = lo + lane;
    return lane < B && p < w.P1 ? p : (lo < w.P1 ? lo : w.P0);
  };
  AcceptPos at{}, atn{};
  accept_desc(accept_pos(wp), at);
  for (int32_t t = t0; t < T; ++t) {
    const WindowPos w2 = gw.window(t + 2, T);
    const int32_t nu = gw.units(wp);
    const uint32_t mark = uint32_t(t + 1) & 0xFFFFu;
    float4 r[kUnroll];
    if (gw.wave < nu) {
#pragma unroll
      for (int v = 0; v < kUnroll; ++v) r[v] = row_load(z, cur.ri[v]);
    }
    if (gw.wave < gw.units(wn)) gw.fill(gw.is_long(wn, gw.wave), nxt);
    const int4 dd = gw.wave < gw.units(w2) ? gw.desc(w2, gw.wave) : make_int4(0, 0, 0, 0);
    const int32_t m = wp.P1 - wp.P0, nblk = (m + B - 1) / B;
    if (gw.wave < nblk) accept_scalars(at);
    if (t + 1 < T) accept_desc(accept_pos(wn), atn);
    if (gw.wave < nu) propose(cur, gw.wave, r);
    for (int32_t u = gw.wave + gw.nw; u < nu; u += gw.nw) {
      Unit x;
      x.d = gw.desc(wp, u);
      gw.fill(gw.is_long(wp, u), x);
#pragma unroll
      for (int v = 0; v < kUnroll; ++v) r[v] = row_load(z, x.ri[v]);
      propose(x, u, r);
    }
    bool unused;
    if (!grid_barrier_marked(ctl, bad, me, members, ++round, own, ~0u, smb, &unused)) return;
    // Accept and scatter
    for (int32_t b = gw.wave; b < nblk; b += gw.nw) {
      const int32_t lo = wp.P0 + b * B, hi = lo + B < wp.P1 ? lo + B : wp.P1;
      float best = INFINITY, bd = 0.0f;
      int32_t bpos = INT32_MAX;
      int4 bds = make_int4(0, 0, 0, 0);
      for (int32_t c0 = lo; c0 < hi; c0 += kWave) {
        const int32_t p = c0 + lane;
        const bool ok = p < hi;
        if (b != gw.wave || c0 != lo) {
          accept_desc(ok ? p : lo, at);
          accept_scalars(at);
        }
        const int4 ds = at.ds;
        const unsigned long long v = agent_load(&prop[(ok ? p : lo) - wp.P0]);
        float ph = __uint_as_float(uint32_t(v >> 32)), d = __uint_as_float(uint32_t(v));
        unsigned long long left = __ballot(ok && at.pe - at.pf > 1);
        while (left) {  // split columns of the block, kSplits of them at once
          int g[kSplits];
          float part[kSplits];
#pragma unroll
          for (int i = 0; i < kSplits; ++i) {
            g[i] = left ? __builtin_ctzll(left) : -1;
            left &= left - 1;  // 0 stays 0
            part[i] = 0.0f;
            if (g[i] < 0) continue;
            const int32_t f = __builtin_amdgcn_readlane(at.pf, g[i]);
            const int32_t np = __builtin_amdgcn_readlane(at.pe, g[i]) - f;
            if (lane < np) part[i] = agent_load(&a.gacc[f + lane]);
            for (int32_t q = lane + kWave; q < np; q += kWave) part[i] += agent_load(&a.gacc[f + q]);
          }
#pragma unroll
          for (int i = 0; i < kSplits; ++i) {
            if (g[i] < 0) break;
            const float grad = rows_sum(row_group_sum<16>(part[i])) / a.n_f;
            float de, pp;
            propose_f32(grad, at.c, at.w, a.lam, de, pp);  // lane g[i]'s is the column's
            if (lane == g[i]) {
              ph = pp;
              d = de;
            }
          }
        }
        if (ok && ph < best) {  // a lane's positions come in increasing order
          best = ph;
          bpos = p;
          bd = d;
          bds = ds;
        }
      }
      float wb = best;
      int32_t wpos = bpos;
#pragma unroll
      for (int off = kWave / 2; off > 0; off >>= 1) {
        const float ob = __shfl_xor(wb, off);
        const int32_t op = __shfl_xor(wpos, off);
        if (ob < wb || (ob == wb && op < wpos)) {
          wb = ob;
          wpos = op;
        }
      }
      uint32_t pub_beg = 0, pub_len = 0;
      float d = 0.0f;
      if (wpos != INT32_MAX) {  // uniform: every lane holds the winner
        const int g = __builtin_ctzll(__ballot(bpos == wpos));
        d = __shfl(bd, g);
        const int32_t j = __shfl(bds.y, g), len0 = __shfl(bds.w, g) & 0x7FFFFFFF;
        uint32_t beg = uint32_t(__shfl(bds.x, g));
        int32_t len = len0;
        if (len0 == 0) {  // a long column
          const int64_t cb = a.col_ptr[j];
          beg = uint32_t(cb);
          len = int32_t(a.col_ptr[j + 1] - cb);
        }
        if (lane == 0) {
          acc_nnz += (unsigned long long)len;
          acc_cnt += 1ull;
          if (d != 0.0f) a.w[j] += d;
        }
        if (d != 0.0f && len > kDirect) {
          pub_beg = beg;
          pub_len = uint32_t(len);
          if (lane == 0) published = mark;
        } else if (d != 0.0f) {
          int32_t ri[kUnroll];
          float vv[kUnroll];
#pragma unroll
          for (int v = 0; v < kUnroll; ++v) {
            const int32_t e = v * kWave + lane;
            const int64_t from = int64_t(beg) + (e < len ? e : 0);
            ri[v] = a.row_idx[from];
            vv[v] = a.val[from];
          }
#pragma unroll
          for (int v = 0; v < kUnroll; ++v)
            if (v * kWave + lane < len) atomicAdd(&a.zs[ri[v]].y, d * vv[v]);
        }
      }
      if (lane == 0) {
        agent_store(&win[2 * b], static_cast<unsigned long long>(pub_beg) << 32 | pub_len);
        agent_store(&win[2 * b + 1], word(0u, d));
      }
    }
    __syncthreads();
    own = published;
    bool spread = false;
    if (!grid_barrier_marked(ctl, bad, me, members, ++round, own, mark, smb, &spread)) return;
    if (spread) {  // the same decision in every workgroup
      int32_t seen = 0;  // chunks handed out so far
      for (int32_t b0 = 0; b0 < nblk; b0 += kWave) {
        const int32_t b = b0 + lane < nblk ? b0 + lane : b0;
        unsigned long long v = agent_load(&win[2 * b]);
        const unsigned long long dv = agent_load(&win[2 * b + 1]);
        if (b0 + lane >= nblk) v = 0;
        unsigned long long left = __ballot(uint32_t(v) != 0);
        while (left) {
          const int g = __builtin_ctzll(left);
          left &= left - 1;
          const uint32_t beg = uint32_t(__builtin_amdgcn_readlane(int(v >> 32), g));
          const int32_t len = __builtin_amdgcn_readlane(int(v), g);
          const float d = __int_as_float(__builtin_amdgcn_readlane(int(dv), g));
          const int32_t nc = (len + kDirect - 1) / kDirect;
          int32_t c = (gw.wave - seen) % gw.nw;
          for (c += c < 0 ? gw.nw : 0; c < nc; c += gw.nw) {
            int32_t ri[kUnroll];
            float vv[kUnroll];
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) {
              const int32_t e = c * kDirect + u * kWave + lane;
              const int64_t from = int64_t(beg) + (e < len ? e : 0);
              ri[u] = a.row_idx[from];
              vv[u] = a.val[from];
            }
#pragma unroll
            for (int u = 0; u < kUnroll; ++u)
              if (c * kDirect + u * kWave + lane < len) atomicAdd(&a.zs[ri[u]].y, d * vv[u]);
          }
          seen = (seen + nc) % gw.nw;
        }
      }
      if (!grid_barrier_marked(ctl, bad, me, members, ++round, own, ~0u, smb, &unused)) return;
    }
    wp = wn;
    wn = w2;
    cur = nxt;
    nxt.d = dd;
    at = atn;
  }
  if (lane == 0 && acc_cnt > 0) {
    atomicAdd(a.counters + 0, acc_nnz);
    atomicAdd(a.counters + 1, acc_cnt);
  }
}

// Workgroups for windows of `nnz` entries on average.  A barrier takes 0.9 us
// among 32, 1.2 among 64 and 1.8 among 128 (every member reads every flag);
// more of them gather and scatter faster.  Per window, 32 / 64 / 128: 2k
// entries 4.6 / 4.8 / 5.9 us, 8k 6.1 / 6.1 / 7.0, 31k 8.6 / 8.1 / 8.6, 61k
// 13.0 / 10.0 / 9.9.  More units than the waves of 32 take 64 as well: 2000
// columns of 3 entries in groups of 32 3.2 -> 2.5 ms (two launches 2.75).
static unsigned grid_size(double nnz, int64_t units) {
  return nnz <= 8192.0 && units <= 32 * (kGridThreads / kWave) ? 32 : 64;
}

template <int GS>
static void launch_grid_g(const IterArgs &a, int mode, GridCtl *ctl, unsigned long long *bad,
                          int32_t t0, int32_t T, int32_t block, unsigned m, hipStream_t s) {
  if (mode == 2)
    hipLaunchKernelGGL(k_greedy_grid<GS>, dim3(m), dim3(kGridThreads), 0, s, a, ctl, bad, t0, T,
                       block);
  else if (mode == 1)
    hipLaunchKernelGGL((k_epoch_grid<GS, 1>), dim3(m), dim3(kGridThreads), 0, s, a, ctl, bad, t0, T);
  else
    hipLaunchKernelGGL((k_epoch_grid<GS, 0>), dim3(m), dim3(kGridThreads), 0, s, a, ctl, bad, t0, T);
}

// Windows of one launch (5 to 20 us each, so at most about 80 ms: other
// streams' work is not held up for long).
constexpr int64_t kGridMaxWindows = 4096;

int launch_epoch_grid(const IterArgs &a, int group, int mode, GridCtl *ctl,
                      unsigned long long *bad, int64_t T, double nnz, int64_t units,
                      int64_t block, hipStream_t s) {
  if (mode == 2 && (T > kGreedyMaxT || block < 2 || block > kGreedyMaxBlock))
    return GENCD_ERR_INVALID_ARG;
  if (a.piece > kWave * kUnroll || T < 1 || a.k_live < 1 || a.nrows * 16 > INT32_MAX)
    return GENCD_ERR_INVALID_ARG;
  const unsigned m = grid_size(nnz, units);
  for (int64_t t0 = 0; t0 < T; t0 += kGridMaxWindows) {
    if (t0 > 0) {  // the next launch's grid enrols anew
      const int st = fill_i32(reinterpret_cast<int32_t *>(ctl), sizeof(GridCtl) / sizeof(int32_t), 0, s);
      if (st) return st;
    }
    const int32_t b = int32_t(t0), e = int32_t(std::min(T, t0 + kGridMaxWindows));
    const int32_t blk = int32_t(block);
    switch (group) {
      case 4: launch_grid_g<4>(a, mode, ctl, bad, b, e, blk, m, s); break;
      case 8: launch_grid_g<8>(a, mode, ctl, bad, b, e, blk, m, s); break;
      case 16: launch_grid_g<16>(a, mode, ctl, bad, b, e, blk, m, s); break;
      default: launch_grid_g<32>(a, mode, ctl, bad, b, e, blk, m, s); break;
    }
  }
  return hipGetLastError() == hipSuccess ? GENCD_OK : GENCD_ERR_HIP;
}

}  // namespace gencd
