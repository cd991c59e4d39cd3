// Whole epochs of a small accept-all problem in one workgroup.
//
// An iteration of Algorithm 1 on a window of a few thousand entries is far
// too little work for a launch: on two launches per iteration a window of 16
// nonzeros costs about 7 us, of which the arithmetic is a few tens of
// nanoseconds.  Here one workgroup keeps the fitted values of every row
// (z_hi, z_lo, y; 12 bytes a row) in LDS and runs Select, Propose and Update
// of a whole epoch, with a workgroup barrier where the two-launch form has a
// kernel boundary; every proposal of a window still reads the state at the
// window's start.  The next window's descriptors, entries and weights are
// loaded while the current one computes, so a window's chain is LDS gather
// -> reduction -> step -> LDS scatter.  Small matrices also take the FP64
// check here, so a solve runs many epochs per launch and the host looks only
// at a check that ends it.
//
// What bounds it: the dependent instructions of that chain on one wave or a
// few (about 250 at 5 to 6 cycles each with |J| = 1), not memory.  Measured
// per window on MI355X, against the two launches it replaces: |J| = 1 of 4
// entries 0.6 us (7.2 us), |J| = 64 of 4 entries, logistic, 1.25 us (10 us),
// |J| = 96 of 20 entries, squared, 2.4 us (10 us).  Whole solves: n = 400,
// k = 1000, cyclic, 60 epochs 434 -> 37 ms; Shotgun |J| = 64 to KKT 1e-6
// 35 -> 6.2 ms; n = 2000, k = 5000 Lasso, |J| = 96, 3.4 -> 1.4 ms.
#include <cmath>

#include "gencd_common.hpp"
#include "gencd_kernels.hpp"
#include "gencd_solver.hpp"

namespace gencd {

constexpr int kSoloThreads = 1024;

// Sum over an aligned group of G lanes, the same bits in every lane: DPP
// moves inside a row of 16 and, for a whole wave, the four row sums by
// readlane.
template <int G>
__device__ __forceinline__ float lanes_sum(float x) {
  if constexpr (G == kWave) {
    x = row_group_sum<16>(x);
    const int b = __float_as_int(x);
    return (__int_as_float(__builtin_amdgcn_readlane(b, 0)) +
            __int_as_float(__builtin_amdgcn_readlane(b, 16))) +
           (__int_as_float(__builtin_amdgcn_readlane(b, 32)) +
            __int_as_float(__builtin_amdgcn_readlane(b, 48)));
  } else {
    return row_group_sum<G>(x);
  }
}

// Barrier for data exchanged through LDS only: the loads in flight (later
// windows') and the weight stores need not complete.  One wave needs no
// barrier, its LDS operations execute in order.
template <bool ONE>
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  if constexpr (!ONE) {
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  }
}

// Block sums (the first NS values) and maxima (the rest) of NV doubles;
// every thread gets them.  Rows of 16 lanes fold by DPP moves, their results
// go through LDS.
template <int NT, int NV, int NS>
__device__ __forceinline__ void block_fold(double (&v)[NV], double (*sm)[8]) {
  constexpr int ROWS = NT / 16;
  __syncthreads();  // the previous use of sm is over
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    v[i] = i < NS ? row_fold<false>(v[i]) : row_fold<true>(v[i]);
    if ((threadIdx.x & 15) == 0) sm[threadIdx.x / 16][i] = v[i];
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    double r = 0.0;  // sums and maxima of non-negative values both start at 0
    for (int q = int(threadIdx.x) & 15; q < ROWS; q += 16) {
      const double o = sm[q][i];
      if (i < NS)
        r += o;
      else
        r = nan_max(r, o);
    }
    v[i] = i < NS ? row_fold<false>(r) : row_fold<true>(r);
  }
}

// A column of the pipeline: its descriptor {first entry, column, length,
// curvature}, weight and first G * U entries (U per lane).
template <int G, int U>
struct ColSlot {
  int4 d;
  float w;
  int32_t ri[U];
  float vv[U];
};

// Entries [base, base + G * U) of the column.  Lanes past the end take its
// first entry with value 0, so the loads need no branch per lane; a wave
// whose columns all end earlier skips the rest (U > 1).
template <int G, int U>
__device__ __forceinline__ void solo_load(const SoloArgs &a, const int4 &d, int32_t base, int gl,
                                          int32_t (&ri)[U], float (&vv)[U]) {
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int32_t e = base + u * G + gl;
    if (u > 0 && !__any(e < d.z)) {
      ri[u] = 0;
      vv[u] = 0.0f;
      continue;
    }
    // byte offsets of 32 bits: solo_plan bounds the nonzeros
    const uint32_t at = 4u * (uint32_t(d.x) + uint32_t(e < d.z ? e : 0));
    ri[u] = *reinterpret_cast<const int32_t *>(reinterpret_cast<const char *>(a.row_idx) + at);
    vv[u] = *reinterpret_cast<const float *>(reinterpret_cast<const char *>(a.val) + at);
  }
}

template <int G, int U>
__device__ __forceinline__ float solo_dot(int loss, int32_t base, int32_t len, int gl,
                                          const int32_t (&ri)[U], const float (&vv)[U],
                                          const float *zh, const float *zl, const float *yy) {
  float s = 0.0f;
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const bool ok = base + u * G + gl < len;
    if (u > 0 && !__any(ok)) continue;
    const int32_t i = ri[u];
    const float r = dloss_f32(loss, yy[i], zh[i] + zl[i]);
    s += ok ? vv[u] * r : 0.0f;
  }
  return s;
}

template <int G, int U>
__device__ __forceinline__ void solo_scatter(int32_t base, int32_t len, int gl,
                                             const int32_t (&ri)[U], const float (&vv)[U], float d,
                                             float *zl) {
#pragma unroll
  for (int u = 0; u < U; ++u)
    if (base + u * G + gl < len) atomicAdd(&zl[ri[u]], d * vv[u]);
}

// FP64 check inside the workgroup (the quantities of k_check_*): z64 = Xw in
// LDS, objective, KKT, gap, drift, and the re-sync of (z_hi, z_lo).  The
// columns without entries come in through o: no step changes their weights,
// and each nonzero one violates Eq. (1)'s conditions by lambda.
template <int NT, int G>
__device__ __forceinline__ void solo_check(const SoloArgs &a, double *z64, float *zh, float *zl, const float *yy,
                           double (*sm)[8], SoloOut &o) {
  const int tid = int(threadIdx.x), n = a.n;
  const int grp = tid / G, gl = tid & (G - 1);
  constexpr int NG = NT / G, V = 4;  // V columns per group and round: their loads overlap
  for (int i = tid; i < n; i += NT) z64[i] = 0.0;
  __syncthreads();
#pragma unroll 1
  for (int64_t p0 = grp; p0 < a.k_live; p0 += V * NG) {
    int4 d[V];
    float wj[V];
#pragma unroll
    for (int u = 0; u < V; ++u) {
      const int64_t p = p0 + u * NG;
      d[u] = a.rec[p < a.k_live ? p : 0];
      wj[u] = p < a.k_live ? 1.0f : 0.0f;
    }
#pragma unroll
    for (int u = 0; u < V; ++u) wj[u] *= a.w[d[u].y];
#pragma unroll
    for (int u = 0; u < V; ++u) {
      if (wj[u] == 0.0f) continue;
      const int64_t beg = int64_t(uint32_t(d[u].x));
#pragma unroll 2
      for (int32_t e = gl; e < d[u].z; e += G)
        atomicAdd(&z64[a.row_idx[beg + e]], double(wj[u]) * double(a.val[beg + e]));
    }
  }
  __syncthreads();
  // sums: loss, z64^2, |w|, nonzeros of w; maxima: drift, KKT, |g|
  double f[7] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
#pragma unroll 1
  for (int i = tid; i < n; i += NT) {
    const double t = z64[i], yi = double(yy[i]);
    f[0] += loss_f64(a.loss, yi, t);
    const double dv = fabs((double(zh[i]) + double(zl[i])) - t);
    f[4] = nan_max(f[4], dv);
    f[1] += t * t;
    const float h = float(t);
    zh[i] = h;
    zl[i] = float(t - double(h));
    a.z64[i] = t;
    z64[i] = dloss_f64(a.loss, yi, t);  // from here on the residual
  }
  __syncthreads();
#pragma unroll 1
  for (int64_t p0 = grp; p0 < a.k_live; p0 += V * NG) {
    int4 d[V];
    double s[V];
    float wj[V];
    int32_t r[V];
    float x[V];
#pragma unroll
    for (int u = 0; u < V; ++u) {
      const int64_t p = p0 + u * NG;
      d[u] = p < a.k_live ? a.rec[p] : make_int4(0, 0, 0, 0);
    }
#pragma unroll
    for (int u = 0; u < V; ++u) {
      const int64_t at = int64_t(uint32_t(d[u].x)) + (gl < d[u].z ? gl : 0);
      wj[u] = a.w[d[u].y];
      r[u] = a.row_idx[at];
      x[u] = gl < d[u].z ? a.val[at] : 0.0f;
    }
#pragma unroll
    for (int u = 0; u < V; ++u) {
      const int64_t beg = int64_t(uint32_t(d[u].x));
      s[u] = gl < d[u].z ? double(x[u]) * z64[r[u]] : 0.0;
#pragma unroll 2
      for (int32_t e = gl + G; e < d[u].z; e += G)
        s[u] += double(a.val[beg + e]) * z64[a.row_idx[beg + e]];
    }
#pragma unroll
    for (int u = 0; u < V; ++u) {
      const double g = group_sum<G>(s[u]) * a.inv_n;
      if (gl != 0 || d[u].z == 0) continue;
      f[6] = nan_max(f[6], fabs(g));
      const double w = double(wj[u]);
      double v;
      if (w != 0.0) {
        v = fabs(g + (w > 0.0 ? a.lam64 : -a.lam64));
        f[2] += fabs(w);
        f[3] += 1.0;
      } else {
        v = fabs(g) - a.lam64;
        if (v < 0.0) v = 0.0;
      }
      f[5] = nan_max(f[5], v);
    }
  }
  block_fold<NT, 7, 4>(f, sm);
  f[2] += o.l1_empty;
  f[3] += double(o.nz_empty);
  if (o.nz_empty > 0) f[5] = nan_max(f[5], a.lam64);
  const double gm = f[6], sc = gm > a.lam64 ? a.lam64 / gm : 1.0;
  double du[1] = {0.0};
#pragma unroll 1
  for (int i = tid; i < n; i += NT) {
    const double v = sc * z64[i], yi = double(yy[i]);
    if (a.loss == GENCD_SQUARED) {
      du[0] -= v * yi + 0.5 * v * v;
    } else {
      const double p = -v * yi;
      double h = 0.0;
      if (p > 0.0) h -= p * log(p);
      if (p < 1.0) h -= (1.0 - p) * log1p(-p);
      du[0] += h;
    }
  }
  block_fold<NT, 1, 1>(du, sm);
  o.objective = f[0] / double(n) + a.lam64 * f[2];
  o.kkt = f[5];
  o.gap = o.objective - du[0] / double(n);
  o.nnz_w = int64_t(f[3]);
  const double rms = sqrt(f[1] / double(n));
  const double dr = rms > 0.0 ? f[4] / rms : 0.0;
  o.drift = nan_max(o.drift, dr);
}

// One launch: from window a.t0 of epoch a.e0 on, until an FP64 check falls due
// that the host takes (a.inner == 0), or (a.inner) until a check that ends the
// solve, calls for the divergence guard or is the last one, or until
// a.max_windows windows have run, where the next launch takes up the epoch.
// G lanes per column, U entries per lane and batch; ONE: a window
// fits one wave, the other waves only take part in the rest of the epoch.
template <int G, int U, bool ONE>
__global__ __launch_bounds__(kSoloThreads) void k_solo(SoloArgs a) {
  constexpr int NT = kSoloThreads;
  extern __shared__ double lds64[];
  __shared__ double sm[NT / 16][8];
  double *z64 = lds64;
  float *zh = reinterpret_cast<float *>(lds64 + (a.inner ? a.n : 0));
  float *zl = zh + a.n, *yy = zl + a.n, *del = yy + a.n;
  const int tid = int(threadIdx.x);
  const int grp = tid / G, gl = tid & (G - 1);
  constexpr int NG = (ONE ? kWave : NT) / G;  // groups, one column each at a time
  for (int i = tid; i < a.n; i += NT) {
    const float4 r = a.zs[i];
    zh[i] = r.x;
    zl[i] = r.y;
    yy[i] = r.z;
  }
  if (a.build_rec)  // live columns in index order, once per solve
    for (int64_t p = tid; p < a.k_live; p += NT) {
      const int32_t j = a.live[p];
      const int64_t b = a.col_ptr[j];
      a.rec[p] = make_int4(int32_t(uint32_t(b)), j, int32_t(a.col_ptr[j + 1] - b),
                           __float_as_int(a.c[j]));
    }
  __syncthreads();
  SoloOut o{};
  o.best = a.best;
  o.l1_empty = a.l1_empty;
  o.nz_empty = a.nz_empty;
  if (a.sum_empty) {
    double em[2] = {0.0, 0.0};
    for (int64_t j = tid; j < a.k; j += NT)
      if (a.col_ptr[j] == a.col_ptr[j + 1]) {
        const double wj = fabs(double(a.w[j]));
        em[0] += wj;
        em[1] += wj != 0.0 ? 1.0 : 0.0;
      }
    block_fold<NT, 2, 2>(em, sm);
    o.l1_empty = em[0];
    o.nz_empty = int64_t(em[1]);
  }
  int64_t e = a.e0, next_check = a.next_check;
  const int32_t S = a.S, kl = int32_t(a.k_live), T = (kl + S - 1) / S;
  int32_t t0 = a.t0, left = a.max_windows;
  const bool overflow = a.max_len > G * U;  // some column needs a second batch
  for (;;) {
    if (t0 == 0) {
      // Select: the epoch's order as one descriptor {first entry, column,
      // length, curvature} per position
      const PermKey pk = make_perm_key(a.k_live, a.seed, e);
#pragma unroll 1
      for (int64_t p = tid; p < a.k_live; p += NT)
        a.desc[p] = a.rec[a.natural ? p : int64_t(perm_apply(pk, uint64_t(p)))];
      __syncthreads();
    }
    const int32_t t1 = T - t0 < left ? T : t0 + left;
    // position of this group in window t, or past the end
    auto desc_at = [&](int32_t t) {
      int4 d = make_int4(0, 0, 0, 0);
      const int32_t p = t * S + grp;
      if (grp < S && p < kl) d = a.desc[p];
      return d;
    };
    auto fetch = [&](ColSlot<G, U> &c) {
      if (!__any(c.d.z > 0)) return;  // a wave without columns loads nothing
      c.w = a.w[c.d.y];
      solo_load<G, U>(a, c.d, 0, gl, c.ri, c.vv);
    };
    // Window t from slot c.  Slots rotate over four windows: the descriptor
    // of window t is loaded at the end of window t - 4, its entries and
    // weight at the start of window t - 2 (slot f at window t; the columns of
    // the two windows between are others, as every column appears once per
    // epoch, so its weight is final).
    auto window = [&](int32_t t, ColSlot<G, U> &c, ColSlot<G, U> &f) {
      const int32_t P0 = t * S;
      const int32_t m = P0 + S < kl ? S : kl - P0;
      fetch(f);
      float d = 0.0f, ph;
      if (c.d.z > 0) {
        float s = solo_dot<G, U>(a.loss, 0, c.d.z, gl, c.ri, c.vv, zh, zl, yy);
#pragma unroll 1
        for (int32_t base = G * U; overflow && base < c.d.z; base += G * U) {
          int32_t ri[U];
          float vv[U];
          solo_load<G, U>(a, c.d, base, gl, ri, vv);
          s += solo_dot<G, U>(a.loss, base, c.d.z, gl, ri, vv, zh, zl, yy);
        }
        s = lanes_sum<G>(s);
        propose_f32(s / a.n_f, __int_as_float(c.d.w), c.w, a.lam, d, ph);
        if (d != 0.0f && gl == 0) a.w[c.d.y] = c.w + d;
      }
#pragma unroll 1
      for (int32_t q = grp + NG; q < m; q += NG) {  // more columns than groups
        const int4 dq = a.desc[P0 + q];
        float s = 0.0f, dd;
        for (int32_t base = 0; base < dq.z; base += G * U) {
          int32_t ri[U];
          float vv[U];
          solo_load<G, U>(a, dq, base, gl, ri, vv);
          s += solo_dot<G, U>(a.loss, base, dq.z, gl, ri, vv, zh, zl, yy);
        }
        s = lanes_sum<G>(s);
        const float wq = a.w[dq.y];
        propose_f32(s / a.n_f, __int_as_float(dq.w), wq, a.lam, dd, ph);
        if (gl == 0) {
          del[q - NG] = dd;
          if (dd != 0.0f) a.w[dq.y] = wq + dd;
        }
      }
      lds_barrier<ONE>();  // every proposal has read the window's starting state
      if (d != 0.0f) {
        solo_scatter<G, U>(0, c.d.z, gl, c.ri, c.vv, d, zl);
#pragma unroll 1
        for (int32_t base = G * U; overflow && base < c.d.z; base += G * U) {
          int32_t ri[U];
          float vv[U];
          solo_load<G, U>(a, c.d, base, gl, ri, vv);
          solo_scatter<G, U>(base, c.d.z, gl, ri, vv, d, zl);
        }
      }
#pragma unroll 1
      for (int32_t q = grp + NG; q < m; q += NG) {
        const float dd = del[q - NG];
        if (dd == 0.0f) continue;
        const int4 dq = a.desc[P0 + q];
        for (int32_t base = 0; base < dq.z; base += G * U) {
          int32_t ri[U];
          float vv[U];
          solo_load<G, U>(a, dq, base, gl, ri, vv);
          solo_scatter<G, U>(base, dq.z, gl, ri, vv, dd, zl);
        }
      }
      lds_barrier<ONE>();
      c.d = desc_at(t + 4);
    };
    if (!ONE || tid < kWave) {
      ColSlot<G, U> c0, c1, c2, c3;
      c0.d = desc_at(t0);
      c1.d = desc_at(t0 + 1);
      c2.d = desc_at(t0 + 2);
      c3.d = desc_at(t0 + 3);
      fetch(c0);
      fetch(c1);
#pragma unroll 1
      for (int32_t t = t0; t < t1; t += 4) {
        window(t, c0, c2);
        if (t + 1 < t1) window(t + 1, c1, c3);
        if (t + 2 < t1) window(t + 2, c2, c0);
        if (t + 3 < t1) window(t + 3, c3, c1);
      }
    }
    __syncthreads();
    left -= t1 - t0;
    t0 = t1 < T ? t1 : 0;
    if (t0 > 0) {  // inside the epoch; the FP32 pairs go through memory as they are
      o.checked = 0;
      break;
    }
    for (int i = tid; i < a.n; i += NT) {  // exact renormalisation, as k_renorm
      const float h = zh[i], l = zl[i];
      zh[i] = h + l;
      zl[i] = twosum_err(h, l);
    }
    ++e;
    const bool due = e >= next_check || e == a.max_epochs;
    if (!a.inner) {
      if (due || left == 0) break;
      __syncthreads();
      continue;
    }
    __syncthreads();
    o.checked = 0;
    if (due) {
      next_check = e + check_interval(a.check_every, e);
      solo_check<NT, G>(a, z64, zh, zl, yy, sm, o);
      o.checked = 1;
      const bool conv = o.kkt <= a.kkt_tol &&
                        (a.gap_tol <= 0.0 || o.gap <= a.gap_tol * fabs(o.objective));
      // the comparison is false for a NaN objective as well
      const bool good = o.objective <= o.best + 1e-3 * fabs(o.best) + 1e-12 &&
                        o.objective >= -1.7e308;
      if (conv || !good || e == a.max_epochs) break;
      if (o.objective <= o.best) {
        o.best = o.objective;
        for (int64_t p = tid; p < a.k; p += NT) a.w_ckpt[p] = a.w[p];
      }
      __syncthreads();
    }
    if (left == 0) break;
  }
  __syncthreads();
  for (int i = tid; i < a.n; i += NT) a.zs[i] = make_float4(zh[i], zl[i], yy[i], 0.0f);
  if (tid == 0) {
    o.epoch = e;
    o.window = t0;
    o.next_check = next_check;
    *a.out = o;
  }
}

// ---------------------------------------------------------------------------
// Which solves run here, and with which shape
// ---------------------------------------------------------------------------
constexpr size_t kSoloLds = 156 * 1024;   // of the 160 KB of a CU; the rest is static
// The FP64 check of 100k entries takes one workgroup about 55 us, which is
// what the seven launches and the read-back of the other form take.
constexpr int64_t kSoloInnerNnz = 131072;
// Expected entries of a window: about 1.2 ns an entry here (3.8k entries
// 4.9 us, 8k 9.7 us) against 10 to 11 us for two launches at any size up to
// this, so the line is drawn well below where they meet.
constexpr int64_t kSoloWindowNnz = 4096;
// Columns of a window, in lanes: one and a half rounds of the workgroup's lane
// groups.  A further round is a chain of its own, while the resident grid
// (gencd_grid.hip) takes the window in one.  2 M entries, n = 13 000, an epoch's
// ms here / there: columns of 3, |J| = 192 10 / 14, 288 11 / 10, 512 9.3 / 6.0
// (two launches 9.3), 1024 8.9 / 3.3 (4.7); of 24, 128 3.5 / 3.7, 160 4.4 / 3.1;
// of 80, 32 4.3 / 4.3, 48 4.3 / 3.0 (4.2).  On a small matrix the checks and
// orders between the launches weigh more: with 50 000 entries the two meet near
// |J| = 300, with 16 000 near 600 (columns of 3).
constexpr double kSoloLanes = 1536.0, kSoloLanesNnz = 81920.0;

SoloPlan solo_plan(int64_t n, int64_t nnz, int64_t k_live, int64_t max_len, int64_t S) {
  SoloPlan p{};
  if (k_live <= 0 || nnz <= 0 || S < 1) return p;
  if (k_live > (1 << 24) || nnz > (1 << 28)) return p;  // 32-bit positions and byte offsets
  const double mean = double(nnz) / double(k_live);
  if (double(S) * mean > double(kSoloWindowNnz)) return p;
  const int wide = mean > 64.0 ? 64 : mean > 32.0 ? 16 : 8;  // lanes a column keeps busy
  if (double(S) * wide > kSoloLanes * std::fmax(1.0, kSoloLanesNnz / double(nnz))) return p;
  if (mean > 64.0) {
    p.G = 64;
  } else if (S <= 4) {
    p.G = 16;  // one wave
  } else {
    p.G = wide == 16 ? 16 : S * 8 <= kSoloThreads ? 8 : 4;
  }
  p.one = S * p.G <= kWave;
  p.U = p.G == 64 ? 4 : max_len <= p.G ? 1 : max_len <= 2 * p.G ? 2 : max_len <= 4 * p.G ? 4 : 6;
  // a group walks its column alone: no column much longer than the mean
  if (max_len > int64_t(p.G) * 32) return p;
  const int64_t groups = (p.one ? kWave : kSoloThreads) / p.G;
  p.inner = nnz <= kSoloInnerNnz;
  auto lds = [&](bool inner) {
    return size_t(n) * (inner ? 20 : 12) + sizeof(float) * size_t(S > groups ? S - groups : 0) + 16;
  };
  if (p.inner && lds(true) > kSoloLds) p.inner = false;
  p.lds = lds(p.inner);
  p.ok = p.lds <= kSoloLds;
  return p;
}

template <int G, int U>
static int launch_solo_u(const SoloArgs &a, const SoloPlan &p, hipStream_t s) {
  void (*const kern)(SoloArgs) = p.one ? k_solo<G, U, true> : k_solo<G, U, false>;
  if (p.lds > 64 * 1024)
    GENCD_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, int(p.lds)));
  hipLaunchKernelGGL(kern, dim3(1), dim3(kSoloThreads), p.lds, s, a);
  return hipGetLastError() == hipSuccess ? GENCD_OK : GENCD_ERR_HIP;
}

template <int G>
static int launch_solo_g(const SoloArgs &a, const SoloPlan &p, hipStream_t s) {
  switch (p.U) {
    case 1: return launch_solo_u<G, 1>(a, p, s);
    case 2: return launch_solo_u<G, 2>(a, p, s);
    case 4: return launch_solo_u<G, 4>(a, p, s);
    default: return launch_solo_u<G, 6>(a, p, s);
  }
}

int launch_solo(const SoloArgs &a, const SoloPlan &p, hipStream_t s) {
  if (!p.ok || a.n <= 0 || a.k_live <= 0 || a.S < 1) return GENCD_ERR_INVALID_ARG;
  switch (p.G) {
    case 4: return launch_solo_g<4>(a, p, s);
    case 8: return launch_solo_g<8>(a, p, s);
    case 16: return launch_solo_g<16>(a, p, s);
    default: return launch_solo_u<64, 4>(a, p, s);
  }
}

}  // namespace gencd
