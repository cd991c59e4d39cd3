// Kernel argument blocks and launchers (implemented in gencd_kernels.hip).
#pragma once

#include "gencd_common.hpp"

namespace gencd {

// Everything one iteration's kernels read or write.  Passed by value.
struct IterArgs {
  const int64_t *col_ptr;
  const int32_t *row_idx;
  const float *val;
  float n_f;
  int32_t loss;
  float lam;
  const float *c;
  float *w;
  float4 *zs;                      // {z_hi, z_lo, y, 0} per row
  float *rs;                       // non-null: refresh l'(y, z) into rs, Propose reads it
  int64_t nrows;
  const int32_t *col_of_pos;
  const int32_t *loff;             // long-piece offsets of the positions
  const int4 *desc_s;              // descriptor of every position (length 0: long column)
  const int4 *desc_l;              // long-piece descriptors of the current order
  const int32_t *wbl;              // window t: long pieces [wbl[t], wbl[t+1])
  int32_t nl;                      // waves walking long pieces (set by the launcher)
  int32_t piece;                   // nonzeros per long piece
  int64_t accept_top;              // > 0: deferred acceptance of the best accept_top of the window
  int32_t improve;                 // extra quadratic-approximation steps per accepted proposal
  const int32_t *win_off;  // per-epoch window offsets, or null: [win_lo, win_hi)
  int32_t t, win_lo, win_hi;
  int32_t S, k_live;       // whole-epoch kernels: window t is [t S, (t + 1) S) of k_live
  float *delta, *phi, *gacc, *gout, *wsnap;
  int32_t *acc;
  int32_t *bw_pos, *bw_phi;  // per-chunk winners of a two-stage global accept (scratch)
  int32_t exact_accum;     // 1: TwoSum per update (returning atomics); 0: low-word accumulation
  unsigned long long *counters;  // [0] accepted nnz, [1] accepted proposals (greedy rules)
  unsigned long long *scat;      // non-null: Update adds the nonzeros it scatters here
                                 // (replica line b % kChkRep of workgroup b, 16 words each)
};

// Control block of a grid of resident workgroups (gencd_grid.hip); all zero
// before each launch.
constexpr int kGridMax = 256;
// Thread-Greedy on the grid: three barriers a window at most, counted in 16
// bits; one wave walks a block, 64 positions a round.
constexpr int64_t kGreedyMaxT = 21000;
constexpr int64_t kGreedyMaxBlock = 256;
struct GridCtl {
  int32_t count, members;
  int32_t pad[30];
  int32_t flag[kGridMax];
};

// All T windows of an epoch whose order is built, in launches of up to 4096
// windows (mode 0: accept all, 1: Coloring, 2: Thread-Greedy with 2 to
// kGreedyMaxBlock positions per block and at most kGreedyMaxT windows; pieces of
// at most 64 * kUnroll entries, rows of at most 2 GiB).  nnz, units: expected
// entries and work units of a window.  A grid barrier that runs out sets bit 16
// of *bad.
int launch_epoch_grid(const IterArgs &a, int group, int mode, GridCtl *ctl,
                      unsigned long long *bad, int64_t T, double nnz, int64_t units,
                      int64_t block, hipStream_t s);

// Whole epochs of a small accept-all problem in one workgroup
// (gencd_solo.hip).
struct SoloOut {
  int64_t epoch, next_check;  // epochs run so far, and the next due check
  int64_t window;             // windows of the next epoch that have run
  double objective, kkt, gap, drift, best;  // the last check; drift: the largest
  int64_t nnz_w, checked;     // checked: the launch ended on a check
  double l1_empty;            // weights of the columns without entries: |w|_1 and
  int64_t nz_empty;           // nonzeros (they never change)
};

struct SoloArgs {
  const int64_t *col_ptr;
  const int32_t *row_idx;
  const float *val;
  const float *c;
  const int32_t *live;
  float *w, *w_ckpt;
  float4 *zs;
  int4 *rec;         // [k_live] column records in index order (build_rec: written first)
  int4 *desc;        // [k_live] scratch: the epoch order
  double *z64;       // [n] Xw of the last check
  SoloOut *out;
  int64_t k, k_live;
  int32_t n, S, loss, natural, inner, build_rec;
  int32_t sum_empty;          // find l1_empty and nz_empty in this launch
  double l1_empty;
  int64_t nz_empty;
  int32_t max_len;   // entries of the longest column
  float lam, n_f;
  double lam64, inv_n, kkt_tol, gap_tol, best;
  uint64_t seed;
  int64_t e0, max_epochs, next_check, check_every;
  int32_t t0, max_windows;    // first window of epoch e0; windows of this launch
};

struct SoloPlan {
  bool ok, inner;    // inner: the FP64 checks run in the same launch
  bool one;          // a window fits one wave
  int G, U;          // lanes per column, entries per lane and batch
  size_t lds;
};

// Shape for windows of S columns of a matrix whose longest column has
// max_len entries (ok = false: the multi-workgroup kernels take it).
SoloPlan solo_plan(int64_t n, int64_t nnz, int64_t k_live, int64_t max_len, int64_t S);
// Rows that fit the LDS of one workgroup (a bound without the other sizes).
constexpr int64_t kSoloMaxRows = 13312;
int launch_solo(const SoloArgs &a, const SoloPlan &p, hipStream_t s);

int fill_f32(float *p, int64_t m, float v, hipStream_t s);
int fill_i32(int32_t *p, int64_t m, int32_t v, hipStream_t s);
int fill_f64(double *p, int64_t m, double v, hipStream_t s);
int copy_f32(float *d, const float *src, int64_t m, hipStream_t s);
int copy_i32(int32_t *d, const int32_t *src, int64_t m, hipStream_t s);

int launch_validate(const gencd_csc *X, const float *y, int loss, bool matrix,
                    unsigned long long *bad, hipStream_t s);
// want_max: leave the longest column's entries in word 11 of w.red.
int launch_preprocess(const gencd_csc *X, int loss, int piece, int short_max, const Ws &w,
                      bool want_max, hipStream_t s);
int launch_curvature(const gencd_csc *X, int loss, int32_t n_short, int32_t n_lpieces,
                     const Ws &w, hipStream_t s);
int launch_select_perm(int64_t m, uint64_t seed, int64_t epoch, int32_t *out, hipStream_t s);
// Writes the epoch order, its piece descriptors and, in w.wbounds[0..T], the
// first piece of every window (S positions per window; colour windows for
// COLORING).  Then the epoch counter steps, and ctl (may be null) is cleared
// for the epoch's grid.
int launch_epoch_order(const Ws &w, int64_t k_live, int rule, uint64_t seed, int64_t *epoch,
                       GridCtl *ctl, int64_t num_colors, int64_t S, int64_t T, hipStream_t s);
int launch_list_order(const Ws &w, const int32_t *J, int64_t nJ, hipStream_t s);
// group: lanes per short column (4, 8, 16 or 32); short_bound / long_bound:
// expected short columns / long pieces of a window (they size the grid; the
// kernels stride over whatever the window holds).
// ev0/ev1 (optional) stamp the Propose dispatch, ev2/ev3 the Update dispatch.
int launch_iteration(const IterArgs &a, int group, int mode, int64_t block, int64_t short_bound,
                     int64_t long_bound, int64_t nblocks_accept, hipStream_t s,
                     hipEvent_t ev0 = nullptr, hipEvent_t ev1 = nullptr,
                     hipEvent_t ev2 = nullptr, hipEvent_t ev3 = nullptr);
// Fused asynchronous Shotgun iteration (accept-all rules): window a.t, plus
// the split columns of window a.t - 1; `flush` applies only the latter
// (a.t = number of windows).
int launch_fused(const IterArgs &a, int group, int64_t short_bound, int64_t long_bound, bool flush,
                 hipStream_t s);
// Power-iteration estimate of the normalised Gram spectral radius; needs the
// column sums of squares in ws.g64 (left there by launch_curvature) and the
// rho arrays of the workspace.  Squared norms land in ws.rho_hist[0..iters).
// beside: other work runs on the device meanwhile.
int launch_rho(const gencd_csc *X, int32_t n_short, int32_t n_lpieces, const Ws &ws, int64_t k_live,
               int64_t max_len, bool beside, int iters, hipStream_t s);
// Block Shotgun: preset blocks (base order, block of every column) and the
// per-block power iteration; needs the column sums of squares in ws.g64.
// Squared norms land in ws.bhist[t][b].
int launch_block_setup(const gencd_csc *X, int32_t n_short, int32_t n_lpieces, const Ws &ws,
                       int64_t k_live, uint64_t seed, int iters, hipStream_t s);
// Per-epoch order of Block Shotgun (col_of_pos, windows win_off[0..T]).
int launch_block_order(const Ws &w, int64_t k_live, uint64_t seed, int64_t *epoch, GridCtl *ctl,
                       int64_t T, hipStream_t s);
int launch_check(const gencd_csc *X, const float *y, int loss, double lam, const float *w,
                 int32_t n_short, int32_t n_lpieces, const Ws &ws, bool resync, hipStream_t s);
int launch_renorm(int64_t n, float4 *zs, hipStream_t s);
// Copy caller-held (z_hi, z_lo) and the labels into the packed rows, and back.
int launch_pack_state(int64_t n, const float *z_hi, const float *z_lo, const float *y, float4 *zs,
                      hipStream_t s);
int launch_unpack_state(int64_t n, const float4 *zs, float *z_hi, float *z_lo, hipStream_t s);
int launch_round_f32(const double *src, float *dst, int64_t m, hipStream_t s);

}  // namespace gencd
