// Host side of the MGRIT-FAS library: argument checks, the level hierarchy, the workspace
// layout and the launch schedule of the FAS V-cycle (forward and adjoint).  Every arithmetic
// step of the method runs in the HIP kernels of mgrit_kernels.hip, mgrit_conv_grad.hip and the three files of sweeps
// (mgrit_sweep.hip, mgrit_wave.hip, mgrit_wide.hip); this file only decides which launch comes next.
#include <math.h>
#include <stdlib.h>
#include <string.h>

#include "../../include/mgrit.h"
#include "mgrit_internal.h"

using namespace mgrit;

namespace {

constexpr size_t ALIGN = 256;
inline size_t align_up(size_t x) { return (x + ALIGN - 1) / ALIGN * ALIGN; }
// MGRIT_ADJ_TRANSPOSED=1 in the environment: the adjoint of dense and fully connected layers runs on a transposed
// copy of the weights in the workspace (diagnostic; by default the kernels read the caller's array k-major)
inline bool adjoint_transposed_copy() {
  const char* e = getenv("MGRIT_ADJ_TRANSPOSED");
  return e && e[0] == '1';
}
// Whether ReLU's act' factors are stored as bits.  They are where their bytes count; taking bits apart costs more than it saves
//   - in dense layers of 8 or 16 features, whose lanes have four factors each;
//   - in float layers wider than 128 that have few of them, and in the widest, whose weights are most of the bytes;
//   - in layers of 8 channels that have few.
// us with values / with bits, adjoint with gradient: float width 8, 8 MB of factors as values 260 / 277, 32 MB 812 / 832; width 16,
// 16 MB 264 / 284, 64 MB 827 / 833; bf16 width 16, 8 MB 192 / 194, 32 MB 525 / 536; float width 24, 3 MB 185 / 182, 96 MB 1954 / 1912;
// width 64, 2 MB 143 / 143, 64 MB 651 / 629; width 136, 2 MB 316 / 323, 68 MB 1405 / 1371; width 256, 1 MB 315 / 317, 16 MB
// 547 / 546, 32 MB 668 / 652, 128 MB 1854 / 1766; width 448, 28 MB 1759 / 1774, 56 MB 2105 / 2061; width 512, 32 MB 1911 / 1940, 128 MB
// 3420 / 3404; width 896, 112 MB 5513 / 5567, 448 MB 18586 / 18473; width 1024, 64 MB 5580 / 5598, 512 MB 22539 / 22636; bf16 width 64,
// 2 MB 112 / 107; 8 channels, 12 MB 316 / 330, 49 MB 702 / 728, 128 MB 1603 / 1573; bf16 24 channels, 2 MB 272 / 259; bf16 40
// channels, 2 MB 446 / 349; bf16 64 channels, 0.4 MB 296 / 296, 2 MB 615 / 601, 2 GB 17093 / 14817.
// MGRIT_ACT_VALUES=1 / 0 in the environment: values / bits whatever the size (diagnostic).
inline bool act_factor_bits(const mgrit_problem_t* p, double bytes_as_values) {
  const char* e = getenv("MGRIT_ACT_VALUES");
  if (e && (e[0] == '0' || e[0] == '1')) return e[0] == '0';
  const double mb = bytes_as_values / (1024.0 * 1024.0);
  if (p->layer == MGRIT_LAYER_CONV3X3) return p->C > 8 || mb >= 64.0;
  if (p->q <= 16) return false;
  return p->dtype == MGRIT_BF16 || p->q <= 128 || (p->q <= 896 && mb >= (p->q <= 448 ? 24.0 : 128.0));
}
inline bool aligned(const void* p) { return (reinterpret_cast<uintptr_t>(p) % ALIGN) == 0; }

// Sweeps (one launch for many layer steps) can be switched off with MGRIT_NO_SWEEP=1 in the environment; the tests run
// both ways.
inline bool sweep_enabled() {
  const char* e = getenv("MGRIT_NO_SWEEP");
  return !(e && e[0] == '1');
}

struct Plan {
  int L;
  int Nl[MGRIT_MAX_LEVELS];
  long long mpow[MGRIT_MAX_LEVELS];
  float hl[MGRIT_MAX_LEVELS];
  long long E, wsize;
  int M, Nf, K, TH;
  size_t esize;                        // bytes per weight element
  size_t off_X[MGRIT_MAX_LEVELS], off_g[MGRIT_MAX_LEVELS], off_R[MGRIT_MAX_LEVELS];
  size_t off_partial, n_partial, off_hist, off_Wt, off_D, off_gpart;
  size_t bytes_fwd, bytes_adj;
  // mixed stacks (Sec. IV-E): every fcP-th layer is fully connected on the flattened sample; 0 = none
  int fcP, nfc, B;
  long long dfc, wsize_fc;             // flattened sample size d and d*d
  size_t off_Wfct;                     // transposed fully connected weights (adjoint)
};

// Level hierarchy (Sec. III-C): coarsen by m while fewer than max_levels levels exist and the
// current level has more than min_coarse steps and at least one whole coarse interval.  Points
// 0, m, 2m, .. of a level are its C-points; a level whose size is not a multiple of m ends in
// fewer than m trailing F-points, and the next level has floor(N_l / m) steps.
int build_levels(const mgrit_problem_t* p, int* L, int* Nl) {
  if (!p) return MGRIT_ERR_POINTER;
  if (p->N < 1 || p->m < 2 || p->max_levels < 1 || p->max_levels > MGRIT_MAX_LEVELS) return MGRIT_ERR_PROBLEM;
  const int minc = p->min_coarse < 1 ? 1 : p->min_coarse;
  int n = 1;
  Nl[0] = p->N;
  while (n < p->max_levels && Nl[n - 1] > minc && Nl[n - 1] >= p->m) {
    Nl[n] = Nl[n - 1] / p->m;
    ++n;
  }
  *L = n;
  return MGRIT_OK;
}

int make_plan(const mgrit_problem_t* p, Plan* pl, int fcP = 0) {
  memset(pl, 0, sizeof(*pl));
  int rc = build_levels(p, &pl->L, pl->Nl);
  if (rc != MGRIT_OK) return rc;
  if (fcP != 0 && (fcP < 2 || p->layer != MGRIT_LAYER_CONV3X3)) return MGRIT_ERR_PROBLEM;
  if (!(p->h > 0.0f) || !isfinite(p->h)) return MGRIT_ERR_PROBLEM;
  if (p->N > 65535) return MGRIT_ERR_UNSUPPORTED;            // layers / points index one grid dimension of the transfer kernels
  if (p->relax != MGRIT_RELAX_F && p->relax != MGRIT_RELAX_FCF) return MGRIT_ERR_PROBLEM;
  if (p->cycle != 0 || p->max_iter < 1) return MGRIT_ERR_PROBLEM;
  if (p->norm_kind != MGRIT_NORM_L2 && p->norm_kind != MGRIT_NORM_RMS) return MGRIT_ERR_PROBLEM;
  if (p->layer != MGRIT_LAYER_DENSE && p->layer != MGRIT_LAYER_CONV3X3) return MGRIT_ERR_PROBLEM;
  if (p->act != MGRIT_ACT_TANH && p->act != MGRIT_ACT_RELU) return MGRIT_ERR_PROBLEM;
  if (p->dtype != MGRIT_FP32 && p->dtype != MGRIT_BF16) return MGRIT_ERR_PROBLEM;
  if (p->init < MGRIT_INIT_ZERO || p->init > MGRIT_INIT_NESTED) return MGRIT_ERR_PROBLEM;
  if (p->layer == MGRIT_LAYER_DENSE) {
    if (p->B < 1 || p->q < 1) return MGRIT_ERR_PROBLEM;
    if (p->q % 8 != 0) return MGRIT_ERR_UNSUPPORTED;       // 16-byte operand pieces
    if ((long long)p->B * p->q > 0x7fffffffLL) return MGRIT_ERR_UNSUPPORTED;   // 32-bit offsets inside a state
    pl->M = p->B; pl->Nf = p->q; pl->K = p->q; pl->TH = 0;
  } else {
    if (p->B < 1 || p->C < 1 || p->Himg < 1 || p->Wimg < 1) return MGRIT_ERR_PROBLEM;
    if (p->C % 8 != 0 || p->C > 64 || p->Wimg > 256) return MGRIT_ERR_UNSUPPORTED;
    if ((long long)p->B * p->Himg * p->Wimg * p->C > 0x7fffffffLL) return MGRIT_ERR_UNSUPPORTED;
    pl->M = p->B * p->Himg * p->Wimg; pl->Nf = p->C; pl->K = 9 * p->C;
    pl->TH = conv_tile_rows(p->Himg, p->Wimg, p->C, p->dtype);
    if (pl->TH < 1) return MGRIT_ERR_UNSUPPORTED;
  }
  pl->E = (long long)pl->M * pl->Nf;
  pl->wsize = (long long)pl->Nf * pl->K;
  pl->esize = p->dtype == MGRIT_FP32 ? 4 : 2;
  pl->B = p->B;
  if (fcP) {
    pl->fcP = fcP;
    pl->nfc = (p->N + fcP - 1) / fcP;
    pl->dfc = (long long)p->Himg * p->Wimg * p->C;
    if (pl->dfc * pl->dfc > 0x7fffffffLL) return MGRIT_ERR_UNSUPPORTED;      // 32-bit offsets inside a weight matrix
    pl->wsize_fc = pl->dfc * pl->dfc;
  }
  long long mp = 1;
  for (int l = 0; l < pl->L; ++l) {
    pl->mpow[l] = mp;
    pl->hl[l] = p->h * (float)mp;
    mp *= p->m;
  }
  // workspace: coarse-level states and right-hand sides, C-point residuals, norm partials,
  // residual history; for the adjoint also the transposed weights and the act' cache
  size_t off = 0;
  for (int l = 1; l < pl->L; ++l) {
    pl->off_X[l] = off; off = align_up(off + (size_t)(pl->Nl[l] + 1) * pl->E * 4);
    pl->off_g[l] = off; off = align_up(off + (size_t)(pl->Nl[l] + 1) * pl->E * 4);
  }
  for (int l = 0; l + 1 < pl->L; ++l) {
    pl->off_R[l] = off; off = align_up(off + (size_t)(pl->Nl[l + 1] + 1) * pl->E * 4);
  }
  StepArgs a;
  memset(&a, 0, sizeof(a));
  a.M = pl->M; a.Nf = pl->Nf; a.K = pl->K; a.Himg = p->Himg; a.Wimg = p->Wimg; a.TH = pl->TH;
  size_t np = (size_t)step_grid_blocks(a, p->layer, p->dtype, p->N) * p->N + diff_sq_blocks(pl->E);
  if (np > 0x7fffffffu) return MGRIT_ERR_UNSUPPORTED;       // the largest launch (all N layers) must fit a 1-D grid
  if (pl->L > 1) {
    size_t np1 = (size_t)step_grid_blocks(a, p->layer, p->dtype, pl->Nl[1]) * pl->Nl[1];
    if (np1 > np) np = np1;
  }
  if (fcP)     // the dense launch of the fully connected groups adds its workgroups (at most 32x32 tiles of each)
    np += (size_t)((p->B + 31) / 32) * (size_t)((pl->dfc + 31) / 32) * (size_t)pl->nfc;
  if (np > 0x7fffffffu) return MGRIT_ERR_UNSUPPORTED;
  pl->n_partial = np;
  pl->off_partial = off; off = align_up(off + np * 4);
  pl->off_hist = off; off = align_up(off + (size_t)(p->max_iter + 1) * 8);
  pl->bytes_fwd = off;
  // transposed weights of the adjoint: convolution layers always; dense layers only on request (their kernels
  // read the caller's array k-major)
  const bool wcopy = p->layer != MGRIT_LAYER_DENSE || adjoint_transposed_copy();
  pl->off_Wt = off;
  if (wcopy) off = align_up(off + (size_t)p->N * pl->wsize * pl->esize);
  pl->off_D = off; off = align_up(off + (size_t)p->N * pl->E * pl->esize);   // act' cache, in the weights' type
  pl->off_gpart = off;                 // partial sums of the conv parameter gradient when layers are split
  if (p->layer == MGRIT_LAYER_CONV3X3)
    off = align_up(off + conv_grad_partial_bytes(p->B, p->Himg, p->Wimg, p->C, p->dtype, p->N));
  pl->off_Wfct = off;
  if (fcP && adjoint_transposed_copy()) off = align_up(off + (size_t)pl->nfc * pl->wsize_fc * pl->esize);
  pl->bytes_adj = off;
  return MGRIT_OK;
}

// The cycle is written once, in "sweep order": sweep point 0 carries the known value and the
// sweep advances to sweep point N_l.  The forward solve sweeps up the layer axis; the adjoint
// solve sweeps down it, so sweep point js of its level l is natural fine point N - js m^l (its
// hierarchy counts from layer N, whatever N mod m is).  Only the caller's fine-level array is
// stored in natural order; all workspace arrays are in sweep order.
struct Solver {
  const mgrit_problem_t* p;
  Plan pl;
  hipStream_t s;
  bool adjoint;
  float* X[MGRIT_MAX_LEVELS];
  float* g[MGRIT_MAX_LEVELS];
  float* R[MGRIT_MAX_LEVELS];
  bool plain_rhs = false;              // nested start: every level carries the right-hand side (first, 0, .., 0)
  bool want_norm = false;              // somebody reads the residual norm of the cycles
  const void* W;
  int wn = 0, wn_fc = 0;               // adjoint on the caller's dense / fully connected weights as stored: W[k][n]
  const float* bias;
  const float* Dm;
  int dbits = 0;                       // the act' factors (input and output) are bits: ReLU's
  const void* Wfc = nullptr;           // fully connected layers of a mixed stack (their transposes in the adjoint)
  const float* bfc = nullptr;
  int act;
  float* partial;
  double* hist_dev;
  // Narrow dense stacks (wave): sweeps that follow one another are collected and launched together (flush).
  bool wave = false;
  WaveProgram prog;
  long long prog_units = 0;
  double prog_bytes = 0.0;
  bool prog_by_slice = false;          // it has norm partials laid out for one workgroup per slice
  int late_norms = 0;                  // > 0: norm partials per cycle that wait in `partial`, cycle by cycle, for one summation
  hipError_t err = hipSuccess;

  void chk(hipError_t e) { if (err == hipSuccess && e != hipSuccess) err = e; }
  // map of a sweep-order index range of level l's state array to its storage order
  PtMap pm(int l, long long base, long long stride) const {
    if (l == 0 && adjoint) return PtMap{pl.Nl[0] - base, -stride};
    return PtMap{base, stride};
  }
  // layer index used by the sweep step that lands on sweep point js of level l
  PtMap layer_map(int l, long long js0, long long jstride) const {
    if (adjoint) return PtMap{p->N - js0 * pl.mpow[l], -jstride * pl.mpow[l]};
    return PtMap{(js0 - 1) * pl.mpow[l], jstride * pl.mpow[l]};
  }
  StepArgs base_args(int l, long long js0, long long jstride) const {
    StepArgs a;
    memset(&a, 0, sizeof(a));
    a.W = W; a.wn = wn; a.bias = bias; a.wm = layer_map(l, js0, jstride);
    a.Dm = Dm; a.dm = a.wm;
    a.sp = 1.0f; a.hs = pl.hl[l]; a.mode = MODE_PHI; a.act = act;
    a.M = pl.M; a.Nf = pl.Nf; a.K = pl.K; a.Himg = p->Himg; a.Wimg = p->Wimg; a.TH = pl.TH;
    a.E = pl.E; a.wsize = pl.wsize;
    a.dbf16 = p->dtype == MGRIT_BF16 ? 1 : 0; a.dbits = dbits;
    // weights that a level touches: above 128 MB they are streamed past the caches, else later sweeps of the
    // same cycle find them in the last-level cache (a coarse level re-reads its few layers several times per cycle)
    a.wstream = (double)pl.Nl[l] * (double)pl.wsize * (double)pl.esize > 128.0 * 1024.0 * 1024.0 ? 1 : 0;
    return a;
  }
  // Groups of a launch whose layer a.wm(gi) is fully connected: gi = g0 + per * j, j < cnt.  The layer index is
  // affine in gi, so the solutions of  layer = 0 (mod fcP)  form an arithmetic progression.
  void fc_subset(const PtMap& wm, int groups, long long* g0, long long* per, int* cnt) const {
    *g0 = 0; *per = 1; *cnt = 0;
    const long long P = pl.fcP;
    if (!P) return;
    const long long st = ((wm.stride % P) + P) % P;
    long long a = st, b = P;                                // gcd(stride mod P, P); gcd(0, P) = P
    while (a) { const long long t = b % a; b = a; a = t; }
    *per = P / b;
    const long long lim = groups < *per ? groups : *per;
    for (long long gi = 0; gi < lim; ++gi)
      if ((((wm.base + gi * wm.stride) % P) + P) % P == 0) {
        *g0 = gi;
        *cnt = (int)((groups - 1 - gi) / *per + 1);
        return;
      }
  }
  StepArgs fc_args(const StepArgs& a, long long g0, long long per) const {
    auto sub = [&](const PtMap& mp) { return PtMap{mp.base + g0 * mp.stride, mp.stride * per}; };
    StepArgs d = a;
    d.xm = sub(a.xm); d.dm = sub(a.dm); d.om = sub(a.om); d.e1m = sub(a.e1m); d.rm = sub(a.rm);
    d.wm = PtMap{(a.wm.base + g0 * a.wm.stride) / pl.fcP, a.wm.stride * per / pl.fcP};
    d.W = Wfc; d.wn = wn_fc; d.bias = a.bias ? bfc : nullptr;
    d.M = pl.B; d.Nf = (int)pl.dfc; d.K = (int)pl.dfc; d.Himg = 0; d.Wimg = 0; d.TH = 0;
    d.wsize = pl.wsize_fc;
    d.wstream = (double)pl.nfc * (double)pl.wsize_fc * (double)pl.esize > 128.0 * 1024.0 * 1024.0 ? 1 : 0;
    d.skip0 = 0; d.skipper = 0;
    return d;
  }
  // workgroups (= norm partials) of a step launch over `groups` groups
  int launch_blocks(const StepArgs& a, int groups) const {
    int nb = step_grid_blocks(a, p->layer, p->dtype, groups) * groups;
    if (pl.fcP) {
      long long g0, per; int cnt;
      fc_subset(a.wm, groups, &g0, &per, &cnt);
      if (cnt) nb += step_grid_blocks(fc_args(a, g0, per), MGRIT_LAYER_DENSE, p->dtype, cnt) * cnt;
    }
    return nb;
  }
  void launch(const StepArgs& a, int groups) {
    flush();
    if (err != hipSuccess) return;
    if (!pl.fcP) { chk(launch_step(a, p->layer, p->dtype, groups, s)); return; }
    // mixed stack: the convolution kernel passes over the fully connected groups, a dense launch serves them
    long long g0, per; int cnt;
    fc_subset(a.wm, groups, &g0, &per, &cnt);
    StepArgs c = a;
    if (cnt) { c.skip0 = (int)g0; c.skipper = (int)per; }
    if (cnt < groups || a.norm_partial) chk(launch_step(c, p->layer, p->dtype, groups, s));
    if (cnt && err == hipSuccess) {
      StepArgs d = fc_args(a, g0, per);
      if (a.norm_partial) d.norm_partial = a.norm_partial + (size_t)step_grid_blocks(a, p->layer, p->dtype, groups) * groups;
      chk(launch_step(d, MGRIT_LAYER_DENSE, p->dtype, cnt, s));
    }
  }
  // states out[om] = Phi(in[im]) + g[l][js] for js = js0 + gi*jstride     (relaxation, coarsest solve)
  void step(int l, long long js0, long long jstride, int groups, const float* in, PtMap im, float* out, PtMap om) {
    StepArgs a = base_args(l, js0, jstride);
    a.X = in; a.xm = im;
    a.Out = out; a.om = om;
    if (g[l] && !plain_rhs) { a.E1 = g[l]; a.e1m = PtMap{js0, jstride}; a.c1 = 1.0f; }
    launch(a, groups);
  }
  void propagate(int l, long long js0, long long jstride, int groups) {
    step(l, js0, jstride, groups, X[l], pm(l, js0 - 1, jstride), X[l], pm(l, js0, jstride));
  }
  // dense layers of the wide sweep (q says nothing of other layers)
  bool wide_layers() const { return p->layer == MGRIT_LAYER_DENSE && wide_supported(p->q, p->dtype); }
  // Layers whose state fits on a CU -- convolution layers on images of at most 1024 pixels, dense layers of width at most
  // 256, in bf16 1024: all relaxation of a level's visit is one launch (march), the closing F-relaxation and the coarsest solve are
  // one launch each.  Whole solves 372 -> 226 us (5 images of 13 x 17 pixels, 24 channels, bf16), 1405 -> 797 us
  // (64 of 28 x 28, 16 channels, float), 16.6 -> 9.3 ms (32 of 32 x 32, 64 channels, bf16);
  // 655 -> 521 us (128 samples, width 256, float); width 8 and 16, where launches are saved as well, 250 -> 67 us (4 samples, width 8).
  // Where a step of a chain is long, a level needs enough chains: a lockstep launch spreads one step over many workgroups.
  // us per step with one chain (images, or slices of 16 rows, on as many CUs), sweep / lockstep, forward and adjoint:
  //   64 channels on more than 512 pixels: 24.5 / 24.4 forward with 128 images, 27.9 / 45 with 256 (32 x 32); adjoint 50 / 42 with
  //   128, 52 / 55 with 144 (32 x 32), 37.3 / 36.2 with 160 and 40 / 50 with 192 (23 x 23); 48 channels adjoint on 32 x 32 17.1 / 16.5
  //   with 8, 20.7 / 21.2 with 32; float of width 136 to 256: 5.5 (and a barrier's wait between two kernels less) / 5.0 for 8
  //   slices, level with 7.4 at 128.
  // bf16 of width 264 to 1024: a workgroup has a CU to itself, so a sweep goes in rounds of 256 of them.  Time of a level's
  // relaxation, lockstep / sweep, forward (adjoint), mean over m = 2, 4 and 16, at widths 1024, 768, 640 and 512, 256 rows:
  //   80 workgroups  0.62 (0.64)   0.93 (1.01)   1.08 (1.11)   1.08 (1.24)
  //   160            1.01 (0.95)   0.96 (1.01)   1.11 (1.15)   1.30 (1.39)
  //   208            1.14 (1.10)   1.44 (1.43)   1.65 (1.57)   1.42 (1.51)
  //   256            1.12 (1.14)   1.59 (1.45)   1.69 (1.56)   1.46 (1.51)
  //   260            0.80 (0.74)   0.93 (0.93)   0.99 (0.93)   1.21 (1.11)
  //   320            0.86 (0.79)   0.97 (0.97)   1.11 (1.08)   1.23 (1.17)
  //   352            0.88 (0.90)   1.20 (1.12)   1.14 (1.12)   1.22 (1.24)
  //   416            1.08 (1.04)   1.28 (1.18)   1.41 (1.27)   1.35 (1.40)
  //   516            0.96 (0.90)   1.12 (1.05)   1.10 (1.07)   1.27 (1.25)
  //   640            1.09 (1.04)   1.27 (1.30)   1.33 (1.28)   1.33 (1.33)
  // and 772 of them, the fourth round begun, 1.10 (1.05) at width 1024, 1.24 (1.19) at 768.  A second or third round is therefore
  // taken up where it is full enough.  64 rows, for which a lockstep launch reads every weight and uses half a tile, lose in the
  // first round alone: 80 workgroups 1.15 (0.89) and 1.01 (0.86) at 1024 and 768, 160 1.39 (1.23) and 1.55 (1.40), 257 1.13 (1.06)
  // and 1.33 (1.20).
  // Every other instance is as fast or faster with a single image at its largest size: float 16 channels on 32 x 32 7.0 / 7.1 and
  // 8.2 / 8.2, 32 on 16 x 32 9.9 / 16.3 and 11.4 / 17.9; bf16 32 channels on 32 x 32 8.0 / 8.9 and 9.2 / 10.3, 48 on 32 x 32
  // 13.3 / 14.3, 64 on 16 x 32 9.9 / 13.3 and 12.8 / 14.6; dense 1.4 .. 2.5 / 4 (float to 128), 0.9 .. 3.0 / 4.4 (bf16).
  bool use_march(int l) const {
    if (!sweep_enabled()) return false;
    const bool conv = p->layer == MGRIT_LAYER_CONV3X3;
    // Mixed stacks, forward: where the fully connected layers of a level open intervals (and on the coarsest level wherever they
    // are) they are launches of their own between sweeps over the convolution layers.  256 layers of 16 channels on 16 x 16
    // pixels, 32 images, one in 64 fully connected: the convolutions' lockstep launches took 1180 of 2300 us.
    if (pl.fcP && (adjoint || (l + 1 < pl.L && pl.fcP % (pl.mpow[l] * p->m) != 0))) return false;
    const bool wide = wide_layers();
    if (!(conv ? conv_sweep_supported(p->Himg, p->Wimg, p->C, p->dtype) : wide || sweep_supported(p->q))) return false;
    // (a launch holds less than 2^32 threads: at most 1024 for 16 rows, 512 for an image or 64 rows, of every chain)
    const long long units = conv ? p->B : wide ? wide_blocks(pl.M, 1) : (pl.M + 15LL) / 16;
    const long long most = units * (pl.L > 1 ? pl.Nl[1] + 1LL : 1LL);
    if (most * (conv ? 512 : 1024) >= 1LL << 32) return false;
    long long need = 1;
    const long long wgs = units * (l + 1 < pl.L ? pl.Nl[l + 1] : 1LL);
    if (wide) {
      const long long rounds = (wgs + 255) / 256;
      need = p->q > 768 ? 160 : p->q > 640 ? 144 : p->q > 512 ? 96 : 72;
      if (units > 1 && adjoint && p->q > 896) need = 200;
      if (units > 1 && p->q > 512 && (rounds == 2 || rounds == 3)) need = rounds * (p->q > 768 ? 200 : p->q > 640 ? 172 : 144);
    } else if (!conv) need = p->dtype == MGRIT_FP32 && p->q > 128 ? 128 : 1;
    else if (conv_sweep_ring(p->Himg, p->Wimg, p->C, p->dtype)) need = !adjoint ? 128 : p->Himg * p->Wimg >= 784 ? 144 : 192;
    else if (adjoint && p->C == 48 && p->Himg * p->Wimg > 900) need = 32;
    return wgs >= need;
  }
  // chains of level l that start at sweep point ci * stride, for every ci
  SweepArgs sweep_args(int l, long long stride) const {
    SweepArgs a;
    memset(&a, 0, sizeof(a));
    const long long mp = pl.mpow[l];
    if (g[l] && !plain_rhs) { a.G = g[l]; a.gb = 0; a.gs = stride; }
    a.W = W; a.wn = wn; a.bias = bias; a.Dm = Dm;
    if (adjoint) { a.lb = p->N - mp; a.ls = -stride * mp; a.lk = -mp; }
    else         { a.lb = 0;         a.ls = stride * mp;  a.lk = mp; }
    a.hs = pl.hl[l]; a.act = act == ACT_IDENT && dbits ? ACT_MASK : act;
    a.M = pl.M; a.q = pl.Nf; a.E = pl.E; a.wsize = pl.wsize;
    if (p->layer == MGRIT_LAYER_CONV3X3) { a.M = pl.B; a.Himg = p->Himg; a.Wimg = p->Wimg; a.C = p->C; }
    return a;
  }
  // the same, steps from + 1, from + 2, .. of the chains
  void start_behind(SweepArgs& a, int from) const {
    a.lb += from * a.lk;
    if (a.G) a.gb += from;
    if (a.X) a.xb += from * a.xk;
  }
  // Mixed stacks: the chains of a, groups of them, whose first layer is fully connected.  That step of theirs as one launch, into
  // out[om]; the sweep then goes on from there.
  void first_steps(SweepArgs& a, int l, long long js0, long long jstride, int groups, float* out, PtMap om) {
    if (!pl.fcP) return;
    StepArgs s1 = base_args(l, js0, jstride);
    long long g0, per; int cnt;
    fc_subset(s1.wm, groups, &g0, &per, &cnt);
    if (!cnt) return;
    s1.X = a.S; s1.xm = a.sm;
    s1.Out = out; s1.om = om;
    if (a.G) { s1.E1 = a.G; s1.e1m = PtMap{js0, jstride}; s1.c1 = 1.0f; }
    if (err == hipSuccess) chk(launch_step(fc_args(s1, g0, per), MGRIT_LAYER_DENSE, p->dtype, cnt, s));
    a.alt0 = (int)g0; a.altper = (int)per; a.Alt = out; a.am = om;
  }
  void keep_states(SweepArgs& a, int l, long long stride) const {   // into the level's own array
    const PtMap unit = pm(l, 0, 1);                                 // storage index of sweep point js = base + js * stride
    a.X = X[l]; a.xb = unit.base; a.xs = unit.stride * stride; a.xk = unit.stride;
  }
  // A sweep joins the ones before it in one launch if a slice's workgroup is done with it before a launch of its own would be:
  // us, measured -- a step takes 0.25 and, with many chains on one CU, 0.08 for each of them; a dependent launch 4 more, spread
  // over the CUs 0.3 a step.
  bool joins(const SweepArgs& a) const {
    const double step = 0.08 * a.nchains > 0.25 * wave_workgroups(a.nchains) ? 0.08 * a.nchains : 0.25 * wave_workgroups(a.nchains);
    return wave && 0.5 + step * a.nsteps <= 4.0 + 0.3 * a.nsteps;
  }
  void flush() {
    if (prog.nops == 0) return;
    // (a sweep that stayed alone gets all the workgroups it can use)
    const int per = prog.nops == 1 && !prog_by_slice ? wave_workgroups(prog.op[0].nchains) : 1;
    if (err == hipSuccess) chk(launch_wave(prog, per, p->dtype, prog_units, prog_bytes, s));
    prog.nops = 0; prog_units = 0; prog_bytes = 0.0; prog_by_slice = false;
  }
  void collect(const SweepArgs& a) {
    const bool join = joins(a);
    if (!join || prog.nops == WAVE_OPS) flush();
    prog.M = a.M; prog.q = a.q; prog.act = a.act; prog.wn = a.wn;
    prog.W = a.W; prog.bias = a.bias; prog.Dm = a.Dm; prog.E = a.E; prog.wsize = a.wsize;
    WaveOp& o = prog.op[prog.nops++];
    o.S = a.S; o.X = a.X; o.Y = a.Y; o.Z = a.Z; o.Ref = a.Ref; o.G = a.G; o.norm_partial = a.norm_partial;
    o.sb = (int)a.sm.base; o.ss = (int)a.sm.stride;
    o.xb = (int)a.xb; o.xs = (int)a.xs; o.xk = (int)a.xk; o.store0 = a.store0;
    o.yb = (int)a.yb; o.ys = (int)a.ys; o.kmid = a.kmid;
    o.zb = (int)a.zb; o.zs = (int)a.zs; o.zfirst = (int)a.zfirst; o.tau = a.tau;
    o.rb = (int)a.rm.base; o.rs = (int)a.rm.stride; o.gb = (int)a.gb; o.gs = (int)a.gs;
    o.lb = (int)a.lb; o.ls = (int)a.ls; o.lk = (int)a.lk;
    o.nsteps = a.nsteps; o.nlast = a.nlast; o.nchains = a.nchains; o.hs = a.hs;
    prog_by_slice |= join && a.norm_partial;
    prog_units += a.units;
    prog_bytes += sweep_bytes(a, p->dtype);
    if (!join) flush();
  }
  // workgroups (= norm partials) of the launch of a
  int march_blocks(const SweepArgs& a) const {
    if (wave) return wave_slices(a.M) * (joins(a) ? 1 : wave_workgroups(a.nchains));
    if (wide_layers()) return wide_blocks(a.M, a.nchains);
    return p->layer == MGRIT_LAYER_CONV3X3 ? conv_sweep_blocks(a, p->dtype) : sweep_blocks(a.M, a.nchains);
  }
  void launch_march(SweepArgs& a, long long units) {
    a.units = units;
    if (err != hipSuccess) return;
    if (wave) { collect(a); return; }
    chk(p->layer == MGRIT_LAYER_CONV3X3 ? launch_conv_sweep(a, p->dtype, s)
        : wide_layers()                 ? launch_wide(a, p->dtype, s)
                                        : launch_sweep(a, p->dtype, s));
  }
  // Where the current values of a level's C-points 0, m, 2m, .. are: point js = j m at p[m.base + j m.stride].
  // They do not live in the level's own array: the relaxation leaves them in R[l], the coarse solve in X[l + 1]
  // (it solves for their corrected values: with injection, U_C + (V_H - U_H) is V_H), and every consumer reads them
  // there.  The level's own array receives them once, when the level is closed.
  struct CPoints { const float* p; PtMap m; };

  void f_relax(int l, const CPoints& c) {                      // Sec. III-C, Fig. 3
    const int Nc = pl.Nl[l + 1];
    const int tail = pl.Nl[l] - Nc * p->m;                     // F-points behind the last C-point (< m)
    step(l, 1, p->m, Nc + (1 <= tail ? 1 : 0), c.p, c.m, X[l], pm(l, 1, p->m));
    for (int k = 2; k < p->m; ++k) propagate(l, k, p->m, Nc + (k <= tail ? 1 : 0));
  }
  // The level's own array, complete: C-points from the level below, F-points by F-relaxation (Alg. 1 ends with the
  // C-points; the F-layers follow by F-relaxation, Sec. III-C).
  void close(int l) {
    if (use_march(l)) {
      // chain ci: the C-point and the F-points behind it; trailing F-points are a chain of their own behind the last C-point,
      // which otherwise the last chain passes on
      SweepArgs a = sweep_args(l, p->m);
      const int Nc = pl.Nl[l + 1];
      a.S = X[l + 1]; a.sm = PtMap{0, 1};
      keep_states(a, l, p->m);
      const int tail = pl.Nl[l] - Nc * p->m;
      a.store0 = tail > 0 ? 1 : 2;
      a.nsteps = p->m - 1; a.nlast = tail > 0 ? tail : p->m - 1; a.nchains = Nc + (tail > 0 ? 1 : 0);
      first_steps(a, l, 1, p->m, a.nchains, X[l], pm(l, 1, p->m));
      launch_march(a, pl.Nl[l] - Nc);
      return;
    }
    flush();
    chk(launch_copy_points(X[l], pm(l, 0, p->m), X[l + 1], PtMap{0, 1}, pl.E, pl.Nl[l + 1] + 1, s));
    f_relax(l, CPoints{X[l + 1], PtMap{0, 1}});
  }

  // The coarsest level: its points in sequence.  X[l][0] holds the known value.
  void serial(int l) {
    if (use_march(l)) {
      for (int j = 0; j < pl.Nl[l];) {                          // (one run, in a mixed stack those between fully connected layers)
        auto fc = [&](int i) { return pl.fcP && layer_map(l, i + 1, 1).base % pl.fcP == 0; };     // step i + 1
        int end = j;
        while (end < pl.Nl[l] && !fc(end)) ++end;
        if (end > j) {
          SweepArgs a = sweep_args(l, 0);
          a.S = X[l]; a.sm = pm(l, j, 0);
          keep_states(a, l, 0);
          start_behind(a, j);
          a.nsteps = a.nlast = end - j; a.nchains = 1;
          launch_march(a, end - j);
        }
        for (j = end; j < pl.Nl[l] && fc(j); ++j) propagate(l, j + 1, 1, 1);
      }
      return;
    }
    for (int j = 1; j <= pl.Nl[l]; ++j) propagate(l, j, 1, 1);
  }

  // Relaxation of level l from the C-points c, and the step P_j that lands on every C-point j, in one launch.  A chain
  // starts at C-point ci.  FCF-relaxation: m - 1 F-steps, the C-step to the new value of C-point ci + 1 (kept in R[l]), and
  // on through the next interval's F-steps to P_{ci + 2}: the new C-point is where the second F-relaxation of that interval
  // starts.  The first interval's C-point does not change, so its second F-relaxation repeats the first and P_1 is the new
  // value of C-point 1; the last chain ends at the last C-point.  F-relaxation: m - 1 F-steps and P_{ci + 1}.
  void march(int l, const CPoints& c) {
    const int m = p->m, Nc = pl.Nl[l + 1];
    SweepArgs a = sweep_args(l, m);
    a.S = c.p; a.sm = c.m;
    a.nchains = Nc;
    a.Z = g[l + 1];
    if (pl.fcP) {
      // Mixed stack: fully connected layers open intervals, so a chain has them in step 1 and, under FCF-relaxation, in step
      // m + 1: two sweeps.  The states behind those steps wait at their F-points in the level's own array, where lockstep
      // relaxation has them too and which no sweep writes before the level is closed.
      first_steps(a, l, 1, m, Nc, X[l], pm(l, 1, m));
      a.nsteps = a.nlast = m;
      a.zb = 1; a.zs = 1;
      if (p->relax == MGRIT_RELAX_FCF) { a.Y = R[l]; a.yb = 1; a.ys = 1; a.kmid = m; a.zfirst = 1; }
      launch_march(a, pl.Nl[l]);
      if (p->relax != MGRIT_RELAX_FCF || Nc < 2) return;
      SweepArgs b = sweep_args(l, m);
      start_behind(b, m);
      b.S = R[l]; b.sm = PtMap{1, 1};
      b.nsteps = b.nlast = m; b.nchains = Nc - 1;
      b.Z = g[l + 1]; b.zb = 2; b.zs = 1;
      first_steps(b, l, m + 1, m, Nc - 1, X[l], pm(l, m + 1, m));
      launch_march(b, pl.Nl[l]);
      return;
    }
    if (p->relax == MGRIT_RELAX_FCF) {
      a.Y = R[l]; a.yb = 1; a.ys = 1; a.kmid = m;
      a.zb = 2; a.zs = 1; a.zfirst = 1;
      a.nsteps = 2 * m; a.nlast = m;
    } else {
      a.zb = 1; a.zs = 1;
      a.nsteps = a.nlast = m;
    }
    // (counted as the relaxation's lockstep launches are: the trailing F-points and the first interval's repeated sweep,
    // which change nothing before the level is closed, among them)
    launch_march(a, (p->relax == MGRIT_RELAX_FCF ? 2 : 1) * (long long)pl.Nl[l]);
  }

  // Nested-iteration start: the coarsest level's own equation is solved in sequence from the known
  // value; going up, the C-points of a level take the coarser level's values and (on the middle
  // levels) the F-points follow by F-relaxation.  The fine level's C-points are then level 1's values.
  void nested_start() {
    plain_rhs = true;
    const int lc = pl.L - 1;
    serial(lc);
    for (int l = lc - 1; l >= 1; --l) close(l);
    plain_rhs = false;
  }

  // the coarse right-hand side of level l as lockstep steps: S_H = P - Phi_H, P in place
  StepArgs rhs_args(int l, const CPoints& c) const {
    StepArgs a = base_args(l + 1, 1, 1);
    a.X = c.p; a.xm = c.m;
    a.Out = g[l + 1]; a.om = PtMap{1, 1};
    a.sp = -1.0f;
    a.E1 = g[l + 1]; a.e1m = PtMap{1, 1}; a.c1 = 1.0f;          // in place, element by element
    return a;
  }
  double norm_scale() const {          // of the C-point residual of the fine level
    return p->norm_kind == MGRIT_NORM_RMS ? 1.0 / sqrt((double)(pl.Nl[1] + 1) * (double)pl.E) : 1.0;
  }

  // One visit of level l, up to the new values of its C-points in X[l + 1] (of all its points on the coarsest level).
  // c: the C-points' current values (unused on the coarsest level).
  void cycle(int l, int iter, CPoints c) {
    const int m = p->m;
    if (l == pl.L - 1) { serial(l); return; }
    const int Nc = pl.Nl[l + 1];
    // Alg. 1 steps 2 and 3.  With P_j the layer step that lands on C-point j (plus the level's right-hand side) the
    // residual there is R_j = P_j - U_j, Eq. (19), and the coarse right-hand side
    // S_H = L_H(U_H) + R_H = U_j - Phi_H(U_{j-1}) + P_j - U_j = P_j - Phi_H(U_{j-1}): the residual itself is needed for
    // its norm only, which the second launch takes of E1 - Ref.
    if (use_march(l)) {
      march(l, c);                                              // Alg. 1 step 1, and P
      if (p->relax == MGRIT_RELAX_FCF) c = CPoints{R[l], PtMap{0, 1}};
    } else {
      f_relax(l, c);                                            // Alg. 1 step 1
      if (p->relax == MGRIT_RELAX_FCF) {
        step(l, m, m, Nc, X[l], pm(l, m - 1, m), R[l], PtMap{1, 1});
        c = CPoints{R[l], PtMap{0, 1}};
        f_relax(l, c);
      }
      step(l, m, m, Nc, X[l], pm(l, m - 1, m), g[l + 1], PtMap{1, 1});
    }
    const bool norm = l == 0 && want_norm;
    const PtMap next = PtMap{c.m.base + c.m.stride, c.m.stride};
    float* sums = partial;                                      // one per workgroup
    int blocks;
    if (use_march(l + 1)) {
      // (the coarse step here and the one of the coarse solve nearly cancel, so they have to round alike and are the same
      // kernel's.  With the lockstep kernel here and sweeps there: float 1.7e-7 from the exact states instead of 1.0e-7;
      // in bf16, where a last bit may flip the rounding of an operand, the residual stays above 2e-6 for ever)
      SweepArgs a = sweep_args(l + 1, 1);
      a.G = nullptr;
      a.S = c.p; a.sm = c.m;
      a.nsteps = a.nlast = 1; a.nchains = Nc;
      a.tau = 1; a.Z = g[l + 1]; a.zb = 1; a.zs = 1;
      // (a slice of 16 rows may be less than a lockstep tile, which `partial` is sized for; a state of every chain that nothing
      // needs at this point holds more: the coarse solve's, or the residual's where only FCF-relaxation uses it)
      sums = p->relax == MGRIT_RELAX_FCF ? X[l + 1] + pl.E : R[l];
      if (norm && iter == 0 && p->tol <= 0.0f && joins(a) && (size_t)wave_slices(pl.M) * p->max_iter <= pl.n_partial)
        late_norms = wave_slices(pl.M);
      if (norm && late_norms) sums = partial + (size_t)iter * late_norms;
      if (norm) { a.Ref = c.p; a.rm = next; a.norm_partial = sums; }
      blocks = march_blocks(a);
      if (pl.fcP) {                                             // the coarse steps of fully connected layers by themselves
        StepArgs d = rhs_args(l, c);
        long long g0, per; int cnt;
        fc_subset(d.wm, Nc, &g0, &per, &cnt);
        if (cnt) {
          a.alt0 = (int)g0; a.altper = (int)per;
          d = fc_args(d, g0, per);
          if (norm) {
            const PtMap rn{next.base + g0 * next.stride, next.stride * per};
            d.Ref = c.p; d.rm = rn; d.norm_partial = sums + blocks;
            blocks += step_grid_blocks(d, MGRIT_LAYER_DENSE, p->dtype, cnt) * cnt;
          }
          if (err == hipSuccess) chk(launch_step(d, MGRIT_LAYER_DENSE, p->dtype, cnt, s));
        }
      }
      launch_march(a, Nc);
    } else {
      StepArgs a = rhs_args(l, c);
      if (norm) { a.Ref = c.p; a.rm = next; a.norm_partial = partial; }
      launch(a, Nc);
      blocks = launch_blocks(a, Nc);
    }
    if (norm && !late_norms) {
      flush();
      chk(launch_norm_final(sums, blocks, norm_scale(), hist_dev + iter, 1, s));
    }
    cycle(l + 1, iter, CPoints{c.p, PtMap{c.m.base, c.m.stride * m}});   // V_H, Alg. 1 steps 3 to 5
    if (l + 1 < pl.L - 1) close(l + 1);
  }
};

int check_finite(const double* h, int n) {
  for (int i = 0; i < n; ++i)
    if (!isfinite(h[i])) return MGRIT_ERR_NONFINITE;
  return MGRIT_OK;
}

// Runs the solve loop shared by the forward and the adjoint entry point.
int run_solver(Solver& sv, const float* first, double* resnorm_hist, int32_t* iters_done) {
  const mgrit_problem_t* p = sv.p;
  const Plan& pl = sv.pl;
  const int m = p->m;
  // the known value, in every array that holds sweep point 0, and the initial guess of the C-points
  sv.wave = p->layer == MGRIT_LAYER_DENSE && !pl.fcP && wave_supported(p->q) && sv.use_march(0) && sv.use_march(pl.L - 1);
  sv.want_norm = p->tol > 0.0f || resnorm_hist;
  float* zero_pt[2 * MGRIT_MAX_LEVELS];
  int nz = 0;
  // MGRIT_INIT_COPY: the known value everywhere, from the coarsest level's copy of it (`first` may be a row of the caller's
  // array, the last state of an earlier solve, that the relaxation writes to)
  Solver::CPoints c{sv.X[pl.L - 1], PtMap{0, 0}};
  if (pl.L == 1) {
    zero_pt[nz++] = sv.X[0] + sv.pm(0, 0, 0).base * pl.E;
  } else {
    zero_pt[nz++] = sv.X[pl.L - 1];
    for (int l = 0; l + 1 < pl.L && p->relax == MGRIT_RELAX_FCF; ++l) zero_pt[nz++] = sv.R[l];
    if (p->init == MGRIT_INIT_ZERO || p->init == MGRIT_INIT_USER) {
      c = Solver::CPoints{sv.X[0], sv.pm(0, 0, m)};
      zero_pt[nz++] = sv.X[0] + c.m.base * pl.E;
    }
  }
  if (sv.wave) {
    for (int i = 0; i < nz; ++i) {                              // chains of no steps
      SweepArgs a = sv.sweep_args(0, 0);
      a.G = nullptr;
      a.S = first; a.sm = PtMap{0, 0};
      a.X = zero_pt[i]; a.store0 = 1;
      a.nchains = 1;
      sv.launch_march(a, 0);
    }
  } else {
    sv.chk(launch_spread_state(zero_pt, nz, first, pl.E, sv.s));
  }
  if (pl.L > 1 && p->init == MGRIT_INIT_ZERO) {
    sv.flush();
    sv.chk(launch_zero_points(sv.X[0], sv.pm(0, m, m), pl.E, pl.Nl[1], sv.s));
  }
  if (pl.L > 1 && p->init == MGRIT_INIT_NESTED) {
    sv.nested_start();
    c = Solver::CPoints{sv.X[1], PtMap{0, 1}};
  }

  int iters = 0;
  int rc = MGRIT_OK;
  if (pl.L == 1) {
    sv.cycle(0, 0, c);
    sv.flush();
    iters = 1;
    if (resnorm_hist) resnorm_hist[0] = 0.0;
    if (sv.err == hipSuccess && (resnorm_hist || iters_done)) sv.chk(hipStreamSynchronize(sv.s));
  } else {
    for (int k = 0; k < p->max_iter && sv.err == hipSuccess; ++k) {
      sv.cycle(0, k, c);
      c = Solver::CPoints{sv.X[1], PtMap{0, 1}};
      ++iters;
      if (p->tol > 0.0f) {
        double v = 0.0;
        sv.flush();
        sv.chk(hipMemcpyAsync(&v, sv.hist_dev + k, sizeof(double), hipMemcpyDeviceToHost, sv.s));
        sv.chk(hipStreamSynchronize(sv.s));
        if (sv.err != hipSuccess) break;
        if (resnorm_hist) resnorm_hist[k] = v;
        if (!isfinite(v)) { rc = MGRIT_ERR_NONFINITE; break; }
        if (v <= (double)p->tol) break;
      }
    }
    if (sv.err == hipSuccess) sv.close(0);
    sv.flush();
    if (sv.late_norms && sv.err == hipSuccess)
      sv.chk(launch_norm_final(sv.partial, sv.late_norms, sv.norm_scale(), sv.hist_dev, iters, sv.s));
    if (!(p->tol > 0.0f) && resnorm_hist && sv.err == hipSuccess) {
      sv.chk(hipMemcpyAsync(resnorm_hist, sv.hist_dev, sizeof(double) * iters, hipMemcpyDeviceToHost, sv.s));
      sv.chk(hipStreamSynchronize(sv.s));
      if (sv.err == hipSuccess) rc = check_finite(resnorm_hist, iters);
    } else if ((iters_done || resnorm_hist) && sv.err == hipSuccess) {
      sv.chk(hipStreamSynchronize(sv.s));
    }
  }
  if (iters_done) *iters_done = iters;
  if (sv.err != hipSuccess) return MGRIT_ERR_HIP;
  return rc;
}

void bind_workspace(Solver& sv, void* workspace) {
  unsigned char* ws = static_cast<unsigned char*>(workspace);
  const Plan& pl = sv.pl;
  for (int l = 1; l < pl.L; ++l) {
    sv.X[l] = reinterpret_cast<float*>(ws + pl.off_X[l]);
    sv.g[l] = reinterpret_cast<float*>(ws + pl.off_g[l]);
  }
  for (int l = 0; l + 1 < pl.L; ++l) {
    sv.R[l] = reinterpret_cast<float*>(ws + pl.off_R[l]);
  }
  sv.partial = reinterpret_cast<float*>(ws + pl.off_partial);
  sv.hist_dev = reinterpret_cast<double*>(ws + pl.off_hist);
}

// checks of the fully connected part of a mixed stack (fc == nullptr: plain stack)
int check_fc(const mgrit_fc_layers_t* fc, bool adjoint, const float* dW, const float* db) {
  if (!fc) return MGRIT_OK;
  if (!fc->Wfc || !fc->bfc || !aligned(fc->Wfc) || !aligned(fc->bfc)) return MGRIT_ERR_POINTER;
  if (adjoint) {
    if ((dW && !fc->dWfc) || (db && !fc->dbfc)) return MGRIT_ERR_POINTER;
    if (!aligned(fc->dWfc) || !aligned(fc->dbfc)) return MGRIT_ERR_POINTER;
  }
  return MGRIT_OK;
}

int forward_impl(const mgrit_problem_t* p, const mgrit_fc_layers_t* fc, const void* W, const float* b,
                 const float* u0, float* U, double* resnorm_hist, int32_t* iters_done, void* workspace,
                 size_t workspace_bytes, void* hip_stream) {
  if (!p || !W || !b || !u0 || !U || !workspace) return MGRIT_ERR_POINTER;
  if (!aligned(W) || !aligned(b) || !aligned(u0) || !aligned(U) || !aligned(workspace)) return MGRIT_ERR_POINTER;
  int rc = check_fc(fc, false, nullptr, nullptr);
  if (rc != MGRIT_OK) return rc;
  Solver sv;
  rc = make_plan(p, &sv.pl, fc ? fc->fc_period : 0);
  if (rc != MGRIT_OK) return rc;
  if (fc && !sv.pl.fcP) return MGRIT_ERR_PROBLEM;
  if (workspace_bytes < sv.pl.bytes_fwd) return MGRIT_ERR_WORKSPACE;
  sv.p = p; sv.s = static_cast<hipStream_t>(hip_stream); sv.adjoint = false;
  memset(sv.X, 0, sizeof(sv.X)); memset(sv.g, 0, sizeof(sv.g)); memset(sv.R, 0, sizeof(sv.R));
  sv.X[0] = U;
  sv.W = W; sv.bias = b; sv.Dm = nullptr; sv.act = p->act;
  if (fc) { sv.Wfc = fc->Wfc; sv.bfc = fc->bfc; }
  bind_workspace(sv, workspace);
  return run_solver(sv, u0, resnorm_hist, iters_done);
}

int adjoint_impl(const mgrit_problem_t* p, const mgrit_fc_layers_t* fc, const void* W, const float* b,
                 const float* U, const float* lamN, float* Lam, float* dW, float* db, double* resnorm_hist,
                 int32_t* iters_done, void* workspace, size_t workspace_bytes, void* hip_stream) {
  if (!p || !W || !b || !U || !lamN || !Lam || !workspace) return MGRIT_ERR_POINTER;
  if (!aligned(W) || !aligned(b) || !aligned(U) || !aligned(lamN) || !aligned(Lam) || !aligned(workspace) ||
      !aligned(dW) || !aligned(db))
    return MGRIT_ERR_POINTER;
  int rc = check_fc(fc, true, dW, db);
  if (rc != MGRIT_OK) return rc;
  Solver sv;
  rc = make_plan(p, &sv.pl, fc ? fc->fc_period : 0);
  if (rc != MGRIT_OK) return rc;
  if (fc && !sv.pl.fcP) return MGRIT_ERR_PROBLEM;
  if (workspace_bytes < sv.pl.bytes_adj) return MGRIT_ERR_WORKSPACE;
  const Plan& pl = sv.pl;
  sv.p = p; sv.s = static_cast<hipStream_t>(hip_stream); sv.adjoint = true;
  memset(sv.X, 0, sizeof(sv.X)); memset(sv.g, 0, sizeof(sv.g)); memset(sv.R, 0, sizeof(sv.R));
  sv.X[0] = Lam;
  bind_workspace(sv, workspace);
  unsigned char* ws = static_cast<unsigned char*>(workspace);
  void* Wt = ws + pl.off_Wt;
  void* Wfct = ws + pl.off_Wfct;
  float* D = reinterpret_cast<float*>(ws + pl.off_D);
  // transposed parameters (convolution layers, whose taps are mirrored as well; dense and fully connected
  // matrices only on request), and act'(A_n U^n + b_n) for every layer in one grouped launch
  const bool copy_dense = adjoint_transposed_copy();
  const bool copy_main = p->layer != MGRIT_LAYER_DENSE || copy_dense;
  if (copy_main) sv.chk(launch_transpose_weights(W, Wt, p->layer, p->dtype, p->N, pl.Nf, sv.s));
  if (fc && copy_dense) sv.chk(launch_transpose_weights(fc->Wfc, Wfct, MGRIT_LAYER_DENSE, p->dtype, pl.nfc, (int)pl.dfc, sv.s));
  {
    sv.W = W; sv.bias = b; sv.Dm = nullptr; sv.act = p->act;
    sv.dbits = p->act == MGRIT_ACT_RELU &&
               act_factor_bits(p, (double)p->N * (double)pl.E * (double)pl.esize);
    if (fc) { sv.Wfc = fc->Wfc; sv.bfc = fc->bfc; }
    StepArgs a = sv.base_args(0, 1, 1);
    a.wm = PtMap{0, 1};
    a.mode = MODE_DACT;
    a.X = U; a.xm = PtMap{0, 1};
    a.Out = D; a.om = PtMap{0, 1};
    sv.launch(a, p->N);
  }
  sv.bias = nullptr; sv.Dm = D; sv.act = ACT_IDENT;
  if (copy_main) sv.W = Wt; else { sv.W = W; sv.wn = 1; }
  if (fc) {
    sv.bfc = nullptr;
    if (copy_dense) sv.Wfc = Wfct; else { sv.Wfc = fc->Wfc; sv.wn_fc = 1; }
  }
  rc = run_solver(sv, lamN, resnorm_hist, iters_done);
  if (rc != MGRIT_OK && rc != MGRIT_ERR_NONFINITE) return rc;
  if (dW || db) {
    GradArgs ga;
    memset(&ga, 0, sizeof(ga));
    ga.U = U; ga.um = PtMap{0, 1};
    ga.Lam = Lam; ga.lm = PtMap{1, 1};
    ga.Dm = D; ga.dm = PtMap{0, 1}; ga.dbits = sv.dbits;
    ga.dW = dW; ga.db = db; ga.hs = p->h;
    ga.M = pl.M; ga.Nf = pl.Nf; ga.K = pl.K; ga.Himg = p->Himg; ga.Wimg = p->Wimg; ga.B = p->B;
    ga.E = pl.E; ga.wsize = pl.wsize;
    ga.partial = reinterpret_cast<float*>(ws + pl.off_gpart);
    if (launch_grad(ga, p->layer, p->dtype, p->N, sv.s) != hipSuccess) return MGRIT_ERR_HIP;
    if (fc) {
      // the convolution gradient ran over every layer: its slots at the fully connected layers are defined as
      // zero; their own gradient is the dense contraction over the batch
      const long long P = pl.fcP;
      if (dW) sv.chk(launch_zero_points(dW, PtMap{0, P}, pl.wsize, pl.nfc, sv.s));
      if (db) sv.chk(launch_zero_points(db, PtMap{0, P}, pl.Nf, pl.nfc, sv.s));
      GradArgs gd;
      memset(&gd, 0, sizeof(gd));
      gd.U = U; gd.um = PtMap{0, P};
      gd.Lam = Lam; gd.lm = PtMap{1, P};
      gd.Dm = D; gd.dm = PtMap{0, P}; gd.dbits = sv.dbits;
      gd.dW = dW ? fc->dWfc : nullptr; gd.db = db ? fc->dbfc : nullptr; gd.hs = p->h;
      gd.M = p->B; gd.Nf = (int)pl.dfc; gd.K = (int)pl.dfc; gd.B = p->B;
      gd.E = pl.E; gd.wsize = pl.wsize_fc;
      if (sv.err != hipSuccess || launch_grad(gd, MGRIT_LAYER_DENSE, p->dtype, pl.nfc, sv.s) != hipSuccess)
        return MGRIT_ERR_HIP;
    }
    if (resnorm_hist || iters_done)
      if (hipStreamSynchronize(sv.s) != hipSuccess) return MGRIT_ERR_HIP;
  }
  return rc;
}

int residual_norm_impl(const mgrit_problem_t* p, const mgrit_fc_layers_t* fc, const void* W, const float* b,
                       const float* u0, const float* U, double* norm_out, void* workspace, size_t workspace_bytes,
                       void* hip_stream) {
  if (!p || !W || !b || !u0 || !U || !norm_out || !workspace) return MGRIT_ERR_POINTER;
  if (!aligned(W) || !aligned(b) || !aligned(u0) || !aligned(U) || !aligned(workspace)) return MGRIT_ERR_POINTER;
  int rc = check_fc(fc, false, nullptr, nullptr);
  if (rc != MGRIT_OK) return rc;
  Solver sv;
  rc = make_plan(p, &sv.pl, fc ? fc->fc_period : 0);
  if (rc != MGRIT_OK) return rc;
  if (fc && !sv.pl.fcP) return MGRIT_ERR_PROBLEM;
  if (workspace_bytes < sv.pl.bytes_fwd) return MGRIT_ERR_WORKSPACE;
  const Plan& pl = sv.pl;
  sv.p = p; sv.s = static_cast<hipStream_t>(hip_stream); sv.adjoint = false;
  memset(sv.X, 0, sizeof(sv.X)); memset(sv.g, 0, sizeof(sv.g)); memset(sv.R, 0, sizeof(sv.R));
  sv.W = W; sv.bias = b; sv.Dm = nullptr; sv.act = p->act;
  if (fc) { sv.Wfc = fc->Wfc; sv.bfc = fc->bfc; }
  bind_workspace(sv, workspace);
  // rows n = 1..N of f_h - L_h(U): Phi(U[n-1]) - U[n]; row 0: u0 - U[0]
  StepArgs a = sv.base_args(0, 1, 1);
  a.X = U; a.xm = PtMap{0, 1};
  a.E1 = U; a.e1m = PtMap{1, 1}; a.c1 = -1.0f;
  a.norm_partial = sv.partial;
  sv.launch(a, p->N);
  const int nb = sv.launch_blocks(a, p->N);
  int nb0 = 0;
  sv.chk(launch_diff_sq(u0, U, pl.E, sv.partial + nb, &nb0, sv.s));
  const double scale = p->norm_kind == MGRIT_NORM_RMS ? 1.0 / sqrt((double)(p->N + 1) * (double)pl.E) : 1.0;
  sv.chk(launch_norm_final(sv.partial, nb + nb0, scale, sv.hist_dev, 1, sv.s));
  double v = 0.0;
  sv.chk(hipMemcpyAsync(&v, sv.hist_dev, sizeof(double), hipMemcpyDeviceToHost, sv.s));
  sv.chk(hipStreamSynchronize(sv.s));
  if (sv.err != hipSuccess) return MGRIT_ERR_HIP;
  *norm_out = v;
  return isfinite(v) ? MGRIT_OK : MGRIT_ERR_NONFINITE;
}

// Workspace of the entry point that allocates nothing: a fixed array in device memory that every GPU the
// library runs on holds until the process ends.  In host code its name is only a handle; the address of a
// device's copy comes from hipGetSymbolAddress, once per device, and only that address is handed to kernels.
__device__ __align__(256) unsigned char scratch[MGRIT_STATIC_SCRATCH_BYTES];
void* g_scratch_ptr[64] = {};

}  // namespace

extern "C" {

int32_t mgrit_level_map(const mgrit_problem_t* p, int32_t* n_levels, int32_t* N_l, int32_t* fine_index) {
  if (!p || !n_levels) return MGRIT_ERR_POINTER;
  int L, Nl[MGRIT_MAX_LEVELS];
  const int rc = build_levels(p, &L, Nl);
  if (rc != MGRIT_OK) return rc;
  *n_levels = L;
  long long mp = 1;
  size_t pos = 0;
  for (int l = 0; l < L; ++l) {
    if (N_l) N_l[l] = Nl[l];
    if (fine_index)
      for (int j = 0; j <= Nl[l]; ++j) fine_index[pos++] = (int32_t)(j * mp);
    mp *= p->m;
  }
  return MGRIT_OK;
}

size_t mgrit_workspace_bytes(const mgrit_problem_t* p) {
  Plan pl;
  if (!p || make_plan(p, &pl) != MGRIT_OK) return 0;
  return pl.bytes_fwd;
}

size_t mgrit_adjoint_workspace_bytes(const mgrit_problem_t* p) {
  Plan pl;
  if (!p || make_plan(p, &pl) != MGRIT_OK) return 0;
  return pl.bytes_adj;
}

int32_t mgrit_fas_forward(const mgrit_problem_t* p, const void* W, const float* b, const float* u0, float* U,
                          double* resnorm_hist, int32_t* iters_done, void* workspace, size_t workspace_bytes,
                          void* hip_stream) {
  return forward_impl(p, nullptr, W, b, u0, U, resnorm_hist, iters_done, workspace, workspace_bytes, hip_stream);
}

int32_t mgrit_fas_adjoint(const mgrit_problem_t* p, const void* W, const float* b, const float* U, const float* lamN,
                          float* Lam, float* dW, float* db, double* resnorm_hist, int32_t* iters_done,
                          void* workspace, size_t workspace_bytes, void* hip_stream) {
  return adjoint_impl(p, nullptr, W, b, U, lamN, Lam, dW, db, resnorm_hist, iters_done, workspace, workspace_bytes,
                      hip_stream);
}

int32_t mgrit_residual_norm(const mgrit_problem_t* p, const void* W, const float* b, const float* u0, const float* U,
                            double* norm_out, void* workspace, size_t workspace_bytes, void* hip_stream) {
  return residual_norm_impl(p, nullptr, W, b, u0, U, norm_out, workspace, workspace_bytes, hip_stream);
}

int32_t mgrit_fas_forward_static(const mgrit_problem_t* p, const void* W, const float* b, const float* u0, float* U,
                                 double* resnorm_hist, int32_t* iters_done, void* hip_stream) {
  Plan pl;
  if (!p) return MGRIT_ERR_POINTER;
  const int rc = make_plan(p, &pl);
  if (rc != MGRIT_OK) return rc;
  if (pl.bytes_fwd > (size_t)MGRIT_STATIC_SCRATCH_BYTES) return MGRIT_ERR_WORKSPACE;
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess) return MGRIT_ERR_HIP;
  if (dev < 0 || dev >= 64) return MGRIT_ERR_UNSUPPORTED;
  if (!g_scratch_ptr[dev]) {                     // first call on this device: look up its copy of the array
    void* ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return MGRIT_ERR_HIP;
    g_scratch_ptr[dev] = ptr;
  }
  // nothing in the workspace has to start at zero: every array in it is written before it is read
  return forward_impl(p, nullptr, W, b, u0, U, resnorm_hist, iters_done, g_scratch_ptr[dev],
                      (size_t)MGRIT_STATIC_SCRATCH_BYTES, hip_stream);
}

size_t mgrit_workspace_bytes_mixed(const mgrit_problem_t* p, int32_t fc_period) {
  Plan pl;
  if (!p || fc_period < 2 || make_plan(p, &pl, fc_period) != MGRIT_OK) return 0;
  return pl.bytes_fwd;
}

size_t mgrit_adjoint_workspace_bytes_mixed(const mgrit_problem_t* p, int32_t fc_period) {
  Plan pl;
  if (!p || fc_period < 2 || make_plan(p, &pl, fc_period) != MGRIT_OK) return 0;
  return pl.bytes_adj;
}

int32_t mgrit_fas_forward_mixed(const mgrit_problem_t* p, const mgrit_fc_layers_t* fc, const void* W, const float* b,
                                const float* u0, float* U, double* resnorm_hist, int32_t* iters_done,
                                void* workspace, size_t workspace_bytes, void* hip_stream) {
  if (!fc) return MGRIT_ERR_POINTER;
  return forward_impl(p, fc, W, b, u0, U, resnorm_hist, iters_done, workspace, workspace_bytes, hip_stream);
}

int32_t mgrit_fas_adjoint_mixed(const mgrit_problem_t* p, const mgrit_fc_layers_t* fc, const void* W, const float* b,
                                const float* U, const float* lamN, float* Lam, float* dW, float* db,
                                double* resnorm_hist, int32_t* iters_done, void* workspace, size_t workspace_bytes,
                                void* hip_stream) {
  if (!fc) return MGRIT_ERR_POINTER;
  return adjoint_impl(p, fc, W, b, U, lamN, Lam, dW, db, resnorm_hist, iters_done, workspace, workspace_bytes,
                      hip_stream);
}

int32_t mgrit_residual_norm_mixed(const mgrit_problem_t* p, const mgrit_fc_layers_t* fc, const void* W,
                                  const float* b, const float* u0, const float* U, double* norm_out,
                                  void* workspace, size_t workspace_bytes, void* hip_stream) {
  if (!fc) return MGRIT_ERR_POINTER;
  return residual_norm_impl(p, fc, W, b, u0, U, norm_out, workspace, workspace_bytes, hip_stream);
}

void mgrit_trace_begin(void) { trace_begin(); }

int32_t mgrit_trace_end(double* ms, int64_t* launches, int64_t* units, double* bytes, int32_t n_classes) {
  if (!ms || !launches || !units || n_classes < 1) return MGRIT_ERR_POINTER;
  long long l[TRACE_NCLASS], u[TRACE_NCLASS];
  double m[TRACE_NCLASS], b[TRACE_NCLASS];
  if (trace_end(m, l, u, b, TRACE_NCLASS) != 0) return MGRIT_ERR_HIP;
  for (int i = 0; i < n_classes; ++i) {
    ms[i] = i < TRACE_NCLASS ? m[i] : 0.0;
    launches[i] = i < TRACE_NCLASS ? l[i] : 0;
    units[i] = i < TRACE_NCLASS ? u[i] : 0;
    if (bytes) bytes[i] = i < TRACE_NCLASS ? b[i] : 0.0;
  }
  return MGRIT_OK;
}

}  // extern "C"
