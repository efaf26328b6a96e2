// Internal declarations shared by the host schedule and the HIP kernels of the MGRIT-FAS
// library.  Not part of the public C ABI.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace mgrit {

// Affine map from the group index of a launch to a point (or layer) index of an array that
// is laid out [points][E]:  idx = base + gi * stride.  A negative stride walks the layer
// axis backwards (adjoint sweeps).
struct PtMap {
  long long base;
  long long stride;
};

// One layer-batched step launch: every group gi evaluates, for its own input point and its
// own layer parameters,
//     z   = A_layer * (Dm ? Dm .* X : X) + bias
//     phi = X + hs * act(z)                                   (Sec. II, Eq. (1))
//     out = sp * phi + c1 * E1                                (mode PHI)
//     out = act'(z)                                           (mode DACT)
// which covers F-/C-relaxation, the C-point residual, the FAS right-hand side and the adjoint
// steps (Sec. III-B, III-C).  If norm_partial is set, every workgroup also writes the sum of
// out^2, with Ref of (E1 - Ref)^2, over its tile to norm_partial[linear block index].
struct StepArgs {
  const float* X;   PtMap xm;
  const float* Dm;  PtMap dm;      // optional elementwise multiplier of the matrix operand (the act' cache);
                                   // its storage type is the weights' type: float, or bf16 when dbf16 is set; bits with dbits
  const void*  W;   PtMap wm;      // weights of layer wm(gi); element type = template parameter
  int wn;                          // dense only, 1: W holds W[k][n] (contraction index slowest), as the adjoint reads the
                                   // caller's weights without a transposed copy; 0: W[n][k].  Needs K == Nf and Dm.
  const float* bias;               // [layers][Nf] or null (same layer index as W)
  float* Out;       PtMap om;      // may be null when only the norm is wanted
  const float* E1;  PtMap e1m;  float c1;
  const float* Ref; PtMap rm;      // norm only: subtracted from E1 (null: the norm is that of out)
  float sp, hs;
  float* norm_partial;
  int mode;                        // MODE_PHI / MODE_DACT
  int act;                         // 0 tanh, 1 relu, 2 identity
  int M;                           // rows per state: B (dense) or B*Himg*Wimg (conv)
  int Nf;                          // features per row: q (dense) or C (conv)
  int K;                           // contraction length per output: q or 9*C
  int Himg, Wimg, TH;              // conv only: image size and rows of an output tile
  unsigned wmagic;                 // conv only: ceil(2^20 / Wimg), filled in by the launch wrapper
  int tiles;                       // workgroups per group (filled in by the launch wrapper)
  int dbf16;                       // 1: Dm (input) and the output of MODE_DACT are bf16 arrays
  int dbits;                       // 1: ... are bits (the factors of ReLU, 0 or 1), whatever dbf16 says
  int wstream;                     // 1: all layers' weights together exceed the last-level cache, load them
                                   // non-temporally; 0: they fit and later launches of the solve find them there
  int skip0, skipper;              // conv only, skipper > 0: groups skip0, skip0 + skipper, ... do nothing (their
                                   // layer is a fully connected one, served by a dense launch) and write 0 to
                                   // their norm partials
  long long E;                     // M * Nf
  long long wsize;                 // Nf * K elements per layer
};

enum { MODE_PHI = 0, MODE_DACT = 1 };
enum { ACT_TANH = 0, ACT_RELU = 1, ACT_IDENT = 2, ACT_MASK = 3 };   // ACT_MASK: identity, the sweep's Dm as bits

// Parameter gradient launch (one group per layer n):
//   G = Dm[n] .* Lam[n+1];  dW[n] = hs * G^T (*) U[n];  db[n] = hs * sum G
struct GradArgs {
  const float* U;   PtMap um;
  const float* Lam; PtMap lm;
  const float* Dm;  PtMap dm;        // act' cache in the weights' type (float, or bf16 for a bf16 problem), or bits
  int dbits;
  float* dW;                        // [layers][Nf][K] float
  float* db;                        // [layers][Nf] or null
  float hs;
  int M, Nf, K, Himg, Wimg, B;
  int tiles;                        // workgroups per layer (filled in by the launch wrapper)
  long long E, wsize;
  // conv, all taps in one workgroup (filled in by the launch wrapper from conv_grad_geom)
  float* partial;                   // [chunks][layers][wsize] partial sums when a layer is split into chunks
  int layers;
  int gWp, gR, gKL, gPU, gPG, gspi, gslabs, gchunks, gspc;
};
// Geometry of the conv gradient kernel that forms all nine taps in one workgroup: a slab is gR image rows
// of one image (row pitch gWp, a multiple of 8), the contraction over a slab runs over gKL pixel slots,
// the layer's slabs are split into `chunks` workgroups whose partial sums a second kernel adds in a fixed order.
struct ConvGradGeom {
  int Wp, R, KL, PU, PG, spi, slabs, chunks, spc;
  size_t smem;
  bool ok;                          // false: image row too wide for this kernel (one workgroup per tap is used)
};
ConvGradGeom conv_grad_geom(int B, int Himg, int Wimg, int C, int dtype, int layers);
// Float layers of at most 32 channels on the bf16 matrix cores: the slab's geometry (false: not these), and the launch, with
// `layers`, `gchunks` and what the geometry gives filled in.
bool       conv_grad_split_geom(int B, int Himg, int Wimg, int C, bool bits, ConvGradGeom* gm);
hipError_t launch_conv_grad_split(const GradArgs& a, size_t smem, hipStream_t s);
size_t     conv_grad_partial_bytes(int B, int Himg, int Wimg, int C, int dtype, int layers);

// ---- launch wrappers (defined in mgrit_kernels.hip, those of sweeps in mgrit_sweep.hip, mgrit_wave.hip and mgrit_wide.hip); all
// enqueue on `s` and return the HIP status
hipError_t launch_step(const StepArgs& a, int layer_kind, int dtype, int groups, hipStream_t s);
int        step_grid_blocks(const StepArgs& a, int layer_kind, int dtype, int groups);  // workgroups per group
int        conv_tile_rows(int Himg, int Wimg, int C, int dtype);            // TH, or 0 if unsupported
hipError_t launch_grad(const GradArgs& a, int layer_kind, int dtype, int groups, hipStream_t s);

// out[om(gi)] = in[im(gi)]                      (C-points handed to the finer level)
hipError_t launch_copy_points(float* out, PtMap om, const float* in, PtMap im, long long E, int groups,
                              hipStream_t s);
// out[i] = in for n <= 32 states
hipError_t launch_spread_state(float* const* out, int n, const float* in, long long E, hipStream_t s);
// out[om(gi)] = 0
hipError_t launch_zero_points(float* out, PtMap om, long long E, int groups, hipStream_t s);
// partial[slot0 + block] = sum over this block's chunk of (a - b)^2 ; returns blocks used
hipError_t launch_diff_sq(const float* a, const float* b, long long n, float* partial, int* blocks_used,
                          hipStream_t s);
int        diff_sq_blocks(long long n);
// out[j] = sqrt(sum_{i<n} partial[j n + i]) * scale for j < count, summed in a fixed order in double
hipError_t launch_norm_final(const float* partial, int n, double scale, double* out, int count, hipStream_t s);
// transposed parameter copies for the adjoint: dense Wt[n][i][o] = W[n][o][i];
// conv Kt[n][i][2-dy][2-dx][o] = K[n][o][dy][dx][i]
hipError_t launch_transpose_weights(const void* W, void* Wt, int layer_kind, int dtype, int layers, int Nf,
                                    hipStream_t s);

// A sweep: chain ci = 0 .. nchains - 1 starts from S[sm(ci)] and performs n layer steps in sequence (n = nsteps, nlast for
// the last chain) with the state on chip:
//   step k = 1..n:  u <- u + hs * act(A_layer (Dm_layer .* u) + bias_layer) + G[gb + ci*gs + k]
//   layer(k) = lb + ci*ls + (k-1)*lk
// One launch replaces n lockstep launches (Sec. III-C, Fig. 3).  What it keeps of the states:
//   X, xk != 0: the state after every step k, in X[xb + ci*xs + k*xk]; with store0 also the start state, k = 0,
//               and with store0 = 2 the point behind the last chain, S[sm(nchains)] to X[xb + nchains*xs]
//   Y:          the state after step kmid, in Y[yb + ci*ys]
//   Z:          the state after the last step, in Z[zb + ci*zs], if n > kmid; chain 0's state after step kmid in Z[zfirst]
//   tau:        single steps (n = 1): Z[zb + ci*zs] <- Z[zb + ci*zs] - state, and with Ref the sum over a workgroup of
//               (Z - Ref[rm(ci)])^2, Z before the update, in norm_partial[workgroup]
//   alt:        chains alt0, alt0 + altper, .. (convolution sweep, altper > 0) have a first layer of another kind: they go on from
//               Alt[am(ci)], the state behind their first step, or with tau do nothing but write 0 to their norm partials
// The launch may not write what it reads of S and Alt, by whichever chain: X, Y, Z are other arrays, or other points of the same
// one.  (A float sweep that meets a value that is not finite starts its chain from them once more, after its stores.)
struct SweepArgs {
  const float* S;  PtMap sm;
  float* X;  long long xb, xs, xk;  int store0;
  float* Y;  long long yb, ys;  int kmid;
  float* Z;  long long zb, zs, zfirst;
  int tau;  const float* Ref;  PtMap rm;  float* norm_partial;
  const float* G;  long long gb, gs;     // optional right-hand side (null: none)
  const void* W;  const float* bias;     // weights in the problem's type; bias may be null
  int wn;                                // dense sweep, 1: W holds W[k][n] (the adjoint on the caller's weights)
  const void* Dm;                        // optional act' factors in the weights' type, [layers][E]; bits with ACT_MASK
  long long lb, ls, lk;
  float hs;
  int act, nsteps, nlast, nchains, M, q;
  long long units;                       // layer steps of the schedule that the launch stands for (launch trace)
  long long E, wsize;
  int alt0, altper;  const float* Alt;  PtMap am;
  int Himg, Wimg, C;                     // convolution sweep only (then M = images per state)
  int ipw;                               // ... images per workgroup (filled in by the launch wrapper)
};
// Dense layers of width at most 256: workgroup (chain, slice of batch rows).
bool       sweep_supported(int q);
int        sweep_blocks(int M, int nchains);             // workgroups of a launch
double     sweep_bytes(const SweepArgs& a, int dtype);   // algorithmic bytes of a launch
hipError_t launch_sweep(const SweepArgs& a, int dtype, hipStream_t s);
// Dense layers of width 257 to 1024, bf16: workgroup (chain, 64 batch rows).
bool       wide_supported(int q, int dtype);
int        wide_blocks(int M, int nchains);
hipError_t launch_wide(const SweepArgs& a, int dtype, hipStream_t s);
// Dense layers of width at most 16: one wavefront per (chain, slice of 16 batch rows), and up to WAVE_OPS sweeps that follow one
// another in one launch.  The fields of a sweep are SweepArgs's; what all of them share is stated once.
struct WaveOp {
  const float* S;  float* X;  float* Y;  float* Z;  const float* Ref;  const float* G;  float* norm_partial;
  int sb, ss;  int xb, xs, xk, store0;  int yb, ys, kmid;  int zb, zs, zfirst, tau;  int rb, rs;  int gb, gs;
  int lb, ls, lk;  int nsteps, nlast, nchains;  float hs;
};
enum { WAVE_OPS = 20 };
struct WaveProgram {
  int nops = 0, nsl, per, M, q, act, wn;       // nsl slices, per workgroups for each (both filled in by the launch wrapper)
  const void* W;  const float* bias;  const void* Dm;
  long long E, wsize;
  WaveOp op[WAVE_OPS];
};
bool       wave_supported(int q);
int        wave_slices(int M);
int        wave_workgroups(int nchains);                 // workgroups of a slice that hold all chains of a sweep at once
// (norm_partial: one per workgroup; `per` workgroups for each slice, 1 if there is more than one sweep)
hipError_t launch_wave(const WaveProgram& p, int per, int dtype, long long units, double bytes, hipStream_t s);
// 3x3 convolution layers: workgroup (chain, images).
bool       conv_sweep_supported(int Himg, int Wimg, int C, int dtype);
bool       conv_sweep_ring(int Himg, int Wimg, int C, int dtype);        // its weights pass through LDS tap by tap
int        conv_sweep_blocks(const SweepArgs& a, int dtype);
hipError_t launch_conv_sweep(const SweepArgs& a, int dtype, hipStream_t s);

// launch tracing (diagnostic): kernel classes, and begin / collect
enum { TRACE_DENSE_F32_64 = 0, TRACE_DENSE_F32_128, TRACE_DENSE_BF16_64, TRACE_DENSE_BF16_128,
       TRACE_CONV_F32, TRACE_CONV_BF16, TRACE_GRAD, TRACE_SWEEP_F32, TRACE_SWEEP_BF16, TRACE_DENSE_F32_KS8,
       TRACE_DENSE_F32_KS, TRACE_DENSE_BF16_KS, TRACE_DENSE_BF16_KS8, TRACE_CONV_SWEEP_F32, TRACE_NCLASS };
void trace_begin();
int  trace_end(double* ms, long long* launches, long long* units, double* bytes, int ncls);
void trace_before(hipStream_t s);
void trace_after(hipStream_t s, int cls, long long units, double bytes);

}  // namespace mgrit
