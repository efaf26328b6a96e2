// Kernels that carry one state through many layer steps in one launch (sweeps): a workgroup owns some samples of one
// coarse interval and keeps their state on chip from step to step.
#include "mgrit_device.h"

namespace mgrit {

// ------------------------------------------------------------------------------------------
// Sweep over 3x3 convolution layers.  A convolution needs its neighbours' rows, so the unit is a whole image: a
// workgroup of eight wavefronts owns `ipw` images of one chain and marches through its layer steps.
//   - The float state stays in registers, in the arrangement of the accumulators of v_mfma_f32_16x16x32_bf16 with the
//     weights as the A operand: lane (c, kq) of a 16-pixel block holds channels 16 cb + 4 kq .. + 3 of pixel c.
//   - The matrix operand (act' .* state) of all pixels sits in LDS as bf16.  Taps that fall off the image read one
//     pixel of zeros, chosen by a 9-bit mask per pixel, so no frame is stored and several small images can share the
//     list of pixels.  The 16-byte pieces of a pixel are permuted by its index where the pixel pitch would put eight
//     neighbours on the same banks.
//   - The contraction runs over k = (tap, input channel) in steps of 32, four 8-channel pieces per step.
// NP = 1: bf16 problems.  NP = 3: float problems; state and weights are split into three bf16 numbers each, x = x1 + x2
// + x3 (8 + 8 + 8 significant bits, so the split is exact for values above about 2^-110; below, x3 and then x2 leave bf16's
// range), and the six products that reach 2^-24 are formed on the bf16 matrix cores with float accumulation -- 6/16 of the time
// of the float instructions.  Two of the products left out, x2 y3 and x3 y2, can reach 2^-25 of the full one each (|x2| <= 2^-8,
// |x3| <= 2^-17 for x near 1), together one rounding of a float addition in the worst case; typically they are 2^-29.
// (Infinite values: repeat_in_float.)
// The weights of a layer: all in LDS (the next layer's are on their way in registers during a step), or, for 64 channels
// on images too large for that (RING), tap by tap through three LDS slots.
// What bounds it: 16 channels float -- the LDS reads of the operand (15 KB per 16 pixels and step against 480 cycles of
// matrix instructions); 64 channels bf16 -- LDS reads and matrix instructions alike (a 64 x 64 tile per wavefront needs
// 8 KB of fragments for 16 instructions).  Global memory sees only what a caller keeps of the states.
// ------------------------------------------------------------------------------------------
typedef unsigned char u8;

// A value that rounds to an infinite bf16 number, 0x1.ffp127 = 3.396e38 or more, has no such parts: in a weight or an operand
// it makes NaN of every sum that it enters.  Float sweeps pass NaN on through the activation, so that it stays in the state,
// and a workgroup that ends with a state that is not finite repeats its chain with products of the float values themselves,
// as the lockstep kernels form them.  (To look at the values where they are split, or at the sums of a step, took 1 to 7 % of
// the sweeps of 16 channels and up to 40 % of those of width 256, in registers and branches more than in instructions; this
// way 64 layers of 16 channels take what they took, 795 us, and 256 of width 256 524 instead of 522.)
template <int NP, int ACT> __device__ __forceinline__ float sweep_act(float z) {
  if constexpr (NP == 3 && ACT == ACT_RELU) return __builtin_elementwise_maximum(z, 0.0f);
  else return act_fn_c<ACT>(z);
}
template <int A, int B> __device__ __forceinline__ bool any_not_finite(const floatx4 (&st)[A][B]) {   // in some lane
  float top = 0.0f;
#pragma unroll
  for (int i = 0; i < A; ++i)
#pragma unroll
    for (int j = 0; j < B; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) top = __builtin_elementwise_maximum(top, __builtin_fabsf(st[i][j][v]));
  return __builtin_amdgcn_ballot_w64(!(top < __builtin_inff())) != 0;
}

// A barrier for what is in LDS: the stores of the last states stay in flight (waiting for them is 1 % of the sweeps of width 256).
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Sum over a workgroup in a fixed order over the wavefronts; valid in thread 0.
template <int NWV> __device__ __forceinline__ float sum_workgroup(float sq, float* red, int tid) {
#pragma unroll
  for (int w = 32; w > 0; w >>= 1) sq += __shfl_xor(sq, w, 64);
  if ((tid & 63) == 0) red[tid >> 6] = sq;
  __syncthreads();
  float t = red[0];
#pragma unroll
  for (int w = 1; w < NWV; ++w) t += red[w];
  return t;
}

// The repeated chain.  A thread holds U groups of four neighbouring values -- channels of a pixel, features of a row, the lanes
// of a wavefront at most eight different ones, so that they share weights -- and the operand of a step is in LDS as it is.
// What bounds it are LDS reads (convolution: the weights too, put there at the start of a step) and weight loads.  With NaN in
// every state a solve of 64 layers of 16 channels takes 7.1 ms (lockstep: 1.4), one of 256 layers of width 256 2.4 ms (0.7); 29
// and 34 ms with the weights loaded value by value.  It takes nothing but the wavefront's number from the sweep and reads its arguments again,
// through a pointer that the compiler cannot follow (kept in scalar registers from the sweep on, they cost 2 % of it in spills).
template <int NWV, int U, int ACT, bool WN, bool CONV>
__device__ __forceinline__ void repeat_in_float(float* X, float* Wl, float* red, int wave) {
  constexpr int NTH = 64 * NWV;
  typedef const unsigned __attribute__((address_space(4))) * ArgWords;
  ArgWords words = (ArgWords)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(words));
  const int tid = 64 * wave + (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
  SweepArgs a;
  static_assert(sizeof(SweepArgs) % 4 == 0, "copied word by word");
#pragma unroll
  for (unsigned i = 0; i < sizeof(SweepArgs) / 4; ++i) reinterpret_cast<unsigned*>(&a)[i] = words[i];
  const int per = CONV ? a.ipw : 16 * U;                            // samples of a workgroup (dense: 16 rows per block)
  const int size = CONV ? a.Himg * a.Wimg * a.C : a.q;              // values of a sample
  const int nwg = (a.M + per - 1) / per, L = logical_block(), r0 = (L % nwg) * per;
  const long long ci = L / nwg, first = (long long)r0 * size;
  const int rows = min(per, a.M - r0), n = a.tau ? 1 : ci == a.nchains - 1 ? a.nlast : a.nsteps;
  const int C = CONV ? a.C : a.q, Wd = a.Wimg, HW = CONV ? a.Himg * Wd : 1, npx = rows * HW, ZP = per * HW;
  const int PX = CONV ? C : C + 4;                                  // floats of a pixel or row in LDS
  auto at = [&](const float* base, long long point) { return const_cast<float*>(base) + point * a.E + first; };
  auto pixel = [&](int i) { const int u = tid + NTH * i; return CONV ? u / (C / 4) : u % (16 * U); };
  auto chan = [&](int i) { const int u = tid + NTH * i; return 4 * (CONV ? u % (C / 4) : u / (16 * U)); };
  auto mine = [&](int i) { return pixel(i) < npx && chan(i) < C; };
  auto elem = [&](int i) { return pixel(i) * C + chan(i); };
  const bool alt = CONV && a.altper > 0 && ci >= a.alt0 && (ci - a.alt0) % a.altper == 0;
  __syncthreads();                                                  // the sweep's stores are done: the same places are written again
  floatx4 st[U];
#pragma unroll
  for (int i = 0; i < U; ++i) {
    st[i] = floatx4{0.f, 0.f, 0.f, 0.f};
    if (mine(i)) st[i] = *reinterpret_cast<const floatx4*>((alt ? at(a.Alt, a.am.base + ci * a.am.stride) : at(a.S, a.sm.base + ci * a.sm.stride)) + elem(i));
  }
  if (CONV && tid < C) X[ZP * C + tid] = 0.0f;
#pragma unroll 1
  for (int k = alt ? 2 : 1; k <= n; ++k) {
    const long long layer = a.lb + ci * a.ls + (long long)(k - 1) * a.lk;
    const float* W = reinterpret_cast<const float*>(a.W) + layer * a.wsize;
#pragma unroll
    for (int i = 0; i < U; ++i)
      if (mine(i)) {
        floatx4 v = st[i];
        if constexpr (ACT == ACT_IDENT || ACT == ACT_MASK) {
          typedef Fac<typename std::conditional<ACT == ACT_MASK, Bit, float>::type> F;
          const float4 d = F::f4(F::load(F::at(a.Dm, layer * a.E + first), elem(i)), elem(i));
          v *= floatx4{d.x, d.y, d.z, d.w};
        }
        *reinterpret_cast<floatx4*>(X + pixel(i) * PX + chan(i)) = v;
      }
    if (CONV)                                                       // a layer's weights, 9 C^2 floats, to LDS
      for (int e = 4 * tid; e < 9 * C * C; e += 4 * NTH) *reinterpret_cast<floatx4*>(Wl + e) = *reinterpret_cast<const floatx4*>(W + e);
    __syncthreads();
    // where the state is kept, as in the sweep
    float* o1 = nullptr;
    float* o2 = nullptr;
    if (a.tau) {}
    else if (a.X && a.xk) o1 = at(a.X, a.xb + ci * a.xs + (long long)k * a.xk);
    else if (k == a.kmid) { o1 = at(a.Y, a.yb + ci * a.ys); if (ci == 0) o2 = at(a.Z, a.zfirst); }
    else if (a.Z && k == n) o1 = at(a.Z, a.zb + ci * a.zs);
#pragma unroll
    for (int i = 0; i < U; ++i)
      if (mine(i)) {
        const int p = pixel(i), ch = chan(i);
        floatx4 z = floatx4{0.f, 0.f, 0.f, 0.f};
        if (a.bias) z = *reinterpret_cast<const floatx4*>(a.bias + layer * C + ch);
        const int y = p % HW / Wd, x = p % HW % Wd;
#pragma unroll 1
        for (int tap = 0; tap < (CONV ? 9 : 1); ++tap) {
          const int yy = y + tap / 3 - 1, xx = x + tap % 3 - 1;
          const bool inside = yy >= 0 && yy < a.Himg && xx >= 0 && xx < Wd;
          const float* xp = X + (CONV ? inside ? p + (yy - y) * Wd + xx - x : ZP : p) * PX;
          const float* w = CONV ? Wl + (ch * 9 + tap) * C : W + (WN ? ch : ch * C);
          const int next = CONV ? 9 * C : C;                        // from one output's weights, or one k's, to the next
#pragma unroll 2
          for (int t = 0; t < C; t += 4) {
            const floatx4 xv = *reinterpret_cast<const floatx4*>(xp + t);
            floatx4 wv[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) wv[r] = *reinterpret_cast<const floatx4*>(WN ? w + (t + r) * next : w + r * next + t);
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
              for (int v = 0; v < 4; ++v) z[v] = __builtin_fmaf(WN ? wv[r][v] : wv[v][r], xv[r], z[v]);
          }
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) st[i][v] += a.hs * act_fn_c<ACT>(z[v]);
        if (a.G) st[i] += *reinterpret_cast<const floatx4*>(at(a.G, a.gb + ci * a.gs + k) + elem(i));
        if (o1) *reinterpret_cast<floatx4*>(o1 + elem(i)) = st[i];
        if (o2) *reinterpret_cast<floatx4*>(o2 + elem(i)) = st[i];
      }
    __syncthreads();
  }
  if (!a.tau) return;
  float sq = 0.0f;
#pragma unroll
  for (int i = 0; i < U; ++i)
    if (mine(i)) {
      floatx4* o = reinterpret_cast<floatx4*>(at(a.Z, a.zb + ci * a.zs) + elem(i));
      const floatx4 p = *o;
      *o = p - st[i];
      if (a.Ref) {
        const floatx4 d = p - *reinterpret_cast<const floatx4*>(at(a.Ref, a.rm.base + ci * a.rm.stride) + elem(i));
        sq += (d[0] * d[0] + d[1] * d[1]) + (d[2] * d[2] + d[3] * d[3]);
      }
    }
  if (a.norm_partial) {
    const float t = sum_workgroup<NWV>(sq, red, tid);
    if (tid == 0) a.norm_partial[L] = t;
  }
}

// LDS layouts of this file suppose that a 16-byte read is served for lanes 0-3, 12-15, 20-27 together, then 4-11, 16-19, 28-31,
// and the same in the upper half (inferred: the layouts made for it measured faster), so for a fragment -- lane (c, kq) reads
// piece kq of row c -- these sixteen should lie in different 16-byte columns of 256 bytes.  Row pitches of 2 modulo 4 columns do
// that; elsewhere the pieces are permuted, by -kq & 3 rather than kq for the weights: 823 -> 797 us for 64 layers of 16 channels
// float, 9.71 -> 9.44 ms for 512 of 64 channels bf16, 531 -> 522 us for 256 of width 256.  Conflicts are left all the same: the
// counters still show 1.4 to 1.8 conflict cycles per LDS cycle in the sweeps of 16 channels, 0.75 in those of 64 and 0.9 in the
// adjoint dense sweep, whose 8-byte staging stores at a pitch of 72 bytes put rows r and r + 4 on the same banks (forward: 0.2 to 0.4).
template <int NP, int CP>
__device__ __forceinline__ int conv_sweep_swz(int p) {          // permutation of a pixel's 16-byte pieces
  if (CP == 64 && NP == 1) return p & 7;                        // pitch 128 bytes
  if (CP == 32 && NP == 1) return (p >> 1) & 3;                 // 64
  if (CP == 32 && NP == 3) return -(p >> 2) & 3;                // 192
  return 0;                                                     // 32, 96: eight neighbours already on distinct banks
}
template <int NP, int CP> constexpr int conv_sweep_ksteps() { return (9 * (CP / 8) + 3) / 4; }
template <int NP, int CP, bool RING> constexpr size_t conv_sweep_wbytes() {
  return (size_t)(RING ? 3 * 2 : conv_sweep_ksteps<NP, CP>()) * 4 * NP * CP * 16;
}
static_assert(conv_sweep_wbytes<3, 16, false>() >= 9 * 16 * 16 * 4 && conv_sweep_wbytes<3, 32, false>() >= 9 * 32 * 32 * 4, "repeat_in_float");

// TAU: the coarse right-hand side, single steps (its epilogue beside the others would cost the sweep registers).  ALT: some chains have
// a first layer of another kind (in every instance: 64 layers of 16 channels 805 -> 830 us)
template <int NP, int CP, int NWV, int NBW, bool RING, int ACT, bool TAU, bool ALT>
__global__ __launch_bounds__(64 * NWV) void conv_sweep_kernel(SweepArgs a) {
  constexpr bool HD = ACT == ACT_IDENT || ACT == ACT_MASK;      // the adjoint: act' factors, no bias
  constexpr bool MASK = ACT == ACT_MASK;                        // ... as bits
  constexpr int NTH = 64 * NWV;
  constexpr int CB = CP / 16, PPT = CP / 8, NPC = 9 * PPT, S = conv_sweep_ksteps<NP, CP>();
  constexpr int PLB = CP * 2, PXB = NP * PLB;                   // LDS bytes of one part of a pixel, of a pixel
  constexpr int GB = 4, NG = NBW / GB;                          // pixel blocks multiplied together, groups of them
  constexpr int WSB = 4 * NP * CP * 16;                         // LDS bytes of the weights of a k step
  constexpr int WS = RING ? 2 : S;                              // k steps loaded together: a tap or the whole layer
  constexpr int WU = (WS * 4 * CP + NTH - 1) / NTH;             // units (8 input channels of one output channel) per thread
  constexpr int WR = NP == 3 ? 2 : 1;                           // 16-byte loads per unit
  // a layer's weight fragments fit in registers (beside factors stored as values not without spills, except for bf16 and 16
  // channels: 1445 us for 64 float layers of 16 channels, 1385 with fragments read from LDS; a step of 32 channels bf16 on
  // 32 x 32 pixels 11.1 -> 9.2 us.  Beside bits they do: 64 float layers of 16 channels, adjoint and gradient, 1370 -> 1304 us)
  constexpr bool HOLD = (CP == 16 && !(HD && !MASK && NP == 3)) || (CP == 32 && NP == 1 && (!HD || MASK));
  // act' factors requested at the start of a step (values of wider layers: only when it is done, for they would be spilled: a step
  // of 48 channels on 28 x 28 pixels 17.8 -> 14.1 us, of 64 on 16 x 32 14.4 -> 12.8).  Bits instead of bf16 values, requested
  // early: 512 layers of 64 channels on 32 x 32 pixels, 32 images, adjoint and gradient, 17.1 -> 14.8 ms; 64 layers on 2 images of 5 x 5
  // 299 -> 296 us.  Above 32 channels registers are short (spilled: 48 channels 14, 64 channels 16 above 512 pixels, else 1), so
  // what write_operand exchanges is addressed by the opaque pixel: 11 to 23 registers spilled otherwise, and those two 310 us, 15.0 ms
  constexpr bool DEARLY = CP <= 32 || MASK;
  static_assert(NBW % GB == 0 && (!RING || (CP == 64 && NP == 1)), "instances");
  typedef typename std::conditional<NP == 3, float, __bf16>::type WT;
  typedef Fac<WT> F;
  typedef typename F::Raw DR;
  extern __shared__ __attribute__((aligned(16))) u8 smem[];
  __shared__ float red[NWV];
  __shared__ int repeat;                                        // float: a state of the chain is not finite

  const int tid = threadIdx.x, lane = tid & 63, c = lane & 15, kq = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int H = a.Himg, Wd = a.Wimg, C = RING ? CP : a.C, HW = H * Wd;
  const int nwg = (a.M + a.ipw - 1) / a.ipw;                    // workgroups per chain
  const int L = logical_block();
  const long long ci = L / nwg;
  const int img0 = (L % nwg) * a.ipw;
  const int npx = min(a.ipw, a.M - img0) * HW;                  // pixels of this workgroup
  const int nblk = (npx + 15) >> 4;
  const int nbw = nblk > wave ? (nblk - wave + NWV - 1) / NWV : 0;     // blocks wave, wave + 8, .. of this wavefront
  const int ngr = ((nblk + NWV - 1) / NWV + GB - 1) / GB;       // groups of the wavefront with the most blocks
  const int n = TAU ? 1 : ci == a.nchains - 1 ? a.nlast : a.nsteps;
  const bool alt = ALT && ci >= a.alt0 && (ci - a.alt0) % a.altper == 0;
  const int k1 = alt ? 2 : 1;                                   // the first step
  if (TAU && alt) {                                             // the whole workgroup
    if (a.norm_partial && tid == 0) a.norm_partial[L] = 0.0f;
    return;
  }
  const int ZP = a.ipw * HW;                                    // the pixel of zeros
  u8* P = smem;
  u8* Wl = smem + ((size_t)(ZP + 1) * PXB + 255) / 256 * 256;
  float* bl = reinterpret_cast<float*>(Wl + conv_sweep_wbytes<NP, CP, RING>());     // [2][CP] bias
  const long long img_off = (long long)img0 * HW * C;
  auto layer_of = [&](int k) __attribute__((always_inline)) { return a.lb + ci * a.ls + (long long)(k - 1) * a.lk; };

  // this lane's pixel in block b and its place in a state
  // (cpx is made opaque to the compiler once per step: everything that follows from a lane's pixel -- the operand addresses
  // of all taps and blocks -- is the same in every step, and kept across the step loop it would take several hundred
  // registers)
  int cpx = c;
  auto px = [&](int b) __attribute__((always_inline)) { return (wave + NWV * b) * 16 + cpx; };
  // (pixels past the last one read that one's values, channels past C those of the pixel's first block: never stored)
  const int chl = CB == 1 && 4 * kq >= C ? 0 : 4 * kq;
  const bool last_ok = 16 * (CB - 1) + 4 * kq < C;              // C % 8 == 0: a lane's four channels are in or out together
  const int chlast = last_ok ? 16 * (CB - 1) : 0;
  auto off = [&](int b, int cb) __attribute__((always_inline)) { return (unsigned)(min(px(b), npx - 1) * C + chl + (cb < CB - 1 ? 16 * cb : chlast)); };
  // which of the nine taps of a pixel lie in its image (bit 9 and above: never)
  unsigned mask[NBW];
#pragma unroll
  for (int b = 0; b < NBW; ++b) {
    const int p = px(b), r = p % HW, y = r / Wd, x = r % Wd;
    const unsigned xm = (x > 0 ? 1u : 0u) | 2u | (x + 1 < Wd ? 4u : 0u);
    unsigned m = xm << 3;
    if (y > 0) m |= xm;
    if (y + 1 < H) m |= xm << 6;
    mask[b] = p < npx ? m : 0u;
  }

  floatx4 st[NBW][CB];
  auto store_state = [&](float* o) __attribute__((always_inline)) {
#pragma unroll
    for (int b = 0; b < NBW; ++b)
      if (px(b) < npx) {
#pragma unroll
        for (int cb = 0; cb < CB - 1; ++cb) *reinterpret_cast<floatx4*>(o + off(b, cb)) = st[b][cb];
        if (last_ok) *reinterpret_cast<floatx4*>(o + off(b, CB - 1)) = st[b][CB - 1];
      }
  };
  auto place = [&](float* base, long long point) __attribute__((always_inline)) { return base + point * a.E + img_off; };
  // the start state (store0 = 2: the last chain first passes on the point behind it)
  for (int t = a.store0 == 2 && ci == a.nchains - 1 ? 1 : 0; t >= 0; --t) {
    const float* sp = a.S + (a.sm.base + (ci + t) * a.sm.stride) * a.E + img_off;
#pragma unroll
    for (int b = 0; b < NBW; ++b)
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) st[b][cb] = *reinterpret_cast<const floatx4*>(sp + off(b, cb));
    if (a.store0) store_state(place(a.X, a.xb + (ci + t) * a.xs));
  }
  if (n < k1) return;                                           // the whole workgroup
  if (alt) {
    const float* sp = a.Alt + (a.am.base + ci * a.am.stride) * a.E + img_off;
#pragma unroll
    for (int b = 0; b < NBW; ++b)
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) st[b][cb] = *reinterpret_cast<const floatx4*>(sp + off(b, cb));
  }

  // ---- weights: unit u = (k step, output channel, piece of the step)
  const WT* Wall = reinterpret_cast<const WT*>(a.W);
  u32x4 wr[WU * WR];
  // (a unit outside the layer -- a padded channel, the k step's pieces past tap 8 -- reads the layer's first values and is
  // cleared on its way into LDS)
  auto unit_ok = [&](int u, int tap0) __attribute__((always_inline)) {
    const int pc = 4 * (u / (4 * CP)) + (u & 3);
    return u < WS * 4 * CP && tap0 + pc / PPT < 9 && (u >> 2) % CP < C && (pc % PPT) * 8 < C;
  };
  auto load_w = [&](u32x4 (&r)[WU * WR], const WT* Wp, int tap0) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < WU; ++i) {
      if constexpr (RING) {                                     // every unit inside: a uniform base and a fixed offset
        const int u = tid + NTH * i;
        const unsigned e = (unsigned)(((u >> 2) & 63) * 9 * CP + (u >> 8) * 32 + (u & 3) * 8);
        r[i] = *reinterpret_cast<const u32x4*>(reinterpret_cast<const char*>(Wp + tap0 * CP) + 2u * e);
        continue;
      }
      const int u = tid + NTH * i, pc = 4 * (u / (4 * CP)) + (u & 3), o = (u >> 2) % CP;
      const unsigned e = (unsigned)((o * 9 + tap0 + pc / PPT) * C + (pc % PPT) * 8);
      const WT* q = Wp + (unit_ok(u, tap0) ? e : 0u);
#pragma unroll
      for (int j = 0; j < WR; ++j) r[i * WR + j] = *reinterpret_cast<const u32x4*>(q + (NP == 3 ? 4 * j : 0));
    }
  };
  auto store_w = [&](u32x4 (&r)[WU * WR], u8* dst, int tap0) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < WU; ++i) {
      const int u = tid + NTH * i, s = u / (4 * CP), kg = u & 3, o = (u >> 2) % CP;
      if (u < WS * 4 * CP) {
        // (the slot of an output channel is permuted by the piece, so that the four pieces a quad of lanes holds go to
        // different banks)
        u8* q = dst + s * WSB + ((kg * NP) * CP + (o ^ (4 * (-kg & 3)))) * 16;
        const unsigned keep = RING || unit_ok(u, tap0) ? ~0u : 0u;
#pragma unroll
        for (int j = 0; j < WR; ++j) r[i * WR + j] &= keep;
        if constexpr (NP == 1) {
          *reinterpret_cast<u32x4*>(q) = r[i];
        } else {
          bf16x8 h, m, l;
          split3<8>([&](int e) { return __uint_as_float(r[i * WR + (e >> 2)][e & 3]); }, h, m, l);
          *reinterpret_cast<bf16x8*>(q) = h;
          *reinterpret_cast<bf16x8*>(q + CP * 16) = m;
          *reinterpret_cast<bf16x8*>(q + 2 * CP * 16) = l;
        }
      }
    }
  };
  const WT* Wc = Wall + layer_of(k1) * a.wsize;
  load_w(wr, Wc, 0);
  float bnext = 0.0f;
  auto load_bias = [&](int k) __attribute__((always_inline)) { if (a.bias && tid < CP && tid < C) bnext = a.bias[layer_of(k) * C + tid]; };
  load_bias(k1);

  // ---- operand of a step: act' .* state, to LDS (a pixel's padded channels are zero)
  // (bits: all of a pixel's channels in one load of up to eight bytes, wherever they start; it may reach into the next pixel,
  // and behind the last layer's factors into the cache's unused part.  Up to 32 channels a lane loads those of its own pixels;
  // above, the four lanes of a pixel load those of a quarter of the blocks each and exchange them when the operand is written:
  // four registers from the start of a step on, not sixteen)
  constexpr bool DSHARE = CB > 2;
  constexpr int NDB = DSHARE ? NBW / 4 : NBW;
  typedef typename std::conditional<CB == 1, unsigned short, typename std::conditional<CB == 2, unsigned, u32x2>::type>::type BW;
  struct __attribute__((packed)) PixelBits { BW w; };
  BW db[MASK ? NDB : 1];
  DR dr[HD && !MASK ? NBW : 1][HD && !MASK ? CB : 1];
  auto load_d = [&](int k) __attribute__((always_inline)) {
    if constexpr (MASK) {
      const u8* dp = Fac<Bit>::at(a.Dm, layer_of(k) * a.E + img_off);
#pragma unroll
      for (int i = 0; i < NDB; ++i)
        db[i] = reinterpret_cast<const PixelBits*>(dp + (unsigned)(min(px(DSHARE ? NDB * kq + i : i), npx - 1) * C) / 8u)->w;
    } else if constexpr (HD) {
      const typename F::Ptr dp = F::at(a.Dm, layer_of(k) * a.E + img_off);
#pragma unroll
      for (int b = 0; b < NBW; ++b)
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) dr[b][cb] = F::load(dp, off(b, cb));
    }
  };
  auto piece = [&](int p, int pc) __attribute__((always_inline)) { return (unsigned)(p * PXB + ((pc ^ conv_sweep_swz<NP, CP>(p)) << 4)); };
  auto write_operand = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int b = 0; b < NBW; ++b) {
      const int p = px(b);
      unsigned bits[2];                                             // channels 32 i + 4 kq and on
      if constexpr (MASK && DSHARE) {
#pragma unroll
        for (int i = 0; i < 2; ++i) bits[i] = (unsigned)__builtin_amdgcn_ds_bpermute(4 * (cpx + 16 * (b / NDB)), (int)db[b % NDB][i]) >> (4 * kq);
      } else if constexpr (MASK) bits[0] = (unsigned)db[b] >> (4 * kq);
      if (p < npx) {
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) {
          float4 v = make_float4(st[b][cb][0], st[b][cb][1], st[b][cb][2], st[b][cb][3]);
          if constexpr (MASK) {
            const unsigned w = bits[cb >> 1];
            const int at = 16 * (cb & 1);
            v.x *= bit_factor(w, at); v.y *= bit_factor(w, at + 1); v.z *= bit_factor(w, at + 2); v.w *= bit_factor(w, at + 3);
          } else if constexpr (HD) { const float4 d = F::f4(dr[b][cb], 0); v.x *= d.x; v.y *= d.y; v.z *= d.z; v.w *= d.w; }
          if (cb == CB - 1 && !last_ok) v = make_float4(0.f, 0.f, 0.f, 0.f);
          // (the permutation of a pixel's pieces repeats every 16 pixels at most: it depends on the lane alone)
          u8* q = P + p * PXB + (((2 * cb + (kq >> 1)) ^ conv_sweep_swz<NP, CP>(cpx)) << 4) + (kq & 1) * 8;
          if constexpr (NP == 1) {
            cvt_store4(reinterpret_cast<__bf16*>(q), v);
          } else {
            bf16x4 h, m, l;
            const floatx4 f = floatx4{v.x, v.y, v.z, v.w};
            split3<4>([&](int e) { return f[e]; }, h, m, l);
            *reinterpret_cast<bf16x4*>(q) = h;
            *reinterpret_cast<bf16x4*>(q + PLB) = m;
            *reinterpret_cast<bf16x4*>(q + 2 * PLB) = l;
          }
        }
      }
    }
  };
  load_d(k1);
  if (tid < PXB / 4) reinterpret_cast<float*>(P + (size_t)ZP * PXB)[tid] = 0.0f;
  if (NP == 3 && tid == 0) repeat = 0;
  write_operand();
  store_w(wr, Wl, 0);
  if constexpr (RING) load_w(wr, Wc, 1);
  if (tid < CP) bl[(k1 & 1) * CP + tid] = bnext;
  __syncthreads();

  const unsigned alane = (unsigned)(((kq * NP) * CP + (c ^ (4 * (-kq & 3)))) * 16);      // this lane's row of a weight fragment
  for (int k = k1; k <= n; ++k) {
    asm volatile("" : "+v"(cpx));
#pragma unroll
    for (int b = 0; b < NBW; ++b) asm volatile("" : "+v"(mask[b]));
    const WT* Wn = Wall + layer_of(k < n ? k + 1 : k) * a.wsize;                  // (past the last step: read, not used)
    if constexpr (!RING) load_w(wr, Wn, 0);
    if (k < n) {
      load_bias(k + 1);
      if constexpr (DEARLY) load_d(k + 1);
    }
    bf16x8 hold[HOLD ? S : 1][HOLD ? CB : 1][NP];
    if constexpr (HOLD) {
#pragma unroll
      for (int s = 0; s < S; ++s)
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
#pragma unroll
          for (int q = 0; q < NP; ++q)
            hold[s][cb][q] = *reinterpret_cast<const bf16x8*>(Wl + alane + s * WSB + q * CP * 16 + cb * 256);
    }
    const float* bp = bl + (k & 1) * CP;
    const float* gp = a.G ? a.G + (a.gb + ci * a.gs + k) * a.E + img_off : nullptr;

    // one k step for NV pixel blocks: base address of each block's pixel for the lane's tap and piece
    // (NP = 3: the five small products have accumulators of their own, so that the large one's sum is rounded once per k
    // step; they are added at the end)
    auto mma = [&](auto nvc, floatx4 (&acc)[GB][CB], floatx4 (&low)[NP == 3 ? GB : 1][NP == 3 ? CB : 1], const unsigned (&pa)[GB], const u8* ws, int s) __attribute__((always_inline)) {
      constexpr int NV = decltype(nvc)::value;
      // (the fragments of one k step at a time: the other wavefront of the SIMD covers their latency, and a second set
      // in flight would not fit beside state and accumulators)
      if constexpr (NBW * CB + NV * CB > 16) __builtin_amdgcn_sched_barrier(0);
      bf16x8 bfr[NV][NP];
#pragma unroll
      for (int i = 0; i < NV; ++i)
#pragma unroll
        for (int q = 0; q < NP; ++q) bfr[i][q] = *reinterpret_cast<const bf16x8*>(P + pa[i] + q * PLB);
      bf16x8 afr[CB][NP];
#pragma unroll
      for (int cb = 0; cb < CB; ++cb)
#pragma unroll
        for (int q = 0; q < NP; ++q) {
          if constexpr (HOLD) afr[cb][q] = hold[s][cb][q];
          else afr[cb][q] = *reinterpret_cast<const bf16x8*>(ws + alane + q * CP * 16 + cb * 256);
        }
      if constexpr (NP == 1) {
#pragma unroll
        for (int i = 0; i < NV; ++i)
#pragma unroll
          for (int cb = 0; cb < CB; ++cb) acc[i][cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(afr[cb][0], bfr[i][0], acc[i][cb], 0, 0, 0);
      } else {
        constexpr int PA[6] = {2, 0, 1, 1, 0, 0}, PB[6] = {0, 2, 1, 0, 1, 0};     // smallest products first
#pragma unroll
        for (int t = 0; t < 5; ++t)
#pragma unroll
          for (int i = 0; i < NV; ++i)
#pragma unroll
            for (int cb = 0; cb < CB; ++cb)
              low[i][cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(afr[cb][PA[t]], bfr[i][PB[t]], low[i][cb], 0, 0, 0);
#pragma unroll
        for (int i = 0; i < NV; ++i)
#pragma unroll
          for (int cb = 0; cb < CB; ++cb) acc[i][cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(afr[cb][0], bfr[i][0], acc[i][cb], 0, 0, 0);
      }
    };
    auto update = [&](auto grpc, auto nvc, floatx4 (&acc)[GB][CB]) __attribute__((always_inline)) {
      constexpr int G0 = decltype(grpc)::value * GB, NV = decltype(nvc)::value;
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) {
#pragma unroll
        for (int i = 0; i < NV; ++i)
#pragma unroll
          for (int v = 0; v < 4; ++v) st[G0 + i][cb][v] += a.hs * sweep_act<NP, ACT>(acc[i][cb][v]);
      }
      if (gp) {                                                     // coarse levels only
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) {
          floatx4 gv[NV];
#pragma unroll
          for (int i = 0; i < NV; ++i) gv[i] = *reinterpret_cast<const floatx4*>(gp + off(G0 + i, cb));
#pragma unroll
          for (int i = 0; i < NV; ++i) st[G0 + i][cb] += gv[i];
        }
      }
    };
    auto group = [&](auto grpc, auto nvc) __attribute__((always_inline)) {
      constexpr int G0 = decltype(grpc)::value * GB, NV = decltype(nvc)::value;
      floatx4 acc[GB][CB];
#pragma unroll
      for (int i = 0; i < NV; ++i)
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) {
          if (!HD) acc[i][cb] = *reinterpret_cast<const floatx4*>(bp + 16 * cb + 4 * kq);        // the bias
          else acc[i][cb] = floatx4{0.f, 0.f, 0.f, 0.f};
        }
      floatx4 low[NP == 3 ? GB : 1][NP == 3 ? CB : 1];
      if constexpr (NP == 3) {
#pragma unroll
        for (int i = 0; i < NV; ++i)
#pragma unroll
          for (int cb = 0; cb < CB; ++cb) low[i][cb] = floatx4{0.f, 0.f, 0.f, 0.f};
      }
      if constexpr (RING) {
        // Tap by tap: a tap's weights are requested two taps and written to LDS one tap before their use, and the barrier at
        // the end of a tap makes the next one's visible.
        const bool last = decltype(grpc)::value + 1 >= ngr;
        bf16x8 af[CB], bf[GB];
        unsigned pa[GB];
        auto tap_addr = [&](int tap) __attribute__((always_inline)) {
          const int ty = (tap * 11) >> 5, dp = (ty - 1) * Wd + (tap - 3 * ty) - 1;        // tap / 3
#pragma unroll
          for (int i = 0; i < GB; ++i) {
            const int pp = (mask[G0 + i] >> tap) & 1u ? px(G0 + i) + dp : ZP;
            pa[i] = piece(pp, kq);
          }
        };
        auto kstep = [&](const u8* ws, unsigned flip) __attribute__((always_inline)) {                 // flip 64: pieces 4 .. 7 of the pixel
#pragma unroll
          for (int cb = 0; cb < CB; ++cb) af[cb] = *reinterpret_cast<const bf16x8*>(ws + alane + cb * 256);
#pragma unroll
          for (int i = 0; i < GB; ++i) bf[i] = *reinterpret_cast<const bf16x8*>(P + (pa[i] ^ flip));
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int i = 0; i < GB; ++i)
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) acc[i][cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[cb], bf[i], acc[i][cb], 0, 0, 0);
        };
        if constexpr (NV > 0) tap_addr(0);
        // (a rolled loop: unrolled, the kernel is larger than the 64 KB instruction cache of two CUs and takes five times as
        // long, waiting for its instructions)
        u8* slot = Wl;                                              // this tap's weights; the next tap's go to the next slot
#pragma unroll 1
        for (int tap = 0; tap < 9; ++tap) {
          u8* next = slot == Wl + 4 * WSB ? Wl : slot + 2 * WSB;
          store_w(wr, next, 0);
          load_w(wr, (tap >= 7 && last) ? Wn : Wc, tap >= 7 ? tap - 7 : tap + 2);
          if constexpr (NV > 0) {
            kstep(slot, 0u);
            __builtin_amdgcn_sched_barrier(0);
            kstep(slot + WSB, 64u);
            if (tap < 8) tap_addr(tap + 1);
          }
          __syncthreads();                                          // next tap complete
          slot = next;
        }
      } else if constexpr (NV > 0) {
        auto kstep = [&](int s) __attribute__((always_inline)) {
          const int pc = 4 * s + kq, tap = pc / PPT, ty = (tap * 11) >> 5;        // tap / 3 for 0 <= tap < 16
          const int dp = (ty - 1) * Wd + (tap - 3 * ty) - 1;
          unsigned pa[GB];
#pragma unroll
          for (int i = 0; i < NV; ++i) {
            const int pp = (mask[G0 + i] >> tap) & 1u ? px(G0 + i) + dp : ZP;
            pa[i] = piece(pp, pc % PPT);
          }
          mma(nvc, acc, low, pa, Wl + s * WSB, s);
        };
        if constexpr (HOLD) {
#pragma unroll
          for (int s = 0; s < S; ++s) kstep(s);
        } else {                                                    // (rolled: the instruction cache again)
#pragma unroll 2
          for (int s = 0; s < S; ++s) kstep(s);
        }
      }
      if constexpr (NP == 3) {
#pragma unroll
        for (int i = 0; i < NV; ++i)
#pragma unroll
          for (int cb = 0; cb < CB; ++cb) acc[i][cb] += low[i][cb];
      }
      if constexpr (NV > 0) update(grpc, nvc, acc);
    };
    auto groups = [&](auto grpc) __attribute__((always_inline)) {
      const int nv = nbw - decltype(grpc)::value * GB;              // the same for all lanes of the wavefront
      if constexpr (RING) {                                         // every wavefront takes part in the ring's barriers
        if (nv > 0) group(grpc, std::integral_constant<int, 4>{});  // (blocks past the last one read zeros)
        else        group(grpc, std::integral_constant<int, 0>{});
      } else {
        if (nv >= 4) group(grpc, std::integral_constant<int, 4>{});
        else if (nv == 3) group(grpc, std::integral_constant<int, CP == 16 ? 3 : 4>{});
        else if (nv == 2) group(grpc, std::integral_constant<int, 2>{});
        else if (nv == 1) group(grpc, std::integral_constant<int, CP == 16 ? 1 : 2>{});
      }
    };
    groups(std::integral_constant<int, 0>{});
    if constexpr (NG > 1) { if (ngr > 1) groups(std::integral_constant<int, 1>{}); }
    if constexpr (NG > 2) { if (ngr > 2) groups(std::integral_constant<int, 2>{}); }
    if constexpr (NG > 3) { if (ngr > 3) groups(std::integral_constant<int, 3>{}); }
    static_assert(NG <= 4, "groups");

    if constexpr (TAU) {                                            // coarse right-hand side: Z <- Z - state, and its norm
      if constexpr (NP == 3) {
        if (any_not_finite(st)) repeat = 1;
        lds_barrier();
        if (repeat) break;
      }
      float* o = place(a.Z, a.zb + ci * a.zs);
      const float* ref = a.Ref ? a.Ref + (a.rm.base + ci * a.rm.stride) * a.E + img_off : nullptr;
      float sq = 0.0f;
#pragma unroll
      for (int b = 0; b < NBW; ++b) {
        floatx4 pv[CB], rv[CB];
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) pv[cb] = *reinterpret_cast<const floatx4*>(o + off(b, cb));
        if (ref) {
#pragma unroll
          for (int cb = 0; cb < CB; ++cb) rv[cb] = *reinterpret_cast<const floatx4*>(ref + off(b, cb));
        }
        if (px(b) < npx) {
#pragma unroll
          for (int cb = 0; cb < CB; ++cb)
            if (cb < CB - 1 || last_ok) {
              *reinterpret_cast<floatx4*>(o + off(b, cb)) = pv[cb] - st[b][cb];
              if (ref) {
                const floatx4 d = pv[cb] - rv[cb];
                sq += (d[0] * d[0] + d[1] * d[1]) + (d[2] * d[2] + d[3] * d[3]);
              }
            }
        }
      }
      if (a.norm_partial) {
        const float t = sum_workgroup<NWV>(sq, red, tid);
        if (tid == 0) a.norm_partial[L] = t;
      }
      break;                                                        // (n = 1)
    }
    float* o1 = nullptr;                                            // where this step's state is kept: at most two places
    float* o2 = nullptr;
    if (a.X && a.xk) o1 = place(a.X, a.xb + ci * a.xs + (long long)k * a.xk);
    else if (k == a.kmid) { o1 = place(a.Y, a.yb + ci * a.ys); if (ci == 0) o2 = place(a.Z, a.zfirst); }
    else if (a.Z && k == n) o1 = place(a.Z, a.zb + ci * a.zs);
    for (; o1; o1 = o2, o2 = nullptr) store_state(o1);
    if (k == n) break;
    if constexpr (!DEARLY) load_d(k + 1);
    __syncthreads();                                                // every wavefront is done with the operand and the weights
    write_operand();
    if constexpr (!RING) store_w(wr, Wl, 0);
    if (tid < CP) bl[((k + 1) & 1) * CP + tid] = bnext;
    Wc = Wn;
    __syncthreads();
  }
  if constexpr (NP == 3) {
    if constexpr (!TAU) {
      if (any_not_finite(st)) repeat = 1;
      lds_barrier();
    }
    if (repeat) repeat_in_float<NWV, NBW * CB, ACT, false, true>(reinterpret_cast<float*>(P), reinterpret_cast<float*>(Wl), red, wave);
  }
}

// Instances: 1 / 2 / 3 / 4 blocks of 16 channels; up to 1024 pixels per workgroup with eight pixel blocks per
// wavefront, 512 with four.
namespace {
struct ConvSweepShape { int cp, np, nwv, nbw; bool ring; size_t smem; };
size_t conv_sweep_smem(int np, int cp, bool ring, int pixels) {
  const size_t op = ((size_t)(pixels + 1) * np * cp * 2 + 255) / 256 * 256;
  const size_t ks = ring ? 6 : (9 * (cp / 8) + 3) / 4;
  return op + ks * 4 * np * cp * 16 + 2 * cp * sizeof(float);
}
bool conv_sweep_shape(int pixels, int C, int dtype, ConvSweepShape* sh) {
  const size_t cap = (size_t)160 * 1024;
  sh->np = dtype == 0 ? 3 : 1;
  sh->cp = (C + 15) / 16 * 16;
  sh->ring = false;
  if (sh->np == 3 && sh->cp > 32) return false;
  sh->nwv = 8;
  sh->nbw = (sh->np == 3 && sh->cp == 32) || sh->cp == 64 ? 4 : 8;
  if (C == 64 && sh->np == 1 && pixels > 512) { sh->ring = true; sh->nwv = 8; sh->nbw = 8; }
  sh->smem = conv_sweep_smem(sh->np, sh->cp, sh->ring, pixels);
  return pixels <= sh->nwv * sh->nbw * 16 && sh->smem <= cap;
}
template <int NP, int CP, int NWV, int NBW, bool RING, int ACT, bool TAU, bool ALT = false>
hipError_t launch_conv_sweep_t(const SweepArgs& a, unsigned blocks, size_t smem, hipStream_t s) {
  if constexpr (!ALT && (ACT == ACT_TANH || ACT == ACT_RELU))
    if (a.altper > 0) return launch_conv_sweep_t<NP, CP, NWV, NBW, RING, ACT, TAU, true>(a, blocks, smem, s);
  if (!ALT && a.altper > 0) return hipErrorInvalidValue;        // forward solves only
  static LdsOptIn opt;
  const hipError_t e = opt.raise(reinterpret_cast<const void*>(conv_sweep_kernel<NP, CP, NWV, NBW, RING, ACT, TAU, ALT>), smem);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((conv_sweep_kernel<NP, CP, NWV, NBW, RING, ACT, TAU, ALT>), dim3(blocks), dim3(64 * NWV), smem, s, a);
  return hipGetLastError();
}
}  // namespace

bool conv_sweep_supported(int Himg, int Wimg, int C, int dtype) {
  ConvSweepShape sh;
  if (Himg < 1 || Wimg < 1 || C < 8 || C > 64 || C % 8 != 0 || (long long)Himg * Wimg > 1024) return false;
  return conv_sweep_shape(Himg * Wimg, C, dtype, &sh);
}
bool conv_sweep_ring(int Himg, int Wimg, int C, int dtype) {
  ConvSweepShape sh;
  return conv_sweep_supported(Himg, Wimg, C, dtype) && conv_sweep_shape(Himg * Wimg, C, dtype, &sh) && sh.ring;
}
// Images per workgroup: a step has fixed costs (two barriers, the weights' way into LDS) and eight wavefronts want at least
// a block of 16 pixels each, so small images share a workgroup as long as every CU still gets one.
static int conv_sweep_images(int Himg, int Wimg, int C, int dtype, int B, int nchains) {
  ConvSweepShape sh;
  int ipw = 1;
  while (2 * ipw <= B && 2 * ipw * Himg * Wimg <= 512 && (long long)nchains * ((B + 2 * ipw - 1) / (2 * ipw)) >= 256 &&
         conv_sweep_shape(2 * ipw * Himg * Wimg, C, dtype, &sh))
    ipw *= 2;
  return ipw;
}

int conv_sweep_blocks(const SweepArgs& a, int dtype) {
  const int ipw = conv_sweep_images(a.Himg, a.Wimg, a.C, dtype, a.M, a.nchains);
  return (a.M + ipw - 1) / ipw * a.nchains;
}
hipError_t launch_conv_sweep(const SweepArgs& a_in, int dtype, hipStream_t s) {
  SweepArgs a = a_in;
  if (a.nchains <= 0) return hipSuccess;
  if (a.tau && (a.nsteps != 1 || a.nlast != 1 || !a.Z)) return hipErrorInvalidValue;
  if ((a.act == ACT_IDENT || a.act == ACT_MASK) != (a.Dm != nullptr)) return hipErrorInvalidValue;     // the adjoint's steps, and only they
  if (a.M < 1 || !conv_sweep_supported(a.Himg, a.Wimg, a.C, dtype)) return hipErrorInvalidValue;
  a.ipw = conv_sweep_images(a.Himg, a.Wimg, a.C, dtype, a.M, a.nchains);
  ConvSweepShape sh;
  if (!conv_sweep_shape(a.ipw * a.Himg * a.Wimg, a.C, dtype, &sh)) return hipErrorInvalidValue;
  const unsigned blocks = (unsigned)((a.M + a.ipw - 1) / a.ipw) * (unsigned)a.nchains;
  trace_before(s);
  hipError_t e = hipErrorInvalidValue;
#define MGRIT_CS(NP_, CP_, NWV_, NBW_, RING_, TAU_)                                                                    \
  if (sh.np == NP_ && sh.cp == CP_ && sh.nwv == NWV_ && sh.nbw == NBW_ && sh.ring == RING_ && (a.tau != 0) == TAU_)    \
    e = a.act == ACT_TANH   ? launch_conv_sweep_t<NP_, CP_, NWV_, NBW_, RING_, ACT_TANH, TAU_>(a, blocks, sh.smem, s)  \
        : a.act == ACT_RELU ? launch_conv_sweep_t<NP_, CP_, NWV_, NBW_, RING_, ACT_RELU, TAU_>(a, blocks, sh.smem, s)  \
        : a.act == ACT_MASK ? launch_conv_sweep_t<NP_, CP_, NWV_, NBW_, RING_, ACT_MASK, TAU_>(a, blocks, sh.smem, s)  \
                            : launch_conv_sweep_t<NP_, CP_, NWV_, NBW_, RING_, ACT_IDENT, TAU_>(a, blocks, sh.smem, s);
  MGRIT_CS(1, 16, 8, 8, false, false) MGRIT_CS(1, 32, 8, 8, false, false) MGRIT_CS(1, 48, 8, 8, false, false)
  MGRIT_CS(1, 64, 8, 4, false, false) MGRIT_CS(1, 64, 8, 8, true, false)
  MGRIT_CS(3, 16, 8, 8, false, false) MGRIT_CS(3, 32, 8, 4, false, false)
  MGRIT_CS(1, 16, 8, 8, false, true) MGRIT_CS(1, 32, 8, 8, false, true) MGRIT_CS(1, 48, 8, 8, false, true)
  MGRIT_CS(1, 64, 8, 4, false, true) MGRIT_CS(1, 64, 8, 8, true, true)
  MGRIT_CS(3, 16, 8, 8, false, true) MGRIT_CS(3, 32, 8, 4, false, true)
#undef MGRIT_CS
  // algorithmic bytes: per layer step the weights and bias, the act' factor, the right-hand side and what is kept of the
  // state; the start state once per chain
  const double es = dtype == 0 ? 4.0 : 2.0, E4 = 4.0 * (double)a.E;
  const double steps = (double)(a.nchains - 1) * a.nsteps + a.nlast;
  const double per = es * (double)a.wsize + (a.bias ? 4.0 * a.C : 0.0) + (a.Dm ? a.act == ACT_MASK ? 0.125 : es : 0.0) * (double)a.E + (a.G ? E4 : 0.0) +
                     (a.X && a.xk ? E4 : 0.0) + (a.tau ? E4 : 0.0) + (a.Ref ? E4 : 0.0);
  trace_after(s, TRACE_CONV_SWEEP_F32, a.units,
              steps * per + (double)a.nchains * E4 * (1.0 + (a.Y ? 1.0 : 0.0) + (a.Z ? 1.0 : 0.0) + (a.store0 ? 1.0 : 0.0)));
  return e;
}

// ------------------------------------------------------------------------------------------
// Sweep over dense layers of width at most 256.  A dense layer acts on every batch row by itself, so a workgroup owns 16 RB
// rows of one chain and marches through its layer steps without talking to any other.
//   - Matrix instructions as in the convolution sweep, weights as the A operand: lane (c, kq) holds features
//     16 fb + 4 kq .. + 3 of batch row c of a block; wavefront w owns the feature blocks w FBW .. + FBW - 1.  The float
//     state stays in registers, the operand (act' .* state) of all rows sits in LDS.
//   - The weights of a layer stream from L2, k step by k step (32 values of k), two k steps ahead in registers and running
//     on into the next layer; every wavefront handles its own features' weights, so the contraction has no barriers.
//     They pass through an LDS area of the wavefront's own: fragments read straight from memory touch a 64-byte segment
//     per lane (38 GB/s per CU against 130 for whole segments).  k-major bf16 weights take LDS's transposing read.
//   - Everything a wavefront does in a k step depends on what it did before, so the chain's latency counts: width 256 runs
//     with sixteen wavefronts of one feature block (four per SIMD) instead of eight of two.
// NP = 3 (float) splits state and weights into three bf16 numbers as the convolution sweep does.
// What bounds it, width 256 float: splitting the weights (every wavefront its own, vector instructions) and the latency of
// a k step; a step takes 9.1 us with 32 rows (float matrix instructions and eight wavefronts before: 12.5) and 5.5 us with
// 16 (a lockstep launch before: 5.1 .. 7.5, and the state through memory).  Global memory sees the weights once per XCD and
// what a caller keeps of the states.
// Requesting a layer's lines ahead of their loads did not pay: 126 us instead of 105 for 16 serial steps.
// ------------------------------------------------------------------------------------------
template <int NP, int FBW, bool WN> constexpr int dense_sweep_stage() {     // bytes of a wavefront's staging area
  return NP == 3 ? (WN ? 32 * (64 * FBW + 8) : 16 * FBW * 160) : (WN ? 32 * (32 * FBW + 32) : 16 * FBW * 96);
}
constexpr int dense_sweep_pitch(int np, int kp) { return np * kp * 2 + 32; }   // bytes of an operand row in LDS
constexpr int DENSE_SWEEP_ZEROS = 512;                                      // bytes of zeros behind the staging areas

template <int NP, int NWV, int FBW, int RB, int ACT, bool WN>
__global__ __launch_bounds__(64 * NWV) void dense_sweep_kernel(SweepArgs a) {
  static_assert(4 * (32 * FBW + 32) + 8 <= DENSE_SWEEP_ZEROS && 64 * NWV >= DENSE_SWEEP_ZEROS / 4, "one lane's reads; its writers");
  constexpr bool HD = ACT == ACT_IDENT || ACT == ACT_MASK;          // the adjoint: act' factors, no bias
  constexpr int NTH = 64 * NWV, R = 16 * RB;
  constexpr int STG = dense_sweep_stage<NP, FBW, WN>();
  constexpr int NL = NP == 3 ? 2 * FBW : FBW;                       // 16-byte loads of a k step per lane
  typedef typename std::conditional<NP == 3, float, __bf16>::type WT;
  typedef Fac<typename std::conditional<ACT == ACT_MASK, Bit, WT>::type> F;
  typedef typename F::Raw DR;
  typedef u32x4 LW;
  extern __shared__ __attribute__((aligned(16))) u8 smem[];
  __shared__ float red[NWV];
  __shared__ int repeat;                                            // float: a state of the chain is not finite

  const int tid = threadIdx.x, lane = tid & 63, c = lane & 15, kq = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int q = a.q, KP = (q + 63) & ~63, KS = KP / 32, OP = dense_sweep_pitch(NP, KP);   // KS is even
  const int nsl = (a.M + R - 1) / R;
  const int L = logical_block();
  const long long ci = L / nsl;
  const int r0 = (L % nsl) * R, rows = min(R, a.M - r0);
  const int n = ci == a.nchains - 1 ? a.nlast : a.nsteps;
  u8* A = smem;                                                     // operand [R][OP]
  u8* Ws = smem + R * OP + wave * STG;
  u8* Zr = smem + R * OP + NWV * STG;
  const long long sl_off = (long long)r0 * q;
  const int f0 = wave * FBW * 16;                                   // this wavefront's first feature
  auto layer_of = [&](int k) __attribute__((always_inline)) { return a.lb + ci * a.ls + (long long)(k - 1) * a.lk; };
  auto place = [&](const float* base, long long point) __attribute__((always_inline)) { return const_cast<float*>(base) + point * a.E + sl_off; };
  // (rows past the batch read the last one's values, features past the width those of feature 0: never stored)
  auto feat = [&](int j) __attribute__((always_inline)) { return f0 + 16 * j + 4 * kq; };
  auto off = [&](int rb, int j) __attribute__((always_inline)) { return (unsigned)(min(16 * rb + c, rows - 1) * q + (feat(j) < q ? feat(j) : 0)); };

  floatx4 st[RB][FBW];
  auto store_state = [&](float* o) __attribute__((always_inline)) {
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
      for (int j = 0; j < FBW; ++j)
        if (16 * rb + c < rows && feat(j) < q) *reinterpret_cast<floatx4*>(o + off(rb, j)) = st[rb][j];
  };
  // the start state (store0 = 2: the last chain first passes on the point behind it)
  for (int t = a.store0 == 2 && ci == a.nchains - 1 ? 1 : 0; t >= 0; --t) {
    const float* sp = place(a.S, a.sm.base + (ci + t) * a.sm.stride);
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
      for (int j = 0; j < FBW; ++j) st[rb][j] = *reinterpret_cast<const floatx4*>(sp + off(rb, j));
    if (a.store0) store_state(place(a.X, a.xb + (ci + t) * a.xs));
  }
  if (n <= 0) return;                                               // the whole workgroup

  // ---- weights of a k step, straight into registers: whole 128-byte (bf16: 64-byte) pieces of the wavefront's rows, or
  // rows of k.  Everything past the width is clamped to a valid address: the lanes that hold it read zeros instead, or its
  // output is not stored.
  const WT* Wall = reinterpret_cast<const WT*>(a.W);
  // (a k step inside the width: a uniform base and offsets that stay the same; the last ones are clamped value by value)
  unsigned wo[NL];
  int wk[NL];
#pragma unroll
  for (int i = 0; i < NL; ++i) {
    int f, k;
    if constexpr (WN) { constexpr int LPR = (NP == 3 ? 4 : 2) * FBW, VEC = NP == 3 ? 4 : 8; const int p = lane + 64 * i; k = p / LPR; f = f0 + (p % LPR) * VEC; }
    else { constexpr int LPR = NP == 3 ? 8 : 4, VEC = NP == 3 ? 4 : 8; const int p = lane + 64 * i; f = f0 + p / LPR; k = (p % LPR) * VEC; }
    f = f < q ? f : 0;
    wk[i] = k;
    wo[i] = (unsigned)(WN ? k * q + f : f * q + k) * (unsigned)sizeof(WT);
  }
  auto load_w = [&](LW (&w)[NL], const WT* Wp, int s) __attribute__((always_inline)) {
    const int k0 = 32 * s;
    if (k0 + 32 <= q) {
      const char* base = reinterpret_cast<const char*>(Wp + (size_t)k0 * (WN ? q : 1));
#pragma unroll
      for (int i = 0; i < NL; ++i) w[i] = *reinterpret_cast<const LW*>(base + wo[i]);
    } else {
      const char* base = reinterpret_cast<const char*>(Wp);
      const unsigned step = (unsigned)(k0 * (WN ? q : 1) * (int)sizeof(WT)), row = (unsigned)((WN ? q : 1) * (int)sizeof(WT));
#pragma unroll
      for (int i = 0; i < NL; ++i) w[i] = *reinterpret_cast<const LW*>(base + (k0 + wk[i] < q ? wo[i] + step : wo[i] - wk[i] * row));
    }
  };
  auto stage_w = [&](const LW (&w)[NL]) __attribute__((always_inline)) {
    {
#pragma unroll
      for (int i = 0; i < NL; ++i) {
        const int p = lane + 64 * i;
        if constexpr (WN && NP == 3) {
          u32x2* d = reinterpret_cast<u32x2*>(Ws + (p / (4 * FBW)) * (64 * FBW + 8) + (p % (4 * FBW)) * 16);
          d[0] = u32x2{w[i][0], w[i][1]}; d[1] = u32x2{w[i][2], w[i][3]};
        } else if constexpr (WN) *reinterpret_cast<u32x4*>(Ws + (p / (2 * FBW)) * (32 * FBW + 32) + (p % (2 * FBW)) * 16) = w[i];
        else if constexpr (NP == 3) *reinterpret_cast<u32x4*>(Ws + (p >> 3) * 160 + ((p & 7) >> 1) * 16 + (p & 1) * 64) = w[i];
        else *reinterpret_cast<u32x4*>(Ws + (p >> 2) * 96 + (p & 3) * 16) = w[i];
      }
    }
  };
  // A wavefront's staging area is its own and its LDS operations execute in order: the fences only keep the compiler from
  // moving accesses across.
  auto wave_sync = [&]() __attribute__((always_inline)) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };
  DR dr[RB][FBW];
  auto load_d = [&](int k) __attribute__((always_inline)) {
    if constexpr (HD) {
      const typename F::Ptr dp = F::at(a.Dm, layer_of(k) * a.E + sl_off);
#pragma unroll
      for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int j = 0; j < FBW; ++j) dr[rb][j] = F::load(dp, off(rb, j));
    }
  };
  auto write_operand = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
      for (int j = 0; j < FBW; ++j)
        if (feat(j) < KP) {
          float4 v = make_float4(st[rb][j][0], st[rb][j][1], st[rb][j][2], st[rb][j][3]);
          if constexpr (HD) { const float4 d = F::f4(dr[rb][j], 4 * kq); v.x *= d.x; v.y *= d.y; v.z *= d.z; v.w *= d.w; }
          if (feat(j) >= q) v = make_float4(0.f, 0.f, 0.f, 0.f);
          u8* p = A + (16 * rb + c) * OP + feat(j) * 2;
          if constexpr (NP == 1) {
            cvt_store4(reinterpret_cast<__bf16*>(p), v);
          } else {
            bf16x4 h, m, l;
            const floatx4 f = floatx4{v.x, v.y, v.z, v.w};
            split3<4>([&](int e) { return f[e]; }, h, m, l);
            *reinterpret_cast<bf16x4*>(p) = h;
            *reinterpret_cast<bf16x4*>(p + KP * 2) = m;
            *reinterpret_cast<bf16x4*>(p + KP * 4) = l;
          }
        }
  };
  const WT* Wc = Wall + layer_of(1) * a.wsize;
  LW w0[NL], w1[NL];
  load_w(w0, Wc, 0);
  load_w(w1, Wc, 1);
  load_d(1);
  if (tid < DENSE_SWEEP_ZEROS / 4) reinterpret_cast<float*>(Zr)[tid] = 0.0f;
  if (NP == 3 && tid == 0) repeat = 0;
  write_operand();
  __syncthreads();

  for (int k = 1; k <= n; ++k) {
    const WT* Wn = Wall + layer_of(k < n ? k + 1 : k) * a.wsize;    // (past the last step: read, not used)
    floatx4 bv[FBW], gv[RB][FBW];
    if constexpr (!HD) {
      const float* bp = a.bias + layer_of(k) * q;
#pragma unroll
      for (int j = 0; j < FBW; ++j) bv[j] = *reinterpret_cast<const floatx4*>(bp + (feat(j) < q ? feat(j) : 0));
    }
    if (a.G) {
      const float* gp = place(a.G, a.gb + ci * a.gs + k);
#pragma unroll
      for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int j = 0; j < FBW; ++j) gv[rb][j] = *reinterpret_cast<const floatx4*>(gp + off(rb, j));
    }
    if (k < n) load_d(k + 1);

    floatx4 acc[RB][FBW], low[RB][FBW];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
      for (int j = 0; j < FBW; ++j) { acc[rb][j] = floatx4{0.f, 0.f, 0.f, 0.f}; low[rb][j] = floatx4{0.f, 0.f, 0.f, 0.f}; }
    auto kstep = [&](LW (&w)[NL], int s) __attribute__((always_inline)) {
      bf16x8 af[FBW][NP];
      {
        stage_w(w);
        wave_sync();
        // bf16: a lane whose eight values of k lie past the width takes zeros: its operand is zero as well, but a clamped
        // weight may be infinite (float: such a chain is repeated)
        const bool in = NP == 3 || 32 * s + 8 * kq < q;
#pragma unroll
        for (int j = 0; j < FBW; ++j) {
          if constexpr (NP == 3 && WN) {
            // rows k of 64 FBW + 8 bytes: the four lane groups, eight rows apart, fall on different banks
            const u8* p = Ws + 8 * kq * (64 * FBW + 8) + (16 * j + c) * 4;
            float x[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) x[e] = *reinterpret_cast<const float*>(p + e * (64 * FBW + 8));
            split3<8>([&](int e) { return x[e]; }, af[j][0], af[j][1 % NP], af[j][2 % NP]);
          } else if constexpr (NP == 3) {
            const u8* p = Ws + (16 * j + c) * 160 + kq * 16;          // pieces 2 kq, 2 kq + 1 of the row
            const floatx4 x0 = *reinterpret_cast<const floatx4*>(p), x1 = *reinterpret_cast<const floatx4*>(p + 64);
            split3<8>([&](int e) { return e < 4 ? x0[e & 3] : x1[e & 3]; }, af[j][0], af[j][1 % NP], af[j][2 % NP]);
          } else if constexpr (WN) {
            // two transposing reads: rows k = 8 kq + 0 .. 3 and + 4 .. 7 of column c of the block
            constexpr int P = 32 * FBW + 32;
            typedef __attribute__((address_space(3))) short4v* lds_s4;
            const u8* p = in ? Ws + (8 * kq + (c >> 2)) * P + 32 * j + 8 * (c & 3) : Zr;
            const short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4)(p));
            const short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4)(p + 4 * P));
            af[j][0] = __builtin_shufflevector(__builtin_bit_cast(bf16x4, lo), __builtin_bit_cast(bf16x4, hi), 0, 1, 2, 3, 4, 5, 6, 7);
          } else {
            af[j][0] = *reinterpret_cast<const bf16x8*>(in ? Ws + (16 * j + c) * 96 + kq * 16 : Zr);
          }
        }
        wave_sync();
      }
      // the k step after next goes into the registers this one has left
      if (s + 2 < KS) load_w(w, Wc, s + 2); else load_w(w, Wn, s + 2 - KS);
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) {
        const u8* p = A + (16 * rb + c) * OP + 64 * s + 16 * kq;
        bf16x8 bf[NP];
#pragma unroll
        for (int t = 0; t < NP; ++t) bf[t] = *reinterpret_cast<const bf16x8*>(p + t * KP * 2);
        if constexpr (NP == 1) {
#pragma unroll
          for (int j = 0; j < FBW; ++j) acc[rb][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[j][0], bf[0], acc[rb][j], 0, 0, 0);
        } else {
          constexpr int PA[5] = {2, 0, 1, 1, 0}, PB[5] = {0, 2, 1, 0, 1};         // smallest products first
#pragma unroll
          for (int t = 0; t < 5; ++t)
#pragma unroll
            for (int j = 0; j < FBW; ++j)
              low[rb][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[j][PA[t] % NP], bf[PB[t] % NP], low[rb][j], 0, 0, 0);
#pragma unroll
          for (int j = 0; j < FBW; ++j) acc[rb][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[j][0], bf[0], acc[rb][j], 0, 0, 0);
        }
      }
    };
    for (int s = 0; s < KS; s += 2) { kstep(w0, s); kstep(w1, s + 1); }

#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
      for (int j = 0; j < FBW; ++j) {
        floatx4 z = acc[rb][j];
        if constexpr (NP == 3) z += low[rb][j];
        if constexpr (!HD) z += bv[j];
#pragma unroll
        for (int v = 0; v < 4; ++v) st[rb][j][v] += a.hs * sweep_act<NP, ACT>(z[v]);
        if (a.G) st[rb][j] += gv[rb][j];
      }

    if (a.tau) {                                                    // coarse right-hand side: Z <- Z - state, and its norm
      if constexpr (NP == 3) {
        if (any_not_finite(st)) repeat = 1;
        lds_barrier();
        if (repeat) break;
      }
      float* o = place(a.Z, a.zb + ci * a.zs);
      const float* ref = a.Ref ? place(a.Ref, a.rm.base + ci * a.rm.stride) : nullptr;
      float sq = 0.0f;
#pragma unroll
      for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int j = 0; j < FBW; ++j)
          if (16 * rb + c < rows && feat(j) < q) {
            const floatx4 p = *reinterpret_cast<const floatx4*>(o + off(rb, j));
            *reinterpret_cast<floatx4*>(o + off(rb, j)) = p - st[rb][j];
            if (ref) {
              const floatx4 d = p - *reinterpret_cast<const floatx4*>(ref + off(rb, j));
              sq += (d[0] * d[0] + d[1] * d[1]) + (d[2] * d[2] + d[3] * d[3]);
            }
          }
      if (a.norm_partial) {
        const float t = sum_workgroup<NWV>(sq, red, tid);
        if (tid == 0) a.norm_partial[L] = t;
      }
      break;                                                        // (n = 1)
    }
    float* o1 = nullptr;                                            // where this step's state is kept: at most two places
    float* o2 = nullptr;
    if (a.X && a.xk) o1 = place(a.X, a.xb + ci * a.xs + (long long)k * a.xk);
    else if (k == a.kmid) { o1 = place(a.Y, a.yb + ci * a.ys); if (ci == 0) o2 = place(a.Z, a.zfirst); }
    else if (a.Z && k == n) o1 = place(a.Z, a.zb + ci * a.zs);
    for (; o1; o1 = o2, o2 = nullptr) store_state(o1);
    if (k == n) break;
    __syncthreads();                                                // every wavefront is done with the operand
    write_operand();
    Wc = Wn;
    __syncthreads();
  }
  if constexpr (NP == 3) {
    if (!a.tau) {
      if (any_not_finite(st)) repeat = 1;
      lds_barrier();
    }
    if (repeat) repeat_in_float<NWV, RB * FBW, ACT, WN, false>(reinterpret_cast<float*>(A), nullptr, red, wave);
  }
}

namespace {
template <int NP, int NWV, int FBW, int RB, int ACT, bool WN>
hipError_t launch_dense_sweep_t(const SweepArgs& a, unsigned blocks, hipStream_t s) {
  const size_t smem = (size_t)16 * RB * dense_sweep_pitch(NP, (a.q + 63) & ~63) + (size_t)NWV * dense_sweep_stage<NP, FBW, WN>() + DENSE_SWEEP_ZEROS;
  static LdsOptIn opt;
  const hipError_t e = opt.raise(reinterpret_cast<const void*>(dense_sweep_kernel<NP, NWV, FBW, RB, ACT, WN>), smem);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((dense_sweep_kernel<NP, NWV, FBW, RB, ACT, WN>), dim3(blocks), dim3(64 * NWV), smem, s, a);
  return hipGetLastError();
}
// Rows of a workgroup: 32 where that still gives three quarters of the CUs a workgroup, else 16.  A CU holds one workgroup
// of sixteen wavefronts, and a step of 16 rows takes 5.5 us against 9.1 us for 32: twice the workgroups pay as long as they
// all run at once (17 chains of 128 rows, three steps: 22 us in 136 workgroups), not in two rounds.
int sweep_rows(int M, int nchains) { return (long long)((M + 31) / 32) * nchains >= 192 ? 32 : 16; }
}  // namespace

bool sweep_supported(int q) { return q >= 8 && q <= 256 && q % 8 == 0; }
int sweep_blocks(int M, int nchains) { const int r = sweep_rows(M, nchains); return (M + r - 1) / r * nchains; }

// Algorithmic bytes: per layer step the weights and bias, the act' factor, the right-hand side and what is kept of the state; the
// start state once per chain.
double sweep_bytes(const SweepArgs& a, int dtype) {
  const double es = dtype == 0 ? 4.0 : 2.0, E4 = 4.0 * (double)a.E;
  const double steps = (double)(a.nchains - 1) * a.nsteps + a.nlast;
  const double per = es * (double)a.wsize + (a.bias ? 4.0 * a.q : 0.0) + (a.Dm ? a.act == ACT_MASK ? 0.125 : es : 0.0) * (double)a.E + (a.G ? E4 : 0.0) +
                     (a.X && a.xk ? E4 : 0.0) + (a.tau ? E4 : 0.0) + (a.Ref ? E4 : 0.0);
  return steps * per + (double)a.nchains * E4 * (1.0 + (a.Y ? 1.0 : 0.0) + (a.Z ? 1.0 : 0.0) + (a.store0 ? 1.0 : 0.0));
}
hipError_t launch_sweep(const SweepArgs& a, int dtype, hipStream_t s) {
  if (a.nchains <= 0) return hipSuccess;
  if (a.M < 1 || !sweep_supported(a.q)) return hipErrorInvalidValue;
  if ((a.act == ACT_IDENT || a.act == ACT_MASK) != (a.Dm != nullptr) || (a.Dm == nullptr && (a.wn || !a.bias))) return hipErrorInvalidValue;  // the adjoint's steps, and only they
  if (a.tau && (a.nsteps != 1 || a.nlast != 1 || !a.Z)) return hipErrorInvalidValue;
  const int rows = sweep_rows(a.M, a.nchains);
  const unsigned blocks = (unsigned)sweep_blocks(a.M, a.nchains);
  trace_before(s);
  hipError_t e = hipErrorInvalidValue;
#define MGRIT_DS_RB(NP_, NWV_, FBW_, RB_)                                                                     \
  e = a.act == ACT_TANH   ? launch_dense_sweep_t<NP_, NWV_, FBW_, RB_, ACT_TANH, false>(a, blocks, s)         \
      : a.act == ACT_RELU ? launch_dense_sweep_t<NP_, NWV_, FBW_, RB_, ACT_RELU, false>(a, blocks, s)         \
      : a.act == ACT_MASK ? (a.wn ? launch_dense_sweep_t<NP_, NWV_, FBW_, RB_, ACT_MASK, true>(a, blocks, s)  \
                                  : launch_dense_sweep_t<NP_, NWV_, FBW_, RB_, ACT_MASK, false>(a, blocks, s)) \
      : a.wn              ? launch_dense_sweep_t<NP_, NWV_, FBW_, RB_, ACT_IDENT, true>(a, blocks, s)         \
                          : launch_dense_sweep_t<NP_, NWV_, FBW_, RB_, ACT_IDENT, false>(a, blocks, s)
#define MGRIT_DS(NP_, NWV_, FBW_) { if (rows == 32) MGRIT_DS_RB(NP_, NWV_, FBW_, 2); else MGRIT_DS_RB(NP_, NWV_, FBW_, 1); }
  // wavefronts x feature blocks of 16 that cover the width
  if (dtype == 0) { if (a.q <= 64) MGRIT_DS(3, 4, 1) else if (a.q <= 128) MGRIT_DS(3, 8, 1) else MGRIT_DS(3, 16, 1) }
  else            { if (a.q <= 64) MGRIT_DS(1, 4, 1) else if (a.q <= 128) MGRIT_DS(1, 8, 1) else MGRIT_DS(1, 16, 1) }
#undef MGRIT_DS
#undef MGRIT_DS_RB
  trace_after(s, dtype == 0 ? TRACE_SWEEP_F32 : TRACE_SWEEP_BF16, a.units, sweep_bytes(a, dtype));
  return e;
}

}  // namespace mgrit
