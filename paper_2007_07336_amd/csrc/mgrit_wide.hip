// Sweep over dense layers of width 257 to 1024, bf16 operands: a workgroup owns 64 batch rows of one chain and carries them through
// its layer steps with the state on chip.
#include "mgrit_device.h"

namespace mgrit {

// ------------------------------------------------------------------------------------------
// Eight wavefronts; 64 rows of 1024 floats are 256 KB, half of a CU's registers, and their bf16 operand 128 KB, most of its LDS.
//   - Features are dealt in blocks of 32: wavefront w forms block w, w + 8, .. of them, one after the other (NP passes), each for
//     all 64 rows.  The accumulators of a pass are 32 registers, so that the state (32 per pass) and the weights in flight fit.
//   - The operand (act' .* state) of all rows stays in LDS for a step; the new state goes to registers pass by pass and to LDS
//     behind the barrier that ends the step.
//   - A layer's weights stream from L2 in pieces of 32 features by 32 values of k, two pairs of them ahead in registers and on into the next
//     pass and layer.  A wavefront's pieces are its own: through 4 KB of LDS, no barrier inside a step.
// LDS is full (128 KB + 32 KB at width 1024), so nothing is padded: 16-byte pieces of the operand's rows and of the staging rows are
// permuted instead, such that the lanes that are served together (0-3, 12-15, 20-27, then the others) find different banks.
// What bounds it at width 1024: the contraction alone takes 31 us a step (LDS: 8 MB a step; the matrix instructions 14), with its
// weights, 2 MB a step and workgroup from L2, 55 (adjoint 67): the first of a chain's slices to ask for a line waits for memory, the
// others with it, and only two pairs of pieces can be requested ahead.  A lockstep launch takes 73 (97) us, reads the weights once per
// 128 rows and the state in and out.  1024 layers of width 1024, 256 samples: forward solve 7.21 -> 5.95 ms, adjoint with gradient
// 13.0 -> 11.1.  Tried: four pieces in flight 6.13; a load per group of pairs that touches the lines of the next group, each
// slice another quarter, 6.4.
// The instances for width 769 to 1024 use all 256 registers and spill (forward 86, adjoint 61 to 64; up to 768 the adjoint about factors
// as values 6 to 8): before and behind the loop over k, which is free of spills, in the writing of the operand, the end of a step and the
// coarse right-hand side.  About 30 of the spilled ones are read in a step, 60 KB of a workgroup's 2 MB.
// ------------------------------------------------------------------------------------------
constexpr int WIDE_NWV = 8, WIDE_RB = 4, WIDE_ROWS = 16 * WIDE_RB, WIDE_STG = 2 * 2048;     // staging bytes of a wavefront, two pieces
constexpr int wide_kp(int q) { return (q + 127) / 128 * 128; }

template <int NP, int ACT, bool WN>
__global__ __launch_bounds__(64 * WIDE_NWV) void wide_sweep_kernel(SweepArgs a) {
  constexpr bool HD = ACT == ACT_IDENT || ACT == ACT_MASK;          // the adjoint: act' factors, no bias
  constexpr int RB = WIDE_RB, FB = 2;
  typedef Fac<typename std::conditional<ACT == ACT_MASK, Bit, __bf16>::type> F;
  typedef typename F::Raw DR;
  typedef u32x4 LW;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63, c = lane & 15, kq = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int q = a.q, KP = wide_kp(q), KS = KP / 32, OP = 2 * KP;    // KS is a multiple of four
  const int nsl = (a.M + WIDE_ROWS - 1) / WIDE_ROWS;
  const int L = logical_block();
  const long long ci = L / nsl;
  const int r0 = (L % nsl) * WIDE_ROWS, rows = min(WIDE_ROWS, a.M - r0);
  const int n = ci == a.nchains - 1 ? a.nlast : a.nsteps;
  unsigned char* Ws = smem + WIDE_ROWS * OP + wave * WIDE_STG;
  const long long sl_off = (long long)r0 * q;
  const int np = min(NP, (q - 32 * wave + 255) / 256);              // passes that have features, >= 1
  auto layer_of = [&](int k) __attribute__((always_inline)) { return a.lb + ci * a.ls + (long long)(k - 1) * a.lk; };
  auto place = [&](const float* base, long long point) __attribute__((always_inline)) { return const_cast<float*>(base) + point * a.E + sl_off; };
  // (rows past the batch read the last one's values, features past the width those of feature 0: never stored)
  auto feat = [&](int p, int j) __attribute__((always_inline)) { return 256 * p + 32 * wave + 16 * j + 4 * kq; };
  // (the row is made opaque to the compiler wherever a state's places are used: kept across the contraction they would take a
  // register each)
  int cx = c;
  auto opaque = [&]() __attribute__((always_inline)) { asm volatile("" : "+v"(cx)); };
  auto off = [&](int p, int rb, int j) __attribute__((always_inline)) {
    return (unsigned)(min(16 * rb + cx, rows - 1) * q + (feat(p, j) < q ? feat(p, j) : 0));
  };

  floatx4 st[NP][RB][FB];
  auto store_state = [&](float* o) __attribute__((always_inline)) {
#pragma unroll
    for (int p = 0; p < NP; ++p)
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) {
        opaque();
#pragma unroll
        for (int j = 0; j < FB; ++j)
          if (16 * rb + cx < rows && feat(p, j) < q) *reinterpret_cast<floatx4*>(o + off(p, rb, j)) = st[p][rb][j];
      }
  };
  // the start state (store0 = 2: the last chain first passes on the point behind it)
  for (int t = a.store0 == 2 && ci == a.nchains - 1 ? 1 : 0; t >= 0; --t) {
    const float* sp = place(a.S, a.sm.base + (ci + t) * a.sm.stride);
#pragma unroll
    for (int p = 0; p < NP; ++p)
#pragma unroll
      for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int j = 0; j < FB; ++j) st[p][rb][j] = *reinterpret_cast<const floatx4*>(sp + off(p, rb, j));
    if (a.store0) store_state(place(a.X, a.xb + (ci + t) * a.xs));
  }
  if (n <= 0) return;                                               // the whole workgroup

  // ---- weights: a pair of pieces (pass p, k steps 2 d and 2 d + 1), four 16-byte loads per lane.  W[n][k]: 8 rows of 128 bytes
  // each, whole lines, the k steps in the lower and the upper lanes, sorted later (part).  W[k][n] (WN): 16 rows of 64 bytes each;
  // the line's other half is the next wavefront's.  What lies past the width reads some other weight of the layer, the last one at most.
  unsigned wo[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int row = WN ? 16 * i + (lane >> 2) : 8 * i + ((lane & 31) >> 2), pc = (lane & 3) * 8;
    wo[i] = 2u * (unsigned)(WN ? row * q + 32 * wave + pc : (32 * wave + row) * q + pc + 32 * (lane >> 5));
  }
  const unsigned wlast = 2u * (unsigned)(q * q - 8);
  // (All slices of a chain take k in the same order, so that a sample's result does not depend on its place in the batch.  With each
  // slice fetching another quarter of every 256 values of k first and finding the others' in the XCD's L2 the forward solve took 5.55
  // ms instead of 5.94, the adjoint 10.7 instead of 11.1.)
  auto load_w = [&](LW (&w)[4], const __bf16* Wp, int p, int d) __attribute__((always_inline)) {
    int s = 2 * d;
    asm volatile("" : "+s"(s));                                     // (or every load gets an address register that counts along)
    const unsigned add = 2u * (unsigned)(WN ? 32 * s * q + 256 * p : 256 * p * q + 32 * s);
    const char* base = reinterpret_cast<const char*>(Wp);
#pragma unroll
    for (int i = 0; i < 4; ++i) w[i] = *reinterpret_cast<const LW*>(base + min(wo[i] + add, wlast));
  };
  // a pair as loaded -> [0], [1]: k step 2 d, [2], [3]: k step 2 d + 1, rows lane / 4 and 16 more
  auto sort_w = [&](LW (&w)[4]) __attribute__((always_inline)) {
    if constexpr (!WN) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const auto lo = __builtin_amdgcn_permlane32_swap(w[0][i], w[1][i], false, false);
        const auto hi = __builtin_amdgcn_permlane32_swap(w[2][i], w[3][i], false, false);
        w[0][i] = lo[0]; w[1][i] = hi[0];
        w[2][i] = lo[1]; w[3][i] = hi[1];
      }
    }
  };
  // staging rows of 64 bytes; the pieces of a row are permuted by h(row), WN by wnf(row), see the reads
  auto h = [](int r) __attribute__((always_inline)) { return -(r >> 2) & 3; };
  auto wnf = [](int r) __attribute__((always_inline)) { return (r >> 3) & 1; };
  unsigned so[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int row = (lane + 64 * i) >> 2, pc = lane & 3;
    so[i] = (unsigned)(row * 64 + (WN ? (((pc >> 1) ^ wnf(row)) * 32 + (pc & 1) * 16) : ((pc ^ h(row & 15)) * 16)));
  }
  auto stage_w = [&](const LW (&w)[4], int odd) __attribute__((always_inline)) {       // a k step's piece, to its half of the area
#pragma unroll
    for (int i = 0; i < 2; ++i) *reinterpret_cast<u32x4*>(Ws + 2048 * odd + so[i]) = w[2 * odd + i];
  };
  // A wavefront's staging area is its own and its LDS operations execute in order: the fences only keep the compiler from
  // moving accesses across.
  auto wave_sync = [&]() __attribute__((always_inline)) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };
  // ---- the operand: piece t (8 values of k) of row r at r OP + 16 (t ^ sigma(r)); OP is a multiple of 256 bytes
  const int sigma = ((c & 3) << 2) | h(c);
  auto write_operand = [&](int k) __attribute__((always_inline)) {  // of step k
    DR dr[2][RB][FB];                                               // the next pass's act' factors are on their way
    auto load_d = [&](int p) __attribute__((always_inline)) {
      if constexpr (HD) {
        opaque();
        const typename F::Ptr dp = F::at(a.Dm, layer_of(k) * a.E + sl_off);
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
          for (int j = 0; j < FB; ++j) dr[p & 1][rb][j] = F::load(dp, off(p, rb, j));
      }
    };
    load_d(0);
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      if (p >= np && 256 * p + 32 * wave >= KP) break;              // (features from the width to KP are zeros)
      if (p + 1 < NP) load_d(p + 1);
      opaque();
#pragma unroll
      for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int j = 0; j < FB; ++j) {
          float4 v = make_float4(st[p][rb][j][0], st[p][rb][j][1], st[p][rb][j][2], st[p][rb][j][3]);
          if constexpr (HD) { const float4 d = F::f4(dr[p & 1][rb][j], 4 * kq); v.x *= d.x; v.y *= d.y; v.z *= d.z; v.w *= d.w; }
          if (feat(p, j) >= q) v = make_float4(0.f, 0.f, 0.f, 0.f);
          const int t = 32 * p + 4 * wave + 2 * j + (kq >> 1);
          cvt_store4(reinterpret_cast<__bf16*>(smem + (16 * rb + cx) * OP + ((t ^ sigma) << 4) + 8 * (kq & 1)), v);
        }
    }
  };

  const __bf16* Wall = reinterpret_cast<const __bf16*>(a.W);
  const __bf16* Wc = Wall + layer_of(1) * a.wsize;
  LW w[2][4];
  load_w(w[0], Wc, 0, 0);
  load_w(w[1], Wc, 0, 1);
  write_operand(1);
  sort_w(w[0]);
  stage_w(w[0], 0);
  __syncthreads();

  const unsigned oc = (unsigned)c * OP, ox = (unsigned)((kq ^ sigma) << 4);    // this lane's row and piece: (4 s + kq) ^ sigma = 4 s ^ (kq ^ sigma)
  // ... and its pieces of the weights in the staging area (W[k][n]: rows 8 kq + c / 4 and four further on)
  unsigned aw[FB];
#pragma unroll
  for (int j = 0; j < FB; ++j)
    aw[j] = WN ? (unsigned)((8 * kq + (c >> 2)) * 64 + ((j ^ wnf(8 * kq)) * 32) + 8 * (c & 3)) : (unsigned)(c * 64 + ((kq ^ h(c)) * 16));
  for (int k = 1; k <= n; ++k) {
    const __bf16* Wn = Wall + layer_of(k < n ? k + 1 : k) * a.wsize;           // (past the last step: read, not used)
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      if (p >= np) break;
      opaque();
      const bool lastp = p + 1 >= np;
      const __bf16* Wx = lastp ? Wn : Wc;                           // the piece after this pass's last
      const int px = lastp ? 0 : p + 1;
      floatx4 acc[RB][FB];
#pragma unroll
      for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int j = 0; j < FB; ++j) acc[rb][j] = floatx4{0.f, 0.f, 0.f, 0.f};
      // k step i of the pass: its fragments, then the next piece's way into the other half of the staging area and, every other time,
      // the request for the pair after the next, then the matrix instructions (the other wavefront of the SIMD covers the reads)
      auto kstep = [&](LW (&w0)[4], LW (&w1)[4], int i, auto oddc) __attribute__((always_inline)) {
        constexpr int odd = decltype(oddc)::value, half = 2048 * odd;
        int s = i;
        asm volatile("" : "+s"(s));
        __builtin_amdgcn_sched_barrier(0);
        bf16x8 af[FB], bf[RB];
#pragma unroll
        for (int j = 0; j < FB; ++j) {
          if constexpr (WN) {
            // two transposing reads: rows k = 8 kq + 0 .. 3 and + 4 .. 7 of column c of the block
            typedef __attribute__((address_space(3))) short4v* lds_s4;
            const short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4)(Ws + half + aw[j]));
            const short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4)(Ws + half + aw[j] + 256));
            af[j] = __builtin_shufflevector(__builtin_bit_cast(bf16x4, lo), __builtin_bit_cast(bf16x4, hi), 0, 1, 2, 3, 4, 5, 6, 7);
          } else {
            af[j] = *reinterpret_cast<const bf16x8*>(Ws + half + aw[0] + 1024 * j);
          }
        }
        const unsigned char* ap = smem + oc + (ox ^ (64u * s));
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) bf[rb] = *reinterpret_cast<const bf16x8*>(ap + rb * 16 * OP);
        __builtin_amdgcn_sched_barrier(0);
        wave_sync();
        if constexpr (odd) {
          sort_w(w1);
          stage_w(w1, 0);
        } else {
          stage_w(w0, 1);
          const int d = (i >> 1) + 2;
          if (2 * d < KS) load_w(w0, Wc, p, d); else load_w(w0, Wx, px, d - KS / 2);
        }
        wave_sync();
        __builtin_amdgcn_sched_barrier(0);
        // a lane whose eight values of k lie past the width takes zeros: its operand is zero as well, but the weight read for it
        // may be infinite
        if (32 * s + 32 > q) {
          asm volatile("");                                         // (a branch, not a select in every step)
#pragma unroll
          for (int j = 0; j < FB; ++j) {
            const u32x4 z = __builtin_bit_cast(u32x4, af[j]);
            af[j] = __builtin_bit_cast(bf16x8, 32 * s + 8 * kq < q ? z : u32x4{0u, 0u, 0u, 0u});
          }
        }
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
          for (int j = 0; j < FB; ++j) acc[rb][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[j], bf[rb], acc[rb][j], 0, 0, 0);
      };
#pragma unroll 1
      for (int i = 0; i < KS; i += 4) {                             // KS is a multiple of four
        kstep(w[0], w[1], i, std::integral_constant<int, 0>{});
        kstep(w[0], w[1], i + 1, std::integral_constant<int, 1>{});
        kstep(w[1], w[0], i + 2, std::integral_constant<int, 0>{});
        kstep(w[1], w[0], i + 3, std::integral_constant<int, 1>{});
      }
      const float* bp = HD ? nullptr : a.bias + layer_of(k) * q;
      const float* gp = a.G ? place(a.G, a.gb + ci * a.gs + k) : nullptr;
#pragma unroll
      for (int j = 0; j < FB; ++j) {
        floatx4 bv = floatx4{0.f, 0.f, 0.f, 0.f};
        if constexpr (!HD) bv = *reinterpret_cast<const floatx4*>(bp + (feat(p, j) < q ? feat(p, j) : 0));
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
          for (int v = 0; v < 4; ++v) st[p][rb][j][v] += a.hs * act_fn_c<ACT>(acc[rb][j][v] + bv[v]);
      }
      if (gp) {                                                     // coarse levels only
        opaque();
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
          for (int j = 0; j < FB; ++j) st[p][rb][j] += *reinterpret_cast<const floatx4*>(gp + off(p, rb, j));
      }
    }

    if (a.tau) {                                                    // coarse right-hand side: Z <- Z - state, and its norm
      float* o = place(a.Z, a.zb + ci * a.zs);
      const float* ref = a.Ref ? place(a.Ref, a.rm.base + ci * a.rm.stride) : nullptr;
      float sq = 0.0f;
#pragma unroll
      for (int p = 0; p < NP; ++p)
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
          for (int j = 0; j < FB; ++j)
            if (16 * rb + cx < rows && feat(p, j) < q) {
              const floatx4 z = *reinterpret_cast<const floatx4*>(o + off(p, rb, j));
              *reinterpret_cast<floatx4*>(o + off(p, rb, j)) = z - st[p][rb][j];
              if (ref) {
                const floatx4 d = z - *reinterpret_cast<const floatx4*>(ref + off(p, rb, j));
                sq += (d[0] * d[0] + d[1] * d[1]) + (d[2] * d[2] + d[3] * d[3]);
              }
            }
      if (a.norm_partial) {
#pragma unroll
        for (int x = 32; x > 0; x >>= 1) sq += __shfl_xor(sq, x, 64);
        __syncthreads();                                            // every wavefront is done with the operand: its first bytes hold the sums
        float* red = reinterpret_cast<float*>(smem);
        if (lane == 0) red[wave] = sq;
        __syncthreads();
        if (tid == 0) {
          float t = red[0];
          for (int x = 1; x < WIDE_NWV; ++x) t += red[x];
          a.norm_partial[L] = t;
        }
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
    write_operand(k + 1);
    Wc = Wn;
    __syncthreads();
  }
}

bool wide_supported(int q, int dtype) { return dtype == 1 && q > 256 && q <= 1024 && q % 8 == 0; }
int  wide_blocks(int M, int nchains) { return (M + WIDE_ROWS - 1) / WIDE_ROWS * nchains; }

namespace {
template <int NP, int ACT, bool WN> hipError_t launch_wide_t(const SweepArgs& a, unsigned blocks, hipStream_t s) {
  const size_t smem = (size_t)WIDE_ROWS * 2 * wide_kp(a.q) + (size_t)WIDE_NWV * WIDE_STG;
  static LdsOptIn opt;
  const hipError_t e = opt.raise(reinterpret_cast<const void*>(wide_sweep_kernel<NP, ACT, WN>), smem);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((wide_sweep_kernel<NP, ACT, WN>), dim3(blocks), dim3(64 * WIDE_NWV), smem, s, a);
  return hipGetLastError();
}
template <int NP> hipError_t launch_wide_np(const SweepArgs& a, unsigned blocks, hipStream_t s) {
  switch (a.act) {
    case ACT_TANH: return launch_wide_t<NP, ACT_TANH, false>(a, blocks, s);
    case ACT_RELU: return launch_wide_t<NP, ACT_RELU, false>(a, blocks, s);
    case ACT_MASK: return a.wn ? launch_wide_t<NP, ACT_MASK, true>(a, blocks, s) : launch_wide_t<NP, ACT_MASK, false>(a, blocks, s);
    default:       return a.wn ? launch_wide_t<NP, ACT_IDENT, true>(a, blocks, s) : launch_wide_t<NP, ACT_IDENT, false>(a, blocks, s);
  }
}
}  // namespace

hipError_t launch_wide(const SweepArgs& a, int dtype, hipStream_t s) {
  if (a.nchains <= 0) return hipSuccess;
  if (a.M < 1 || !wide_supported(a.q, dtype)) return hipErrorInvalidValue;
  if ((a.act == ACT_IDENT || a.act == ACT_MASK) != (a.Dm != nullptr) || (a.Dm == nullptr && (a.wn || !a.bias))) return hipErrorInvalidValue;
  if (a.tau && (a.nsteps != 1 || a.nlast != 1 || !a.Z)) return hipErrorInvalidValue;
  const unsigned blocks = (unsigned)wide_blocks(a.M, a.nchains);
  trace_before(s);
  const hipError_t e = a.q <= 512 ? launch_wide_np<2>(a, blocks, s) : a.q <= 768 ? launch_wide_np<3>(a, blocks, s) : launch_wide_np<4>(a, blocks, s);
  trace_after(s, TRACE_SWEEP_BF16, a.units, sweep_bytes(a, dtype));
  return e;
}

}  // namespace mgrit
