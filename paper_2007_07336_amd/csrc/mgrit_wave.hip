// Sweeps over narrow dense layers: one wavefront carries sixteen batch rows of a chain through its layer steps, and one launch
// can hold many sweeps that follow one another.
#include "mgrit_device.h"

namespace mgrit {

// ------------------------------------------------------------------------------------------
// A unit is (chain, slice of 16 batch rows) of layers of width 8 or 16, and a wavefront does a whole step of it by itself:
//   - Lane (c, kq) holds features 4 kq .. + 3 of batch row c, which is where the matrix instructions with the weights as the A
//     operand leave them.  The instructions that contract over 4 (float) or 16 (bf16) values of k take their B operand from the
//     same place: k = 4 kq + t is what lane (c, kq) has in st[t].  So the state never leaves its registers between steps: no LDS,
//     no barrier, no exchange between lanes.
//   - Float layers run on the float matrix instructions: at this width splitting the operands (the wider sweeps' way) would take
//     longer than the instructions it saves.
//   - A layer's weights, bias, act' factors and right-hand side are requested PD steps ahead.
// Every slice of a dense stack is independent of all others for a whole solve.  Where the sweeps that follow one another are
// short, a workgroup therefore takes all chains of its slice, wavefront by wavefront, and goes on to the next sweep behind a
// barrier instead of a launch: between two dependent launches 4 to 5 us pass, between two sweeps of a workgroup about 1.5.
// What bounds it is latency, and with many wavefronts on a CU the addresses: a lane's 16 bytes lie 64 from its neighbour's, and
// such an access takes the CU 64 cycles.  (That is why it ends at width 16: with two blocks of features a layer's weights are four
// such accesses, and 64 layers of width 32 took 138 us, as sweeps of four wavefronts 100.)
// 16 layers of width 8, 4 samples, four cycles with the residual history, against sweeps of four wavefronts and a launch each: 141 -> 67
// us; 1024 layers on 256 samples, two cycles, three levels with m = 4: 359 -> 127 us forward, 536 -> 255 adjoint and gradient.
// ------------------------------------------------------------------------------------------
constexpr int WAVE_NW = 8;                                          // wavefronts of a workgroup

template <int NW> __device__ __forceinline__ float wave_block_sum(float sq, float* red, int tid) {   // fixed order; valid in thread 0
#pragma unroll
  for (int w = 32; w > 0; w >>= 1) sq += __shfl_xor(sq, w, 64);
  if ((tid & 63) == 0) red[tid >> 6] = sq;
  __syncthreads();
  float t = red[0];
#pragma unroll
  for (int w = 1; w < NW; ++w) t += red[w];
  __syncthreads();
  return t;
}

// WN: weights W[k][n] (the adjoint on the caller's array).
template <typename WT, int ACT, bool WN>
__global__ __launch_bounds__(64 * WAVE_NW) void dense_wave_kernel(WaveProgram p) {
  constexpr bool HD = ACT == ACT_IDENT || ACT == ACT_MASK, BF = sizeof(WT) == 2;
  constexpr int PD = 4;                                             // steps requested ahead
  typedef Fac<typename std::conditional<ACT == ACT_MASK, Bit, WT>::type> F;
  typedef typename F::Raw DR;
  typedef typename std::conditional<BF, bf16x4, floatx4>::type WV;  // four values of k of one output feature
  __shared__ float red[WAVE_NW];
  const int tid = threadIdx.x, lane = tid & 63, c = lane & 15, kq = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int q = p.q, slice = blockIdx.x % p.nsl, part = blockIdx.x / p.nsl;
  const int r0 = slice * 16, rows = min(16, p.M - r0);
  const long long sl_off = (long long)r0 * q;
  const WT* W = reinterpret_cast<const WT*>(p.W);
  // (rows past the batch read the last one's values, features past the width those of feature 0: never stored, and zero as an operand)
  const bool in = 4 * kq < q;                                       // q % 8 == 0: a lane's four are in or out together
  const int k4 = in ? 4 * kq : 0, cw = c < q ? c : 0;
  const unsigned off = 4u * (unsigned)(min(c, rows - 1) * q + k4);  // bytes into a state of floats
  const unsigned wo = (unsigned)sizeof(WT) * (unsigned)(WN ? k4 * q + cw : cw * q + k4);       // into a layer's weights
  // (global memory, said explicitly: the compiler does not know it of a pointer that it has seen copied as words; a uniform base
  // and a 32-bit offset of a lane)
  typedef char __attribute__((address_space(1))) * GBase;
  auto place = [&](const float* base, long long point) __attribute__((always_inline)) { return (GBase)(char*)const_cast<float*>(base + point * p.E + sl_off); };
  auto get4 = [&](GBase b, unsigned o) __attribute__((always_inline)) { return *(const floatx4 __attribute__((address_space(1)))*)(b + o); };
  auto put4 = [&](GBase b, unsigned o, floatx4 v) __attribute__((always_inline)) { *(floatx4 __attribute__((address_space(1)))*)(b + o) = v; };

  typedef const unsigned __attribute__((address_space(4))) * ArgWords;
  const ArgWords args = (ArgWords)__builtin_amdgcn_kernarg_segment_ptr();
#pragma unroll 1
  for (int op = 0; op < p.nops; ++op) {
    WaveOp a;                                                       // (read through the argument segment: the index is not constant)
    static_assert(sizeof(WaveOp) % 4 == 0 && offsetof(WaveProgram, op) % 4 == 0, "copied word by word");
#pragma unroll
    for (unsigned i = 0; i < sizeof(WaveOp) / 4; ++i) reinterpret_cast<unsigned*>(&a)[i] = args[offsetof(WaveProgram, op) / 4 + op * (sizeof(WaveOp) / 4) + i];
    float sq = 0.0f;
#pragma unroll 1
    for (int ci = part * WAVE_NW + wave; ci < a.nchains; ci += p.per * WAVE_NW) {
      const int n = ci == a.nchains - 1 ? a.nlast : a.nsteps;
      floatx4 st;
      auto store_state = [&](GBase o) __attribute__((always_inline)) {
        if (c < rows && in) put4(o, off, st);
      };
      // the start state (store0 = 2: the last chain first passes on the point behind it)
      for (int t = a.store0 == 2 && ci == a.nchains - 1 ? 1 : 0; t >= 0; --t) {
        st = get4(place(a.S, a.sb + (long long)(ci + t) * a.ss), off);
        if (a.store0) store_state(place(a.X, a.xb + (long long)(ci + t) * a.xs));
      }
      // ---- a step's inputs
      auto run = [&](auto with_g) __attribute__((always_inline)) {
      constexpr bool WG = decltype(with_g)::value;                  // there is a right-hand side
      struct In { WV w; floatx4 bias, g; DR d; };
      In ring[PD];
      auto request = [&](In& r, int k) __attribute__((always_inline)) {
        const long long layer = a.lb + (long long)ci * a.ls + (long long)(k - 1) * a.lk;
        const char* wp = reinterpret_cast<const char*>(W + layer * p.wsize);
        if constexpr (WN) {
#pragma unroll
          for (int t = 0; t < 4; ++t) r.w[t] = *reinterpret_cast<const WT*>(wp + (wo + (unsigned)(t * q * (int)sizeof(WT))));
        } else {
          r.w = *reinterpret_cast<const WV*>(wp + wo);
        }
        if constexpr (HD) r.d = F::load_bytes(reinterpret_cast<const char*>(F::at(p.Dm, layer * p.E + sl_off)), off >> 2);
        else r.bias = *reinterpret_cast<const floatx4*>(reinterpret_cast<const char*>(p.bias + layer * q) + 4u * k4);
        if constexpr (WG) {
          r.g = get4(place(a.G, a.gb + (long long)ci * a.gs + k), off);
        }
      };
      auto step = [&](In& r, int k) __attribute__((always_inline)) {
        floatx4 acc = floatx4{0.f, 0.f, 0.f, 0.f}, x = st;
        if constexpr (!HD) acc = r.bias;
        if constexpr (HD) { const float4 d = F::f4(r.d, 4 * kq); x *= floatx4{d.x, d.y, d.z, d.w}; }
        // (past the width both factors of a product are zero: a clamped weight may be infinite)
        if (!in) x = floatx4{0.f, 0.f, 0.f, 0.f};
        if constexpr (BF) {
          bf16x4 xb;
#pragma unroll
          for (int t = 0; t < 4; ++t) xb[t] = static_cast<__bf16>(x[t]);
          u32x2 w = __builtin_bit_cast(u32x2, r.w);
          if (!in) w = u32x2{0u, 0u};
          acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(short4v, w), __builtin_bit_cast(short4v, xb), acc, 0, 0, 0);
        } else {
#pragma unroll
          for (int t = 0; t < 4; ++t) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(in ? (float)r.w[t] : 0.0f, x[t], acc, 0, 0, 0);
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) st[v] += a.hs * act_fn_c<ACT>(acc[v]);
        if constexpr (WG) st += r.g;
        if (a.tau) return;
        GBase o1 = nullptr, o2 = nullptr;                           // where this step's state is kept: at most two places
        if (a.X && a.xk) o1 = place(a.X, a.xb + (long long)ci * a.xs + (long long)k * a.xk);
        else if (k == a.kmid) { o1 = place(a.Y, a.yb + (long long)ci * a.ys); if (ci == 0) o2 = place(a.Z, a.zfirst); }
        else if (a.Z && k == n) o1 = place(a.Z, a.zb + (long long)ci * a.zs);
        if (o1) store_state(o1);
        if (o2) store_state(o2);
      };
#pragma unroll
        for (int i = 0; i < PD; ++i) request(ring[i], min(1 + i, n));   // (past the last step: read, not used)
        for (int k0 = 1; k0 <= n; k0 += PD) {
#pragma unroll
          for (int i = 0; i < PD; ++i) {
            const int k = k0 + i;
            if (k > n) break;
            step(ring[i], k);
            request(ring[i], min(k + PD, n));
          }
        }
      };
      if (n <= 0) continue;
      if (a.G) run(std::true_type{});
      else run(std::false_type{});
      if (a.tau) {                                                  // coarse right-hand side: Z <- Z - state, and its norm
        const GBase o = place(a.Z, a.zb + (long long)ci * a.zs), ref = a.Ref ? place(a.Ref, a.rb + (long long)ci * a.rs) : nullptr;
        const floatx4 z = get4(o, off), d = ref ? z - get4(ref, off) : floatx4{0.f, 0.f, 0.f, 0.f};
        if (c < rows && in) {
          put4(o, off, z - st);
          sq += (d[0] * d[0] + d[1] * d[1]) + (d[2] * d[2] + d[3] * d[3]);
        }
      }
    }
    if (a.norm_partial) {
      const float t = wave_block_sum<WAVE_NW>(sq, red, tid);
      if (tid == 0) *((float __attribute__((address_space(1)))*)(float*)a.norm_partial + blockIdx.x) = t;
    }
    __syncthreads();                                                // this slice's states are written: the next sweep reads them
  }
}

bool wave_supported(int q) { return q >= 8 && q <= 16 && q % 8 == 0; }
int  wave_slices(int M) { return (M + 15) / 16; }
int  wave_workgroups(int nchains) { return (nchains + WAVE_NW - 1) / WAVE_NW; }

hipError_t launch_wave(const WaveProgram& p_in, int per, int dtype, long long units, double bytes, hipStream_t s) {
  if (p_in.nops <= 0) return hipSuccess;
  WaveProgram p = p_in;
  if (p.M < 1 || per < 1 || (per > 1 && p.nops > 1) || p.nops > WAVE_OPS || !wave_supported(p.q)) return hipErrorInvalidValue;
  if ((p.act == ACT_IDENT || p.act == ACT_MASK) != (p.Dm != nullptr) || (p.Dm == nullptr && (p.wn || !p.bias))) return hipErrorInvalidValue;
  p.nsl = wave_slices(p.M);
  p.per = per;
  const dim3 grid((unsigned)p.nsl * (unsigned)per);
  trace_before(s);
#define MGRIT_WV(WT_, ACT_, WN_) hipLaunchKernelGGL((dense_wave_kernel<WT_, ACT_, WN_>), grid, dim3(64 * WAVE_NW), 0, s, p)
#define MGRIT_WV_ACT(WT_)                                                                                    \
  { if (p.act == ACT_TANH)      MGRIT_WV(WT_, ACT_TANH, false);                                              \
    else if (p.act == ACT_RELU) MGRIT_WV(WT_, ACT_RELU, false);                                              \
    else if (p.act == ACT_MASK) { if (p.wn) MGRIT_WV(WT_, ACT_MASK, true); else MGRIT_WV(WT_, ACT_MASK, false); }   \
    else                        { if (p.wn) MGRIT_WV(WT_, ACT_IDENT, true); else MGRIT_WV(WT_, ACT_IDENT, false); } }
  if (dtype == 0) MGRIT_WV_ACT(float) else MGRIT_WV_ACT(__bf16)
#undef MGRIT_WV_ACT
#undef MGRIT_WV
  const hipError_t e = hipGetLastError();
  trace_after(s, dtype == 0 ? TRACE_SWEEP_F32 : TRACE_SWEEP_BF16, units, bytes);
  return e;
}

}  // namespace mgrit
