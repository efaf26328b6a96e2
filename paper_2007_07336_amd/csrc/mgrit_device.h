// Device-side helpers shared by the kernel files: operand and accumulator types, activations, the XCD-aware
// workgroup order and the LDS opt-in.
#pragma once
#include "mgrit_internal.h"

#include <type_traits>

namespace mgrit {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef short short4v __attribute__((ext_vector_type(4)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));

// Operand traits.  Matrix-core operands live in LDS as rows of KSTEP-multiples, k fastest.
//   float : v_mfma_f32_32x32x2_f32, a lane feeds 4 consecutive k over 4 instructions
//   bf16  : v_mfma_f32_32x32x16_bf16, a lane feeds 8 consecutive k per instruction
template <typename T> struct Op;
template <> struct Op<float> {
  static constexpr int KSTEP = 8;   // k consumed by one mma_step
  static constexpr int VEC = 4;     // elements per 16-byte piece
  static constexpr int PAD = 4;     // row padding in LDS (elements)
};
template <> struct Op<__bf16> {
  static constexpr int KSTEP = 16;
  static constexpr int VEC = 8;
  static constexpr int PAD = 8;
};

// 16-byte load of layer weights.  STREAM: non-temporal, for parameter sets larger than the 256 MB last-level
// cache -- a weight is used once per launch and must not push out the states, which the next launch reads
// again.  Otherwise a plain load: the whole parameter set stays cached across the launches of a solve
// (measured: 6 % on the q=256 workload with 64 MB of weights, the other way round -0.5 % with 2 GB).
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
template <bool STREAM, typename T>
__device__ __forceinline__ uint4 ld_weights(const T* p) {
  if (STREAM) {
    const u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
    return make_uint4(v.x, v.y, v.z, v.w);
  }
  return *reinterpret_cast<const uint4*>(p);
}
// The act' cache of the adjoint sweep (and of the parameter gradient) is stored in the weights' type: float, or
// bf16 when the matrix-core operands are bf16 anyway (half the bytes of its many reads).  Four consecutive
// values are loaded raw -- no conversion next to the load, which would make the compiler wait for it -- and
// widened when they are used.
// ReLU's are 0 or 1 and are stored as bits, value i of a state in bit i % 8 of byte i / 8 (a state has a multiple of 8 values):
// Fac<Bit>.  A wide adjoint sweep spends a third to a half of its memory traffic on the factors, the gradient a fifth.
struct Bit {};
template <typename T> struct Fac {                                  // T = float or __bf16
  typedef const T* Ptr;                                             // of a layer's factors
  typedef typename std::conditional<sizeof(T) == 4, float4, uint2>::type Raw;
  static __device__ __forceinline__ Ptr at(const void* base, long long value) { return reinterpret_cast<const T*>(base) + value; }
  static __device__ __forceinline__ Raw load(Ptr p, unsigned off) { return *reinterpret_cast<const Raw*>(p + off); }   // four, off % 4 == 0
  // (byte offsets from a uniform base, as the unmasked kernels address memory)
  static __device__ __forceinline__ Raw load_bytes(const char* p, unsigned off) { return *reinterpret_cast<const Raw*>(p + (unsigned)sizeof(T) * off); }
  // the four as floats; off: their offset again, any number of eights left out
  static __device__ __forceinline__ float4 f4(float4 r, unsigned) { return r; }
  static __device__ __forceinline__ float4 f4(uint2 r, unsigned) {
    return make_float4(__uint_as_float(r.x << 16), __uint_as_float(r.x & 0xffff0000u),
                       __uint_as_float(r.y << 16), __uint_as_float(r.y & 0xffff0000u));
  }
};
// bit i of n as a factor 0 or 1
__device__ __forceinline__ float bit_factor(unsigned n, int i) {
  return __uint_as_float((unsigned)((int)(n << (31 - i)) >> 31) & 0x3f800000u);
}
template <> struct Fac<Bit> {
  typedef const unsigned char* Ptr;
  typedef unsigned Raw;
  static __device__ __forceinline__ Ptr at(const void* base, long long value) { return reinterpret_cast<Ptr>(base) + (value >> 3); }
  // (four bytes, of which the first counts and the others may lie past the last layer's factors, in the cache's unused part: a byte
  // that waits in a register until it is used is masked right behind its load, and the wavefront waits for it there.  Float width
  // 64, 32 layers on 16384 samples, adjoint with gradient: 2170 us with bytes, 1887 so, 1950 with values)
  struct __attribute__((packed)) Word { unsigned w; };
  static __device__ __forceinline__ Raw load(Ptr p, unsigned off) { return reinterpret_cast<const Word*>(p + (off >> 3))->w; }
  static __device__ __forceinline__ Raw load_bytes(const char* p, unsigned off) { return load(reinterpret_cast<Ptr>(p), off); }
  static __device__ __forceinline__ float4 f4(Raw r, unsigned off) {
    const unsigned n = r >> (off & 4u);
    return make_float4(bit_factor(n, 0), bit_factor(n, 1), bit_factor(n, 2), bit_factor(n, 3));
  }
};
// The byte of the factors of this lane's four values o and of its odd or even neighbour's (lanes 2 i and 2 i + 1 hold eight
// consecutive ones); both lanes get it.
__device__ __forceinline__ unsigned char factor_byte(float4 o, int lane) {
  const unsigned n = (o.x != 0.0f ? 1u : 0u) | (o.y != 0.0f ? 2u : 0u) | (o.z != 0.0f ? 4u : 0u) | (o.w != 0.0f ? 8u : 0u);
  const unsigned other = (unsigned)__builtin_amdgcn_mov_dpp((int)n, 0xB1, 0xF, 0xF, true);   // quad_perm [1, 0, 3, 2]
  return (unsigned char)((lane & 1) ? (n << 4) | other : n | (other << 4));
}
__device__ __forceinline__ void cvt_store4(float* dst, float4 v) { *reinterpret_cast<float4*>(dst) = v; }
__device__ __forceinline__ void cvt_store4(__bf16* dst, float4 v) {
  bf16x4 o;
  o[0] = static_cast<__bf16>(v.x);   // round to nearest even
  o[1] = static_cast<__bf16>(v.y);
  o[2] = static_cast<__bf16>(v.z);
  o[3] = static_cast<__bf16>(v.w);
  *reinterpret_cast<bf16x4*>(dst) = o;
}

// x = h + m + l, each representable in bf16 (rounded to nearest each time; exact, since a float has 24 significant
// bits), for a vector of floats: two values per conversion instruction.
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ floatx2 widen2(bf16x2 v) {
  const unsigned u = __builtin_bit_cast(unsigned, v);
  return floatx2{__uint_as_float(u << 16), __uint_as_float(u & 0xffff0000u)};
}
template <int N, typename F, typename V>
__device__ __forceinline__ void split3(F f, V& h, V& m, V& l) {               // f(i) = value i
#pragma unroll
  for (int i = 0; i < N; i += 2) {
    const floatx2 x = floatx2{f(i), f(i + 1)};
    const bf16x2 a = __builtin_convertvector(x, bf16x2);
    const floatx2 wa = widen2(a), r = floatx2{x[0] - wa[0], x[1] - wa[1]};
    const bf16x2 b = __builtin_convertvector(r, bf16x2);
    const floatx2 wb = widen2(b);
    const bf16x2 c = __builtin_convertvector((floatx2{r[0] - wb[0], r[1] - wb[1]}), bf16x2);
    h[i] = a[0]; h[i + 1] = a[1];
    m[i] = b[0]; m[i + 1] = b[1];
    l[i] = c[0]; l[i + 1] = c[1];
  }
}

__device__ __forceinline__ floatx16 zero16() {
  floatx16 z;
#pragma unroll
  for (int r = 0; r < 16; ++r) z[r] = 0.0f;
  return z;
}
// tanh(z) = 1 - 2 / (e^{2z} + 1) on the hardware exp2 / rcp units: absolute error about 2e-7
// (the library tanhf costs ~100 instructions per element, which dominated the epilogue).  The
// result enters the state scaled by h, so the absolute error is what matters.
__device__ __forceinline__ float fast_tanh(float z) {
  const float e = __builtin_amdgcn_exp2f(z * 2.885390081777927f);      // e^{2z}; inf / 0 saturate correctly
  return 1.0f - 2.0f * __builtin_amdgcn_rcpf(e + 1.0f);
}
__device__ __forceinline__ float act_fn(float z, int act) {
  if (act == ACT_TANH) return fast_tanh(z);
  if (act == ACT_RELU) return fmaxf(z, 0.0f);
  return z;
}
__device__ __forceinline__ float act_prime(float z, int act) {
  if (act == ACT_TANH) { float t = fast_tanh(z); return 1.0f - t * t; }
  if (act == ACT_RELU) return z > 0.0f ? 1.0f : 0.0f;
  return 1.0f;
}
// The same with the activation as a compile-time value: the epilogues of the tiled kernels branch on it once
// per workgroup instead of once per element (a chain of scalar compares and branches around every one of a
// lane's 64 output values took longer than their arithmetic).
template <int ACT> __device__ __forceinline__ float act_fn_c(float z) {
  if (ACT == ACT_TANH) return fast_tanh(z);
  if (ACT == ACT_RELU) return fmaxf(z, 0.0f);
  return z;
}
template <int ACT> __device__ __forceinline__ float act_prime_c(float z) {
  if (ACT == ACT_TANH) { float t = fast_tanh(z); return 1.0f - t * t; }
  if (ACT == ACT_RELU) return z > 0.0f ? 1.0f : 0.0f;
  return 1.0f;
}

// (In the kernels below the wavefront index is read with readfirstlane: the compiler cannot see that tid >> 6 is
// the same in all lanes, and with a scalar index the address arithmetic and conditions that depend on it stay on
// the scalar unit.)
// XCD-aware workgroup order: hardware deals consecutive workgroup ids round-robin to the 8
// XCDs; remap so that consecutive logical tiles (which share a group's state and weights)
// land on the same XCD and meet in its L2.  With a count that is no multiple of 8 the first
// XCDs get one more.
__device__ __forceinline__ int logical_block() {
  const int total = gridDim.x, L = blockIdx.x, x = L & 7, r = total & 7;
  return x * (total >> 3) + (x < r ? x : r) + (L >> 3);
}

// p / w for 0 <= p < 4096 and 1 <= w <= 256 with magic = ceil(2^20 / w): exact because p * (magic * w - 2^20) < 2^20
__device__ __forceinline__ int div_small(int p, unsigned magic) { return (int)(((unsigned)p * magic) >> 20); }

// A kernel that uses more than 64 KB of dynamic LDS has to opt in, once per device (the attribute belongs to
// the device's copy of the kernel).  One of these per kernel instance remembers the largest size each device
// has been raised to -- once that is done, so that another thread's first launch does not run ahead of it.
struct LdsOptIn {
  size_t seen[64] = {};
  hipError_t raise(const void* kernel, size_t smem) {
    if (smem <= 64 * 1024) return hipSuccess;
    int dev = 0;
    const bool known = hipGetDevice(&dev) == hipSuccess && dev >= 0 && dev < 64;
    if (known && smem <= seen[dev]) return hipSuccess;
    const hipError_t e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    if (e == hipSuccess && known) seen[dev] = smem;
    return e;
  }
};

}  // namespace mgrit
