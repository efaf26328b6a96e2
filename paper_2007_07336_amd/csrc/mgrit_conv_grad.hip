// Parameter gradient of narrow float convolution layers on the bf16 matrix cores.
#include "mgrit_device.h"

namespace mgrit {

// ------------------------------------------------------------------------------------------
// dK[o][tap][i] = hs * sum over pixels p of G[p][o] U[p + tap][i], G = Dm .* Lam, and db[o] = hs * sum G: conv_grad_kernel's
// contraction over slabs of gR image rows, for float layers of at most 32 channels (NB = 1 or 2 blocks of 16).
//   - G and U are split into three bf16 numbers where a slab goes to LDS, [part][channel][pixel slot], and six products of parts
//     stand for one, the five small ones in sums of their own (as in the float sweeps).
//   - U is in LDS once: a lane that holds the eight slots s .. s + 7 of an image row for dx = 0 makes those for dx = -1 and + 1
//     from them and their two neighbours, which lie in an array of their own, [part][channel][eight slots] (read from the rows
//     themselves they meet in a sixteenth of the LDS banks); dy is a row's offset.
//   - NB = 1: each of the four wavefronts has all nine taps and the bias of every fourth step of 32 slots, and their sums are
//     added in wavefront order at the end; NB = 2: a wavefront per pair of channel blocks.
// 64 layers of 16 channels, 64 images of 28 x 28: 174 us (281 on the float matrix instructions, whose 143 it spent in matrix cores and
// the rest in three shifted copies of U), errors against 64 bits 2e-7 instead of 1e-6.  Of the 174 the matrix instructions take 43,
// the vector instructions that split and shift 78, the bytes 103 at the copy rate; what bounds it is that a slab's load, split and
// product follow one another with two workgroups per CU to overlap them (the sums take 80 registers).  Tried: the neighbours read
// from the rows, with four-way bank conflicts, 179; pixels instead of channel groups along the lanes of a load 179.
// Infinite values (and finite ones of 3.396e38 or more) have no such parts and make NaN of the sums they enter: a workgroup that
// ends with a sum that is not finite forms its sums again from the float values.  The gradient above with a NaN in every layer 168 ->
// 870 us (25.7 ms with a thread per output that walked the pixels in global memory), 32 channels on 16 images of 32 x 32 148 -> 1040
// (26.8 ms).  So does one that ends with sums of less than 2^-90 and not zero, whose operands may be so small, below about 1e-34, that
// their lower parts are no bf16 numbers any more: at 1e-37 the error would be 3e-4 of the result instead of 2e-7.
// ------------------------------------------------------------------------------------------
constexpr int CGS_NTH = 256;
// 4 x 4 blocks of U per thread, at most (two, and the factors as values, spill beside the sums of NB = 1)
constexpr int cgs_ub(int nb, bool bits) { return nb == 1 && !bits ? 1 : 2; }

// 32-bit words of a channel's neighbours: an odd multiple of four, so that 16 channels' four words lie on 64 banks
constexpr int cgs_ep(int PU) { return 4 * ((PU / 8 + 3) / 4 | 1); }

template <typename DT, int NB>
__global__ __launch_bounds__(CGS_NTH, 2) void conv_grad_split_kernel(GradArgs a) {
  constexpr int NTH = CGS_NTH, UB = cgs_ub(NB, std::is_same<DT, Bit>::value), NW = NTH / 64;
  static_assert(NB == 1 || NB * NB == NW, "a wavefront per pair of channel blocks");
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  __shared__ int bad;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int bl = lane & 15, kq = lane >> 4;
  const int C = a.Nf, H = a.Himg, Wd = a.Wimg, Wp = a.gWp, R = a.gR, PU = a.gPU, PG = a.gPG, KL = a.gKL;
  __bf16* Ut = reinterpret_cast<__bf16*>(smem_raw);                 // [3][C][PU]
  __bf16* Gt = Ut + 3 * C * PU;                                     // [3][C][PG]
  const int EP = cgs_ep(PU);
  unsigned* Et = reinterpret_cast<unsigned*>(Gt + 3 * C * PG);      // [3][C][EP]: slots s - 1 and s + 8 of the eight from s = 8 g, zero past a row's ends
  const int L = logical_block();
  const int gi = L / a.gchunks, ch = L % a.gchunks;
  const float* Up = a.U + (a.um.base + gi * a.um.stride) * a.E;
  const float* Lp = a.Lam + (a.lm.base + gi * a.lm.stride) * a.E;
  typedef Fac<DT> F;
  const typename F::Ptr Dp = F::at(a.Dm, (a.dm.base + gi * a.dm.stride) * a.E);
  typedef typename F::Raw DR;

  // slots that no block covers (row padding, the rest of the last step of 32) stay zero
  for (int p = tid; p < 3 * C * (PU + PG + 2 * EP) / 8; p += NTH) reinterpret_cast<uint4*>(smem_raw)[p] = make_uint4(0u, 0u, 0u, 0u);

  // this thread's 4 (pixels) x 4 (channels) blocks: one of G, up to UB of U, the latter counted from the last thread.
  // Channel groups fastest: four lanes load 64 bytes in a row, and their stores, rows 64 times an odd number of bytes apart, are on other banks
  const int CG = C >> 2, XG = (Wd + 3) >> 2;
  const int nGb = R * XG * CG, nUb = (R + 2) * XG * CG;
  const bool gact = tid < nGb;
  const int gb = gact ? tid : 0;
  const int g_cg = gb % CG, g_xg = (gb / CG) % XG, g_r = gb / (CG * XG);
  bool uact[UB];
  int u_cg[UB], u_xg[UB], u_r[UB];
#pragma unroll
  for (int t = 0; t < UB; ++t) {
    const int blk = NTH - 1 - tid + NTH * t;
    uact[t] = blk < nUb;
    const int ub = uact[t] ? blk : 0;
    u_cg[t] = ub % CG; u_xg[t] = (ub / CG) % XG; u_r[t] = ub / (CG * XG);
  }
  floatx4 lv[4], uv[UB][4];
  DR dv[4];
  unsigned gmask = 0, umask[UB] = {};
  auto load_slab = [&](int sl) __attribute__((always_inline)) {
    const int b = sl / a.gspi, y0 = (sl % a.gspi) * R;
    {
      const int y = y0 + g_r;
      const bool rok = gact && y < H;
      gmask = 0;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int x = 4 * g_xg + j;
        const bool ok = rok && x < Wd;
        gmask |= ok ? (1u << j) : 0u;
        const unsigned off = ok ? (unsigned)((((long long)b * H + y) * Wd + x) * C + 4 * g_cg) : 0u;
        dv[j] = F::load(Dp, off);
        lv[j] = *reinterpret_cast<const floatx4*>(Lp + off);
      }
    }
#pragma unroll
    for (int t = 0; t < UB; ++t) {
      if (NTH * t >= nUb) break;                                    // uniform
      const int y = y0 - 1 + u_r[t];
      const bool rok = uact[t] && y >= 0 && y < H;
      umask[t] = 0;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int x = 4 * u_xg[t] + j;
        const bool ok = rok && x < Wd;
        umask[t] |= ok ? (1u << j) : 0u;
        const unsigned off = ok ? (unsigned)((((long long)b * H + y) * Wd + x) * C + 4 * u_cg[t]) : 0u;
        uv[t][j] = *reinterpret_cast<const floatx4*>(Up + off);
      }
    }
  };
  // four pixels' values of one channel, split, to the channel's row of each part
  auto put = [&](__bf16* row, int part, floatx4 x, bf16x4 (&y)[3]) __attribute__((always_inline)) {
    split3<4>([&](int e) { return x[e]; }, y[0], y[1], y[2]);
#pragma unroll
    for (int q = 0; q < 3; ++q) *reinterpret_cast<bf16x4*>(row + q * part) = y[q];
  };
  // (places in LDS are made opaque once per slab: kept in registers from slab to slab, all of them, they spill)
  auto opaque = [](int v) __attribute__((always_inline)) { asm volatile("" : "+v"(v)); return v; };
  auto store_slab = [&]() __attribute__((always_inline)) {
    if (gact) {
      __bf16* g0 = Gt + opaque(4 * g_cg * PG + g_r * Wp + 4 * g_xg);
      floatx4 x[4];                                                 // [pixel]
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float4 d = F::f4(dv[j], 4 * g_cg);
        x[j] = (gmask >> j) & 1u ? floatx4{d.x, d.y, d.z, d.w} * lv[j] : floatx4{0.f, 0.f, 0.f, 0.f};
      }
#pragma unroll
      for (int cc = 0; cc < 4; ++cc) {
        bf16x4 y[3];
        put(g0 + cc * PG, C * PG, floatx4{x[0][cc], x[1][cc], x[2][cc], x[3][cc]}, y);
      }
    }
#pragma unroll
    for (int t = 0; t < UB; ++t) {
      if (NTH * t >= nUb) break;                                    // uniform
      if (!uact[t]) continue;
      // its last slot is the left neighbour of the eight behind it, or its first one the right neighbour of the eight before
      const bool odd = u_xg[t] & 1, edge = odd ? 4 * u_xg[t] + 4 < Wp : u_xg[t] > 0;
      const int slot = u_r[t] * Wp + 4 * u_xg[t];
      __bf16* u0 = Ut + opaque(4 * u_cg[t] * PU + slot);
      unsigned short* e0 = reinterpret_cast<unsigned short*>(Et) + opaque(2 * (4 * u_cg[t] * EP + (slot >> 3)) + (odd ? 2 : -1));
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (!((umask[t] >> j) & 1u)) uv[t][j] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int cc = 0; cc < 4; ++cc) {
        bf16x4 y[3];
        put(u0 + cc * PU, C * PU, floatx4{uv[t][0][cc], uv[t][1][cc], uv[t][2][cc], uv[t][3][cc]}, y);
        if (edge) {
#pragma unroll
          for (int q = 0; q < 3; ++q) {
            const u32x2 w = __builtin_bit_cast(u32x2, y[q]);
            e0[2 * (cc + q * C) * EP] = (unsigned short)(odd ? w[1] >> 16 : w[0]);
          }
        }
      }
    }
  };

  const int ob = NB == 1 ? 0 : wave / NB, ib = NB == 1 ? 0 : wave % NB;
  // (channels past the last repeat it: never stored)
  const __bf16* arow = Gt + min(16 * ob + bl, C - 1) * PG;
  const __bf16* brow = Ut + min(16 * ib + bl, C - 1) * PU;
  const unsigned* erow = Et + min(16 * ib + bl, C - 1) * EP;
  floatx4 acc[10], low[10];                                         // taps, and the bias (wavefronts with ib = 0)
#pragma unroll
  for (int j = 0; j < 10; ++j) acc[j] = low[j] = floatx4{0.f, 0.f, 0.f, 0.f};
  const unsigned one2 = 0x3f803f80u;
  const bf16x8 ones = __builtin_bit_cast(bf16x8, u32x4{one2, one2, one2, one2});
  const int s_begin = ch * a.gspc, s_end = min(s_begin + a.gspc, a.gslabs);
  if (s_begin < s_end) load_slab(s_begin);
  for (int sl = s_begin; sl < s_end; ++sl) {
    __syncthreads();
    store_slab();
    __syncthreads();
    if (sl + 1 < s_end) load_slab(sl + 1);
#pragma unroll 1
    for (int ks = NB == 1 ? 32 * wave : 0; ks < KL; ks += NB == 1 ? 32 * NW : 32) {
      const int s = ks + 8 * kq;                                    // the lane's first slot
      bf16x8 af[3];
#pragma unroll
      for (int q = 0; q < 3; ++q) af[q] = *reinterpret_cast<const bf16x8*>(arow + q * C * PG + s);
      constexpr int PA[5] = {2, 0, 1, 1, 0}, PB[5] = {0, 2, 1, 0, 1};   // smallest products first
#pragma unroll
      for (int dy = 0; dy < 3; ++dy) {
        bf16x8 bf[3][3];                                            // [dx][part]
#pragma unroll
        for (int q = 0; q < 3; ++q) {
          const __bf16* b = brow + q * C * PU + dy * Wp;
          const u32x4 w = *reinterpret_cast<const u32x4*>(b + s);
          const unsigned e = erow[q * C * EP + ((dy * Wp + s) >> 3)];
          const unsigned w01 = __builtin_amdgcn_alignbit(w[1], w[0], 16), w12 = __builtin_amdgcn_alignbit(w[2], w[1], 16),
                         w23 = __builtin_amdgcn_alignbit(w[3], w[2], 16);
          bf[0][q] = __builtin_bit_cast(bf16x8, u32x4{__builtin_amdgcn_perm(w[0], e, 0x05040100u), w01, w12, w23});
          bf[1][q] = __builtin_bit_cast(bf16x8, w);
          bf[2][q] = __builtin_bit_cast(bf16x8, u32x4{w01, w12, w23, __builtin_amdgcn_perm(e, w[3], 0x07060302u)});
        }
#pragma unroll
        for (int t = 0; t < 5; ++t)
#pragma unroll
          for (int dx = 0; dx < 3; ++dx)
            low[3 * dy + dx] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[PA[t]], bf[dx][PB[t]], low[3 * dy + dx], 0, 0, 0);
#pragma unroll
        for (int dx = 0; dx < 3; ++dx)
          acc[3 * dy + dx] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[0], bf[dx][0], acc[3 * dy + dx], 0, 0, 0);
      }
      if (NB == 1 || ib == 0) {
        low[9] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[2], ones, low[9], 0, 0, 0);
        low[9] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[1], ones, low[9], 0, 0, 0);
        acc[9] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[0], ones, acc[9], 0, 0, 0);
      }
    }
  }
#pragma unroll
  for (int j = 0; j < 10; ++j) acc[j] += low[j];
  __syncthreads();
  if (tid == 0) bad = 0;
  if constexpr (NB == 1) {                                          // block j's sum over the wavefronts ends in wavefront j % NW
    floatx4* red = reinterpret_cast<floatx4*>(smem_raw);            // [NW][10][64]
#pragma unroll
    for (int j = 0; j < 10; ++j) red[(wave * 10 + j) * 64 + lane] = acc[j];
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 10; ++j) {
      if (j % NW != wave) continue;                                 // uniform
      floatx4 t = red[j * 64 + lane];
#pragma unroll
      for (int w = 1; w < NW; ++w) t += red[(w * 10 + j) * 64 + lane];
      acc[j] = t;
    }
  } else {
    __syncthreads();
  }
  const bool direct = a.gchunks == 1;
  const int NC = 9 * C;
  const long long pstride = a.wsize + C;                            // a partial-sum record: dK of the layer, then db
  float* dKd = direct ? (a.dW ? a.dW + (long long)gi * a.wsize : nullptr) : a.partial + ((long long)ch * a.layers + gi) * pstride;
  float* dbd = direct ? (a.db ? a.db + (long long)gi * C : nullptr) : a.partial + ((long long)ch * a.layers + gi) * pstride + a.wsize;
  const float scale = direct ? a.hs : 1.0f;
  float top = 0.0f;
  // register v of lane (bl, kq) holds output channel 4 kq + v, input channel bl of its blocks
#pragma unroll
  for (int j = 0; j < 10; ++j) {
    if (NB == 1 ? j % NW != wave : j == 9 && ib != 0) continue;     // uniform
    const int i = 16 * ib + bl;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int o = 16 * ob + 4 * kq + v;
      top = __builtin_elementwise_maximum(top, __builtin_fabsf(acc[j][v]));
      if (o >= C) continue;
      if (j < 9) { if (i < C && dKd) dKd[(long long)o * NC + j * C + i] = scale * acc[j][v]; }
      else if (bl == 0 && dbd) dbd[o] = scale * acc[j][v];
    }
  }
  if (!(top < __builtin_inff()) || (top > 0.0f && top < 0x1p-90f)) bad = 1;
  __syncthreads();                                                  // (and the stores above before those below)
  if (!bad) return;
  // The sums from the float values: slab by slab through LDS, [pixel][channel], a thread per pair of channels (o, i) with its nine
  // taps; a slab's sums by themselves, then added to those before.
  constexpr int PAIRS = NB * NB;                                    // C C <= NTH NB NB
  float* Gf = reinterpret_cast<float*>(smem_raw);                   // [R][Wd][C]
  float* Uf = Gf + R * Wd * C;                                      // [R + 2][Wd][C]
  float tot[PAIRS][10];
#pragma unroll
  for (int p = 0; p < PAIRS; ++p)
#pragma unroll
    for (int t = 0; t < 10; ++t) tot[p][t] = 0.0f;
  for (int sl = s_begin; sl < s_end; ++sl) {
    const int b = sl / a.gspi, y0 = (sl % a.gspi) * R, rows = min(R, H - y0), RC = Wd * CG;
    const unsigned first = (unsigned)(((long long)b * H + y0) * Wd * C);
    __syncthreads();
    for (int e = tid; e < rows * RC; e += NTH) {
      const floatx4 l = *reinterpret_cast<const floatx4*>(Lp + first + 4 * e);
      const float4 d = F::f4(F::load(Dp, first + 4 * e), 4 * e);    // (a multiple of eight values before this slab)
      *reinterpret_cast<floatx4*>(Gf + 4 * e) = floatx4{d.x, d.y, d.z, d.w} * l;
    }
    for (int e = tid; e < (rows + 2) * RC; e += NTH) {
      const int y = y0 - 1 + e / RC;
      floatx4 u = floatx4{0.f, 0.f, 0.f, 0.f};
      if (y >= 0 && y < H) u = *reinterpret_cast<const floatx4*>(Up + first + 4 * e - Wd * C);
      *reinterpret_cast<floatx4*>(Uf + 4 * e) = u;
    }
    __syncthreads();
#pragma unroll
    for (int p = 0; p < PAIRS; ++p) {
      const int pair = tid + NTH * p, o = pair / C, i = pair % C;
      if (o >= C) continue;
      float sum[10] = {};
      for (int r = 0; r < rows; ++r) {
        const float* g = Gf + r * Wd * C + o;
        const float* u = Uf + r * Wd * C + i;
        float w[3][3];                                              // U around the pixel, zero outside the image
#pragma unroll
        for (int dy = 0; dy < 3; ++dy) { w[dy][1] = 0.0f; w[dy][2] = u[dy * Wd * C]; }
#pragma unroll 4
        for (int x = 0; x < Wd; ++x) {
          const float gx = g[x * C];
#pragma unroll
          for (int dy = 0; dy < 3; ++dy) {
            w[dy][0] = w[dy][1]; w[dy][1] = w[dy][2];
            w[dy][2] = x + 1 < Wd ? u[(dy * Wd + x + 1) * C] : 0.0f;
#pragma unroll
            for (int dx = 0; dx < 3; ++dx) sum[3 * dy + dx] = __builtin_fmaf(gx, w[dy][dx], sum[3 * dy + dx]);
          }
          sum[9] += gx;
        }
      }
#pragma unroll
      for (int t = 0; t < 10; ++t) tot[p][t] += sum[t];
    }
  }
#pragma unroll
  for (int p = 0; p < PAIRS; ++p) {
    const int pair = tid + NTH * p, o = pair / C, i = pair % C;
    if (o >= C) continue;
    if (dKd)
#pragma unroll
      for (int t = 0; t < 9; ++t) dKd[(long long)o * NC + t * C + i] = scale * tot[p][t];
    if (dbd && i == 0) dbd[o] = scale * tot[p][9];
  }
}

// Slab height: a thread has at most one block of G and one or two of U, and a workgroup half of a CU's LDS.  Among those the one whose
// slabs of an image take the fewest cycles: 57 matrix instructions of 16 for every 32 slots, about 500 for the blocks of a
// thread, 600 for the barriers and the loads' latency.
bool conv_grad_split_geom(int B, int Himg, int Wimg, int C, bool bits, ConvGradGeom* gm) {
  if (C > 32 || C % 8 != 0 || Wimg > 64) return false;
  const int nb = C > 16 ? 2 : 1, Wp = (Wimg + 7) & ~7, bpr = ((Wimg + 3) / 4) * (C / 4);
  double best = 0.0;
  for (int R = 1; R <= Himg; ++R) {
    const int KL = (R * Wp + 31) / 32 * 32, PU = 8 * (((2 * Wp + KL) / 8 + 1) | 1), PG = 8 * ((KL / 8) | 1);
    size_t smem = (size_t)3 * C * (PU + PG + 2 * cgs_ep(PU)) * 2;
    if (nb == 1 && smem < 4 * 10 * 64 * 16) smem = 4 * 10 * 64 * 16;        // the wavefronts' sums
    if (R * bpr > CGS_NTH || (R + 2) * bpr > cgs_ub(nb, bits) * CGS_NTH || smem > 72 * 1024) break;
    const int spi = (Himg + R - 1) / R, steps = nb == 1 ? (KL / 32 + 3) / 4 : KL / 32;
    const double cost = spi * (steps * 57.0 * 16.0 + (2 * R + 2) * bpr * 500.0 / CGS_NTH + 600.0);
    if (best != 0.0 && cost >= best) continue;
    best = cost;
    gm->Wp = Wp; gm->R = R; gm->KL = KL; gm->PU = PU; gm->PG = PG; gm->spi = spi; gm->slabs = B * spi; gm->smem = smem;
  }
  return best != 0.0;
}

template <typename DT, int NB> static hipError_t launch_split(const GradArgs& a, size_t smem, hipStream_t s) {
  static LdsOptIn opt;
  const hipError_t e = opt.raise(reinterpret_cast<const void*>(conv_grad_split_kernel<DT, NB>), smem);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((conv_grad_split_kernel<DT, NB>), dim3((unsigned)a.gchunks * (unsigned)a.layers), dim3(CGS_NTH), smem, s, a);
  return hipGetLastError();
}
hipError_t launch_conv_grad_split(const GradArgs& a, size_t smem, hipStream_t s) {
  if (a.dbits) return a.Nf > 16 ? launch_split<Bit, 2>(a, smem, s) : launch_split<Bit, 1>(a, smem, s);
  return a.Nf > 16 ? launch_split<float, 2>(a, smem, s) : launch_split<float, 1>(a, smem, s);
}

}  // namespace mgrit
