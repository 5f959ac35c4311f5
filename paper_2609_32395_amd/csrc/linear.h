// Linear maps y = x W^T (W stored [out, in], a linear layer's layout) on
// MFMA for the whole-model runtime: a few-row kernel and an LDS-tiled GEMM
// that share one reduction order, and the host dispatch between them.
// Both MFMA operands run along the reduction dimension, so a lane's 8
// k-values are 16 contiguous bytes of an x row and of a W row.
#pragma once

#include <algorithm>
#include <type_traits>

#include "common.h"
#include "linear_plan.h"

namespace smem {

typedef __bf16 bf16x8m __attribute__((ext_vector_type(8)));

enum LinEpi : int { kLinStore = 0, kLinGelu = 1, kLinResid = 2, kLinF32 = 3, kLinSplit = 4 };

struct LinArgs {
  const uint16_t* x;   // [M][ldx], K used
  const uint16_t* w;   // output rows n < n2: w + n*K
  const uint16_t* w2;  // output rows n >= n2: w2 + (n - n2)*K
  const uint16_t* res; // residual [M][ldy] (kLinResid; may equal y)
  uint16_t* y;         // [M][ldy]
  uint16_t* y1;        // kLinSplit: columns [ns, 2ns) -> y1, [2ns, 3ns) -> y2 (each [M][ns])
  uint16_t* y2;
  float* yf;           // kLinF32: [M][ldy]
  const uint16_t* lng; // y = LN(x) W^T when set: LayerNorm gain and bias [K]
  const uint16_t* lnb;
  uint16_t* lnout;     // many rows: LN(x) written here ([M][K]) before the map
  int32_t M, N, K, ldx, ldy, n2, ns;
};

// erf by Abramowitz and Stegun, Handbook of Mathematical Functions, formula
// 7.1.26: erf(x) = 1 - (a1 t + a2 t^2 + a3 t^3 + a4 t^4 + a5 t^5) exp(-x^2),
// t = 1 / (1 + p x), x >= 0, absolute error <= 1.5e-7 (odd extension for
// x < 0); far below the bf16 rounding of the activations it feeds.
__device__ __forceinline__ float erf_as(float x) {
  const float ax = fabsf(x);
  const float t = __builtin_amdgcn_rcpf(1.f + 0.3275911f * ax);
  const float poly = ((((1.061405429f * t - 1.453152027f) * t + 1.421413741f) * t - 0.284496736f) * t + 0.254829592f) * t;
  const float e = __builtin_amdgcn_exp2f(-ax * ax * 1.4426950408889634f);
  return copysignf(1.f - poly * e, x);
}

// GELU, exact (erf) form: x * Phi(x) = x/2 * (1 + erf(x / sqrt 2)).
__device__ __forceinline__ float gelu_erf(float x) { return 0.5f * x * (1.f + erf_as(x * 0.70710678118654752f)); }

// Reduction order of every linear map, whatever kernel computes it: the
// K-range is cut into chunks of lin_chunk(K) (a multiple of 256); inside a
// chunk, one 16x16x32 bf16 MFMA per 32-wide k step accumulates from zero in
// ascending k; the chunk sums are then added in ascending chunk order to a
// total that starts at zero.  Each output element therefore sees the same
// operations in the same order for any M and any tiling, which keeps a
// row's result independent of the other rows in the call (block-skip serving
// reproduces the cold pass bit for bit).

// LayerNorm of a row of width d (d % 64 == 0, d <= 2048), eps 1e-5, with the
// statistics summed in one fixed order, so the stand-alone kernel below and
// the few-row map that normalizes its own x rows give the same bits.  The row
// is cut as a linear map cuts K: chunks of 256, each of 32 pieces of 8 values
// (16 bytes).  A piece adds its values in ascending order; a chunk adds its
// pieces as a binary tree (ln_tree32; missing pieces of a short last chunk as
// zeros); the chunk totals add in ascending order from zero.  mean = total / d;
// the second moment sums (x - mean)^2 the same way; rstd = 1 / sqrt(m2 / d +
// eps), each operation correctly rounded (the hardware's reciprocal square root
// is not, and saves 0.1 to 0.25 us of a fused map's 6 to 9, within what a call
// of many of them differs by: a 64-row read of 15 reader layers takes 787 to 794
// us with the division and 783 to 800 with the instruction, 8192 rows of
// LayerNorm, q|k|v and attention 80.0 and 79.8).
__device__ __forceinline__ void ln_unpack(const u32x4& c, float (&f)[8]) { Chunk<uint16_t>::unpack(c, f); }
__device__ __forceinline__ float ln_piece(const float (&f)[8]) {
  float s = f[0];
#pragma unroll
  for (int e = 1; e < 8; ++e) s += f[e];
  return s;
}
// f becomes f - mean; returns the sum of the squares
__device__ __forceinline__ float ln_centre(float (&f)[8], float mean) {
  float s = 0.f;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    f[e] -= mean;
    s = __builtin_fmaf(f[e], f[e], s);
  }
  return s;
}
// (x - mean) already in f: f * rstd * gain + bias, packed to bf16
__device__ __forceinline__ u32x4 ln_scale(const float (&f)[8], const float (&g)[8], const float (&b)[8], float rstd) {
  uint32_t w[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const float y0 = __builtin_fmaf(f[2 * e] * rstd, g[2 * e], b[2 * e]);
    const float y1 = __builtin_fmaf(f[2 * e + 1] * rstd, g[2 * e + 1], b[2 * e + 1]);
    w[e] = (uint32_t)f32_to_bf16_bits(y0) | ((uint32_t)f32_to_bf16_bits(y1) << 16);
  }
  return u32x4{w[0], w[1], w[2], w[3]};
}
// The tree over a chunk's 32 pieces, a piece per lane of a half-wave (or per
// lane under an exclusive or of the index): partners 16, 8, 7, 3 and 1 apart
// by exclusive or, each one exchange of the lanes.  Every lane gets the total.
template <int CTRL>
__device__ __forceinline__ float dpp_of(float x) {
  return __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(x), CTRL, 0xf, 0xf, true));
}
constexpr int kXor8 = 0x128, kXor7 = 0x141, kXor3 = 0x1B, kXor1 = 0xB1;   // row_ror:8, row_half_mirror, quad_perm
__device__ __forceinline__ float add_swap16(float x, float y) {  // lanes 0-15: x of both, lanes 16-31: y of both
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float ln_tree32(float x) {
  x = add_swap16(x, x);
  x += dpp_of<kXor8>(x);
  x += dpp_of<kXor7>(x);
  x += dpp_of<kXor3>(x);
  return x + dpp_of<kXor1>(x);
}
// The same tree for R rows at once, each level handing half of the rows to
// each half of its lanes: lane s of a half-wave ends up with row (s >> 2) /
// (8 / R) (bit 4 of s the row's highest).
template <int R>
__device__ __forceinline__ float ln_tree_rows(const float (&t)[R], int s) {
  static_assert(R == 4 || R == 8, "two or three levels hand rows on");
  float u[R / 2];
#pragma unroll
  for (int i = 0; i < R / 2; ++i) u[i] = add_swap16(t[i], t[i + R / 2]);
  auto pick = [&](float x, float y, int bit) { return (s & bit) ? y : x; };
  float v[R / 4];
#pragma unroll
  for (int i = 0; i < R / 4; ++i)
    v[i] = pick(u[i] + dpp_of<kXor8>(u[i]), u[i + R / 4] + dpp_of<kXor8>(u[i + R / 4]), 8);
  float x = v[0] + dpp_of<kXor7>(v[0]);
  if constexpr (R == 8) x = pick(x, v[1] + dpp_of<kXor7>(v[1]), 4);
  x += dpp_of<kXor3>(x);
  return x + dpp_of<kXor1>(x);
}
// The tree where a lane holds pieces 4 t + g in u[t] (g = lane / 16 of an MFMA
// operand): its first two levels are between registers.
__device__ __forceinline__ float ln_tree_operand(const float (&u)[8]) {
  const float w0 = (u[0] + u[4]) + (u[2] + u[6]), w1 = (u[1] + u[5]) + (u[3] + u[7]);
  const float v = w0 + __shfl_xor(w1, 48);
  const float z = v + __shfl_xor(v, 48);
  return z + __shfl_xor(z, 16);
}
__device__ __forceinline__ float ln_rstd(float m2, int d) { return 1.f / sqrtf(m2 / d + 1e-5f); }

// Stand-alone LayerNorm (rows x[row * ldx .. + d) -> y[row * ldy ..)): one
// wave per row, a half-wave per chunk, every load and store 512 contiguous
// bytes of the row per half-wave.
__global__ void __launch_bounds__(256) k_ln_rows(const uint16_t* __restrict__ x, int ldx,
                                                 const uint16_t* __restrict__ g, const uint16_t* __restrict__ b,
                                                 uint16_t* __restrict__ y, int ldy, int rows, int d) {
  const int lane = threadIdx.x & 63, row = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= rows) return;
  const int NC = (d + 255) / 256, half = lane >> 5, k0 = half * 256 + (lane & 31) * 8;
  const uint16_t* xr = x + (size_t)row * ldx;
  float f[4][8];
  u32x4 gv[4], bv[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    u32x4 v = {0u, 0u, 0u, 0u};
    if (k0 + 512 * i < d) v = *(const u32x4*)(xr + k0 + 512 * i);
    ln_unpack(v, f[i]);
  }
#pragma unroll
  for (int i = 0; i < 4; ++i)
    if (k0 + 512 * i < d) {
      gv[i] = *(const u32x4*)(g + k0 + 512 * i);
      bv[i] = *(const u32x4*)(b + k0 + 512 * i);
    }
  auto total = [&](const float (&t)[4]) {
    float s = 0.f;
#pragma unroll
    for (int c = 0; c < 8; ++c)
      if (c < NC) s += __shfl(t[c >> 1], (c & 1) * 32);
    return s;
  };
  float t[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) t[i] = 512 * i < d ? ln_tree32(ln_piece(f[i])) : 0.f;
  const float mean = total(t) / d;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float q = ln_centre(f[i], mean);
    t[i] = 512 * i < d ? ln_tree32(k0 + 512 * i < d ? q : 0.f) : 0.f;
  }
  const float rstd = ln_rstd(total(t), d);
  uint16_t* yr = y + (size_t)row * ldy;
#pragma unroll
  for (int i = 0; i < 4; ++i)
    if (k0 + 512 * i < d) {
      float gf[8], bf[8];
      ln_unpack(gv[i], gf);
      ln_unpack(bv[i], bf);
      *(u32x4*)(yr + k0 + 512 * i) = ln_scale(f[i], gf, bf, rstd);
    }
}

inline void launch_ln(const uint16_t* x, int ldx, const uint16_t* g, const uint16_t* b, uint16_t* y, int ldy, int rows,
                      int d, hipStream_t s) {
  hipLaunchKernelGGL(k_ln_rows, dim3((rows + 3) / 4), dim3(256), 0, s, x, ldx, g, b, y, ldy, rows, d);
}

template <int EPI>
__device__ __forceinline__ void lin_store(const LinArgs& a, int m, int n, float v) {
  if constexpr (EPI == kLinF32) {
    a.yf[(size_t)m * a.ldy + n] = v;
  } else if constexpr (EPI == kLinGelu) {
    a.y[(size_t)m * a.ldy + n] = f32_to_bf16_bits(gelu_erf(v));
  } else if constexpr (EPI == kLinResid) {
    const size_t o = (size_t)m * a.ldy + n;
    a.y[o] = f32_to_bf16_bits(v + bf16_bits_to_f32(a.res[o]));
  } else if constexpr (EPI == kLinSplit) {
    const int g = n / a.ns, c = n - g * a.ns;
    uint16_t* dst = g == 0 ? a.y : (g == 1 ? a.y1 : a.y2);
    dst[(size_t)m * a.ns + c] = f32_to_bf16_bits(v);
  } else {
    a.y[(size_t)m * a.ldy + n] = f32_to_bf16_bits(v);
  }
}

// Four consecutive outputs n .. n+3 of row m (n % 4 == 0; bf16 rows have
// ldy % 4 == 0, so the four share one 8-byte word; a split's column groups
// are multiples of 4 wide).  Columns >= N are dropped.  res: the residual's
// word where it is at hand already.
template <int EPI>
__device__ __forceinline__ void lin_store4(const LinArgs& a, int m, int n, const f32x4& v, const u32x2* res = nullptr) {
  if constexpr (EPI == kLinF32) {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (n + e < a.N) a.yf[(size_t)m * a.ldy + n + e] = v[e];
  } else {
    if (n + 3 >= a.N) {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (n + e < a.N) lin_store<EPI>(a, m, n + e, v[e]);
      return;
    }
    float o[4];
    uint16_t* dst;
    if constexpr (EPI == kLinSplit) {
      const int g = n / a.ns, c = n - g * a.ns;
      dst = (g == 0 ? a.y : (g == 1 ? a.y1 : a.y2)) + (size_t)m * a.ns + c;
    } else {
      dst = a.y + (size_t)m * a.ldy + n;
    }
    if constexpr (EPI == kLinResid) {
      const u32x2 r = res ? *res : *(const u32x2*)(a.res + (size_t)m * a.ldy + n);
      o[0] = v[0] + bf16_bits_to_f32(r.x & 0xffffu);
      o[1] = v[1] + bf16_bits_to_f32(r.x >> 16);
      o[2] = v[2] + bf16_bits_to_f32(r.y & 0xffffu);
      o[3] = v[3] + bf16_bits_to_f32(r.y >> 16);
    } else if constexpr (EPI == kLinGelu) {
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = gelu_erf(v[e]);
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = v[e];
    }
    *(u32x2*)dst = u32x2{(uint32_t)f32_to_bf16_bits(o[0]) | ((uint32_t)f32_to_bf16_bits(o[1]) << 16),
                         (uint32_t)f32_to_bf16_bits(o[2]) | ((uint32_t)f32_to_bf16_bits(o[3]) << 16)};
  }
}

__device__ __forceinline__ const uint16_t* lin_wrow(const LinArgs& a, int n) {
  return n < a.n2 ? a.w + (size_t)n * a.K : a.w2 + (size_t)(n - a.n2) * a.K;
}

// One 16x16x32 step with the W tile as the MFMA's row operand and the x
// tile as its column operand: lane l then holds outputs (x row l % 16,
// W rows 4 (l / 16) .. +3), four consecutive output columns of one row.
__device__ __forceinline__ f32x4 mfma16(const u32x4& A, const u32x4& B, const f32x4& c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8m, A), __builtin_bit_cast(bf16x8m, B), c,
                                                 0, 0, 0);
}

// Few rows (one or two blocks, or a batch of decoded tokens): a workgroup
// owns 16 rows and 16 G columns, and its waves take the reduction chunks side
// by side, so the loads of the whole tile are in flight at once.  An MFMA
// operand asks for 64 bytes of each of 16 rows; loaded like that from memory,
// every instruction touches 16 lines by halves, and the time went into those
// requests (16 rows x 4096 from L2 by 256 workgroups: 3.0 us against 0.65 for
// 512 contiguous bytes per half-wave).  So a wave loads its 256-wide piece of
// a 16-row tile as 8 instructions of two 512-byte rows, and passes it through
// 8 KB of LDS of its own (no barrier) to turn it into the operand.  The
// residual is asked for with the first loads.  Weights out of the caches, us
// per call at 64 rows, before (fragments straight from memory) and now:
// 1024 -> 1024 + residual 5.0 -> 3.7 (1.7 of it the launch), 4096 -> 1024 11.3
// -> 7.2, 8192 -> 2048 27.6 -> 16.7; with the LayerNorm 1024 -> 1024 6.6 ->
// 5.2, 1024 -> 3072 10.5 -> 8.1, 1024 -> 4096 + GELU 10.8 -> 8.2 (2.6 us of it
// waits for the weights, 0.9 the statistics).

// The 8 instructions of a 16-row piece: rows row(2 i + lane / 32), chunk
// lane % 32 of the nt * 4 valid ones from column k (a short last piece
// re-reads its first chunk; its products are not formed).
template <class Row>
__device__ __forceinline__ void few_load(u32x4 (&v)[8], int lane, int k, int nt, Row row) {
  const int s = lane & 31, q = s < 4 * nt ? s : 0;
#pragma unroll
  for (int i = 0; i < 8; ++i) v[i] = *(const u32x4*)(row(2 * i + (lane >> 5)) + k + q * 8);
}
__device__ __forceinline__ void few_put(uint8_t* tile, const u32x4 (&v)[8], int lane) {
#pragma unroll
  for (int i = 0; i < 8; ++i) *(u32x4*)(tile + FewTile::put(2 * i + (lane >> 5), lane & 31)) = v[i];
}
__device__ __forceinline__ void few_get(u32x4 (&o)[8], const uint8_t* tile, int lane) {
#pragma unroll
  for (int t = 0; t < 8; ++t) o[t] = *(const u32x4*)(tile + FewTile::get(lane, t));
}
// LDS operations of one wave run in order; this keeps the compiler to it.
__device__ __forceinline__ void wave_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
__device__ __forceinline__ void few_turn(u32x4 (&o)[8], uint8_t* tile, const u32x4 (&v)[8], int lane) {
  wave_order();
  few_put(tile, v, lane);
  wave_order();
  few_get(o, tile, lane);
}
// The steps that a short last piece does not have become zero operands.
__device__ __forceinline__ void few_clip(u32x4 (&o)[8], int nt) {
  if (nt == 8) return;
#pragma unroll
  for (int t = 1; t < 8; ++t)
    if (t >= nt) o[t] = u32x4{0u, 0u, 0u, 0u};
}
__device__ __forceinline__ void few_mfma(f32x4& acc, const u32x4 (&B)[8], const u32x4 (&A)[8]) {
#pragma unroll
  for (int t = 0; t < 8; ++t) acc = mfma16(B[t], A[t], acc);
}

// The residual of the thread's first four outputs, asked for at the start.
template <int EPI, int RT, int G>
__device__ __forceinline__ u32x2 few_res(const LinArgs& a, int m0, int n0) {
  if constexpr (EPI == kLinResid) {
    const int q = threadIdx.x, m = m0 + q / (4 * G), n = n0 + (q % (4 * G)) * 4;
    if (q < 64 * RT * G && m < a.M && n < a.N) return *(const u32x2*)(a.res + (size_t)m * a.ldy + n);
  }
  return u32x2{0u, 0u};
}
// The chunk sums in LDS ([n_chunks][16 RT][16 G]) added in chunk order, stored;
// res: few_res's word (not AHEAD: loaded here instead).
template <int EPI, int RT, int G, bool AHEAD = true>
__device__ __forceinline__ void few_finish(const LinArgs& a, const float* part, int NC, int m0, int n0,
                                           const u32x2& res) {
  for (int q = threadIdx.x; q < 64 * RT * G; q += blockDim.x) {
    const int row = q / (4 * G), c0 = (q % (4 * G)) * 4;
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
    for (int c4 = 0; c4 < NC; c4 += 4) {
      f32x4 p[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) p[e] = *(const f32x4*)(part + (min(c4 + e, NC - 1) * 16 * RT + row) * 16 * G + c0);
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (c4 + e < NC) v += p[e];
    }
    const int m = m0 + row;
    if (m < a.M) lin_store4<EPI>(a, m, n0 + c0, v, AHEAD && q < (int)blockDim.x ? &res : nullptr);
  }
}
// A lane's sums of tile (row tile i, column tile j) of chunk c.
template <int RT, int G>
__device__ __forceinline__ void few_part(float* part, int c, int i, int j, const f32x4& acc, int lane) {
  *(f32x4*)(part + ((c * RT + i) * 16 + (lane & 15)) * 16 * G + j * 16 + 4 * (lane >> 4)) = acc;
}

// RT row tiles by G column tiles.  LOOP: a wave takes the 8-step pieces of
// chunks w, w + nw, .. (each chunk's in order), the next piece's loads issued
// as soon as the registers are free; else one piece each.
// Dynamic LDS: a tile of 8 KB per wave, then n_chunks x RT x G KB of chunk sums.
template <int EPI, int RT, int G, int NW, bool LOOP>
__global__ void __launch_bounds__(64 * NW) k_linear_few(LinArgs a, int row_tiles, int col_groups) {
  extern __shared__ __attribute__((aligned(16))) uint8_t few_lds[];
  const int pid = xcd_order(blockIdx.x, row_tiles * col_groups);
  if (pid < 0) return;
  const int m0 = (pid % row_tiles) * 16 * RT, n0 = (pid / row_tiles) * 16 * G;
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nw = blockDim.x >> 6, KS = a.K / 32, CS = lin_chunk(a.K) / 32, NC = (KS + CS - 1) / CS;
  uint8_t* tile = few_lds + w * FewTile::BYTES;
  float* part = (float*)(few_lds + nw * FewTile::BYTES);
  auto xrow = [&](int r) { return a.x + (size_t)min(m0 + r, a.M - 1) * a.ldx; };
  auto wrow = [&](int r) { return lin_wrow(a, min(n0 + r, a.N - 1)); };
  auto load_x = [&](u32x4 (&v)[8], int i, int st, int nt) {
    few_load(v, lane, st * 32, nt, [&](int r) { return xrow(i * 16 + r); });
  };
  auto load_w = [&](u32x4 (&v)[8], int j, int st, int nt) {
    few_load(v, lane, st * 32, nt, [&](int r) { return wrow(j * 16 + r); });
  };
  const u32x2 res = few_res<EPI, RT, G>(a, m0, n0);
  u32x4 X[RT][8], W[G][8];
  int c = w, st = c * CS;
  auto steps = [&](int s0, int ch) { return min(8, min(KS, (ch + 1) * CS) - s0); };
  if (c < NC) {
    const int nt = steps(st, c);
#pragma unroll
    for (int i = 0; i < RT; ++i) load_x(X[i], i, st, nt);
#pragma unroll
    for (int j = 0; j < G; ++j) load_w(W[j], j, st, nt);
  }
  f32x4 acc[RT][G];
#pragma unroll
  for (int i = 0; i < RT; ++i)
#pragma unroll
    for (int j = 0; j < G; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  while (c < NC) {                       // (once, unless LOOP)
    const int nt = steps(st, c);
    int c2 = c, st2 = st + 8;            // the next piece
    if (st2 >= min(KS, (c + 1) * CS)) {
      c2 = c + nw;
      st2 = c2 * CS;
    }
    const bool more = LOOP && c2 < NC;
    const int nt2 = more ? steps(st2, c2) : 1;
    u32x4 A[RT][8], B[8];
#pragma unroll
    for (int i = 0; i < RT; ++i) {
      few_turn(A[i], tile, X[i], lane);
      if (more) load_x(X[i], i, st2, nt2);
    }
#pragma unroll
    for (int j = 0; j < G; ++j) {
      few_turn(B, tile, W[j], lane);
      if (more) load_w(W[j], j, st2, nt2);
#pragma unroll
      for (int t = 0; t < 8; ++t)
        if (t < nt) {
#pragma unroll
          for (int i = 0; i < RT; ++i) acc[i][j] = mfma16(B[t], A[i][t], acc[i][j]);
        }
    }
    if (!LOOP || c2 != c) {
#pragma unroll
      for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int j = 0; j < G; ++j) {
          few_part<RT, G>(part, c, i, j, acc[i][j], lane);
          acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
    }
    c = LOOP ? c2 : NC;
    st = st2;
  }
  __syncthreads();
  few_finish<EPI, RT, G>(a, part, NC, m0, n0, res);
}

// The same with the LayerNorm fused (y = LN(x) W^T, K <= 2048, so every chunk
// is 256 wide): WPC waves per chunk, each loading and normalizing 16 / WPC of
// the rows and computing G / WPC of the column tiles; the chunk totals of the
// row statistics meet in LDS in the stand-alone kernel's order, and the
// normalized rows go into the chunk's tile.  A lane holds the same 8 columns
// of all its rows, so it unpacks the gain and the bias once, and each value
// once.  The weights, issued first, are in flight meanwhile.  The sums are
// those of k_linear_few on LN(x) rows: bitwise the unfused pair's.
// Dynamic LDS: n_chunks x WPC tiles, two planes [8][16] of statistics,
// then n_chunks x G KB of chunk sums.
template <int EPI, int G, int WPC>
__global__ void __launch_bounds__(512) k_linear_few_ln(LinArgs a, int row_tiles, int col_groups) {
  constexpr int GW = G / WPC, RI = 8 / WPC;              // column tiles, row pairs per wave
  extern __shared__ __attribute__((aligned(16))) uint8_t few_lds[];
  const int pid = xcd_order(blockIdx.x, row_tiles * col_groups);
  if (pid < 0) return;
  const int m0 = (pid % row_tiles) * 16, n0 = (pid / row_tiles) * 16 * G;
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c = w / WPC, h = w % WPC, half = lane >> 5, s = lane & 31;
  const int KS = a.K / 32, NC = (KS + 7) / 8, nt = min(8, KS - 8 * c), k0 = c * 256;
  uint8_t* xt = few_lds + c * WPC * FewTile::BYTES;      // the chunk's normalized rows
  uint8_t* tile = few_lds + w * FewTile::BYTES;          // this wave's (h = 0: the rows' own, once they are read)
  float* st0 = (float*)(few_lds + NC * WPC * FewTile::BYTES);
  float* st1 = st0 + 128;
  float* part = st1 + 128;
  constexpr bool AHEAD = GW < 4;                         // four tiles of weights leave no registers for it
  u32x2 res = {0u, 0u};
  if constexpr (AHEAD) res = few_res<EPI, 1, G>(a, m0, n0);
  const bool in = s < 4 * nt;
  const int q = in ? s : 0;
  u32x4 X[RI], W[GW][8], g16, b16;
#pragma unroll
  for (int i = 0; i < RI; ++i)
    X[i] = *(const u32x4*)(a.x + (size_t)min(m0 + h * 2 * RI + 2 * i + half, a.M - 1) * a.ldx + k0 + q * 8);
  g16 = *(const u32x4*)(a.lng + k0 + q * 8);
  b16 = *(const u32x4*)(a.lnb + k0 + q * 8);
  __builtin_amdgcn_sched_barrier(0);     // the rows, gain and bias are waited for without the weights
#pragma unroll
  for (int j = 0; j < GW; ++j)
    few_load(W[j], lane, k0, nt, [&](int r) { return lin_wrow(a, min(n0 + (h * GW + j) * 16 + r, a.N - 1)); });
  if (NC < 8)
    for (int e = NC * 16 + threadIdx.x; e < 128; e += blockDim.x) st0[e] = st1[e] = 0.f;
  // the row whose total the tree leaves in this lane (4 / (8 / RI) lanes hold it)
  const int tr = h * 2 * RI + 2 * ((s >> 2) / (8 / RI)) + half;
  float f[RI][8], z[RI];
#pragma unroll
  for (int i = 0; i < RI; ++i) {
    ln_unpack(X[i], f[i]);
    z[i] = in ? ln_piece(f[i]) : 0.f;
  }
  const float t0 = ln_tree_rows<RI>(z, s);
  if ((s & 3) == 0) st0[c * 16 + tr] = t0;
  // lane r finishes row r % 16 for the whole wave; its result is then fetched
  // (chunks past the last are zeros)
  auto total = [&](const float* st) {
    float t = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) t += st[e * 16 + (lane & 15)];
    return t;
  };
  auto fetch = [&](float (&o)[RI], float v) {
#pragma unroll
    for (int i = 0; i < RI; ++i) o[i] = __shfl(v, h * 2 * RI + 2 * i + half);
  };
  float rv[RI];
  __syncthreads();
  fetch(rv, total(st0) / a.K);
#pragma unroll
  for (int i = 0; i < RI; ++i) {
    const float q2 = ln_centre(f[i], rv[i]);
    z[i] = in ? q2 : 0.f;
  }
  const float t1 = ln_tree_rows<RI>(z, s);
  if ((s & 3) == 0) st1[c * 16 + tr] = t1;
  __syncthreads();
  fetch(rv, ln_rstd(total(st1), a.K));
  float gf[8], bf[8];
  ln_unpack(g16, gf);
  ln_unpack(b16, bf);
#pragma unroll
  for (int i = 0; i < RI; ++i)
    *(u32x4*)(xt + FewTile::put(h * 2 * RI + 2 * i + half, s)) = ln_scale(f[i], gf, bf, rv[i]);
  if constexpr (WPC > 1) __syncthreads();
  else wave_order();
  u32x4 A[8], B[2][8];
  few_get(A, xt, lane);
  few_clip(A, nt);
  if constexpr (WPC > 1) __syncthreads();                // the rows are read; h = 0 reuses their tile
  f32x4 acc[GW];
  few_turn(B[0], tile, W[0], lane);
#pragma unroll
  for (int j = 0; j < GW; ++j) {
    acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (j + 1 < GW) few_turn(B[(j + 1) & 1], tile, W[j + 1], lane);
    few_clip(B[j & 1], nt);
    few_mfma(acc[j], B[j & 1], A);
  }
#pragma unroll
  for (int j = 0; j < GW; ++j) few_part<1, G>(part, c, 0, h * GW + j, acc[j], lane);
  __syncthreads();
  few_finish<EPI, 1, G, AHEAD>(a, part, NC, m0, n0, res);
}

// An empty asm that claims to rewrite the packed x rows, so the compiler
// unpacks them again where they are next used instead of keeping 8 floats
// per register live across the statistics barriers.
template <int T, int R>
__device__ __forceinline__ void opaque(u32x4 (&X)[T][R]) {
#pragma unroll
  for (int t = 0; t < T; ++t)
#pragma unroll
    for (int i = 0; i < R; ++i) asm volatile("" : "+v"(X[t][i]));
}

// The same for wide rows (K > 1024) and many columns, and for rows of at most
// 128 values: RT x 16 rows and G x 16 columns per workgroup, one wave per chunk,
// x and W loaded as MFMA fragments (a lane of step t holds piece 4 t + l / 16 of
// its row, so the statistics' tree is partly between registers), U steps of W in
// flight.
// Dynamic LDS: gain and bias (4 K bytes) and two statistics planes of
// n_chunks x 16 RT floats, then, in the same space, n_chunks x RT x G KiB of
// partial sums.
template <int EPI, int RT, int G, int U>
__global__ void __launch_bounds__(512) k_linear_skinny_ln(LinArgs a, int row_tiles, int col_groups) {
  constexpr int W16 = 16 * G;
  extern __shared__ float part[];   // [n_chunks][16 RT][16 G]
  const int pid = xcd_order(blockIdx.x, row_tiles * col_groups);
  if (pid < 0) return;
  const int m0 = (pid % row_tiles) * 16 * RT, n0 = (pid / row_tiles) * W16;
  const int lane = threadIdx.x & 63;
  const int c = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // wave c computes chunk c
  const int kofs = (lane >> 4) * 8;
  const int KS = a.K / 32, NC = (KS + 7) / 8;
  uint16_t* gb = (uint16_t*)part;                                // gain [K], bias [K] (until the MFMAs)
  float* st0 = (float*)(gb + 2 * a.K);                           // [n_chunks][16 RT] sums, then second moments
  float* st1 = st0 + NC * 16 * RT;
  const int s0 = c * 8, ns = min(8, KS - s0);
  const uint16_t* ap[RT];
  const uint16_t* bp[G];
#pragma unroll
  for (int i = 0; i < RT; ++i) ap[i] = a.x + (size_t)min(m0 + i * 16 + (lane & 15), a.M - 1) * a.ldx + kofs;
#pragma unroll
  for (int j = 0; j < G; ++j) bp[j] = lin_wrow(a, min(n0 + j * 16 + (lane & 15), a.N - 1)) + kofs;
  u32x4 X[8][RT], B[U][G];
#pragma unroll
  for (int t = 0; t < 8; ++t)
#pragma unroll
    for (int i = 0; i < RT; ++i) X[t][i] = *(const u32x4*)(ap[i] + (s0 + min(t, ns - 1)) * 32);
  const int q8 = threadIdx.x * 8;
  u32x4 g16 = {0, 0, 0, 0}, b16 = {0, 0, 0, 0};
  if (q8 < a.K) {
    g16 = *(const u32x4*)(a.lng + q8);
    b16 = *(const u32x4*)(a.lnb + q8);
  }
#pragma unroll
  for (int t = 0; t < U; ++t)
#pragma unroll
    for (int j = 0; j < G; ++j) B[t][j] = *(const u32x4*)(bp[j] + (s0 + min(t, ns - 1)) * 32);
  if (q8 < a.K) {
    *(u32x4*)(gb + q8) = g16;
    *(u32x4*)(gb + a.K + q8) = b16;
  }
  float mean[RT], rstd[RT];
#pragma unroll
  for (int i = 0; i < RT; ++i) {
    float u[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      float f[8];
      ln_unpack(X[t][i], f);
      u[t] = t < ns ? ln_piece(f) : 0.f;
    }
    const float v = ln_tree_operand(u);
    if (lane < 16) st0[c * 16 * RT + i * 16 + lane] = v;
  }
  opaque(X);
  __syncthreads();
#pragma unroll
  for (int i = 0; i < RT; ++i) {
    float tot = 0.f;
    for (int q = 0; q < NC; ++q) tot += st0[q * 16 * RT + i * 16 + (lane & 15)];
    mean[i] = tot / a.K;
    float u[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      float f[8];
      ln_unpack(X[t][i], f);
      const float q = ln_centre(f, mean[i]);
      u[t] = t < ns ? q : 0.f;
    }
    const float v = ln_tree_operand(u);
    if (lane < 16) st1[c * 16 * RT + i * 16 + lane] = v;
  }
  opaque(X);
  __syncthreads();
#pragma unroll
  for (int i = 0; i < RT; ++i) {
    float tot = 0.f;
    for (int q = 0; q < NC; ++q) tot += st1[q * 16 * RT + i * 16 + (lane & 15)];
    rstd[i] = ln_rstd(tot, a.K);
  }
#pragma unroll
  for (int t = 0; t < 8; ++t) {
    const int k = (s0 + min(t, ns - 1)) * 32 + kofs;
    float gf[8], bf[8];
    ln_unpack(*(const u32x4*)(gb + k), gf);
    ln_unpack(*(const u32x4*)(gb + a.K + k), bf);
#pragma unroll
    for (int i = 0; i < RT; ++i) {
      float f[8];
      ln_unpack(X[t][i], f);
      ln_centre(f, mean[i]);
      X[t][i] = ln_scale(f, gf, bf, rstd[i]);
    }
  }
  __syncthreads();                       // gain, bias and statistics are read; part may be written
  f32x4 acc[RT][G];
#pragma unroll
  for (int i = 0; i < RT; ++i)
#pragma unroll
    for (int j = 0; j < G; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int t = 0; t < 8; ++t) {
    if (t < ns) {
#pragma unroll
      for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int j = 0; j < G; ++j) acc[i][j] = mfma16(B[t % U][j], X[t][i], acc[i][j]);
    }
    if (t + U < 8) {                     // refill this step's W registers with step t + U
#pragma unroll
      for (int j = 0; j < G; ++j) B[t % U][j] = *(const u32x4*)(bp[j] + (s0 + min(t + U, ns - 1)) * 32);
    }
  }
  float* pc = part + c * (256 * RT * G);
#pragma unroll
  for (int i = 0; i < RT; ++i)
#pragma unroll
    for (int j = 0; j < G; ++j)
      *(f32x4*)(pc + (i * 16 + (lane & 15)) * W16 + j * 16 + 4 * (lane >> 4)) = acc[i][j];
  __syncthreads();
  for (int q = threadIdx.x; q < 64 * RT * G; q += blockDim.x) {
    const int row = q / (4 * G), c0 = (q % (4 * G)) * 4;
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
    for (int ch = 0; ch < NC; ++ch) v += *(const f32x4*)(part + ch * (256 * RT * G) + row * W16 + c0);
    const int m = m0 + row;
    if (m < a.M) lin_store4<EPI>(a, m, n0 + c0, v);
  }
}

template <int EPI, FewKind KIND>
static void launch_few_as(const LinArgs& a, hipStream_t s) {
  constexpr FewPlan p = kFewPlans[KIND];
  const int rt = ceil_div(a.M, 16 * p.rt), cg = ceil_div(a.N, 16 * p.g);
  hipLaunchKernelGGL((k_linear_few<EPI, p.rt, p.g, p.nw, p.loop>), dim3(xcd_grid(rt * cg)),
                     dim3(64 * few_waves(p, a.K)), few_lds_bytes(p, a.K), s, a, rt, cg);
}
template <int EPI>
static void launch_few(const LinArgs& a, hipStream_t s) {
  switch (few_kind(a.M, a.N, a.K)) {
    case kFew1x1: launch_few_as<EPI, kFew1x1>(a, s); break;
    case kFew2x2: launch_few_as<EPI, kFew2x2>(a, s); break;
    case kFew2x4: launch_few_as<EPI, kFew2x4>(a, s); break;
    case kFewDeep1x1: launch_few_as<EPI, kFewDeep1x1>(a, s); break;
    case kFewDeep2x1: launch_few_as<EPI, kFewDeep2x1>(a, s); break;
    case kFewLong1x1: launch_few_as<EPI, kFewLong1x1>(a, s); break;
    case kFewLong1x2: launch_few_as<EPI, kFewLong1x2>(a, s); break;
  }
}

template <int EPI, FewLnKind KIND>
static void launch_few_ln_as(const LinArgs& a, hipStream_t s) {
  constexpr FewLnPlan p = kFewLnPlans[KIND];
  const int rt = ceil_div(a.M, 16 * p.rt), cg = ceil_div(a.N, 16 * p.g);
  const dim3 grid(xcd_grid(rt * cg)), block(few_ln_threads(p, a.K));
  if constexpr (p.wpc > 0)
    hipLaunchKernelGGL((k_linear_few_ln<EPI, p.g, p.wpc>), grid, block, few_ln_lds_bytes(p, a.K), s, a, rt, cg);
  else
    hipLaunchKernelGGL((k_linear_skinny_ln<EPI, p.rt, p.g, p.u>), grid, block, few_ln_lds_bytes(p, a.K), s, a, rt, cg);
}
template <int EPI>
static void launch_few_ln(const LinArgs& a, hipStream_t s) {
  switch (few_ln_kind(a.M, a.N, a.K)) {
    case kLn1x1: launch_few_ln_as<EPI, kLn1x1>(a, s); break;
    case kLn1x2: launch_few_ln_as<EPI, kLn1x2>(a, s); break;
    case kLn1x4: launch_few_ln_as<EPI, kLn1x4>(a, s); break;
    case kLn1x2Two: launch_few_ln_as<EPI, kLn1x2Two>(a, s); break;
    case kLn1x4Two: launch_few_ln_as<EPI, kLn1x4Two>(a, s); break;
    case kLnFrag1x1: launch_few_ln_as<EPI, kLnFrag1x1>(a, s); break;
    case kLnFrag1x2: launch_few_ln_as<EPI, kLnFrag1x2>(a, s); break;
    case kLnFrag2x4: launch_few_ln_as<EPI, kLnFrag2x4>(a, s); break;
  }
}

// Many rows: BM x BN tiles, WAVES_M x WAVES_N waves (each (BM/WAVES_M) x
// (BN/WAVES_N) as 16x16 MFMA tiles), K in BK-wide stages moved global -> LDS
// by DMA through a ring of NS stages, so no register holds an operand in
// transit and NS - 1 stages are in flight during each stage's MFMAs.  An LDS
// row is BK bf16 = BK/8 chunks of 16 B; chunk c of row r sits at slot
// c ^ swz(r), so the 16 rows one MFMA operand read touches cover every bank
// once.  Tiles are visited in groups of 8 row tiles, and consecutive groups
// of the launch order land on one XCD, so the A and W tiles a group shares
// stay in that XCD's L2.  Two operand register sets: the fragments of the
// next 32-wide step are read from LDS under the current step's MFMAs, and the
// stage's one barrier sits between its two steps, with a step's products
// ready to run behind it.  A chunk's first products start from a zero operand
// and its sums join the totals under the last step's MFMAs.  (A ring of two
// stages waits for a stage where it is first read and keeps one operand set:
// fetched ahead, operands have to land half a stage earlier.  us with and
// without, 128 x 128 tiles: 8192 x 2304 x 768 45.8 and 43.1, 1536 x 8192 x 1024
// 34.6 and 33.6, 1024 x 1024 x 4096 49.9 and 44.4.)  Where one workgroup fills
// a CU, it takes tile after tile, and the next tile's first stages are fetched
// while the last one's outputs are formed and stored.
// Measured, us (before: 128 x 128 tiles of 4 waves, one operand set): 8192 x
// 2048 x 8192 with the residual 285 -> 250 (1100 TFLOP/s), 8192 x 8192 x 2048
// with GELU 321 -> 299, 8192 x 4096 x 1024 with GELU 90 -> 85, 8192 x 3072 x
// 1024 64 -> 61, 4096 x 1024 x 1024 18.8 -> 14.6.
template <int N>
__device__ __forceinline__ void wait_stages(int ahead) {
  if (ahead >= 3) wait_vm<3 * N < 63 ? 3 * N : 63>();
  else if (ahead == 2) wait_vm<2 * N>();
  else if (ahead == 1) wait_vm<N>();
  else wait_vm<0>();
}

template <int EPI, class C>
__global__ void __launch_bounds__(C::NT, 2) k_gemm(LinArgs a, int tiles_m, int tiles_n) {
  constexpr int BM = C::BM, BN = C::BN, BK = C::BK, NS = C::NS, WM = C::WM, WN = C::WN;
  constexpr int TM = C::TM, TN = C::TN, IA = C::IA, IB = C::IB, STAGE = C::STAGE, KSS = BK / 32;
  static_assert(KSS % 2 == 0, "the next stage's first step goes to operand set 0");
  __shared__ __attribute__((aligned(1024))) uint16_t lds[NS * STAGE];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm = wave % (BM / WM), wn = wave / (BM / WM);
  const int KT = a.K / BK, CT = lin_chunk(a.K) / BK;
  const uint16_t* ga[IA];
  const uint16_t* gb[IB];
  int m0 = 0, n0 = 0;
  auto place = [&](int i) {              // false: no tile at order index i
    const GemmPlace p = gemm_place(i, tiles_m, tiles_n);
    if (!p.ok) return false;
    m0 = p.tm * BM;
    n0 = p.tn * BN;
#pragma unroll
    for (int i = 0; i < IA; ++i) {
      const int r = (wave * IA + i) * C::RPI + lane / C::CPR, c = (lane % C::CPR) ^ C::swz(r);
      ga[i] = a.x + (size_t)min(m0 + r, a.M - 1) * a.ldx + c * 8;
    }
#pragma unroll
    for (int i = 0; i < IB; ++i) {
      const int r = (wave * IB + i) * C::RPI + lane / C::CPR, c = (lane % C::CPR) ^ C::swz(r);
      gb[i] = lin_wrow(a, min(n0 + r, a.N - 1)) + c * 8;
    }
    return true;
  };
  int order = blockIdx.x;
  if (!place(order)) return;
  const uint32_t lbase = (uint32_t)(uintptr_t)lds;
  // the ring's stages in LDS bytes: the one read next, the one filled next
  uint32_t rd = 0, wr = 0;
  auto turn = [](uint32_t x) { return x + STAGE * 2 == NS * STAGE * 2 ? 0u : x + STAGE * 2; };
  auto issue = [&]() {                   // the next stage of K
    const uint32_t sb = lbase + wr;
#pragma unroll
    for (int i = 0; i < IA; ++i) {
      dma16(ga[i], __builtin_amdgcn_readfirstlane(sb + (wave * IA + i) * 1024));
      ga[i] += BK;
    }
#pragma unroll
    for (int i = 0; i < IB; ++i) {
      dma16(gb[i], __builtin_amdgcn_readfirstlane(sb + BM * BK * 2 + (wave * IB + i) * 1024));
      gb[i] += BK;
    }
    wr = turn(wr);
  };
  f32x4 acc[TM][TN], tot[TM][TN];
  // operand registers, two sets: one 32-wide step's fragments are read from
  // LDS while the other's MFMAs run
  u32x4 A[2][TM], B[2][TN];
  // A tile's operand rows are 16 apart, which leaves their swizzle alone (swz
  // has period 16), and the second step's slots are the first's with bit 2
  // flipped: one LDS address per operand and step, the tiles at fixed offsets.
  static_assert(C::swz(16) == 0 && C::CPR == 8, "operand addresses");
  const int la = (wm * WM + (lane & 15)) * BK, lb = BM * BK + (wn * WN + (lane & 15)) * BK;
  const int sl = ((lane >> 4) ^ C::swz(lane & 15)) << 3;
  auto read = [&](int set, int ks) {
    const uint16_t* st = lds + rd / 2 + (sl ^ (ks << 5));
#pragma unroll
    for (int j = 0; j < TN; ++j) B[set][j] = *(const u32x4*)(st + lb + j * 16 * BK);
#pragma unroll
    for (int i = 0; i < TM; ++i) A[set][i] = *(const u32x4*)(st + la + i * 16 * BK);
  };
  // One stage of a chunk.  FIRST: its first step starts the chunk's sums from
  // zero; LAST: its last step adds them to the totals, each row of tiles
  // behind the next row's MFMAs.
  auto stage = [&](auto first, auto last, int kt) {
    constexpr bool FIRST = decltype(first)::value, LAST = decltype(last)::value;
    if (kt + NS - 1 < KT) issue();
#pragma unroll
    for (int ks = 0; ks < KSS; ++ks) {
      if (ks + 1 < KSS) {
        read((ks + 1) & 1, ks + 1);
      } else {
        // stage kt + 1 has landed for every wave, and every wave has read
        // stage kt (behind the last stage this reads a stale one, unused)
        wait_stages<IA + IB>(min(NS - 2, KT - 2 - kt));
        lds_barrier();
        rd = turn(rd);
        read((ks + 1) & 1, 0);
      }
#pragma unroll
      for (int i = 0; i < TM; ++i) {
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[i][j] = mfma16(B[ks & 1][j], A[ks & 1][i], FIRST && ks == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : acc[i][j]);
        if (LAST && ks + 1 == KSS && i > 0) {
#pragma unroll
          for (int j = 0; j < TN; ++j) tot[i - 1][j] += acc[i - 1][j];
        }
      }
      if (LAST && ks + 1 == KSS) {
#pragma unroll
        for (int j = 0; j < TN; ++j) tot[TM - 1][j] += acc[TM - 1][j];
      }
    }
  };
  auto fill = [&]() {                    // the ring's first stages of a tile
    for (int p = 0; p < NS - 1 && p < KT; ++p) issue();
  };
  constexpr std::true_type yes{};
  constexpr std::false_type no{};
  fill();
  for (bool more = true; more;) {
    wait_stages<IA + IB>(min(NS - 2, KT - 1));
    lds_barrier();
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) tot[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    int kt = 0;
    if constexpr (C::PLAIN) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
      for (; kt < KT; ++kt) {
        if (kt > 0) {
          wait_stages<IA + IB>(min(NS - 2, KT - 1 - kt));
          lds_barrier();                 // stage kt is in LDS; every wave is done with stage kt - 1
        }
        if (kt + NS - 1 < KT) issue();
#pragma unroll
        for (int ks = 0; ks < KSS; ++ks) {
          read(0, ks);
#pragma unroll
          for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) acc[i][j] = mfma16(B[0][j], A[0][i], acc[i][j]);
        }
        rd = turn(rd);
        if ((kt + 1) % CT == 0 || kt + 1 == KT) {
#pragma unroll
          for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) {
              tot[i][j] += acc[i][j];
              acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
            }
        }
      }
    } else {
      read(0, 0);
      for (const int full = KT - KT % CT; kt < full;) {
        stage(yes, no, kt);
        for (int e = kt + CT - 1; ++kt < e;) stage(no, no, kt);
        stage(no, yes, kt++);
      }
      if (kt < KT) {                     // a last, shorter chunk
        stage(yes, no, kt);
        while (++kt < KT) stage(no, no, kt);
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j) tot[i][j] += acc[i][j];
      }
    }
    // The next tile's first stages are fetched while this one is stored (the
    // last stage's barrier left the ring free).
    const int sm = m0, sn = n0;
    more = C::PER_CU == 1 && place(order += gridDim.x);
    if (more) {
      wr = rd;
      fill();
    }
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int m = sm + wm * WM + i * 16 + (lane & 15);
      if (m < a.M) {
#pragma unroll
        for (int j = 0; j < TN; ++j) lin_store4<EPI>(a, m, sn + wn * WN + j * 16 + 4 * (lane >> 4), tot[i][j]);
      }
    }
  }
}

// Few rows by a very wide map (the output head: tens of thousands of
// columns): the x rows (at most 64 when K <= 1024, 32 at K = 2048) are
// loaded into LDS once per workgroup and stay there, and each wave computes
// two 16-column tiles side by side, streaming their weights a reduction
// chunk (8 steps) at a time with the next chunk's loads (16 KB) issued
// before the current chunk's MFMAs; each x fragment read from LDS feeds both
// tiles.  The weights are read from HBM once and x once per workgroup, where
// the few-row kernel re-reads x once per column group.  A wave sums every
// chunk of its tiles itself -- one MFMA per 32-wide step from zero inside a
// chunk, the chunk sums added in chunk order -- the reduction order of every
// linear map.  LDS rows are padded by 16 bytes so the 16 rows one operand
// read touches start on different banks.
template <int NCH, int RT>
__global__ void __launch_bounds__(512) k_linear_wide(LinArgs a, int n_tiles) {
  constexpr int K = 256 * NCH, XP = K + 8;
  __shared__ __attribute__((aligned(16))) uint16_t xs[RT * 16 * XP];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  for (int q = tid; q < RT * 16 * (K / 8); q += 512) {
    const int r = q / (K / 8), c8 = q % (K / 8);
    u32x4 v = {0u, 0u, 0u, 0u};
    if (r < a.M) v = *(const u32x4*)(a.x + (size_t)r * a.ldx + c8 * 8);
    *(u32x4*)(xs + r * XP + c8 * 8) = v;     // rows M .. 16 RT - 1 are zero
  }
  __syncthreads();                           // the only barrier
  const int t0 = (blockIdx.x * 8 + wave) * 2;
  if (t0 >= n_tiles) return;
  const bool second = t0 + 1 < n_tiles;      // else the second tile re-reads the first and is not stored
  const int kofs = (lane >> 4) * 8;
  auto wrow = [&](int t) { return lin_wrow(a, min(t * 16 + (lane & 15), a.N - 1)) + kofs; };
  const uint16_t* wp[2] = {wrow(t0), wrow(second ? t0 + 1 : t0)};
  u32x4 W[2][2][8];                          // [chunk parity][tile][step]
  auto fetch = [&](u32x4 (&Wd)[2][8], int c) {
#pragma unroll
    for (int u = 0; u < 8; ++u)
#pragma unroll
      for (int j = 0; j < 2; ++j) Wd[j][u] = *(const u32x4*)(wp[j] + c * 256 + u * 32);
  };
  fetch(W[0], 0);
  f32x4 tot[2][RT];
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int i = 0; i < RT; ++i) tot[j][i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int c = 0; c < NCH; ++c) {
    if (c + 1 < NCH) fetch(W[(c + 1) & 1], c + 1);
    __builtin_amdgcn_sched_barrier(0);     // the next chunk's loads go out before this chunk's MFMAs
    // an opaque copy of the x offset keeps the compiler from holding x
    // fragments in registers across chunks (an offset, not a pointer, so
    // the reads stay LDS reads)
    int xv = (lane & 15) * XP + kofs + c * 256;
    asm volatile("" : "+v"(xv));
    const uint16_t* xt = xs + xv;
    f32x4 acc[2][RT];
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int i = 0; i < RT; ++i) acc[j][i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int st = 0; st < 8; ++st)
#pragma unroll
      for (int i = 0; i < RT; ++i) {
        const u32x4 xf = *(const u32x4*)(xt + i * 16 * XP + st * 32);
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[j][i] = mfma16(W[c & 1][j][st], xf, acc[j][i]);
      }
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int i = 0; i < RT; ++i) tot[j][i] += acc[j][i];
  }
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    if (j == 1 && !second) break;
#pragma unroll
    for (int i = 0; i < RT; ++i) {
      const int m = i * 16 + (lane & 15);
      if (m < a.M) lin_store4<kLinF32>(a, m, (t0 + j) * 16 + 4 * (lane >> 4), tot[j][i]);
    }
  }
}

template <int NCH, int RT>
static void launch_wide_rt(const LinArgs& a, int n_tiles, dim3 grid, hipStream_t s) {
  if constexpr (wide_lds(RT, 256 * NCH) <= kWideLds)
    hipLaunchKernelGGL((k_linear_wide<NCH, RT>), grid, dim3(512), 0, s, a, n_tiles);
}

template <int NCH>
static void launch_wide_nch(const LinArgs& a, hipStream_t s) {
  const int n_tiles = (a.N + 15) / 16;
  const dim3 grid((n_tiles + 15) / 16);                      // 8 waves of two tiles each
  switch ((a.M + 15) / 16) {
    case 1: launch_wide_rt<NCH, 1>(a, n_tiles, grid, s); break;
    case 2: launch_wide_rt<NCH, 2>(a, n_tiles, grid, s); break;
    case 3: launch_wide_rt<NCH, 3>(a, n_tiles, grid, s); break;
    default: launch_wide_rt<NCH, 4>(a, n_tiles, grid, s); break;
  }
}

static void launch_wide(const LinArgs& a, hipStream_t s) {
  switch (a.K / 256) {
    case 1: launch_wide_nch<1>(a, s); break;
    case 2: launch_wide_nch<2>(a, s); break;
    case 3: launch_wide_nch<3>(a, s); break;
    case 4: launch_wide_nch<4>(a, s); break;
    case 5: launch_wide_nch<5>(a, s); break;
    case 6: launch_wide_nch<6>(a, s); break;
    case 7: launch_wide_nch<7>(a, s); break;
    default: launch_wide_nch<8>(a, s); break;
  }
}

template <int EPI, class C>
static void launch_gemm(const LinArgs& a, hipStream_t s) {
  const int tm = (a.M + C::BM - 1) / C::BM, tn = (a.N + C::BN - 1) / C::BN;
  hipLaunchKernelGGL((k_gemm<EPI, C>), dim3(gemm_grid(C::PER_CU, tm * tn)), dim3(C::NT), 0, s, a, tm, tn);
}

template <int EPI>
static hipError_t linear(const LinArgs& a, hipStream_t s) {
  if (a.M <= 0 || a.N <= 0) return hipSuccess;
  if (a.K <= 0 || a.K % 64) return hipErrorInvalidValue;
  if (EPI != kLinF32 && (a.ldy % 4 || (EPI == kLinSplit && a.ns % 4))) return hipErrorInvalidValue;
  if (a.lng) {
    if (!a.lnb || a.K > 2048 || a.ldx % 8) return hipErrorInvalidValue;
    if (a.M <= 128) {
      launch_few_ln<EPI>(a, s);
      return hipGetLastError();
    }
    if (!a.lnout) return hipErrorInvalidValue;
    launch_ln(a.x, a.ldx, a.lng, a.lnb, a.lnout, a.K, a.M, a.K, s);
    LinArgs n = a;
    n.x = a.lnout;
    n.ldx = a.K;
    n.lng = n.lnb = nullptr;
    return linear<EPI>(n, s);
  }
  if (EPI == kLinF32 && a.ldx % 8 == 0 && wide_fits(a.M, a.N, a.K)) {
    launch_wide(a, s);
  } else if (a.M <= 128) {
    launch_few<EPI>(a, s);
  } else {
    switch (gemm_tile(a.M, a.N, a.K)) {
      case kGemmWide: launch_gemm<EPI, GemmWide>(a, s); break;
      case kGemmTall: launch_gemm<EPI, GemmTall>(a, s); break;
      case kGemmPair: launch_gemm<EPI, GemmPair>(a, s); break;
      case kGemmSmall: launch_gemm<EPI, GemmSmall>(a, s); break;
      default: launch_gemm<EPI, GemmBrief>(a, s); break;
    }
  }
  return hipGetLastError();
}

}  // namespace smem
