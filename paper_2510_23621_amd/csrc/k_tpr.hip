// Edge tensor product of Eq. 26 with the last radial layer computed in place,
// fused with the receiver neighbour sum; and its vector-Jacobian product.
//
//   R[e][p][k]  = sum_j a3[e][j] W3[j][p K + k]                 (last radial layer)
//   At[i][p][m3][k] = inv_c * sum_{e: rcv_e = i} R[e][p][k]
//                     * sum_{m1,m2} C^{lo}_{lh ly}[m1][m2][m3] h[src_e][lh,m1][k] Y[e][ly,m2]
//
// R is never stored: for a K = 128 model with ten paths it would be 5 KB per
// edge each way; the backward forms it again, and R' = dR/dr with it. One wave
// owns a (receiver, 16-channel tile) pair and walks the receiver's edges (CSR
// order) in tiles of 16. For each tile the forward forms R
// with FP32 MFMA (v_mfma_f32_16x16x4_f32; lane l supplies A[l%16][l/16] and
// B[l/16][l%16], result register r holds D[4(l/16)+r][l%16]): rows are the
// tile's edges in transposed order, columns the wave's channels. Lane l
// therefore holds R for channel l%16 and the four edges e0 + 4 q + l/16,
// q = 0..3, and contracts exactly those edges; the four lane groups are summed
// by a fixed butterfly at the end of the receiver, so the result does not
// depend on scheduling.
//
// A block is a few waves on as many receivers, sharing one channel tile; the
// tile's slice of W3 (64 x P x 16 floats) sits in LDS for the block's life,
// and each wave stages the Y rows of its current edge tile in LDS.
#include <algorithm>

#include "mace_internal.h"
#include "static_loops.h"

namespace mace {

typedef float f4 __attribute__((ext_vector_type(4)));

constexpr int kWPitch = 68;   // LDS row pitch of the W3 slice: 64 + 4 (4 mod 32)
constexpr int kYPitch = 20;   // Y tile row: 16 floats + 4 (float4-aligned)
// Launch shape per (l_max, direction): waves per block (all on one channel
// tile) and the waves per SIMD the register budget is cut for. Forward: two
// 8-wave blocks per CU fit the LDS below l = 2 and give four waves per SIMD at
// 128 VGPRs; for l = 2 the W3 slice fills most of the LDS and one 8-wave block
// runs two per SIMD. Backward: two waves per SIMD at l = 1 and 2 (206 to 240
// registers), three at l = 0 (in 4-wave blocks; two or four per SIMD were 3 to
// 7% slower). By the counters (36,864 atoms, K = 128, l = 2) a 16-edge tile and
// channel tile of the backward takes 2,365 vector instructions (the contraction's
// multiply-adds are 2,176) and 408 MFMAs of 16 cycles, in 15,400 cycles of its
// SIMD; the forward 1,371 and 204 in 7,480. The matrix cores work in 42 and 44%
// of the cycles. A vector instruction of two or more waves takes its SIMD 2.3 to
// 4.1 cycles, by its form (measured), and a BF16 MFMA keeps it from vector issue
// for 7 of its 16: at 4 cycles the two together would fill 81 and 93% of the
// time, and how many instructions take less is not known. Operand rings of other
// depths changed nothing. Under this load the clock is 1.74 GHz in the backward
// and 1.80 in the forward, where the sender sum runs at 2.4. The MFMA phases
// raise the wave's priority so that they issue ahead of the other waves' vector
// work on the SIMD.
// At 36,864 atoms (3.18 M edges): forward 7.46 -> 7.07 ms, backward 18.55 ->
// 15.2 ms (and no radial backward); at 1,536 atoms (l = 1) 126 -> 100 us and
// 230 -> 204 us.
template <int LHMAX, bool BWD, int RM = 0>
struct TprShape {
  static constexpr int waves = BWD && LHMAX == 0 ? 4 : 8;
  static constexpr int per_simd = BWD ? (LHMAX == 0 ? 3 : 2) : (LHMAX == 2 ? 2 : 4);
  // waves that share a receiver and its G table, taking its edge tiles in turn
  // (two where eight tables do not fit beside W3's slice)
  static constexpr int share = (BWD && LHMAX == 2 && RM != 1) ? 2 : 1;
  static constexpr int blocks_per_cu = 4 * per_simd / waves;
};

__device__ __forceinline__ f4 mfma4(float a, float b, f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// The block's slice of W3, W3[j][p K + 16 ct + kk] for kk = 0..15: put(p, j,
// kk, v) for four consecutive kk per call. A thread's float4 loads are all in
// flight together (one 4-byte load at a time, each waiting on the last-level
// cache, cost the block 10 to 20 us before its first receiver).
template <int P, int NT, class F>
__device__ __forceinline__ void load_w3_quads(const float* __restrict__ W3, int K, int ct, F&& put) {
  constexpr int NQ = P * 64 * 4, CNT = (NQ + NT - 1) / NT;
  const int PK = P * K;
  f4 v[CNT];
#pragma unroll
  for (int u = 0; u < CNT; ++u) {
    const int q = min((int)threadIdx.x + u * NT, NQ - 1);
    v[u] = *reinterpret_cast<const f4*>(W3 + (size_t)((q >> 2) & 63) * PK + (q >> 8) * K + 16 * ct + 4 * (q & 3));
  }
#pragma unroll
  for (int u = 0; u < CNT; ++u) {
    const int q = threadIdx.x + u * NT;
    if (NQ % NT == 0 || q < NQ) put(q >> 8, (q >> 2) & 63, 4 * (q & 3), v[u]);
  }
}

// sW[(p*16 + kk)*kWPitch + j] = W3[j][p K + 16 ct + kk]
template <int P, int NT>
__device__ __forceinline__ void load_w3_slice(const float* __restrict__ W3, int K, int ct, float* sW) {
  load_w3_quads<P, NT>(W3, K, ct, [&](int p, int j, int kk, f4 v) {
#pragma unroll
    for (int c = 0; c < 4; ++c) sW[(p * 16 + kk + c) * kWPitch + j] = v[c];
  });
}

// Edge (from e0) that MFMA row rho of a tile carries: the transposed order
// 4 (rho % 4) + rho / 4 puts edge e0 + 4 q + (l/16) in result register q of lane
// l, so that a tile of n edges needs ceil(n / 4) edge iterations per lane, where
// the order of the rows would need min(n, 4).
__device__ __forceinline__ int tile_edge(int rho) { return 4 * (rho & 3) + (rho >> 2); }

// R of the 16 edges e0 .. e0+15 (edges at or past e_end get R = 0) for the
// wave's channel tile: r[p][q] = R[e0 + 4 q + l/16][p][16 ct + l%16].
// The 64-long reduction runs in the order j = 16 qq + 4 s + c so that every
// lane reads its A operand as four float4.
template <int P>
__device__ __forceinline__ void tile_radial(const float* __restrict__ a3, int e0, int e_end,
                                            const float* __restrict__ sW, f4* r) {
  const int l = threadIdx.x & 63;
  const int row = e0 + tile_edge(l & 15);
  const float keep = row < e_end ? 1.f : 0.f;
  const f4* arow = reinterpret_cast<const f4*>(a3 + (size_t)min(row, e_end - 1) * 64 + 4 * (l >> 4));
  f4 a[4];
#pragma unroll
  for (int qq = 0; qq < 4; ++qq) a[qq] = arow[4 * qq] * keep;
  const float* wb = sW + (l & 15) * kWPitch + 4 * (l >> 4);
  __builtin_amdgcn_s_setprio(1);
#pragma unroll
  for (int p = 0; p < P; ++p) {
    __builtin_amdgcn_sched_barrier(0);   // B fragments are loaded path by path
    f4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int qq = 0; qq < 4; ++qq) {
      const f4 b = *reinterpret_cast<const f4*>(wb + p * 16 * kWPitch + 16 * qq);
      acc = mfma4(a[qq][0], b[0], acc);
      acc = mfma4(a[qq][1], b[1], acc);
      acc = mfma4(a[qq][2], b[2], acc);
      acc = mfma4(a[qq][3], b[3], acc);
    }
    r[p] = acc;
  }
  __builtin_amdgcn_s_setprio(0);
}

// ---- BF16 radial mode: R = bf16(a3) bf16(W3) on v_mfma_f32_16x16x32_bf16
// (FP32 accumulation); lane l supplies A[l%16][8(l/16)+i] and
// B[8(l/16)+i][l%16], i = 0..7. a3 arrives as its split parts, whose first is
// the bfloat16 rounding.
typedef __bf16 bf8v __attribute__((ext_vector_type(8)));
typedef unsigned short us8v __attribute__((ext_vector_type(8)));
constexpr int kWbPitch = 72;   // bf16 per row of the forward slice: 64 + 8 (36 dwords, 4 mod 32)

__device__ __forceinline__ f4 mfma_bf16(us8v a, us8v b, f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf8v, a), __builtin_bit_cast(bf8v, b), c, 0, 0,
                                                 0);
}
// Forward slice sWb[(p*16 + kk)*kWbPitch + j] = bf16(W3[j][p K + 16 ct + kk])
template <int P, int NT>
__device__ __forceinline__ void load_w3_slice_bf16(const float* __restrict__ W3, int K, int ct, unsigned short* sWb) {
  load_w3_quads<P, NT>(W3, K, ct, [&](int p, int j, int kk, f4 v) {
#pragma unroll
    for (int c = 0; c < 4; ++c) sWb[(p * 16 + kk + c) * kWbPitch + j] = bf16_bits(v[c]);
  });
}

// As tile_radial, on BF16 operands: two MFMAs (k = 32 each) per path. The W3
// operands are read kBf16Ahead paths ahead of their MFMAs, so that the LDS
// reads do not stall each path's pair of products.
constexpr int kBf16Ahead = 4;
template <int P>
__device__ __forceinline__ void tile_radial_bf16(const unsigned short* __restrict__ a3x, int e0, int e_end,
                                                 const unsigned short* __restrict__ sWb, f4* r) {
  const int l = threadIdx.x & 63;
  const int row = e0 + tile_edge(l & 15);
  const unsigned short* arow = a3x + (size_t)min(row, e_end - 1) * 192 + 8 * (l >> 4);
  const unsigned short* wb = sWb + (l & 15) * kWbPitch + 8 * (l >> 4);
  constexpr int D = kBf16Ahead < P ? kBf16Ahead : P;
  us8v bw[D][2];
  auto load_b = [&](int p, us8v (&b)[2]) {
    b[0] = *reinterpret_cast<const us8v*>(wb + p * 16 * kWbPitch);
    b[1] = *reinterpret_cast<const us8v*>(wb + p * 16 * kWbPitch + 32);
  };
#pragma unroll
  for (int p = 0; p < D; ++p) load_b(p, bw[p]);
  us8v a[2];
#pragma unroll
  for (int ks = 0; ks < 2; ++ks)
    a[ks] = row < e_end ? *reinterpret_cast<const us8v*>(arow + 32 * ks) : us8v{0, 0, 0, 0, 0, 0, 0, 0};
  __builtin_amdgcn_s_setprio(1);
  static_for<0, P>([&](auto PI) {
    constexpr int p = decltype(PI)::value;
    __builtin_amdgcn_sched_barrier(0);
    const us8v b0 = bw[p % D][0], b1 = bw[p % D][1];
    if constexpr (p + D < P) load_b(p + D, bw[p % D]);
    r[p] = mfma_bf16(a[1], b1, mfma_bf16(a[0], b0, f4{0.f, 0.f, 0.f, 0.f}));
  });
  __builtin_amdgcn_s_setprio(0);
}

// ---- Split-BF16 radial layer (FP32-accurate): every FP32 operand x is carried
// as x0 + x1 + x2 with x0 = bf16(x), x1 = bf16(x - x0), x2 = bf16(x - x0 - x1)
// (each difference is exact in FP32, so the three parts hold all 24
// significand bits), and a b = a0 b0 + (a0 b1 + a1 b0) + (a0 b2 + a1 b1 + a2 b0)
// up to terms of relative size 2^-27, on v_mfma_f32_16x16x32_bf16 with FP32
// accumulation: six BF16 MFMAs (16 cycles each) in place of eight FP32 ones
// (32 cycles each) per 16 x 16 x 32 block.
__device__ __forceinline__ void split3(float x, unsigned short& b0, unsigned short& b1, unsigned short& b2) {
  const __bf16 h0 = (__bf16)x;
  const float r1 = x - (float)h0;
  const __bf16 h1 = (__bf16)r1;
  const float r2 = r1 - (float)h1;
  const __bf16 h2 = (__bf16)r2;
  b0 = __builtin_bit_cast(unsigned short, h0);
  b1 = __builtin_bit_cast(unsigned short, h1);
  b2 = __builtin_bit_cast(unsigned short, h2);
}

// The parts of a3[row][32 ks + 8 (l/16) .. +7] from the pre-split rows
// ([E][3][64] bfloat16), zero where keep is false (rows past the tile's end).
__device__ __forceinline__ void load_a3_parts(const unsigned short* __restrict__ a3x, int row, bool keep, int ks,
                                              us8v& a0, us8v& a1, us8v& a2) {
  const int l = threadIdx.x & 63;
  const unsigned short* base = a3x + (size_t)row * 192 + 32 * ks + 8 * (l >> 4);
  const us8v z = {0, 0, 0, 0, 0, 0, 0, 0};
  a0 = keep ? *reinterpret_cast<const us8v*>(base) : z;
  a1 = keep ? *reinterpret_cast<const us8v*>(base + 64) : z;
  a2 = keep ? *reinterpret_cast<const us8v*>(base + 128) : z;
}

// The three parts of the forward slice, part q at sWx + q P 16 kWbPitch, in the
// layout of load_w3_slice_bf16.
template <int P, int NT>
__device__ __forceinline__ void load_w3_slice_x3(const float* __restrict__ W3, int K, int ct, unsigned short* sWx) {
  constexpr int part = P * 16 * kWbPitch;
  load_w3_quads<P, NT>(W3, K, ct, [&](int p, int j, int kk, f4 v) {
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int o = (p * 16 + kk + c) * kWbPitch + j;
      split3(v[c], sWx[o], sWx[part + o], sWx[2 * part + o]);
    }
  });
}

// tile_radial_x3 below l = 2 (described there)
template <int P>
__device__ __forceinline__ void tile_radial_x3_chain(const unsigned short* __restrict__ a3x, int e0, int e_end,
                                                     const unsigned short* __restrict__ sWx, f4* r) {
  constexpr int part = P * 16 * kWbPitch;
  const int l = threadIdx.x & 63;
  const int row = e0 + tile_edge(l & 15);
  const int crow = min(row, e_end - 1);
  const unsigned short* wb = sWx + (l & 15) * kWbPitch + 8 * (l >> 4);
#pragma unroll
  for (int p = 0; p < P; ++p) r[p] = f4{0.f, 0.f, 0.f, 0.f};
  __builtin_amdgcn_s_setprio(1);
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) {
    __builtin_amdgcn_sched_barrier(0);
    us8v a0, a1, a2;
    load_a3_parts(a3x, crow, row < e_end, ks, a0, a1, a2);
#pragma unroll
    for (int p = 0; p < P; ++p) {
      __builtin_amdgcn_sched_barrier(0);   // one path's B parts live at a time
      const unsigned short* q = wb + p * 16 * kWbPitch + 32 * ks;
      const us8v b0 = *reinterpret_cast<const us8v*>(q);
      const us8v b1 = *reinterpret_cast<const us8v*>(q + part);
      const us8v b2 = *reinterpret_cast<const us8v*>(q + 2 * part);
      f4 acc = r[p];
      acc = mfma_bf16(a2, b0, acc);
      acc = mfma_bf16(a1, b1, acc);
      acc = mfma_bf16(a0, b2, acc);
      acc = mfma_bf16(a1, b0, acc);
      acc = mfma_bf16(a0, b1, acc);
      r[p] = mfma_bf16(a0, b0, acc);
    }
  }
  __builtin_amdgcn_s_setprio(0);
}

// As tile_radial, FP32-accurate on split BF16 operands (a3x: the parts of a3,
// [E][3][64] bfloat16, written by the edge prologue): within each K step the
// terms are added from the smallest to the largest.
// Below l = 2 (P <= 10, four waves per SIMD at 128 registers) one path's chain
// of six products at a time, only one K step's A parts live; at l = 2 (P = 17,
// two waves per SIMD) both K steps' A parts are loaded first and the paths go
// in pairs (below).
template <int P>
__device__ __forceinline__ void tile_radial_x3(const unsigned short* __restrict__ a3x, int e0, int e_end,
                                               const unsigned short* __restrict__ sWx, f4* r) {
  if constexpr (P <= 10) {
    tile_radial_x3_chain<P>(a3x, e0, e_end, sWx, r);
    return;
  }
  constexpr int part = P * 16 * kWbPitch;
  const int l = threadIdx.x & 63;
  const int row = e0 + tile_edge(l & 15);
  const int crow = min(row, e_end - 1);
  const unsigned short* wb = sWx + (l & 15) * kWbPitch + 8 * (l >> 4);
#pragma unroll
  for (int p = 0; p < P; ++p) r[p] = f4{0.f, 0.f, 0.f, 0.f};
  __builtin_amdgcn_s_setprio(1);
  us8v a[2][3];
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) load_a3_parts(a3x, crow, row < e_end, ks, a[ks][0], a[ks][1], a[ks][2]);
  // Steps s = ks P + p taken in pairs: the next pair's W3 parts are requested
  // before this pair's MFMAs, and the two paths' six-product chains alternate
  // so that neither waits on its own previous product. Each path's products
  // are added in the same order as in a single chain.
  constexpr int NS = 2 * P;   // even: the pairs are (2t, 2t + 1), t < P
  us8v bb[2][2][3];
  auto load_b = [&](int s, us8v (&b)[3]) {
    const int ks = s / P, p = s % P;
    const unsigned short* q = wb + p * 16 * kWbPitch + 32 * ks;
    b[0] = *reinterpret_cast<const us8v*>(q);
    b[1] = *reinterpret_cast<const us8v*>(q + part);
    b[2] = *reinterpret_cast<const us8v*>(q + 2 * part);
  };
  load_b(0, bb[0][0]);
  load_b(1, bb[0][1]);
  static_for<0, P>([&](auto TI) {
    constexpr int t = decltype(TI)::value;
    constexpr int s0 = 2 * t, s1 = 2 * t + 1;
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (s1 + 2 < NS) {
      load_b(s0 + 2, bb[(t + 1) & 1][0]);
      load_b(s1 + 2, bb[(t + 1) & 1][1]);
    }
    constexpr int ks0 = s0 / P, p0 = s0 % P, ks1 = s1 / P, p1 = s1 % P;
    const us8v(&b0)[3] = bb[t & 1][0];
    const us8v(&b1)[3] = bb[t & 1][1];
    f4 x = r[p0], y = r[p1];
    x = mfma_bf16(a[ks0][2], b0[0], x);
    y = mfma_bf16(a[ks1][2], b1[0], y);
    x = mfma_bf16(a[ks0][1], b0[1], x);
    y = mfma_bf16(a[ks1][1], b1[1], y);
    x = mfma_bf16(a[ks0][0], b0[2], x);
    y = mfma_bf16(a[ks1][0], b1[2], y);
    x = mfma_bf16(a[ks0][1], b0[0], x);
    y = mfma_bf16(a[ks1][1], b1[0], y);
    x = mfma_bf16(a[ks0][0], b0[1], x);
    y = mfma_bf16(a[ks1][0], b1[1], y);
    x = mfma_bf16(a[ks0][0], b0[0], x);
    y = mfma_bf16(a[ks1][0], b1[0], y);
    r[p0] = x;
    r[p1] = y;
  });
  __builtin_amdgcn_s_setprio(0);
}

// Split parts in the backward, without row padding: a 16-byte chunk c of row r
// sits at chunk c ^ s(r), so that the 16 lanes of an MFMA operand read hit 16
// distinct 16-byte bank groups: row r = p 16 + kk of 64 elements (8 chunks of
// j), s(r) = (r >> 1) & 7.
__device__ __forceinline__ int swz_fwd(int r, int c) { return r * 64 + 8 * (c ^ ((r >> 1) & 7)); }

// The precision study's operand rounding of the edge product (rnd: 0 none,
// 1 bfloat16, 2 binary16, round to nearest even) of the radial weights of a
// tile; the harmonics and the sender features arrive rounded (the host runtime
// rounds those buffers in place).
template <int P>
__device__ __forceinline__ void round_tile(f4* r, int rnd) {
  if (!rnd) return;
#pragma unroll
  for (int p = 0; p < P; ++p) {
    if (rnd == 1) {   // the packed hardware conversion: round to nearest even
      const f2v lo = bf16_unpack2(bf16_pack2(f2v{r[p][0], r[p][1]})), hi = bf16_unpack2(bf16_pack2(f2v{r[p][2], r[p][3]}));
      r[p] = f4{lo[0], lo[1], hi[0], hi[1]};
    } else {
#pragma unroll
      for (int q = 0; q < 4; ++q) r[p][q] = fp16_round(r[p][q]);
    }
  }
}

// Y rows of the wave's 16-edge tile into LDS: sy[row][m], row pitch kYPitch.
// Lane l moves float4 number l%4 of row l/4.
__device__ __forceinline__ void stage_y(const float* __restrict__ Y, int e0, int e_end, float* sy) {
  const int l = threadIdx.x & 63;
  const int row = l >> 2, ch = l & 3;
  const int e = min(e0 + row, e_end - 1);
  const f4 v = reinterpret_cast<const f4*>(Y + (size_t)e * 16)[ch];
  *reinterpret_cast<f4*>(sy + row * kYPitch + 4 * ch) = v;
}

__device__ __forceinline__ void read_y(const float* sy, int row, float* y) {
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const f4 t4 = *reinterpret_cast<const f4*>(sy + row * kYPitch + 4 * v);
    y[4 * v] = t4[0];
    y[4 * v + 1] = t4[1];
    y[4 * v + 2] = t4[2];
    y[4 * v + 3] = t4[3];
  }
}

template <int DIN>
__device__ __forceinline__ void load_h_row(const float* __restrict__ h, int src, int K, int k, float* hv) {
#pragma unroll
  for (int c = 0; c < DIN; ++c) hv[c] = h[((size_t)src * DIN + c) * K + k];
}

// RM, the operands of the last radial layer: 0 FP32, 1 BF16, 3 split BF16
// (FP32-accurate). In modes 1 and 3 a3 arrives as its three parts (the a3
// argument then points at [E][3][64] bfloat16 written by the edge prologue).
// KC: K as a compile-time constant (0: the argument K), so that the sender
// rows' component strides become immediate load offsets.
template <int LHMAX, int RM, int NW = TprShape<LHMAX, false>::waves, int KC = 0>
__global__ void __launch_bounds__(64 * NW)
__attribute__((amdgpu_waves_per_eu(TprShape<LHMAX, false>::per_simd, TprShape<LHMAX, false>::per_simd)))
tpr_fwd_kernel(
    int N, int K_arg, const int* __restrict__ rcv_off, const int* __restrict__ snd, const int* __restrict__ src_map,
    const float* __restrict__ a3, const float* __restrict__ W3, const float* __restrict__ Y,
    const float* __restrict__ h, float inv_c, float* __restrict__ At, int rnd) {
  const int K = KC ? KC : K_arg;
  constexpr int P = path_count(LHMAX);
  constexpr int MID = mid_count(LHMAX);
  constexpr int DIN = (LHMAX + 1) * (LHMAX + 1);
  constexpr bool SPLIT = RM == 3;
  constexpr int kSlice = RM == 1 ? (P * 16 * kWbPitch + 1) / 2
                        : (SPLIT ? (3 * P * 16 * kWbPitch + 1) / 2 : P * 16 * kWPitch);   // floats
  __shared__ __align__(16) float sW[kSlice];
  __shared__ float sY[NW][16 * kYPitch];
  const int ct = blockIdx.y;
  if constexpr (RM == 1) load_w3_slice_bf16<P, 64 * NW>(W3, K, ct, reinterpret_cast<unsigned short*>(sW));
  else if constexpr (SPLIT) load_w3_slice_x3<P, 64 * NW>(W3, K, ct, reinterpret_cast<unsigned short*>(sW));
  else load_w3_slice<P, 64 * NW>(W3, K, ct, sW);
  __syncthreads();
  const unsigned short* a3x = reinterpret_cast<const unsigned short*>(a3);
  const int l = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int g = l >> 4;
  const int k = 16 * ct + (l & 15);
  float* sy = sY[w];
  // (a receiver's edge range is requested while the wave's previous receiver is worked on)
  const int stride = gridDim.x * NW;
  int i = blockIdx.x * NW + w;
  if (i >= N) return;
  int nb = rcv_off[i], ne = rcv_off[i + 1];
  for (; i < N; i += stride) {
    constexpr int H2 = (MID + 3) / 4, H1 = 2 * H2;
    float acc[2 * H1];
#pragma unroll
    for (int c = 0; c < 2 * H1; ++c) acc[c] = 0.f;
    const int e_beg = nb, e_end = ne;
    const int i_next = min(i + stride, N - 1);
    nb = rcv_off[i_next];
    ne = rcv_off[i_next + 1];
    for (int e0 = e_beg; e0 < e_end; e0 += 16) {
      // sender rows of the lane's four edges (edges past e_end carry R = 0),
      // requested before the radial MFMAs so that their latency is hidden
      // edge e0 + 4 q + g is the lane's q-th (transposed tile rows)
      int srcq[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int sq = snd[min(e0 + 4 * q + g, e_end - 1)];
        srcq[q] = src_map ? src_map[sq] : sq;
      }
      stage_y(Y, e0, e_end, sy);
      f4 r[P];
      if constexpr (RM == 1) tile_radial_bf16<P>(a3x, e0, e_end, reinterpret_cast<const unsigned short*>(sW), r);
      else if constexpr (SPLIT) tile_radial_x3<P>(a3x, e0, e_end, reinterpret_cast<const unsigned short*>(sW), r);
      else tile_radial<P>(a3, e0, e_end, sW, r);
      round_tile<P>(r, rnd);
      // a tile of n edges fills registers q < ceil(n / 4) (edges past e_end
      // carry R = 0); the scheduling barrier keeps one edge's operands live at
      // a time, and the next edge's h row is requested while this one is contracted
      const int nq = min(4, (e_end - e0 + 3) >> 2);
      // the sender rows of edges q and q + 1 (in flight); at l = 2 the two
      // buffers alternate, below it the next row is copied over (fewer registers)
      constexpr bool ALT = LHMAX == 2;
      float hb[2][DIN];
      load_h_row<DIN>(h, srcq[0], K, k, hb[0]);
      static_for<0, 4>([&](auto QI) {
        constexpr int q = decltype(QI)::value;
        constexpr int cur = ALT ? (q & 1) : 0, nxt = ALT ? ((q + 1) & 1) : 1;
        __builtin_amdgcn_sched_barrier(0);
        if (q >= nq) return;
        const int row = 4 * q + g;   // the lane's edge e0 + row
        if constexpr (q < 3) load_h_row<DIN>(h, srcq[q + 1], K, k, hb[nxt]);
        const float(&hv)[DIN] = hb[cur];
        float y[16];
        read_y(sy, row, y);
        for_paths<LHMAX>([&](auto tag) {
          using T = decltype(tag);
          constexpr int lh = T::lh, ly = T::ly, lo = T::lo;
          // R folded into the sender features (R h[m1]), and each coefficient
          // carried as +-ratio * scale[m3]: acc[m3] += (+-R h[m1]) (ratio Y[m2]),
          // one multiply-add per coefficient with its sign on an operand, one
          // product per distinct (m2, ratio != 1) of the path, and the scales
          // at the end of the receiver
          using C = mt::CG<lh, ly, lo>;
          const float rv = r[T::index][q];
          float hr[2 * lh + 1];
#pragma unroll
          for (int m = 0; m < 2 * lh + 1; ++m) hr[m] = rv * hv[lh * lh + m];
          float yc[C::nyc ? C::nyc : 1];
          C::each_yc([&](int m2, float ratio, int u) { yc[u] = ratio * y[ly * ly + m2]; });
          C::each_ys([&](int m1, int m2, int m3, int sg, int u) {
            const float yv = u >= 0 ? yc[u >= 0 ? u : 0] : y[ly * ly + m2];
            acc[T::offset + m3] = __builtin_fmaf(sg > 0 ? hr[m1] : -hr[m1], yv, acc[T::offset + m3]);
          });
        });
        if constexpr (!ALT && q < 3) {
#pragma unroll
          for (int c = 0; c < DIN; ++c) hb[0][c] = hb[1][c];
        }
      });
    }
    // the components' scales, then the sum over the lane groups (0+1 and 2+3,
    // then the two pairs) with the components halved twice: group g ends with
    // components c0 .. c0 + H2 - 1
    for_paths<LHMAX>([&](auto tag) {
      using T = decltype(tag);
#pragma unroll
      for (int m3 = 0; m3 < 2 * T::lo + 1; ++m3) acc[T::offset + m3] *= mt::CG<T::lh, T::ly, T::lo>::scale(m3);
    });
#pragma unroll
    for (int c = 0; c < H1; ++c) acc[c] = swap_add16(acc[c], acc[c + H1]);
#pragma unroll
    for (int c = 0; c < H2; ++c) acc[c] = swap_add32(acc[c], acc[c + H2]);
    const int c0 = H1 * (g & 1) + H2 * (g >> 1);
    float* out = At + ((size_t)i * MID + c0) * K + k;
#pragma unroll
    for (int c = 0; c < H2; ++c)
      if (c0 + c < MID || MID % 4 == 0) out[c * K] = acc[c] * inv_c;
  }
}

// VJP of tpr_fwd. Given g = dE/dAt, per edge e (receiver i) and channel k,
// with G_p[m1][m2] = sum_m3 C g[i][p][m3] (per receiver and channel, kept in
// LDS for the receiver's edges, one value per coupled (m1, m2) pair) and
// Dm_p[m1] = sum_m2 G_p[m1][m2] Y[m2]:
//   dY[e][ly,m2]  += inv_c sum_k sum_p sum_m1 G_p[m1][m2] R h[m1]    (channel-tile partial)
//   Q[e][lh,m1][k] = inv_c sum_p R Dm_p[m1]                          (per-edge sender gradient)
//   dr[e]         += inv_c sum_k sum_p R'[e][p][k] sum_m1 h[m1] Dm_p[m1]
//                                                                    (channel-tile partial)
// R depends on the edge's length alone, so what the radial MLP's backward needs
// from here is one number per edge, dE/dr through R, with R' = dR/dr:
// R'[e][p][k] = sum_j a3'[e][j] W3[j][p K + k], a3' = da3/dr carried through the
// hidden layers by the edge prologue. R' is a second product with the same W3
// operands as R. (The reverse form, dE/da3 = dR W3^T stored per channel tile
// and taken back through the hidden layers in a kernel of its own, spent as
// many matrix instructions, plus the split of dR into bfloat16 parts, transposed
// reads of W3, 256 bytes written and read per edge and channel tile, and three
// recomputed and three transposed hidden layers.)
// The partials of channel tile ct go to dYp[ct][e][16]: dr in element 0 (the
// l = 0 harmonic is constant and has no gradient) and dY[1..15]; their sum over
// tiles and layers (fixed order) is taken by the geometry's backward.
//
// Edge-lane layout: the radial MFMAs take the weight slice as the A operand and
// a3 (a3') as B, so the result puts the edge on l%16: lane l holds R for edge
// e0 + l%16 and the four channels 16 ct + 4(l/16) .. +3. Each lane contracts
// one edge over four channels:
//   - the Y row and the sender's h rows are the lane's own (float4 loads);
//   - the couplings come from the receiver's G table in LDS, one float4 over
//     the four channels per (m1, m2) pair: Dm[m1] += G Y[m2] and
//     dY[m2] += G (R h[m1]), two multiply-adds per pair and channel;
//   - dr and dY are summed over the lane's four channels in registers and over
//     the four lane groups by two halving exchange steps.
// The paths go in groups of one l_h: the group's R and R' products, then its
// contraction, then its block of Q.
// No divergence: lanes past the receiver's last edge work on that edge; their
// values equal the last valid lane's, so they store the same values to the same
// rows and the stores need no branch.

// The radial operands of one edge (a3 or a3'), per mode: RM 0 the FP32 row,
// v[q] = a3[e][16 q + 4 g .. +3]; RM 1 and 3 its first NQ bfloat16 parts,
// x[ks][q] = part q of a3[e][32 ks + 8 g .. +7] ([E][3][64]).
template <int RM, int NQ>
struct RadOp {
  us8v x[2][NQ];
  __device__ __forceinline__ void load(const float* __restrict__ a3, int e, int g) {
    const unsigned short* row = reinterpret_cast<const unsigned short*>(a3) + (size_t)e * 192 + 8 * g;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int q = 0; q < NQ; ++q) x[ks][q] = *reinterpret_cast<const us8v*>(row + 64 * q + 32 * ks);
  }
};
template <int NQ>
struct RadOp<0, NQ> {
  f4 v[4];
  __device__ __forceinline__ void load(const float* __restrict__ a3, int e, int g) {
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = *reinterpret_cast<const f4*>(a3 + (size_t)e * 64 + 16 * q + 4 * g);
  }
};

// W3's slice in LDS for the backward: FP32 rows (RM 0), or the bfloat16 parts
// (one for RM 1, three for RM 3) in the swizzled layout
template <int P, int RM, int NT>
__device__ __forceinline__ void load_w3_bwd(const float* __restrict__ W3, int K, int ct, void* sW) {
  if constexpr (RM == 0) {
    load_w3_slice<P, NT>(W3, K, ct, reinterpret_cast<float*>(sW));
  } else {
    unsigned short* s = reinterpret_cast<unsigned short*>(sW);
    constexpr int part = P * 16 * 64;
    load_w3_quads<P, NT>(W3, K, ct, [&](int p, int j, int kk, f4 v) {
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const int o = swz_fwd(p * 16 + kk + c, j >> 3) + (j & 7);
        if constexpr (RM == 1) s[o] = bf16_bits(v[c]);
        else split3(v[c], s[o], s[part + o], s[2 * part + o]);
      }
    });
  }
}

constexpr int kRingR = 3;   // W3 operand sets in flight in the radial products
constexpr int kRingG = 4;   // G-table entries in flight (one coupling pair each)

// R and R' of the paths PA .. PB - 1 in the edge-lane layout. RM 3: six partial
// products per operand pair, the smallest first. RM 1: bf16(a3) bf16(W3) for R,
// and for R' the first two parts of a3' (16 significand bits) with bf16(W3). The
// two products of an operand set alternate, so that neither chain waits on its
// own previous MFMA.
template <int PA, int PB, int P, int RM, class XA, class XT>
__device__ __forceinline__ void radial_group(const void* __restrict__ sW, const XA& a, const XT& t, f4* r, f4* rp) {
  const int l = threadIdx.x & 63, g = l >> 4, kk = l & 15;
  __builtin_amdgcn_s_setprio(1);
  if constexpr (RM == 0) {
    const float* wb = reinterpret_cast<const float*>(sW) + kk * kWPitch + 4 * g;
#pragma unroll
    for (int p = PA; p < PB; ++p) {
      __builtin_amdgcn_sched_barrier(0);
      r[p - PA] = rp[p - PA] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const f4 b = *reinterpret_cast<const f4*>(wb + p * 16 * kWPitch + 16 * q);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          r[p - PA] = mfma4(b[c], a.v[q][c], r[p - PA]);
          rp[p - PA] = mfma4(b[c], t.v[q][c], rp[p - PA]);
        }
      }
    }
  } else {
    constexpr int part = P * 16 * 64, NB = RM == 1 ? 1 : 3, F0 = 2 * PA, F1 = 2 * PB;
    const unsigned short* s = reinterpret_cast<const unsigned short*>(sW);
    // operand set of step f = 2 p + ks: row p 16 + kk, chunk 4 ks + g
    auto w_at = [&](int f, us8v* o) {
      const unsigned short* q = s + swz_fwd((f >> 1) * 16 + kk, 4 * (f & 1) + g);
#pragma unroll
      for (int b = 0; b < NB; ++b) o[b] = *reinterpret_cast<const us8v*>(q + b * part);
    };
    us8v ring[kRingR][NB];
#pragma unroll
    for (int f = 0; f < kRingR; ++f)
      if (F0 + f < F1) w_at(F0 + f, ring[f]);
    static_for<F0, F1>([&](auto F) {
      constexpr int f = decltype(F)::value, p = (f >> 1) - PA, ks = f & 1;
      __builtin_amdgcn_sched_barrier(0);   // keeps each read kRingR steps ahead of its use
      us8v b[NB];
#pragma unroll
      for (int q = 0; q < NB; ++q) b[q] = ring[(f - F0) % kRingR][q];
      if constexpr (f + kRingR < F1) w_at(f + kRingR, ring[(f - F0) % kRingR]);
      f4 u = ks == 0 ? f4{0.f, 0.f, 0.f, 0.f} : r[p], v = ks == 0 ? f4{0.f, 0.f, 0.f, 0.f} : rp[p];
      if constexpr (RM == 1) {
        v = mfma_bf16(b[0], t.x[ks][1], v);
        u = mfma_bf16(b[0], a.x[ks][0], u);
        v = mfma_bf16(b[0], t.x[ks][0], v);
      } else {
        constexpr int ib[6] = {0, 1, 2, 0, 1, 0}, ia[6] = {2, 1, 0, 1, 0, 0};
#pragma unroll
        for (int n = 0; n < 6; ++n) {
          u = mfma_bf16(b[ib[n]], a.x[ks][ia[n]], u);
          v = mfma_bf16(b[ib[n]], t.x[ks][ia[n]], v);
        }
      }
      // both products stay in this step (left free, the compiler moves those of
      // R', whose use comes later, behind all of R's and keeps every operand set)
      __asm__ volatile("" : "+v"(u), "+v"(v));
      r[p] = u;
      rp[p] = v;
    });
  }
  __builtin_amdgcn_s_setprio(0);
}

// G_p of receiver i for channel 16 ct + l%16: sg[pair][channel]. Wave ws of
// SHARE takes every SHARE-th path; its dE/dAt values are all requested before
// the first is used (path by path, the receiver paid a memory latency for each).
// The four lane groups compute the same values and the first one stores.
template <int LHMAX, int SHARE>
__device__ __forceinline__ void build_g(const float* __restrict__ gsrc, int K, float inv_c, int ws,
                                        float* __restrict__ sg) {
  const int l = threadIdx.x & 63, g = l >> 4, kk = l & 15;
  static_for<0, SHARE>([&](auto WS) {
    if (SHARE > 1 && ws != decltype(WS)::value) return;
    float gv[mid_count(LHMAX)];
    for_paths<LHMAX>([&](auto tag) {
      using T = decltype(tag);
      if constexpr (T::index % SHARE == decltype(WS)::value) {
#pragma unroll
        for (int m = 0; m < 2 * T::lo + 1; ++m) gv[T::offset + m] = gsrc[(size_t)(T::offset + m) * K + kk];
      }
    });
    __builtin_amdgcn_sched_barrier(0);
    for_paths<LHMAX>([&](auto tag) {
      using T = decltype(tag);
      if constexpr (T::index % SHARE == decltype(WS)::value) {
        using C = mt::CG<T::lh, T::ly, T::lo>;
        constexpr int goff = PathPairOffset<T::index>::value;
#pragma unroll
        for (int m = 0; m < 2 * T::lo + 1; ++m) gv[T::offset + m] *= inv_c;
        float Gp[C::npair];
#pragma unroll
        for (int u = 0; u < C::npair; ++u) Gp[u] = 0.f;
        C::each_p([&](int m1, int m2, int m3, float cg, int pi) { Gp[pi] += cg * gv[T::offset + m3]; });
        if (g == 0) {
#pragma unroll
          for (int u = 0; u < C::npair; ++u) sg[(goff + u) * 16 + kk] = Gp[u];
        }
      }
    });
  });
}

// Wait until every one of the SHARE waves of a group has come here as often as
// this one (cnt: their arrivals, in LDS; due: the count to wait for). All waves
// of a group are resident in the block and take the same receivers, so each
// makes the same number of arrivals and the wait ends. For one wave, only the
// order of its own LDS accesses.
template <int SHARE>
__device__ __forceinline__ void group_sync(int* cnt, int& due) {
  if constexpr (SHARE == 1) {
    __builtin_amdgcn_wave_barrier();
  } else {
    due += SHARE;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    if ((threadIdx.x & 63) == 0) __hip_atomic_fetch_add(cnt, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    while (__hip_atomic_load(cnt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) < due) __builtin_amdgcn_s_sleep(1);
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
  }
}

// RND: the precision study's rounding of R (0 none, 1 bfloat16, 2 binary16; a
// template value, since a branch on it would split the tile); R' is that of the
// unrounded R, gradients passing through the rounding unchanged.
// FIRST: the first layer, whose sender features are rows of the species table
// (through src_map) and take no gradient; otherwise they are the senders' own
// rows of h and Q is written.
template <int LHMAX, int RM, int RND, bool FIRST, int NW = TprShape<LHMAX, true, RM>::waves>
__global__ void __launch_bounds__(64 * NW)
__attribute__((amdgpu_waves_per_eu(TprShape<LHMAX, true, RM>::per_simd, TprShape<LHMAX, true, RM>::per_simd)))
tpr_bwd_kernel(
    int N, int K, int E, const int* __restrict__ rcv_off, const int* __restrict__ snd,
    const int* __restrict__ src_map, const float* __restrict__ a3, const float* __restrict__ t3,
    const float* __restrict__ W3, const float* __restrict__ Y, const float* __restrict__ h, float inv_c,
    const float* __restrict__ dAt, float* __restrict__ dYp, float* __restrict__ Q) {
  constexpr int P = path_count(LHMAX);
  constexpr int MID = mid_count(LHMAX);
  constexpr int DIN = (LHMAX + 1) * (LHMAX + 1);
  constexpr int NPAIR = PairCount<LHMAX>::value;
  constexpr int kSlice = RM == 0 ? P * 16 * kWPitch * 2 : (RM == 1 ? 1 : 3) * P * 16 * 64;   // 2-byte units
  __shared__ __align__(16) unsigned short sW[kSlice];
  constexpr int SH = TprShape<LHMAX, true, RM>::share, NG = NW / SH;   // groups of SH waves, one receiver each
  __shared__ __align__(16) float sG[NG][NPAIR * 16];   // [pair][channel]
  __shared__ int s_cnt[NG];
  const int ct = blockIdx.y;
  load_w3_bwd<P, RM, 64 * NW>(W3, K, ct, sW);
  if (threadIdx.x < NG) s_cnt[threadIdx.x] = 0;
  __syncthreads();
  const int l = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int g = l >> 4, kk = l & 15;
  const int kb = 16 * ct + 4 * g;   // the lane's four channels
  const int wg = w / SH, ws = w % SH;   // the wave's group, and its number there
  float* sg = sG[wg];
  int due = 0;
  float* dYc = dYp + (size_t)ct * E * 16;
  // The next tile's edge and sender index are requested before a tile's last
  // contraction, and a receiver's edge range and first sender index while the
  // wave's previous receiver is worked on. (Conditional loads or stores in the
  // middle of a tile would split it into basic blocks, and the compiler then
  // moves the dY sums to the last one, keeping the G table in registers: it
  // spilled 1.3 to 2.8 KB.)
  int e = 0, src = 0;
  auto fetch = [&](int edge) {
    e = edge;
    src = snd[e];
    if constexpr (FIRST) src = src_map[src];
  };
  const int stride = gridDim.x * NG;
  int i = blockIdx.x * NG + wg;
  if (i >= N) return;   // the whole group
  int nb = rcv_off[i], ne = rcv_off[i + 1];
  auto first_edge = [&]() { return max(min(nb + 16 * ws + kk, ne - 1), 0); };
  int nsrc = snd[first_edge()];
  for (; i < N; i += stride) {
    const int e_beg = nb, e_end = ne;
    e = first_edge();
    src = nsrc;
    if constexpr (FIRST) src = src_map[src];
    const int i_next = min(i + stride, N - 1);
    nb = rcv_off[i_next];
    ne = rcv_off[i_next + 1];
    if (e_beg < e_end) {
      group_sync<SH>(&s_cnt[wg], due);   // the previous receiver's reads come first
      build_g<LHMAX, SH>(dAt + (size_t)i * MID * K + 16 * ct, K, inv_c, ws, sg);
      group_sync<SH>(&s_cnt[wg], due);
    }
    nsrc = snd[first_edge()];
    for (int e0 = e_beg + 16 * ws; e0 < e_end; e0 += 16 * SH) {
      int e_next = min(e0 + 16 * SH + kk, e_end - 1);   // (after the last tile: unused)
      // an offset of zero the compiler cannot see through: W3's operands and the
      // G table are read per tile, not held in registers across tiles
      int z0 = 0;
      __asm__ volatile("" : "+v"(z0), "+v"(e_next)::"memory");
      const int ec = e;
      RadOp<RM, RM == 1 ? 1 : 3> a;
      RadOp<RM, RM == 1 ? 2 : 3> t;
      a.load(a3, e, g);
      t.load(t3, e, g);
      const float* hrow = h + (size_t)src * DIN * K + kb;
      f4 y4[4];
#pragma unroll
      for (int v = 0; v < 4; ++v) y4[v] = reinterpret_cast<const f4*>(Y + (size_t)e * 16)[v];
      float y[16], dy[16];
#pragma unroll
      for (int m = 0; m < 16; ++m) {
        y[m] = y4[m >> 2][m & 3];
        dy[m] = 0.f;
      }
      static_for<0, LHMAX + 1>([&](auto LHI) {
        constexpr int LH = decltype(LHI)::value;
        constexpr int PA = LH == 0 ? 0 : path_count(LH - 1), PB = path_count(LH);
        f4 r[PB - PA], rp[PB - PA], hv[2 * LH + 1], dh[2 * LH + 1];
#pragma unroll
        for (int m = 0; m < 2 * LH + 1; ++m) hv[m] = *reinterpret_cast<const f4*>(hrow + (LH * LH + m) * K);
        radial_group<PA, PB, P, RM>(sW + z0, a, t, r, rp);
        if constexpr (RND != 0) round_tile<PB - PA>(r, RND);
        if constexpr (LH == LHMAX) {
          fetch(e_next);
        }
#pragma unroll
        for (int m = 0; m < 2 * LH + 1; ++m) dh[m] = f4{0.f, 0.f, 0.f, 0.f};
        constexpr int G0 = PathPairOffset<PA>::value, G1 = PathPairOffset<PB>::value;
        const float* gq = sg + 4 * g + z0;
        f4 gring[kRingG];
#pragma unroll
        for (int u = 0; u < kRingG; ++u)
          if (G0 + u < G1) gring[u] = *reinterpret_cast<const f4*>(gq + (G0 + u) * 16);
        static_for<PA, PB>([&](auto PI) {
          using T = PathAt<decltype(PI)::value>;
          constexpr int ly = T::ly;
          constexpr int goff = PathPairOffset<T::index>::value;
          const f4 rv = r[T::index - PA];
          f4 Dm[2 * LH + 1], Rh[2 * LH + 1];
#pragma unroll
          for (int m = 0; m < 2 * LH + 1; ++m) {
            Dm[m] = f4{0.f, 0.f, 0.f, 0.f};
            Rh[m] = rv * hv[m];
          }
          mt::CG<LH, ly, T::lo>::each_pair([&](int m1, int m2, int pi) {
            const int gi = goff + pi;   // a constant after inlining
            __builtin_amdgcn_sched_barrier(0);   // keeps each read kRingG pairs ahead of its use
            const f4 G = gring[(gi - G0) % kRingG];
            if (gi + kRingG < G1) gring[(gi - G0) % kRingG] = *reinterpret_cast<const f4*>(gq + (gi + kRingG) * 16);
            if constexpr (ly == 0) {
              Dm[m1] += G;   // Y[0] = 1, and dY[0] is not wanted
            } else {
              Dm[m1] += G * y[ly * ly + m2];
              float s = dy[ly * ly + m2];
#pragma unroll
              for (int c = 0; c < 4; ++c) s += G[c] * Rh[m1][c];
              dy[ly * ly + m2] = s;
            }
          });
          f4 d = f4{0.f, 0.f, 0.f, 0.f};   // dE/dR
#pragma unroll
          for (int m = 0; m < 2 * LH + 1; ++m) {
            d += hv[m] * Dm[m];
            dh[m] += rv * Dm[m];
          }
          float s = dy[0];
#pragma unroll
          for (int c = 0; c < 4; ++c) s += d[c] * rp[T::index - PA][c];
          dy[0] = s;
        });
        if constexpr (!FIRST) {
#pragma unroll
          for (int m = 0; m < 2 * LH + 1; ++m)
            *reinterpret_cast<f4*>(Q + ((size_t)ec * DIN + LH * LH + m) * K + kb) = dh[m];
        }
      });
      // over the tile's 16 channels: the lane groups halve the elements twice;
      // group q ends with elements 4q .. 4q + 3
#pragma unroll
      for (int m = 0; m < 8; ++m) dy[m] = swap_add32(dy[m], dy[m + 8]);
#pragma unroll
      for (int m = 0; m < 4; ++m) dy[m] = swap_add16(dy[m], dy[m + 4]);
      *reinterpret_cast<f4*>(dYc + (size_t)ec * 16 + 4 * g) = f4{dy[0], dy[1], dy[2], dy[3]};
    }
  }
}

namespace {
// blocks per channel tile: the resident blocks of the whole chip shared
// among the channel tiles, a multiple of 8 where possible so that the channel
// tiles of one receiver group land on the same XCD (same L2)
int tpr_grid_x(int N, int n_ct, int waves, int blocks_per_cu) {
  const int want = std::max(8, (256 * blocks_per_cu / n_ct) & ~7);
  return std::max(1, std::min(want, (N + waves - 1) / waves));
}

template <int LH, int RM>
void tpr_fwd_launch(hipStream_t s, int N, int K, const int* rcv_off, const int* snd, const int* src_map,
                    const float* a3, const float* W3, const float* Y, const float* h, float inv_c, float* At,
                    int rnd) {
  using S = TprShape<LH, false>;
  const int n_ct = K / 16;
  dim3 grid(tpr_grid_x(N, n_ct, S::waves, S::blocks_per_cu), n_ct);
  if constexpr (RM == 3 || RM == 1) {
    if (K == 128) {
      tpr_fwd_kernel<LH, RM, S::waves, 128><<<grid, 64 * S::waves, 0, s>>>(N, K, rcv_off, snd, src_map, a3, W3, Y, h,
                                                                            inv_c, At, rnd);
      return;
    }
  }
  tpr_fwd_kernel<LH, RM><<<grid, 64 * S::waves, 0, s>>>(N, K, rcv_off, snd, src_map, a3, W3, Y, h, inv_c, At, rnd);
}

template <int LH, int RM>
void tpr_bwd_launch(hipStream_t s, int N, int K, int E, const int* rcv_off, const int* snd, const int* src_map,
                    const float* a3, const float* t3, const float* W3, const float* Y, const float* h, float inv_c,
                    const float* dAt, float* dYp, float* Q, int rnd) {
  using S = TprShape<LH, true, RM>;
  const int n_ct = K / 16;
  dim3 grid(tpr_grid_x(N, n_ct, S::waves / S::share, S::blocks_per_cu), n_ct);
  auto go = [&](auto F) {
    auto run = [&](auto R) {
      tpr_bwd_kernel<LH, RM, decltype(R)::value, decltype(F)::value><<<grid, 64 * S::waves, 0, s>>>(
          N, K, E, rcv_off, snd, src_map, a3, t3, W3, Y, h, inv_c, dAt, dYp, Q);
    };
    if (rnd == 1) run(std::integral_constant<int, 1>{});
    else if (rnd == 2) run(std::integral_constant<int, 2>{});
    else run(std::integral_constant<int, 0>{});
  };
  if constexpr (LH == 0) {
    if (!Q) {
      go(std::true_type{});
      return;
    }
  }
  go(std::false_type{});
}
}  // namespace

// Instances built: every l_h <= 2 with radial mode 0 (FP32), 1 (BF16) or 3
// (split BF16). The backward takes src_map and no Q (the first layer, l_h = 0) or
// Q and no src_map.
bool tpr_supported(int lh_max, int radial_mode) {
  return lh_max >= 0 && lh_max <= 2 && (radial_mode == 0 || radial_mode == 1 || radial_mode == 3);
}

bool launch_tpr_fwd(hipStream_t s, int lh_max, int N, int K, const int* rcv_off, const int* snd,
                    const int* src_map, const float* a3, const float* W3, const float* Y, const float* h,
                    float inv_c, float* At, int radial_mode, int tp_round) {
  if (!tpr_supported(lh_max, radial_mode)) return false;
  if (N <= 0) return true;
#define MACE_TPRF(LH)                                                                                              \
  if (radial_mode == 0) tpr_fwd_launch<LH, 0>(s, N, K, rcv_off, snd, src_map, a3, W3, Y, h, inv_c, At, tp_round);      \
  else if (radial_mode == 1) tpr_fwd_launch<LH, 1>(s, N, K, rcv_off, snd, src_map, a3, W3, Y, h, inv_c, At, tp_round); \
  else tpr_fwd_launch<LH, 3>(s, N, K, rcv_off, snd, src_map, a3, W3, Y, h, inv_c, At, tp_round)
  if (lh_max == 0) { MACE_TPRF(0); }
  else if (lh_max == 1) { MACE_TPRF(1); }
  else { MACE_TPRF(2); }
#undef MACE_TPRF
  return true;
}

bool launch_tpr_bwd(hipStream_t s, int lh_max, int N, int K, int E, const int* rcv_off, const int* snd,
                    const int* src_map, const float* a3, const float* t3, const float* W3, const float* Y,
                    const float* h, float inv_c, const float* dAt, float* dYp, float* Q, int radial_mode,
                    int tp_round) {
  if (!tpr_supported(lh_max, radial_mode) || !Q != !!src_map || (lh_max > 0 && !Q)) return false;
  if (N <= 0 || E <= 0) return true;
#define MACE_TPRB(LH, RM) tpr_bwd_launch<LH, RM>(s, N, K, E, rcv_off, snd, src_map, a3, t3, W3, Y, h, inv_c, dAt, dYp, Q, tp_round)
#define MACE_TPRB_ALL(LH)                  \
  if (radial_mode == 0) MACE_TPRB(LH, 0);      \
  else if (radial_mode == 1) MACE_TPRB(LH, 1); \
  else MACE_TPRB(LH, 3)
  if (lh_max == 0) { MACE_TPRB_ALL(0); }
  else if (lh_max == 1) { MACE_TPRB_ALL(1); }
  else { MACE_TPRB_ALL(2); }
#undef MACE_TPRB_ALL
#undef MACE_TPRB
  return true;
}

}  // namespace mace
