// Radial MLP of the edge weights (conv_tp_weights): e [E][nb] -> 64 -> 64 ->
// 64 -> R [E][P*K], bias-free, SiLU between layers, and its derivative with
// respect to the edge length. Weights are consecutive in the blob: W0
// [nb][64], W1 [64][64], W2 [64][64], W3 [64][P*K], each row-major [in][out].
//
// The three hidden layers run here (a3 [E][64] is written out); the wide last
// layer is computed inside the tensor-product kernels. The MLP's only input is
// the edge length r, so for forces the hidden layers are differentiated
// forward: the tangents de/dr -> da1/dr -> da2/dr -> a3' = da3/dr go through
// the same products as the values, as more rows of the same tile, and the
// backward kernels turn a3' into dE/dr. That is six 64-wide layer products per
// edge for value and derivative together, where recomputing the values and
// taking dE/da3 back through the transposed layers needs nine, and nothing of
// width 64 per channel tile goes through memory.
//
// A block owns a 64-edge tile and has 4 waves, wave w the 16 columns 16w ..
// 16w + 15 of a layer; a pass covers 64 rows (4 row tiles of 16): 64 edges'
// values, or 32 edges' values and then their tangents, so that a lane holds an
// edge's value and tangent in row tiles rt and rt + 2. The 64-wide layers run
// as FP32-accurate products on the bfloat16 MFMA pipe
// (v_mfma_f32_16x16x32_bf16; each FP32 operand carried as three bfloat16
// parts, six partial products, as in the edge product): lane l supplies
// A[l%16][8(l/16) + i] and B[8(l/16) + i][l%16], i = 0..7, and result register
// r holds D[4(l/16) + r][l%16]. The weights are the A operand and the
// activations of 16 rows the B operand, so that a lane's results are four
// consecutive columns of one row, which it splits into parts once for the
// next layer. The narrow input layer (nb <= 16 inputs) runs on FP32 MFMA
// (v_mfma_f32_16x16x4_f32, A[l%16][l/16], B[l/16][l%16]), with the same
// operand roles; the precision study's rounded instances run every layer on
// FP32 MFMA with the activations as A (results: rows 4(l/16) + r of column
// l%16).
#include <cmath>
#include <type_traits>

#include "mace_internal.h"

namespace mace {

typedef float f4 __attribute__((ext_vector_type(4)));

constexpr int kTE = 64;     // edges per block
// Up to this many edges a block takes half a tile (with tangents) and one
// interaction layer: four times the blocks, each with a quarter of the serial
// layers, at the cost of repeating the geometry per layer. Two layers with
// tangents: 342 edges 11 against 24 us, 82,900 edges 59 against 65; 249,000
// edges 155 against 150, 3.1 million 2,140 against 1,850.
constexpr int kSmallEdges = 131072;
constexpr int kRows = 64;   // rows of a pass: 64 edges, or 32 edges and their tangents
constexpr int kH = 64;      // hidden width
constexpr int kPad = kH + 4;   // row pitch = 4 (mod 32): A-fragment reads hit 2 lanes per bank
constexpr int kXPad = 20;  // padded row of the radial-basis tile (nb <= 16)

__device__ __forceinline__ f4 mfma4(float a, float b, f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// SiLU and its derivative from one evaluation of the logistic function; value
// and derivative as silu and silu_grad give them
__device__ __forceinline__ float silu_both(float x, float& d) {
  const float s = recip_ge1(1.f + exp_neg(x));
  d = s * (1.f + x * (1.f - s));
  return x * s;
}

// The activation of a pass: z -> silu(z), in place; with tangents (TAN) row
// tiles 2 and 3 hold dz/dr of row tiles 0 and 1 and become d silu(z)/dr
template <bool TAN>
__device__ __forceinline__ void activate(f4* z) {
#pragma unroll
  for (int rt = 0; rt < (TAN ? 2 : 4); ++rt)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      if constexpr (TAN) {
        float d;
        z[rt][r] = silu_both(z[rt][r], d);
        z[rt + 2][r] *= d;
      } else {
        z[rt][r] = silu(z[rt][r]);
      }
    }
}

template <int NIN_PAD, bool RND = false>
__device__ __forceinline__ void load_b_frag(const float* __restrict__ W, int nin, float* b, int rnd = 0) {
  const int l = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int col = 16 * w + (l & 15);
#pragma unroll
  for (int ks = 0; ks < NIN_PAD / 4; ++ks) {
    const int k = 4 * ks + (l >> 4);
    b[ks] = (k < nin) ? W[k * kH + col] : 0.f;
    if constexpr (RND) b[ks] = lowp_round(b[ks], rnd);
  }
}

// The rounded instances' layer: z = in W of the wave's columns (in: LDS rows of
// stride ldin), activated, the values rounded (the tangents are not: gradients
// pass through the rounding unchanged) and stored to out (stride kPad)
template <int NIN_PAD, bool TAN>
__device__ __forceinline__ void hidden_rnd(const float* __restrict__ in, int ldin, const float* b,
                                           float* __restrict__ out, int rnd) {
  const int l = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int col = 16 * w + (l & 15);
  f4 z[4];
#pragma unroll
  for (int rt = 0; rt < 4; ++rt) z[rt] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int ks = 0; ks < NIN_PAD / 4; ++ks) {
    const int k = 4 * ks + (l >> 4);
#pragma unroll
    for (int rt = 0; rt < 4; ++rt) z[rt] = mfma4(in[(16 * rt + (l & 15)) * ldin + k], b[ks], z[rt]);
  }
  activate<TAN>(z);
#pragma unroll
  for (int rt = 0; rt < 4; ++rt)
#pragma unroll
    for (int r = 0; r < 4; ++r)
      out[(16 * rt + 4 * (l >> 4) + r) * kPad + col] = (TAN && rt >= 2) ? z[rt][r] : lowp_round(z[rt][r], rnd);
}

// ---- 64-wide layers on split-BF16 MFMA
typedef unsigned short us8v __attribute__((ext_vector_type(8)));
typedef __bf16 bf8v __attribute__((ext_vector_type(8)));

__device__ __forceinline__ f4 mfma_b16(us8v a, us8v b, f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf8v, a), __builtin_bit_cast(bf8v, b), c, 0, 0, 0);
}

// A operand parts of a 64 x 64 layer for this wave's 16 columns: W[k][col] for
// k = 32 ks + 8 (l/16) + i, from the copy split at setup ([64/8][64][8] per part)
__device__ __forceinline__ void load_w_parts64(const unsigned short* __restrict__ W, int64_t part, us8v (&b)[2][3]) {
  const int l = threadIdx.x & 63, w = threadIdx.x >> 6;
  const unsigned short* f = W + ((l >> 4) * kH + 16 * w + (l & 15)) * 8;
#pragma unroll
  for (int ks = 0; ks < 2; ++ks)
#pragma unroll
    for (int q = 0; q < 3; ++q) b[ks][q] = *reinterpret_cast<const us8v*>(f + q * part + 4 * 8 * kH * ks);
}

// ---- layers with the operands' roles swapped: A = the weights' column
// fragment of the wave's 16 columns, B = the activations of 16 rows, so that
// result register r of lane l holds column 16w + 4(l/16) + r of row
// 16 rt + l%16 (four consecutive columns of one row per lane). Each layer's
// output is split into its three bfloat16 parts once, by the wave that
// produced it, into part planes in LDS (pitch kPP), which every wave of the
// next layer reads as its B operand.
constexpr int kPP = kH + 8;          // 72 bfloat16 per plane row (36 dwords, 4 mod 32)
constexpr int kPlane = kRows * kPP;  // elements per part plane

__device__ __forceinline__ void store_parts_t(const f4* z, unsigned short* __restrict__ P) {
  const int l = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
  for (int rt = 0; rt < 4; ++rt) {
    unsigned p0[2], p1[2], p2[2];
    split3_pair(f2v{z[rt][0], z[rt][1]}, p0[0], p1[0], p2[0]);
    split3_pair(f2v{z[rt][2], z[rt][3]}, p0[1], p1[1], p2[1]);
    unsigned short* d = P + (16 * rt + (l & 15)) * kPP + 16 * w + 4 * (l >> 4);
    *reinterpret_cast<uint2*>(d) = make_uint2(p0[0], p0[1]);
    *reinterpret_cast<uint2*>(d + kPlane) = make_uint2(p1[0], p1[1]);
    *reinterpret_cast<uint2*>(d + 2 * kPlane) = make_uint2(p2[0], p2[1]);
  }
}

// the narrow input layer on FP32 MFMA, operands swapped: z = (x W0) of the
// wave's columns for the pass's 64 rows (x: LDS rows of stride kXPad)
template <int NIN_PAD>
__device__ __forceinline__ void input_mma_t(const float* __restrict__ xs, const float* b, f4* z) {
  const int l = threadIdx.x & 63;
#pragma unroll
  for (int rt = 0; rt < 4; ++rt) z[rt] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int ks = 0; ks < NIN_PAD / 4; ++ks)
#pragma unroll
    for (int rt = 0; rt < 4; ++rt) z[rt] = mfma4(b[ks], xs[(16 * rt + (l & 15)) * kXPad + 4 * ks + (l >> 4)], z[rt]);
}

// a 64-input layer on split-BF16 products from part planes, operands swapped;
// within each K step the six partial products go from the smallest to the
// largest
__device__ __forceinline__ void mma64_x3t(const unsigned short* __restrict__ P, const us8v (&b)[2][3], f4* z) {
  const int l = threadIdx.x & 63;
#pragma unroll
  for (int rt = 0; rt < 4; ++rt) z[rt] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int ks = 0; ks < 2; ++ks)
#pragma unroll
    for (int rt = 0; rt < 4; ++rt) {
      const unsigned short* ar = P + (16 * rt + (l & 15)) * kPP + 32 * ks + 8 * (l >> 4);
      const us8v a0 = *reinterpret_cast<const us8v*>(ar);
      const us8v a1 = *reinterpret_cast<const us8v*>(ar + kPlane);
      const us8v a2 = *reinterpret_cast<const us8v*>(ar + 2 * kPlane);
      f4 c = z[rt];
      c = mfma_b16(b[ks][0], a2, c);
      c = mfma_b16(b[ks][1], a1, c);
      c = mfma_b16(b[ks][2], a0, c);
      c = mfma_b16(b[ks][0], a1, c);
      c = mfma_b16(b[ks][1], a0, c);
      z[rt] = mfma_b16(b[ks][0], a0, c);
    }
}

// Four consecutive columns c0 .. c0 + 3 of edge e of a hidden output: FP32
// [E][64], or (x) its three bfloat16 parts [E][3][64]
__device__ __forceinline__ void store_row4(float* __restrict__ a, unsigned short* __restrict__ x, int e, int c0, f4 v) {
  if (x) {
    unsigned p0[2], p1[2], p2[2];
    split3_pair(f2v{v[0], v[1]}, p0[0], p1[0], p2[0]);
    split3_pair(f2v{v[2], v[3]}, p0[1], p1[1], p2[1]);
    unsigned short* row = x + (size_t)e * 3 * kH + c0;
    *reinterpret_cast<uint2*>(row) = make_uint2(p0[0], p0[1]);
    *reinterpret_cast<uint2*>(row + kH) = make_uint2(p1[0], p1[1]);
    *reinterpret_cast<uint2*>(row + 2 * kH) = make_uint2(p2[0], p2[1]);
  } else {
    *reinterpret_cast<f4*>(a + (size_t)e * kH + c0) = v;
  }
}

// Edge prologue for a tile of TE edges: geometry of every edge (Y, written out,
// and the radial basis e; the first wave computes one edge per lane in FP64),
// then the hidden layers a3 = SiLU(SiLU(SiLU(e W0) W1) W2) of the radial MLP of
// the interaction layers in rs, all from the same e; with TAN also a3' =
// da3/dr from de/dr. RND: the precision study's rounding of every layer's
// input and weights (rs.rnd: 1 bfloat16, 2 binary16). ONE: one interaction
// layer per block (blockIdx.y), the first one's blocks write Y.
template <int NBP, bool TAN, bool RND, int TE, bool ONE>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3)))
edge_prologue_kernel(int E, const float* __restrict__ pos, const int* __restrict__ snd, const int* __restrict__ rcv,
                     const double4* __restrict__ shift, RadialBasis rb, float* __restrict__ Y, RadialSet rs,
                     int* __restrict__ status) {
  constexpr int EP = TAN ? kRows / 2 : kRows, NPASS = TE / EP;   // passes of EP edges
  static_assert(NPASS >= 1 && TE <= 64, "whole passes, one edge per lane of a wave");
  __shared__ float xs[NPASS * kRows * kXPad];
  // RND: two FP32 activation tiles; otherwise the three part planes
  __shared__ __align__(16) float hbuf[RND ? 2 * kRows * kPad : 3 * kPlane / 2];
  unsigned short* P = reinterpret_cast<unsigned short*>(hbuf);
  const int e0 = blockIdx.x * TE;
  const int l = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int t0 = ONE ? blockIdx.y : 0, t1 = ONE ? t0 + 1 : rs.n;
  const int nb = rb.nb;
  // one 64-wide layer's weights in registers at a time, each requested while
  // the values before it are still being computed
  us8v b[2][3];
  if constexpr (!RND) load_w_parts64(rs.Wx[t0], rs.wx_part, b);
  if (threadIdx.x < TE) {
    const int e = e0 + threadIdx.x;
    float row[NBP], trow[NBP];
#pragma unroll
    for (int i = 0; i < NBP; ++i) row[i] = trow[i] = 0.f;
    if (e < E) {
      float y[16];
      const int bad = edge_geometry<NBP, TAN>(e, pos, snd, rcv, shift, rb, y, row, trow);
      if (t0 == 0) {
        if (bad) atomicOr(status, bad);
        float4* Yv = reinterpret_cast<float4*>(Y + (size_t)e * 16);
#pragma unroll
        for (int v = 0; v < 4; ++v) Yv[v] = make_float4(y[4 * v], y[4 * v + 1], y[4 * v + 2], y[4 * v + 3]);
      }
    }
    float* x = xs + ((threadIdx.x / EP) * kRows + threadIdx.x % EP) * kXPad;
#pragma unroll
    for (int i = 0; i < NBP; ++i) {
      x[i] = RND ? lowp_round(row[i], rs.rnd) : row[i];
      if constexpr (TAN) x[EP * kXPad + i] = trow[i];
    }
  }
  __syncthreads();
  for (int t = t0; t < t1; ++t) {
    const float* W0 = rs.W[t];
    if constexpr (RND) {
      const float* W1 = W0 + nb * kH;
      const float* W2 = W1 + kH * kH;
      float* ha = hbuf;
      float* hb = hbuf + kRows * kPad;
      float b0[NBP / 4], b1[kH / 4], b2[kH / 4];
      load_b_frag<NBP, RND>(W0, nb, b0, rs.rnd);
      load_b_frag<kH, RND>(W1, kH, b1, rs.rnd);
      load_b_frag<kH, RND>(W2, kH, b2, rs.rnd);
      for (int ps = 0; ps < NPASS; ++ps) {
        hidden_rnd<NBP, TAN>(xs + ps * kRows * kXPad, kXPad, b0, ha, rs.rnd);
        __syncthreads();
        hidden_rnd<kH, TAN>(ha, kPad, b1, hb, rs.rnd);
        __syncthreads();
        hidden_rnd<kH, TAN>(hb, kPad, b2, ha, rs.rnd);
        __syncthreads();
        for (int idx = threadIdx.x; idx < kRows * kH / 4; idx += blockDim.x) {
          const int row = idx >> 4, c4 = idx & 15;
          const bool tan = TAN && row >= EP;
          const int e = e0 + ps * EP + (tan ? row - EP : row);
          if (e < E)
            store_row4(tan ? rs.t3[t] : rs.a3[t], tan ? rs.t3x[t] : rs.a3x[t], e, 4 * c4,
                       *reinterpret_cast<const f4*>(ha + row * kPad + 4 * c4));
        }
        __syncthreads();   // ha is rewritten by the next pass
      }
    } else {
      // the 64-wide layers on split-BF16 products from part planes split once
      // by their producer. Bound by issue (67 % of the cycles vector, 28 % MFMA)
      // beside 1.3 KB written per edge. The weights split at setup and one layer
      // of them in registers (116 in all, four waves per SIMD in place of three)
      // took 3.1 million edges of two layers from 2.10 to 1.85 ms, 445,000 from
      // 0.378 to 0.315
      float b0[NBP / 4];
      load_b_frag<NBP>(W0, nb, b0);
#pragma unroll
      for (int ps = 0; ps < NPASS; ++ps) {
        f4 z[4];
        input_mma_t<NBP>(xs + ps * kRows * kXPad, b0, z);
        activate<TAN>(z);
        if (t + ps > t0) __syncthreads();   // the previous pass's reads of the planes are done
        store_parts_t(z, P);
        __syncthreads();
        mma64_x3t(P, b, z);
        load_w_parts64(rs.Wx[t] + kH * kH, rs.wx_part, b);
        activate<TAN>(z);
        __syncthreads();   // every wave has read the planes
        store_parts_t(z, P);
        __syncthreads();
        mma64_x3t(P, b, z);
        if (ps + 1 < NPASS || t + 1 < t1) load_w_parts64(rs.Wx[ps + 1 < NPASS ? t : t + 1], rs.wx_part, b);
        activate<TAN>(z);
        // four consecutive columns of one edge per lane, straight to memory
        const int c0 = 16 * w + 4 * (l >> 4);
#pragma unroll
        for (int rt = 0; rt < 4; ++rt) {
          const bool tan = TAN && rt >= 2;
          const int e = e0 + ps * EP + 16 * (tan ? rt - 2 : rt) + (l & 15);
          if (e < E) store_row4(tan ? rs.t3[t] : rs.a3[t], tan ? rs.t3x[t] : rs.a3x[t], e, c0, z[rt]);
        }
      }
    }
  }
}

void launch_edge_prologue(hipStream_t s, int E, const float* pos, const int* snd, const int* rcv,
                          const double4* shift, double rc, int p, int nb, float* Y, const RadialSet& rs, int* status) {
  if (E <= 0) return;
  const RadialBasis rb = radial_basis(rc, p, nb);
  auto go = [&](auto T, auto R) {
    constexpr bool TAN = decltype(T)::value, RND = decltype(R)::value;
    auto run = [&](auto TE, auto ONE) {
      constexpr int te = decltype(TE)::value;
      constexpr bool one = decltype(ONE)::value;
      const dim3 g((E + te - 1) / te, one ? rs.n : 1);
      if (nb <= 8) edge_prologue_kernel<8, TAN, RND, te, one><<<g, 256, 0, s>>>(E, pos, snd, rcv, shift, rb, Y, rs, status);
      else edge_prologue_kernel<16, TAN, RND, te, one><<<g, 256, 0, s>>>(E, pos, snd, rcv, shift, rb, Y, rs, status);
    };
    if constexpr (!RND) {
      if (E <= kSmallEdges) {
        run(std::integral_constant<int, TAN ? 32 : 64>{}, std::true_type{});
        return;
      }
    }
    run(std::integral_constant<int, kTE>{}, std::false_type{});
  };
  const bool tan = rs.tangent;
  if (rs.rnd) tan ? go(std::true_type{}, std::true_type{}) : go(std::false_type{}, std::true_type{});
  else tan ? go(std::true_type{}, std::false_type{}) : go(std::false_type{}, std::false_type{});
}

}  // namespace mace
