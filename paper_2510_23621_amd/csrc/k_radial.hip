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
#include <type_traits>

#include "mace_internal.h"

namespace mace {

typedef float f4 __attribute__((ext_vector_type(4)));

constexpr int kTE = 64;     // edges per block
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
typedef unsigned u4v __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f4 mfma_b16(us8v a, us8v b, f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf8v, a), __builtin_bit_cast(bf8v, b), c, 0, 0, 0);
}

// the three bfloat16 parts of eight FP32 values, element i of each operand
// word holding value i (two values per conversion)
__device__ __forceinline__ void split8(f4 lo, f4 hi, us8v& p0, us8v& p1, us8v& p2) {
  u4v w0, w1, w2;
#pragma unroll
  for (int h = 0; h < 4; ++h) {
    const f2v x = h < 2 ? f2v{lo[2 * h], lo[2 * h + 1]} : f2v{hi[2 * h - 4], hi[2 * h - 3]};
    unsigned a, b, c;
    split3_pair(x, a, b, c);
    w0[h] = a;
    w1[h] = b;
    w2[h] = c;
  }
  p0 = __builtin_bit_cast(us8v, w0);
  p1 = __builtin_bit_cast(us8v, w1);
  p2 = __builtin_bit_cast(us8v, w2);
}

// A operand parts of a 64 x 64 layer for this wave's 16 columns: W[k][col] for
// k = 32 ks + 8 (l/16) + i
__device__ __forceinline__ void load_w_parts64(const float* __restrict__ W, us8v (&b)[2][3]) {
  const int l = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int col = 16 * w + (l & 15);
  float v[2][8];
#pragma unroll
  for (int ks = 0; ks < 2; ++ks)
#pragma unroll
    for (int i = 0; i < 8; ++i) v[ks][i] = W[(32 * ks + 8 * (l >> 4) + i) * kH + col];
#pragma unroll
  for (int ks = 0; ks < 2; ++ks)
    split8(f4{v[ks][0], v[ks][1], v[ks][2], v[ks][3]}, f4{v[ks][4], v[ks][5], v[ks][6], v[ks][7]}, b[ks][0], b[ks][1],
           b[ks][2]);
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

// Edge prologue for a 64-edge tile: geometry of every edge (Y, written out, and
// the radial basis e; the first wave computes one edge per lane in FP64), then
// the hidden layers a3 = SiLU(SiLU(SiLU(e W0) W1) W2) of the radial MLP of
// every interaction layer in rs, all from the same e; with TAN also a3' =
// da3/dr from de/dr. RND: the precision study's rounding of every layer's
// input and weights (rs.rnd: 1 bfloat16, 2 binary16).
template <int NBP, bool TAN, bool RND>
__global__ void __launch_bounds__(256) edge_prologue_kernel(int E, const float* __restrict__ pos,
                                                            const int* __restrict__ snd, const int* __restrict__ rcv,
                                                            const double4* __restrict__ shift, double rc, int p,
                                                            int nb, float* __restrict__ Y, RadialSet rs,
                                                            int* __restrict__ status) {
  constexpr int NPASS = TAN ? 2 : 1, EP = kTE / NPASS;   // passes of EP edges
  __shared__ float xs[NPASS * kRows * kXPad];
  // RND: two FP32 activation tiles; otherwise the three part planes
  __shared__ __align__(16) float hbuf[RND ? 2 * kRows * kPad : 3 * kPlane / 2];
  unsigned short* P = reinterpret_cast<unsigned short*>(hbuf);
  const int e0 = blockIdx.x * kTE;
  const int l = threadIdx.x & 63, w = threadIdx.x >> 6;
  if (threadIdx.x < kTE) {
    const int e = e0 + threadIdx.x;
    float row[kXPad], trow[kXPad];
#pragma unroll
    for (int i = 0; i < kXPad; ++i) row[i] = trow[i] = 0.f;
    if (e < E) {
      float y[16];
      const int bad = edge_geometry<TAN>(e, pos, snd, rcv, shift, rc, p, nb, y, row, trow);
      if (bad) atomicOr(status, bad);
      float4* Yv = reinterpret_cast<float4*>(Y + (size_t)e * 16);
#pragma unroll
      for (int v = 0; v < 4; ++v) Yv[v] = make_float4(y[4 * v], y[4 * v + 1], y[4 * v + 2], y[4 * v + 3]);
    }
    float* x = xs + ((threadIdx.x / EP) * kRows + threadIdx.x % EP) * kXPad;
#pragma unroll
    for (int i = 0; i < kXPad; ++i) {
      x[i] = RND ? lowp_round(row[i], rs.rnd) : row[i];
      if constexpr (TAN) x[EP * kXPad + i] = trow[i];
    }
  }
  __syncthreads();
  for (int t = 0; t < rs.n; ++t) {
    const float* W0 = rs.W[t];
    const float* W1 = W0 + nb * kH;
    const float* W2 = W1 + kH * kH;
    if constexpr (RND) {
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
      // by their producer; the layer's weights stay in registers over the passes
      us8v b1[2][3], b2[2][3];
      float b0[NBP / 4];
      load_b_frag<NBP>(W0, nb, b0);
      load_w_parts64(W1, b1);
      load_w_parts64(W2, b2);
#pragma unroll
      for (int ps = 0; ps < NPASS; ++ps) {
        f4 z[4];
        input_mma_t<NBP>(xs + ps * kRows * kXPad, b0, z);
        activate<TAN>(z);
        if (t + ps > 0) __syncthreads();   // the previous pass's reads of the planes are done
        store_parts_t(z, P);
        __syncthreads();
        mma64_x3t(P, b1, z);
        activate<TAN>(z);
        __syncthreads();   // every wave has read the planes
        store_parts_t(z, P);
        __syncthreads();
        mma64_x3t(P, b2, z);
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
  const int g = (E + kTE - 1) / kTE;
  auto go = [&](auto T, auto R) {
    constexpr bool TAN = decltype(T)::value, RND = decltype(R)::value;
    if (nb <= 8) edge_prologue_kernel<8, TAN, RND><<<g, 256, 0, s>>>(E, pos, snd, rcv, shift, rc, p, nb, Y, rs, status);
    else edge_prologue_kernel<16, TAN, RND><<<g, 256, 0, s>>>(E, pos, snd, rcv, shift, rc, p, nb, Y, rs, status);
  };
  const bool tan = rs.tangent;
  if (rs.rnd) tan ? go(std::true_type{}, std::true_type{}) : go(std::false_type{}, std::true_type{});
  else tan ? go(std::true_type{}, std::false_type{}) : go(std::false_type{}, std::false_type{});
}

}  // namespace mace
