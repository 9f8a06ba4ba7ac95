// Device neighbour list for the graph problem statement: sender j -> receiver
// i with image shift S is an edge iff
//   0 < (d_x^2 + d_y^2) + d_z^2 < r_c^2,  d = (x_j - x_i) + ((S_0 a_0 + S_1 a_1) + S_2 a_2),
// evaluated in FP64 with this operation order and no fused multiply-adds (the
// same expression as the host list, so both produce the same edge set), every
// periodic image enumerated, graphs never joined, output sorted by
// (receiver, sender, S_0, S_1, S_2).
//
// Method (hashed cell list):
//  1. every atom of a periodic graph is wrapped into its cell, x = x_w + n.cell
//     with n = floor(fractional coordinates); the wrapped fractional
//     coordinates lie in [0, 1), so images S' with |S'_a| <= floor(r_c |b_a| + 1)
//     (b_a the reciprocal row) cover every pair within r_c, and of those only
//     the images whose fractional coordinates lie within r_c |b_a| of [0, 1);
//  2. every such image p = x_w + S'.cell of every atom (a candidate) is binned in
//     Cartesian cubes of edge r_c + 1e-6, the cube (with the graph) hashed into
//     a power-of-two slot table; a counting sort groups candidates by slot, with
//     a 16-byte record for the distance pre-test (the place inside the cube in
//     FP32, and the cube's coordinates mod 4);
//  3. one wave per receiver visits the 27 cubes around it. A candidate whose
//     record names another cube mod 4 is not of the visited cube (mod 4 tells
//     the 27 apart, so none is taken twice); the FP32 distance discards pairs
//     beyond r_c with a margin for its rounding; what is left (little more than
//     the edges) takes the exact test above with the shift of the given
//     (unwrapped) positions, S = S' - n_j + n_i. A first pass counts, a scan gives
//     each receiver its output segment, a second pass writes it sorted by
//     (sender, S), which is the order of the candidates' numbers.
// Binning and the pre-test only select candidates; the cube edge exceeds r_c, so
// no pair within r_c is missed, and every edge passes the exact FP64 test.
//
// 36,864 periodic atoms (3.18 M edges): 0.23 ms per call (1.66 ms with all 27
// images of every atom binned and each candidate searched for its cube and
// gathered through five dependent loads); 1,536 atoms: 94 us (144 us), the
// launches and the wait for the count.
#pragma clang fp contract(off)

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <mutex>
#include <vector>

#include "../../include/mace.h"

namespace {

struct NlGraph {
  double cell[9];     // rows = lattice vectors; zero without periodicity
  double inv[9];      // cell^-1: fractional coordinate a = x . column a
  float slack[3];     // how far outside [0, 1) a useful image's fractional coordinates lie
  int16_t nr[3];      // wrapped-image range per lattice direction (below 10^4)
  int16_t periodic;
  int a0, a1;         // atoms [a0, a1)
  int nimg;           // images per atom, prod (2 nr_a + 1)
  int64_t c0;         // first candidate of the graph
};
static_assert(sizeof(NlGraph) == 184, "counted on by the workspace's size (plan_nl)");

constexpr int kNlThreads = 256;
constexpr int kScanPerThread = 16;
constexpr int kScanTile = kNlThreads * kScanPerThread;
constexpr int kScanOneBlock = 65536;  // atoms up to which one block scans the counts (one launch in place of three)
constexpr double kCoordLimit = 1e9;   // |coordinate| bound (keeps cube indices in int32)
constexpr int kFlagNonFinite = 1, kFlagRange = 2;

// Graph of candidate c; one graph comes by value (g0), several in memory.
__device__ __forceinline__ const NlGraph& graph_of_cand(const NlGraph& g0, const NlGraph* gs, int G, int64_t c,
                                                        int& gi) {
  gi = 0;
  if (G == 1) return g0;
  int lo = 0, hi = G - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (gs[mid].c0 <= c) lo = mid;
    else hi = mid - 1;
  }
  gi = lo;
  return gs[lo];
}

__device__ __forceinline__ uint32_t slot_of(int g, int bx, int by, int bz, uint32_t mask) {
  uint64_t h = (uint64_t)(uint32_t)g;
  h = h * 0x100000001B3ull + (uint32_t)bx;
  h = h * 0x100000001B3ull + (uint32_t)by;
  h = h * 0x100000001B3ull + (uint32_t)bz;
  h ^= h >> 33;   // splitmix64 finaliser
  h *= 0xFF51AFD7ED558CCDull;
  h ^= h >> 33;
  h *= 0xC4CEB9FE1A85EC53ull;
  h ^= h >> 33;
  return (uint32_t)h & mask;
}

__device__ __forceinline__ int cube(double p, double bs) { return (int)floor(p / bs); }

// A candidate's record of the pre-test: its place inside its cube (FP32), and the
// cube's coordinates mod 4 with the graph's low bits.
__device__ __forceinline__ uint32_t cube_code(int g, int bx, int by, int bz) {
  return (uint32_t)(bx & 3) | (uint32_t)(by & 3) << 2 | (uint32_t)(bz & 3) << 4 | (uint32_t)g << 6;
}

// One thread per (atom j, image S'), in the order of the candidates' numbers c:
// wrap the atom, drop images out of reach, find the cube and its slot.
// SCATTER = false counts the slots' populations (the thread of S' = 0 also
// stores the atom's own records and flags non-finite or huge coordinates),
// SCATTER = true places the candidates: `cursor` holds each slot's next place.
template <bool SCATTER>
__global__ void __launch_bounds__(kNlThreads)
nl_bin_kernel(int64_t C, const double* __restrict__ pos, NlGraph g0, const NlGraph* __restrict__ gs, int G,
              double bs, uint32_t mask, int4* __restrict__ nsh, int4* __restrict__ rcube, float4* __restrict__ rplace,
              int* __restrict__ flags, int* __restrict__ count, int* __restrict__ cursor, float4* __restrict__ place,
              int4* __restrict__ rec, int* __restrict__ num) {
  const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= C) return;
  int gi;
  const NlGraph& g = graph_of_cand(g0, gs, G, c, gi);
  const uint32_t local = (uint32_t)(c - g.c0);   // candidates number at most 2^30
  const int j = g.a0 + (int)(local / (uint32_t)g.nimg);
  uint32_t s = local % (uint32_t)g.nimg;
  const uint32_t w2 = 2 * g.nr[2] + 1, w1 = 2 * g.nr[1] + 1;
  const int s2 = (int)(s % w2) - g.nr[2];
  s /= w2;
  const int s1 = (int)(s % w1) - g.nr[1];
  const int s0 = (int)(s / w1) - g.nr[0];
  const bool home = s0 == 0 && s1 == 0 && s2 == 0;
  const double x[3] = {pos[3 * (size_t)j], pos[3 * (size_t)j + 1], pos[3 * (size_t)j + 2]};
  int bad = 0;
  for (int q = 0; q < 3; ++q) {
    if (!isfinite(x[q])) bad |= kFlagNonFinite;
    else if (fabs(x[q]) > kCoordLimit) bad |= kFlagRange;
  }
  if (bad) {   // the call fails: no candidate, no receiver
    if (!SCATTER && home) {
      atomicOr(flags, bad);
      nsh[j] = make_int4(0, 0, 0, -1);
    }
    return;
  }
  int n[3] = {0, 0, 0};
  double w[3] = {x[0], x[1], x[2]};
  if (g.periodic) {
    for (int a = 0; a < 3; ++a) n[a] = (int)floor((x[0] * g.inv[0 * 3 + a] + x[1] * g.inv[1 * 3 + a]) + x[2] * g.inv[2 * 3 + a]);
    for (int q = 0; q < 3; ++q)
      w[q] = x[q] - (((double)n[0] * g.cell[0 * 3 + q] + (double)n[1] * g.cell[1 * 3 + q]) + (double)n[2] * g.cell[2 * 3 + q]);
    const int S[3] = {s0, s1, s2};
    bool near = true;
    for (int a = 0; a < 3; ++a) {
      const double f = ((w[0] * g.inv[0 * 3 + a] + w[1] * g.inv[1 * 3 + a]) + w[2] * g.inv[2 * 3 + a]) + (double)S[a];
      near = near && f >= -(double)g.slack[a] && f <= 1.0 + (double)g.slack[a];
    }
    if (!near && !home) return;
  }
  int b[3];
  float r[3];
  for (int q = 0; q < 3; ++q) {
    const double p = w[q] + (((double)s0 * g.cell[0 * 3 + q] + (double)s1 * g.cell[1 * 3 + q]) +
                             (double)s2 * g.cell[2 * 3 + q]);
    b[q] = cube(p, bs);
    r[q] = (float)(p - (double)b[q] * bs);
  }
  const uint32_t slot = slot_of(gi, b[0], b[1], b[2], mask);
  if constexpr (!SCATTER) {
    atomicAdd(&count[slot], 1);
    if (home) {
      nsh[j] = make_int4(n[0], n[1], n[2], gi);
      rcube[j] = make_int4(b[0], b[1], b[2], 0);
      rplace[j] = make_float4(r[0], r[1], r[2], 0.f);
    }
  } else {
    const int at = atomicAdd(&cursor[slot], 1);
    place[at] = make_float4(r[0], r[1], r[2], __uint_as_float(cube_code(gi, b[0], b[1], b[2])));
    rec[at] = make_int4(s0 - n[0], s1 - n[1], s2 - n[2], j);
    num[at] = (int)c;
  }
}

// Receiver pass, one wave per receiver: WRITE = false counts the edges of
// receiver i, WRITE = true writes them to [off_i, off_{i+1}) sorted by (sender,
// S), unless the total exceeds max_edges or a coordinate was bad. Each half-wave
// takes every second non-empty cube, 32 candidates at a time; pairs that pass
// the pre-test go to a list in LDS, which takes the exact test 64 at a time. The
// count pass keeps up to found_cap of each receiver's finds, as many as the
// workspace has left over, and the write pass searches again where there are
// more: in periodic systems that is room for 249 and more, all of them as a
// rule; without images, from a few hundred atoms on, 5 to 10, so that those
// lists are searched twice (512 molecules 151 us per call, 65,536 atoms in one
// cluster 330; a larger find list was not measured). A segment is sorted by rank
// (a candidate's place = the number of candidates of the segment with a lower
// number), in LDS up to kNlSortCap edges, beyond it through the segment's own
// output arrays.
constexpr int kNlWaves = 4;        // receivers per block
constexpr int kNlSortCap = 256;    // edges per receiver sorted through LDS
constexpr int kNlList = 256;       // pre-test list entries from which it is emptied

__device__ __forceinline__ void wave_fence() {
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
}
__device__ __forceinline__ int lanes_below(uint64_t mask) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0));
}

template <bool WRITE>
__global__ void __launch_bounds__(64 * kNlWaves)
nl_receiver_kernel(int N, const double* __restrict__ pos, NlGraph g0, const NlGraph* __restrict__ gs, int G,
                   double bs, double rc2, float pre2, uint32_t mask, const int4* __restrict__ nsh,
                   const int4* __restrict__ rcube, const float4* __restrict__ rplace, const int* __restrict__ slot_cnt,
                   const int* __restrict__ slot_end, const float4* __restrict__ place, const int4* __restrict__ rec,
                   const int* __restrict__ num, int* __restrict__ found, int found_cap, int* __restrict__ count,
                   const int64_t* __restrict__ off, int64_t max_edges, int32_t* __restrict__ sender, int32_t* __restrict__ receiver,
                   int32_t* __restrict__ shifts) {
  __shared__ int s_first[kNlWaves][27], s_len[kNlWaves][27];
  __shared__ uint32_t s_code[kNlWaves][27];
  __shared__ float s_shift[kNlWaves][27][3];
  __shared__ int s_list[kNlWaves][kNlList + 64];
  __shared__ __align__(16) int s_key[WRITE ? kNlWaves : 1][WRITE ? kNlSortCap + 4 : 4];   // candidates' numbers
  __shared__ int s_at[WRITE ? kNlWaves : 1][WRITE ? kNlSortCap : 1];                      // and places
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int i = blockIdx.x * kNlWaves + w;
  if (i >= N) return;   // whole wave; no block-wide barrier below
  int64_t base = 0, n_expect = 0;
  if (WRITE) {
    if (off[N] > max_edges || off[N + 1] != 0) return;   // (the flags sit behind the total)
    base = off[i];
    n_expect = off[i + 1] - base;
    if (n_expect == 0) return;
  }
  const bool in_lds = n_expect <= kNlSortCap;
  const int4 ni = nsh[i];
  int64_t n = 0;
  const int* mine = found + (size_t)i * found_cap;   // the count pass's finds
  if (WRITE && n_expect <= found_cap) {
    for (int a = lane; a < (int)n_expect; a += 64) {
      const int at = mine[a];
      s_at[w][a] = at;
      s_key[w][a] = num[at];
    }
  } else if (ni.w >= 0) {
    const int gi = ni.w;
    const NlGraph& g = G == 1 ? g0 : gs[gi];
    const int4 bi = rcube[i];
    const float4 ri = rplace[i];
    const double xi[3] = {pos[3 * (size_t)i], pos[3 * (size_t)i + 1], pos[3 * (size_t)i + 2]};
    // lanes 0..26: one neighbouring cube each; the non-empty ones to LDS
    int len = 0, first = 0, bx = 0, by = 0, bz = 0;
    if (lane < 27) {
      bx = lane / 9 - 1;
      by = (lane / 3) % 3 - 1;
      bz = lane % 3 - 1;
      const uint32_t slot = slot_of(gi, bi.x + bx, bi.y + by, bi.z + bz, mask);
      len = slot_cnt[slot];
      first = slot_end[slot] - len;
    }
    const uint64_t filled = __ballot(len > 0);
    if (len > 0) {
      const int at = lanes_below(filled);
      s_first[w][at] = first;
      s_len[w][at] = len;
      s_code[w][at] = cube_code(gi, bi.x + bx, bi.y + by, bi.z + bz);
      s_shift[w][at][0] = (float)(bx * bs) - ri.x;
      s_shift[w][at][1] = (float)(by * bs) - ri.y;
      s_shift[w][at][2] = (float)(bz * bs) - ri.z;
    }
    wave_fence();
    const int m = __popcll(filled);
    int listed = 0;
    // the exact test of the listed candidates
    auto empty_list = [&]() {
      wave_fence();
      for (int k0 = 0; k0 < listed; k0 += 64) {
        const int k = k0 + lane;
        bool hit = false;
        int at = 0, j = 0;
        if (k < listed) {
          at = s_list[w][k];
          const int4 t = rec[at];
          j = t.w;
          const int S[3] = {t.x + ni.x, t.y + ni.y, t.z + ni.z};
          double d[3];
          for (int q = 0; q < 3; ++q) {
            const double sv = g.periodic ? ((double)S[0] * g.cell[0 * 3 + q] + (double)S[1] * g.cell[1 * 3 + q]) +
                                               (double)S[2] * g.cell[2 * 3 + q]
                                         : 0.0;
            d[q] = (pos[3 * (size_t)j + q] - xi[q]) + sv;
          }
          const double r2 = (d[0] * d[0] + d[1] * d[1]) + d[2] * d[2];
          hit = r2 < rc2 && r2 > 0.0 && j >= g.a0 && j < g.a1;
        }
        const uint64_t bal = __ballot(hit);
        if (hit) {
          const int64_t to = n + lanes_below(bal);
          if constexpr (!WRITE) {
            if (to < found_cap) found[(size_t)i * found_cap + to] = at;
          } else if (in_lds) {
            if (to < kNlSortCap) {
              s_key[w][to] = num[at];
              s_at[w][to] = at;
            }
          } else {
            sender[base + to] = num[at];
            shifts[3 * (base + to)] = at;
          }
        }
        n += __popcll(bal);
      }
      listed = 0;
      wave_fence();
    };
    // A step is 32 candidates of one cube for each half-wave (a cube of more
    // takes several); the next step's records are requested before this one's
    // are tested.
    const int half = lane >> 5, hl = lane & 31;
    struct Step {
      float4 v;
      int at;
      uint32_t code;   // no record's code where the lane has no candidate
      float sx, sy, sz;
    };
    int c0 = 0, t = 0, longest = 0, cl = 0, cf = 0;
    auto next = [&](Step& st) {   // false past the last cube
      if (t >= longest) {
        if (c0 >= m) return false;
        const int c = min(c0 + half, m - 1);
        cl = c0 + half < m ? s_len[w][c] : 0;
        cf = s_first[w][c];
        st.code = s_code[w][c];
        st.sx = s_shift[w][c][0];
        st.sy = s_shift[w][c][1];
        st.sz = s_shift[w][c][2];
        longest = max(__builtin_amdgcn_readlane(cl, 0), __builtin_amdgcn_readlane(cl, 32));
        t = 0;
        c0 += 2;
      }
      st.at = t + hl < cl ? cf + t + hl : -1;
      st.v = place[max(st.at, 0)];
      t += 32;
      return true;
    };
    Step st;
    bool more = next(st);
    while (more) {
      const Step now = st;
      more = next(st);
      const float dx = now.v.x + now.sx, dy = now.v.y + now.sy, dz = now.v.z + now.sz;
      // (not >=: a place beyond FP32, where the cutoff is, gives NaN and goes to the exact test)
      const bool pass = now.at >= 0 && __float_as_uint(now.v.w) == now.code && !((dx * dx + dy * dy) + dz * dz >= pre2);
      const uint64_t bal = __ballot(pass);
      if (pass) s_list[w][listed + lanes_below(bal)] = now.at;
      listed += __popcll(bal);
      if (listed >= kNlList) empty_list();
    }
    empty_list();
  }
  if (!WRITE) {
    if (lane == 0) count[i] = (int)n;
    return;
  }
  const int4* recs = rec;
  auto put = [&](int64_t e, int at) {
    const int4 t = recs[at];
    sender[e] = t.w;
    receiver[e] = i;
    shifts[3 * e] = t.x + ni.x;
    shifts[3 * e + 1] = t.y + ni.y;
    shifts[3 * e + 2] = t.z + ni.z;
  };
  if (in_lds) {
    const int ne = (int)n_expect;
    if (lane < 4) s_key[w][ne + lane] = 0x7fffffff;   // past the end: below no number
    wave_fence();
    int rank[kNlSortCap / 64] = {}, key[kNlSortCap / 64];
#pragma unroll
    for (int u = 0; u < kNlSortCap / 64; ++u) key[u] = s_key[w][min(lane + 64 * u, ne)];
    for (int b = 0; b < ne; b += 4) {
      const int4 kb = *reinterpret_cast<const int4*>(&s_key[w][b]);
#pragma unroll
      for (int u = 0; u < kNlSortCap / 64; ++u) {
        if (64 * u >= ne) break;   // uniform
        rank[u] += (kb.x < key[u]) + (kb.y < key[u]) + (kb.z < key[u]) + (kb.w < key[u]);
      }
    }
#pragma unroll
    for (int u = 0; u < kNlSortCap / 64; ++u)
      if (lane + 64 * u < ne) s_list[w][rank[u]] = s_at[w][lane + 64 * u];
    wave_fence();
    for (int a = lane; a < ne; a += 64) put(base + a, s_list[w][a]);
    return;
  }
  // long segment: the numbers lie in sender[], the places in shifts[3 e]; the
  // places go to receiver[] in sorted order, then every edge is written
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
  __builtin_amdgcn_wave_barrier();
  for (int64_t a = lane; a < n_expect; a += 64) {
    const int32_t key = sender[base + a];
    int64_t rank = 0;
    for (int64_t b = 0; b < n_expect; ++b) rank += sender[base + b] < key;
    receiver[base + rank] = shifts[3 * (base + a)];
  }
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
  __builtin_amdgcn_wave_barrier();
  for (int64_t a = lane; a < n_expect; a += 64) put(base + a, receiver[base + a]);
}

// Every slot's first place: a block's slots in order, the blocks in any order
// (nothing depends on the candidates' order). cursor[slot] = first place;
// after the scatter it is one past the slot's last.
constexpr int kSlotPerThread = 4;
__global__ void __launch_bounds__(kNlThreads) nl_slot_kernel(const int* __restrict__ count, int* __restrict__ cursor,
                                                              int* __restrict__ taken) {
  __shared__ int sh[kNlThreads / 64 + 1];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int4 c = reinterpret_cast<const int4*>(count)[blockIdx.x * kNlThreads + threadIdx.x];
  const int sum = (c.x + c.y) + (c.z + c.w);
  int incl = sum;
  for (int st = 1; st < 64; st <<= 1) {
    const int v = __shfl_up(incl, st);
    if (lane >= st) incl += v;
  }
  if (lane == 63) sh[w] = incl;
  __syncthreads();
  if (threadIdx.x == 0) {
    int run = 0;
    for (int q = 0; q < kNlThreads / 64; ++q) {
      const int v = sh[q];
      sh[q] = run;
      run += v;
    }
    sh[kNlThreads / 64] = atomicAdd(taken, run);
  }
  __syncthreads();
  const int at = sh[kNlThreads / 64] + sh[w] + incl - sum;
  reinterpret_cast<int4*>(cursor)[blockIdx.x * kNlThreads + threadIdx.x] =
      make_int4(at, at + c.x, at + c.x + c.y, at + c.x + c.y + c.z);
}

// Exclusive scan of n <= kScanOneBlock counts by one block (out[n] = total):
// every wave sums its run of counts, then scans it 256 counts at a time.
__global__ void __launch_bounds__(1024) nl_scan_one_kernel(int n, const int* __restrict__ in,
                                                             int64_t* __restrict__ out) {
  __shared__ int64_t sh[16];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int run = 256 * ((n + 4095) / 4096);   // counts per wave, a multiple of 256
  const int b0 = w * run, b1 = min(b0 + run, n);
  auto load = [&](int at) {   // counts at .. at + 3, zero from n on
    if (at + 3 < n) return *reinterpret_cast<const int4*>(in + at);
    return make_int4(at < n ? in[at] : 0, at + 1 < n ? in[at + 1] : 0, at + 2 < n ? in[at + 2] : 0, 0);
  };
  int64_t sum = 0;
#pragma unroll 4
  for (int b = b0; b < b1; b += 256) {
    const int4 v = load(b + 4 * lane);
    sum += ((int64_t)v.x + v.y) + ((int64_t)v.z + v.w);
  }
  for (int st = 1; st < 64; st <<= 1) sum += __shfl_xor((long long)sum, st);
  if (lane == 0) sh[w] = sum;
  __syncthreads();
  int64_t before = 0;
  for (int q = 0; q < w; ++q) before += sh[q];
  if (threadIdx.x == 1023) out[n] = before + sh[15];
  for (int b = b0; b < b1; b += 256) {
    const int at = b + 4 * lane;
    const int4 v = load(at);
    const int64_t s4 = ((int64_t)v.x + v.y) + ((int64_t)v.z + v.w);
    int64_t incl = s4;
    for (int st = 1; st < 64; st <<= 1) {
      const long long u = __shfl_up((long long)incl, st);
      if (lane >= st) incl += u;
    }
    int64_t e = before + incl - s4;
    const int c[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (at + q < n) out[at + q] = e;
      e += c[q];
    }
    before += __shfl((long long)incl, 63);
  }
}

// Exclusive scan of n int32 counts into out[0..n] (out[n] = total), int64.
// Tile pass (kScanTile elements per block, tile totals to bsum), one-block
// pass over the tile totals, then the tile offsets added.
__device__ __forceinline__ int64_t block_exclusive_scan(int64_t v, int64_t* sh, int64_t* total) {
  const int t = threadIdx.x;
  sh[t] = v;
  __syncthreads();
  for (int st = 1; st < kNlThreads; st <<= 1) {
    const int64_t add = t >= st ? sh[t - st] : 0;
    __syncthreads();
    sh[t] += add;
    __syncthreads();
  }
  const int64_t incl = sh[t];
  *total = sh[kNlThreads - 1];
  __syncthreads();
  return incl - v;
}

__global__ void __launch_bounds__(kNlThreads) nl_scan_tile_kernel(int64_t n, const int* __restrict__ in,
                                                                    int64_t* __restrict__ out,
                                                                    int64_t* __restrict__ bsum) {
  __shared__ int64_t sh[kNlThreads];
  const int64_t t0 = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanPerThread;
  int64_t s = 0;
  for (int u = 0; u < kScanPerThread; ++u)
    if (t0 + u < n) s += in[t0 + u];
  int64_t total;
  int64_t run = block_exclusive_scan(s, sh, &total);
  for (int u = 0; u < kScanPerThread; ++u)
    if (t0 + u < n) {
      out[t0 + u] = run;
      run += in[t0 + u];
    }
  if (threadIdx.x == 0) bsum[blockIdx.x] = total;
}

__global__ void __launch_bounds__(kNlThreads) nl_scan_top_kernel(int nb, int64_t* __restrict__ bsum) {
  __shared__ int64_t sh[kNlThreads];
  int64_t carry = 0;
  for (int c0 = 0; c0 < nb; c0 += kNlThreads) {
    const int idx = c0 + threadIdx.x;
    const int64_t v = idx < nb ? bsum[idx] : 0;
    int64_t total;
    const int64_t ex = block_exclusive_scan(v, sh, &total);
    if (idx < nb) bsum[idx] = carry + ex;
    carry += total;
  }
  if (threadIdx.x == 0) bsum[nb] = carry;
}

__global__ void nl_scan_add_kernel(int64_t n, int64_t* __restrict__ out, const int64_t* __restrict__ bsum,
                                   int nb) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] += bsum[i / kScanTile];
  if (i == 0) out[n] = bsum[nb];
}

void scan(hipStream_t s, int64_t n, const int* in, int64_t* out, int64_t* bsum) {
  if (n <= kScanOneBlock) {
    nl_scan_one_kernel<<<1, 1024, 0, s>>>((int)n, in, out);
    return;
  }
  const int nb = (int)((n + kScanTile - 1) / kScanTile);
  if (nb > 0) nl_scan_tile_kernel<<<nb, kNlThreads, 0, s>>>(n, in, out, bsum);
  nl_scan_top_kernel<<<1, kNlThreads, 0, s>>>(nb, bsum);
  const int64_t blocks = std::max<int64_t>(1, (n + kNlThreads - 1) / kNlThreads);
  nl_scan_add_kernel<<<(unsigned)blocks, kNlThreads, 0, s>>>(n, out, bsum, nb);
}

bool invert3(const double* c, double* inv) {
  const double det = c[0] * (c[4] * c[8] - c[5] * c[7]) - c[1] * (c[3] * c[8] - c[5] * c[6]) +
                     c[2] * (c[3] * c[7] - c[4] * c[6]);
  if (!(std::fabs(det) > 0) || !std::isfinite(det)) return false;
  inv[0] = (c[4] * c[8] - c[5] * c[7]) / det;
  inv[1] = (c[2] * c[7] - c[1] * c[8]) / det;
  inv[2] = (c[1] * c[5] - c[2] * c[4]) / det;
  inv[3] = (c[5] * c[6] - c[3] * c[8]) / det;
  inv[4] = (c[0] * c[8] - c[2] * c[6]) / det;
  inv[5] = (c[2] * c[3] - c[0] * c[5]) / det;
  inv[6] = (c[3] * c[7] - c[4] * c[6]) / det;
  inv[7] = (c[1] * c[6] - c[0] * c[7]) / det;
  inv[8] = (c[0] * c[4] - c[1] * c[3]) / det;
  return true;
}

// a[0 .. na) = 0, b[0] = 0, c[0] = 0: the counters a list starts from (a kernel
// rather than memsets, so that a captured call replays correctly)
__global__ void nl_zero_kernel(int* __restrict__ a, uint32_t na, int* __restrict__ b, int64_t* __restrict__ c) {
  const uint32_t stride = gridDim.x * blockDim.x;
  for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < na; i += stride) a[i] = 0;
  if (blockIdx.x == 0 && threadIdx.x == 0) b[0] = 0, c[0] = 0;
}

constexpr int64_t kMaxCandidates = int64_t(1) << 30;

// Host plan: per-graph records, candidate count, slot table size and the
// workspace layout (256-byte aligned pieces). `bytes` is the size asked of the
// caller, which is also what the calls without a workspace are held to.
struct NlPlan {
  std::vector<NlGraph> gs;
  int64_t C = 0;
  uint32_t n_slots = 0;
  size_t o_gs, o_nsh, o_rcube, o_rplace, o_place, o_rec, o_num, o_scnt, o_scur, o_taken, o_rcnt, o_roff, o_bsum,
      o_found, bytes;
  int found_cap = 0;   // finds kept per receiver, at most kNlSortCap
};

mace_status plan_nl(int64_t N, const double* cells, const int32_t* goff, int32_t G, double r_cut, NlPlan& p) {
  if (N < 0 || N > (int64_t(1) << 30) || !(r_cut > 0) || !std::isfinite(r_cut) || G < 1) return MACE_EINVAL;
  if (!goff && G != 1) return MACE_EINVAL;
  p.gs.assign(G, NlGraph{});
  int64_t C = 0;
  for (int g = 0; g < G; ++g) {
    NlGraph& r = p.gs[g];
    std::memset(&r, 0, sizeof(r));
    r.a0 = goff ? goff[g] : 0;
    r.a1 = goff ? goff[g + 1] : (int)N;
    if (r.a0 < 0 || r.a1 < r.a0 || r.a1 > N || (g == 0 && r.a0 != 0)) return MACE_ERANGE;
    if (g > 0 && r.a0 != p.gs[g - 1].a1) return MACE_ERANGE;
    int64_t nimg = 1;
    if (cells) {
      r.periodic = 1;
      std::memcpy(r.cell, cells + 9 * g, sizeof(r.cell));
      if (!invert3(r.cell, r.inv)) return MACE_EINVAL;
      for (int a = 0; a < 3; ++a) {
        const double bn = std::sqrt(r.inv[0 * 3 + a] * r.inv[0 * 3 + a] + r.inv[1 * 3 + a] * r.inv[1 * 3 + a] +
                                    r.inv[2 * 3 + a] * r.inv[2 * 3 + a]);
        const double m = std::floor(r_cut * bn + 1.0 + 1e-6);
        if (!(m < 1e4)) return MACE_EUNSUPPORTED;
        r.nr[a] = (int16_t)m;
        nimg *= 2 * r.nr[a] + 1;
        // (far above the rounding of fractional coordinates: at most about 1e-3,
        // for coordinates of 1e9 in the most skewed cells accepted, and of the
        // slack itself: below 1e-3 at its limit of 10^4)
        r.slack[a] = (float)(r_cut * bn + 1e-2);
      }
    }
    if (nimg > kMaxCandidates) return MACE_EUNSUPPORTED;
    r.nimg = (int)nimg;
    r.c0 = C;
    C += (int64_t)(r.a1 - r.a0) * nimg;
    if (C > kMaxCandidates) return MACE_EUNSUPPORTED;
  }
  if (!goff && p.gs[0].a1 != N) return MACE_ERANGE;
  if (p.gs[G - 1].a1 != N) return MACE_ERANGE;
  p.C = C;
  const size_t n1 = (size_t)std::max<int64_t>(N, 1), c1 = (size_t)std::max<int64_t>(C, 1);
  size_t o = 0;
  auto take = [&](size_t bytes) {
    const size_t at = o;
    o += (bytes + 255) & ~size_t(255);
    return at;
  };
  // The size asked of the caller: per graph its record, per image 40 bytes, per
  // atom 52, and 16 bytes per slot of a table of at least twice the images. The
  // pieces below fit in it for every input: the same record, 36 bytes per image,
  // 60 per atom (4 more than are saved where an atom has one image only: there
  // the smaller slot table pays for them), and 8 bytes per slot.
  uint32_t ns = 1024;
  while ((int64_t)ns < 2 * C) ns <<= 1;
  const int64_t tiles = (std::max<int64_t>(ns, n1) + kScanTile - 1) / kScanTile;
  for (size_t b : {sizeof(NlGraph) * G, sizeof(double) * 3 * n1, sizeof(int4) * n1, sizeof(int) * c1, sizeof(int4) * c1,
                   sizeof(int4) * c1, sizeof(int) * ns, sizeof(int) * ns, sizeof(int64_t) * (ns + 1), sizeof(int) * c1,
                   sizeof(int) * n1, sizeof(int64_t) * (n1 + 1), sizeof(int64_t) * (tiles + 1), sizeof(int)})
    take(b);
  p.bytes = o;
  // slots: few enough to clear and number cheaply, enough for the occupied
  // cubes (at most one per candidate in reach, about one per 20 at liquid density)
  p.n_slots = 1024;
  while (p.n_slots < ns && (int64_t)p.n_slots < std::max<int64_t>(N, C / 16)) p.n_slots <<= 1;
  o = 0;
  p.o_gs = take(sizeof(NlGraph) * G);
  p.o_nsh = take(sizeof(int4) * n1);
  p.o_rcube = take(sizeof(int4) * n1);
  p.o_rplace = take(sizeof(float4) * n1);
  p.o_place = take(sizeof(float4) * c1);
  p.o_rec = take(sizeof(int4) * c1);
  p.o_num = take(sizeof(int) * c1);
  p.o_scnt = take(sizeof(int) * p.n_slots);
  p.o_scur = take(sizeof(int) * p.n_slots);
  p.o_taken = take(sizeof(int));
  p.o_rcnt = take(sizeof(int) * n1);
  p.o_roff = take(sizeof(int64_t) * (n1 + 2));   // offsets, total, flags
  p.o_bsum = take(sizeof(int64_t) * ((n1 + kScanTile - 1) / kScanTile + 1));
  p.o_found = o;
  p.bytes = std::max(p.bytes, o);
  p.found_cap = (int)std::min<size_t>((p.bytes - o) / (sizeof(int) * n1), kNlSortCap);
  return MACE_OK;
}

}  // namespace

extern "C" size_t mace_neighbor_workspace_bytes(int64_t n_atoms, const double* cells, const int32_t* graph_offsets,
                                                int32_t n_graphs, double r_cut) {
  NlPlan p;
  if (plan_nl(n_atoms, cells, graph_offsets, n_graphs, r_cut, p) != MACE_OK) return 0;
  return p.bytes;
}

namespace {

// The list built in the device buffer w (at least p.bytes), planned by plan_nl.
mace_status nl_run(const NlPlan& p, int64_t n_atoms, const double* positions, int32_t n_graphs, double r_cut,
                   int64_t max_edges, int32_t* sender, int32_t* receiver, int32_t* shifts, int64_t* n_edges,
                   void* workspace, void* stream) {
  *n_edges = 0;
  if (n_atoms == 0) return MACE_OK;
  hipStream_t s = (hipStream_t)stream;
  char* w = reinterpret_cast<char*>(workspace);
  auto* gs = reinterpret_cast<NlGraph*>(w + p.o_gs);
  auto* nsh = reinterpret_cast<int4*>(w + p.o_nsh);
  auto* rcube = reinterpret_cast<int4*>(w + p.o_rcube);
  auto* rplace = reinterpret_cast<float4*>(w + p.o_rplace);
  auto* place = reinterpret_cast<float4*>(w + p.o_place);
  auto* rec = reinterpret_cast<int4*>(w + p.o_rec);
  auto* num = reinterpret_cast<int*>(w + p.o_num);
  auto* scnt = reinterpret_cast<int*>(w + p.o_scnt);
  auto* scur = reinterpret_cast<int*>(w + p.o_scur);
  auto* taken = reinterpret_cast<int*>(w + p.o_taken);
  auto* rcnt = reinterpret_cast<int*>(w + p.o_rcnt);
  auto* roff = reinterpret_cast<int64_t*>(w + p.o_roff);
  auto* bsum = reinterpret_cast<int64_t*>(w + p.o_bsum);
  auto* found = reinterpret_cast<int*>(w + p.o_found);
  auto* flags = reinterpret_cast<int*>(roff + n_atoms + 1);
  const int N = (int)n_atoms, G = n_graphs;
  const double bs = r_cut + 1e-6, rc2 = r_cut * r_cut;
  // The pre-test's distance: r_c, and what the FP32 places (rounded to 2^-24 of
  // a cube edge, differences and cube offsets to a few times that) and the FP64
  // positions behind them (1e-6 at coordinates of 1e9) can be off. Cubes below
  // 1 A could overflow their int32 indices at such coordinates: no pre-test.
  const double pre = r_cut + 2e-6 * bs + 4e-6;
  const float pre2 = bs >= 1.0 ? (float)(pre * pre * (1.0 + 1e-6)) : INFINITY;
  const uint32_t mask = p.n_slots - 1;
  hipError_t err = hipSuccess;
  if (G > 1) err = hipMemcpyAsync(gs, p.gs.data(), sizeof(NlGraph) * G, hipMemcpyHostToDevice, s);
  if (err != hipSuccess) {
    (void)hipStreamSynchronize(s);   // the plan's host copy must outlive the upload
    return MACE_EHIP;
  }
  const NlGraph& g0 = p.gs[0];
  nl_zero_kernel<<<std::min<unsigned>(256, p.n_slots / kNlThreads), kNlThreads, 0, s>>>(scnt, p.n_slots, taken,
                                                                                       roff + n_atoms + 1);
  const unsigned cblk = (unsigned)((p.C + kNlThreads - 1) / kNlThreads);   // (C >= N > 0)
  nl_bin_kernel<false><<<cblk, kNlThreads, 0, s>>>(p.C, positions, g0, gs, G, bs, mask, nsh, rcube, rplace, flags, scnt,
                                                   scur, place, rec, num);
  nl_slot_kernel<<<p.n_slots / (kNlThreads * kSlotPerThread), kNlThreads, 0, s>>>(scnt, scur, taken);
  nl_bin_kernel<true><<<cblk, kNlThreads, 0, s>>>(p.C, positions, g0, gs, G, bs, mask, nsh, rcube, rplace, flags, scnt,
                                                  scur, place, rec, num);
  const unsigned rblk = (unsigned)((N + kNlWaves - 1) / kNlWaves);
  nl_receiver_kernel<false><<<rblk, 64 * kNlWaves, 0, s>>>(N, positions, g0, gs, G, bs, rc2, pre2, mask, nsh, rcube,
                                                         rplace, scnt, scur, place, rec, num, found, p.found_cap, rcnt, nullptr,
                                                         0, nullptr, nullptr, nullptr);
  scan(s, N, rcnt, roff, bsum);
  // The write pass goes before the count is read back: it checks the capacity
  // and the flags itself, so that the device does not wait for the host between
  // the two.
  if (max_edges > 0)
    nl_receiver_kernel<true><<<rblk, 64 * kNlWaves, 0, s>>>(N, positions, g0, gs, G, bs, rc2, pre2, mask, nsh, rcube,
                                                          rplace, scnt, scur, place, rec, num, found, p.found_cap, nullptr, roff,
                                                          max_edges, sender, receiver, shifts);
  int64_t back[2] = {0, 0};   // total, flags
  err = hipGetLastError();
  if (err == hipSuccess) err = hipMemcpyAsync(back, roff + N, sizeof(back), hipMemcpyDeviceToHost, s);
  const hipError_t serr = hipStreamSynchronize(s);
  if (err == hipSuccess) err = serr;
  if (err != hipSuccess) return MACE_EHIP;
  if (back[1] & kFlagNonFinite) return MACE_ENONFINITE;
  if (back[1] & kFlagRange) return MACE_ERANGE;
  *n_edges = back[0];
  return back[0] > max_edges ? MACE_ENOSPACE : MACE_OK;
}

}  // namespace

extern "C" mace_status mace_neighbor_list_device(int64_t n_atoms, const double* positions, const double* cells,
                                                 const int32_t* graph_offsets, int32_t n_graphs, double r_cut,
                                                 int64_t max_edges, int32_t* sender, int32_t* receiver,
                                                 int32_t* shifts, int64_t* n_edges, void* workspace,
                                                 size_t workspace_bytes, void* stream) {
  if (!n_edges || (n_atoms > 0 && !positions) || max_edges < 0) return MACE_EINVAL;
  NlPlan p;
  mace_status st = plan_nl(n_atoms, cells, graph_offsets, n_graphs, r_cut, p);
  if (st != MACE_OK) return st;
  if (!workspace || workspace_bytes < p.bytes) return MACE_ENOSPACE;
  if (max_edges > 0 && (!sender || !receiver || !shifts)) return MACE_EINVAL;
  return nl_run(p, n_atoms, positions, n_graphs, r_cut, max_edges, sender, receiver, shifts, n_edges, workspace,
                stream);
}

// ---- the same list without a workspace argument: a file-scope device array
// serves as the workspace. Every GPU holds its own copy until the process
// ends; host code addresses it only through the pointer hipGetSymbolAddress
// returns for the current device (the array's name on the host is not a
// device address).
constexpr size_t kNlScratchBytes = MACE_NEIGHBOR_SCRATCH_BYTES;
static __device__ __align__(256) unsigned char scratch[kNlScratchBytes];

namespace {
constexpr int kMaxScratchDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxScratchDevices] = {};

// this device's scratch, looked up once per device
void* device_scratch() {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxScratchDevices) return nullptr;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return nullptr;
    g_scratch_ptr[dev] = ptr;
  }
  return g_scratch_ptr[dev];
}
}  // namespace

extern "C" mace_status mace_neighbor_list_device_noalloc(int64_t n_atoms, const double* positions,
                                                         const double* cells, const int32_t* graph_offsets,
                                                         int32_t n_graphs, double r_cut, int64_t max_edges,
                                                         int32_t* sender, int32_t* receiver, int32_t* shifts,
                                                         int64_t* n_edges, void* stream) {
  if (!n_edges || (n_atoms > 0 && !positions) || max_edges < 0) return MACE_EINVAL;
  NlPlan p;
  mace_status st = plan_nl(n_atoms, cells, graph_offsets, n_graphs, r_cut, p);
  if (st != MACE_OK) return st;
  if (p.bytes > kNlScratchBytes) return MACE_ENOSPACE;
  if (max_edges > 0 && (!sender || !receiver || !shifts)) return MACE_EINVAL;
  void* w = device_scratch();
  if (!w) return MACE_EHIP;
  return nl_run(p, n_atoms, positions, n_graphs, r_cut, max_edges, sender, receiver, shifts, n_edges, w, stream);
}
