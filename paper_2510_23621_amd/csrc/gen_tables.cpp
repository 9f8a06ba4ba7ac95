// Build-time generator: writes the device header with the real CG
// couplings and the selected coupling trees as compile-time visitors, so the
// kernels carry every coupling constant as an immediate and index register
// arrays with constants only.
//
// usage: gen_tables <FP32 header> <FP64 header>
#include <vector>
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <set>
#include <string>
#include <tuple>

#include "so3_tables.hpp"

int main(int argc, char** argv) {
  if (argc != 3) {
    std::fprintf(stderr, "usage: %s <out.h> <out64.h>\n", argv[0]);
    return 2;
  }
  std::set<std::tuple<int, int, int>> need;
  for (int a = 0; a <= 3; ++a)
    for (int b = 0; b <= 3; ++b)
      for (int c = std::abs(a - b); c <= std::min(a + b, 3); ++c) need.insert({a, b, c});
  struct TL { int nu, L; std::vector<so3h::Tree> t; };
  std::vector<TL> trees;
  for (int L = 0; L <= 3; ++L) {
    int parity = (L % 2) ? -1 : 1;
    for (int nu = 1; nu <= 3; ++nu) {
      auto sel = so3h::select_trees(nu, L, parity);
      for (auto& t : sel) {
        if (nu == 2) need.insert({t.l1, t.l2, L});
        if (nu == 3) {
          need.insert({t.l1, t.l2, t.l12});
          need.insert({t.l12, t.l3, L});
        }
      }
      trees.push_back({nu, L, sel});
    }
  }
  // the FP32 tables (namespace mt, float immediates) and the FP64 ones of the
  // debug precision (namespace mt64, double immediates to 17 digits)
  for (int dbl = 0; dbl < 2; ++dbl) {
    const char* path = dbl ? argv[2] : argv[1];
    const char* ns = dbl ? "mt64" : "mt";
    const char* vf = dbl ? "%.17g" : "%.9ef";
    FILE* f = std::fopen(path, "w");
    if (!f) return 1;
    auto val = [&](double v) {
      char buf[64];
      std::snprintf(buf, sizeof(buf), vf, v);
      return std::string(buf);
    };
    std::fprintf(f,
                 "// Generated by gen_tables.cpp from so3_tables.hpp: real CG couplings and the\n"
                 "// coupling trees of the symmetric contraction (%s). Do not edit.\n"
                 "#pragma once\n\nnamespace %s {\n\n"
                 "template <int L1, int L2, int L3> struct CG;\n"
                 "template <int NU, int A, int B, int C, int D> struct TreeT {\n"
                 "  static constexpr int nu = NU, l1 = A, l2 = B, l3 = C, l12 = D;\n};\n"
                 "template <int NU, int L> struct Trees;\n\n",
                 dbl ? "FP64" : "FP32", ns);
    for (auto [a, b, c] : need) {
      auto C = so3h::real_cg(a, b, c);
      int nnz = 0;
      for (double v : C.v) nnz += (v != 0.0);
      // pairs (m1, m2) carrying at least one nonzero coupling, numbered in
      // lexicographic order
      std::vector<int> pid((2 * a + 1) * (2 * b + 1), -1);
      int npair = 0;
      for (int m1 = 0; m1 < 2 * a + 1; ++m1)
        for (int m2 = 0; m2 < 2 * b + 1; ++m2)
          for (int m3 = 0; m3 < 2 * c + 1; ++m3)
            if (C.at(m1, m2, m3) != 0.0 && pid[m1 * (2 * b + 1) + m2] < 0) pid[m1 * (2 * b + 1) + m2] = npair++;
      std::fprintf(f, "template <> struct CG<%d, %d, %d> {\n  static constexpr int nnz = %d, npair = %d;\n", a, b,
                   c, nnz, npair);
      // each(f): f(m1, m2, m3, C) per nonzero; each_p adds the pair number
      for (int withp = 0; withp < 2; ++withp) {
        std::fprintf(f, "  template <class F> __host__ __device__ __forceinline__ static void %s(F&& f) {\n",
                     withp ? "each_p" : "each");
        for (int m1 = 0; m1 < 2 * a + 1; ++m1)
          for (int m2 = 0; m2 < 2 * b + 1; ++m2)
            for (int m3 = 0; m3 < 2 * c + 1; ++m3) {
              double v = C.at(m1, m2, m3);
              if (v == 0.0) continue;
              if (withp)
                std::fprintf(f, "    f(%d, %d, %d, %s, %d);\n", m1, m2, m3, val(v).c_str(), pid[m1 * (2 * b + 1) + m2]);
              else
                std::fprintf(f, "    f(%d, %d, %d, %s);\n", m1, m2, m3, val(v).c_str());
            }
        std::fprintf(f, "  }\n");
      }
      // The forward's form of the coefficients, C = sign * ratio * scale[m3]:
      // scale[m3] is applied once per receiver, and each distinct (m2, ratio)
      // with ratio != 1 is one product ratio * Y[m2] per edge. The scales are
      // picked among each m3's magnitudes for the fewest such products (55
      // over the paths of l_h <= 2, where |C| Y[m2] itself takes 112).
      // each_yc(f): f(m2, ratio, product number); each_ys(f): f(m1, m2, m3,
      // sign, product number or -1 for Y[m2] itself) per nonzero; scale(m3).
      {
        const int n3 = 2 * c + 1;
        auto mag = [&](int m1, int m2, int m3) { return std::fabs(C.at(m1, m2, m3)); };
        auto same = [](double x, double y) { return std::fabs(x - y) < 1e-9 * std::fabs(y); };
        std::vector<double> scale(n3, 1.0);
        std::vector<std::vector<double>> cand(n3);
        for (int m3 = 0; m3 < n3; ++m3) {
          int best = 0;
          for (int m1 = 0; m1 < 2 * a + 1; ++m1)
            for (int m2 = 0; m2 < 2 * b + 1; ++m2) {
              const double v = mag(m1, m2, m3);
              if (v == 0.0) continue;
              int count = 0;
              for (int q1 = 0; q1 < 2 * a + 1; ++q1)
                for (int q2 = 0; q2 < 2 * b + 1; ++q2) count += same(mag(q1, q2, m3), v);
              if (std::none_of(cand[m3].begin(), cand[m3].end(), [&](double x) { return same(x, v); })) cand[m3].push_back(v);
              if (count > best) {
                best = count;
                scale[m3] = v;
              }
            }
        }
        using Prod = std::pair<int, double>;   // (m2, ratio)
        auto find = [&](const std::vector<Prod>& ps, int m2, double ratio) {
          for (size_t u = 0; u < ps.size(); ++u)
            if (ps[u].first == m2 && same(ps[u].second, ratio)) return (int)u;
          return -1;
        };
        auto products = [&](const std::vector<double>& sc) {
          std::vector<Prod> ps;
          for (int m1 = 0; m1 < 2 * a + 1; ++m1)
            for (int m2 = 0; m2 < 2 * b + 1; ++m2)
              for (int m3 = 0; m3 < n3; ++m3) {
                const double v = mag(m1, m2, m3);
                if (v == 0.0 || same(v, sc[m3]) || find(ps, m2, v / sc[m3]) >= 0) continue;
                ps.push_back({m2, v / sc[m3]});
              }
          return ps;
        };
        for (int sweep = 0; sweep < 3; ++sweep)
          for (int m3 = 0; m3 < n3; ++m3)
            for (double v : cand[m3]) {
              std::vector<double> t = scale;
              t[m3] = v;
              if (products(t).size() < products(scale).size()) scale = t;
            }
        const std::vector<Prod> yc = products(scale);
        std::string ys, sc;
        for (int m1 = 0; m1 < 2 * a + 1; ++m1)
          for (int m2 = 0; m2 < 2 * b + 1; ++m2)
            for (int m3 = 0; m3 < n3; ++m3) {
              const double v = C.at(m1, m2, m3);
              if (v == 0.0) continue;
              char buf[96];
              std::snprintf(buf, sizeof(buf), "    f(%d, %d, %d, %d, %d);\n", m1, m2, m3, v > 0 ? 1 : -1,
                            find(yc, m2, std::fabs(v) / scale[m3]));
              ys += buf;
            }
        for (int m3 = 0; m3 < n3; ++m3)
          sc += std::string(m3 ? " : " : "") + (m3 + 1 < n3 ? "m3 == " + std::to_string(m3) + " ? " : "") + val(scale[m3]);
        std::fprintf(f, "  static constexpr int nyc = %d;\n", (int)yc.size());
        std::fprintf(f, "  template <class F> __host__ __device__ __forceinline__ static void each_yc(F&& f) {\n");
        for (size_t u = 0; u < yc.size(); ++u) std::fprintf(f, "    f(%d, %s, %d);\n", yc[u].first, val(yc[u].second).c_str(), (int)u);
        if (yc.empty()) std::fprintf(f, "    (void)f;\n");
        std::fprintf(f, "  }\n");
        std::fprintf(f, "  template <class F> __host__ __device__ __forceinline__ static void each_ys(F&& f) {\n%s  }\n", ys.c_str());
        std::fprintf(f, "  __host__ __device__ __forceinline__ static constexpr %s scale(int m3) { return %s; }\n",
                     dbl ? "double" : "float", sc.c_str());
      }
      // each_pair(f): f(m1, m2, pair number) per pair
      std::fprintf(f, "  template <class F> __host__ __device__ __forceinline__ static void each_pair(F&& f) {\n");
      for (int m1 = 0; m1 < 2 * a + 1; ++m1)
        for (int m2 = 0; m2 < 2 * b + 1; ++m2)
          if (pid[m1 * (2 * b + 1) + m2] >= 0)
            std::fprintf(f, "    f(%d, %d, %d);\n", m1, m2, pid[m1 * (2 * b + 1) + m2]);
      std::fprintf(f, "  }\n};\n");
    }
    for (auto& tl : trees) {
      std::fprintf(f, "template <> struct Trees<%d, %d> {\n  static constexpr int n = %d;\n", tl.nu, tl.L,
                   (int)tl.t.size());
      std::fprintf(f, "  template <class F> __host__ __device__ __forceinline__ static void each(F&& f) {\n");
      int eta = 0;
      for (auto& t : tl.t)
        std::fprintf(f, "    f(TreeT<%d, %d, %d, %d, %d>{}, %d, %s);\n", t.nu, t.l1, t.l2, t.l3, t.l12, eta++,
                     val(t.scale).c_str());
      if (tl.t.empty()) std::fprintf(f, "    (void)f;\n");
      std::fprintf(f, "  }\n};\n");
    }
    std::fprintf(f, "\n}  // namespace %s\n", ns);
    std::fclose(f);
  }
  return 0;
}
