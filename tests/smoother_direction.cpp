// The Chebyshev steps of the multigrid smoother, run on the host on one vector
// per node: the functions of mg.hip are compiled for the host as well here.
// With A = 0 the residual is b whatever x is, so a step's direction cannot
// depend on x, and x_out is x plus that direction, rounded once.  Prints, for a
// step that stores its direction and for a last step, on a stored level and on
// level 0, how many entries differ from that; see test_smoother_direction.py.
#include <hip/hip_runtime.h>
#undef __device__
#define __device__ __attribute__((host)) __attribute__((device))
#include "mg.hip"

#include <cstdio>
#include <random>
#include <vector>

using namespace etm;

template <typename T>
struct Case {
  static constexpr size_t n = 5000;
  std::vector<T> D = std::vector<T>(6 * n), b = std::vector<T>(3 * n), d0 = std::vector<T>(3 * n),
                 x = std::vector<T>(3 * n);
  MgLevel<T> L{};
  static V3<T> vec(std::vector<T> &v) { return V3<T>{{v.data(), v.data() + n, v.data() + 2 * n}}; }

  Case() {
    std::mt19937_64 rng(7);
    std::uniform_real_distribution<double> u(-1.0, 1.0);
    for (T &v : D) v = T(u(rng));
    for (T &v : b) v = T(u(rng));
    for (T &v : d0) v = T(u(rng));
    for (T &v : x) v = T(1000.0 * u(rng));
    L.n = int64_t(n);
    L.Dinv = D.data();
  }
  // one step from `xin` with the direction d0 before it: x_out and the new direction
  template <bool KEEP>
  void step(bool level0, std::vector<T> xin, std::vector<T> &xout, std::vector<T> &d) {
    const T y[3] = {T(0), T(0), T(0)}, c1 = T(0.813), c2 = T(3.21);
    d = d0;
    xout = d0;  // (a last step finds the direction where its result goes)
    for (int64_t i = 0; i < L.n; ++i) {
      if (level0) {
        const NodeAt at{i, 0u};
        const T xc[3] = {xin[i], xin[n + i], xin[2 * n + i]};
        const EpiSmooth0<T, KEEP> e{L, vec(b), vec(xout), vec(d), c1, c2, kDirKept};
        e(at, y, xc, e.load(at), nullptr);
      } else {
        const OpSmooth<T, KEEP> op{L, vec(b), vec(xin), vec(xout), vec(d), c1, c2, kDirKept};
        op(i, y, op.load(i), nullptr);
      }
    }
  }
  template <bool KEEP>
  void run(const char *name) {
    for (int level0 = 0; level0 < 2; ++level0) {
      std::vector<T> dir, dz, xo, dx;
      step<KEEP>(level0 != 0, std::vector<T>(3 * n, T(0)), dir, dz);  // from x = 0: the direction
      step<KEEP>(level0 != 0, x, xo, dx);
      size_t bad_x = 0, bad_d = 0;
      for (size_t q = 0; q < 3 * n; ++q) {
        bad_x += xo[q] != T(x[q] + dir[q]);
        bad_d += KEEP && (dx[q] != dz[q] || dx[q] != dir[q]);
      }
      std::printf("%s keep=%d level0=%d %zu %zu\n", name, int(KEEP), level0, bad_x, bad_d);
    }
  }
};

int main() {
  Case<float> f;
  f.run<true>("fp32");
  f.run<false>("fp32");
  Case<double> g;
  g.run<true>("fp64");
  g.run<false>("fp64");
  return 0;
}
