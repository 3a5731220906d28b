// What a plan's launches would be and what its workspace holds, on a machine
// without a GPU.  Reads one query per line and answers each with one line; see
// test_launch_rules.py.  Linked with the library; nothing is launched.
//   partials PREC NX NY NZ -> rows the solve's partials hold, and the blocks of
//                             the HEX8 operator in FP32 and FP64
//   tiles PREC NX NY NZ    -> blocks along x and y and z-chunks of one plane of
//                             the march on its own
//   chunk PREC NX NY NZ    -> planes per block of the HEX8 operator, and the
//                             nanoseconds that choosing them takes
#include <chrono>
#include <cstdio>
#include <string>
#include <vector>

#include "mech_common.h"
#include "plan.h"

static etm_plan *make_plan(int prec, int nx, int ny, int nz) {
  const std::vector<double> dx(nx, 1e-6), dy(ny, 1e-6), dz(nz, 1e-6);
  const std::vector<uint8_t> mat(size_t(nx) * ny * nz, 0);
  const etm_material m{11.7, 10.0, 0.0, 148.0, 1.63e6, 130e9, 0.28, 2.6e-6, 0, 0};
  etm_mesh mesh{};
  mesh.nx = nx; mesh.ny = ny; mesh.nz = nz;
  mesh.dx = dx.data(); mesh.dy = dy.data(); mesh.dz = dz.data(); mesh.mat = mat.data();
  etm_opts o;
  if (etm_opts_default(&o) != ETM_OK) return nullptr;
  o.precision = prec;
  etm_plan *p = nullptr;
  return etm_plan_create(&mesh, &m, 1, nullptr, &o, &p) == ETM_OK ? p : nullptr;
}

int main() {
  char what[32];
  int prec, nx, ny, nz;
  while (std::scanf("%31s %d %d %d %d", what, &prec, &nx, &ny, &nz) == 5) {
    DevGrid g{};
    g.nx = nx; g.ny = ny; g.nz = nz;
    if (std::string(what) == "partials") {
      etm_plan *p = make_plan(prec, nx, ny, nz);
      if (!p) {
        std::printf("error %s\n", etm_last_error());
        continue;
      }
      std::printf("%lld %lld %lld\n", (long long)(p->r_partm.bytes / (kRedWidth * 8)),
                  (long long)mech::cell_blocks<float>(g), (long long)mech::cell_blocks<double>(g));
      etm_plan_destroy(p);
    } else if (std::string(what) == "tiles") {
      g.sy = (nx + 1 + kPad - 1) / kPad * kPad;
      g.sz = g.sy * (ny + 1);
      g.ntot = g.sz * (nz + 1);
      int ntx, nty, nkc;
      em_tiles(g, prec, 1, &ntx, &nty, &nkc);
      std::printf("%d %d %d\n", ntx, nty, nkc);
    } else if (std::string(what) == "chunk") {
      const int n = 200;
      volatile int kc = 0;
      const auto t0 = std::chrono::steady_clock::now();
      for (int q = 0; q < n; ++q) kc = prec == ETM_PREC_FP64 ? mech::cell_kchunk<double>(g) : mech::cell_kchunk<float>(g);
      const auto ns = std::chrono::duration_cast<std::chrono::nanoseconds>(std::chrono::steady_clock::now() - t0);
      std::printf("%d %lld\n", int(kc), (long long)ns.count() / n);
    } else {
      std::printf("error unknown query\n");
    }
  }
  return 0;
}
