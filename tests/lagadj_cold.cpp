// Products of the Rusanov and HLL fluxes (paper_1408_3719_amd/csrc/lagadj.h,
// host build, no GPU) where one side's sound speed plays no part: the left
// trace has a pressure below zero, so that the flux takes the right side's
// speeds, or the flux is the upwind one and the normal has no part in space.
// Prints "<case> <max relative deviation>" from central differences of the
// flux that the same functions return; a product that is no number prints nan.
#include <cmath>
#include <cstdio>

#include "lagadj.h"

using namespace aw::lag;

static void flux(bool hll, const double z[11], double F[4]) {
  const double none[4] = {};
  double a[4] = {}, b[4] = {}, n[3] = {};
  (hll ? hll_flux_vjp : rusanov_flux_vjp)(z, z + 4, z + 8, 1.4, none, a, b, n, F);
}

static void check(const char* name, bool hll, const double z[11]) {
  const double Fb[4] = {0.7, -0.4, 0.9, 0.3};
  double zb[11] = {}, F[4];
  (hll ? hll_flux_vjp : rusanov_flux_vjp)(z, z + 4, z + 8, 1.4, Fb, zb, zb + 4, zb + 8, F);
  double dev = 0.0, scale = 1e-300;
  for (int k = 0; k < 11; ++k) {
    const double h = 1e-6;
    double zp[11], zm[11], fp[4], fm[4], fd = 0.0;
    for (int i = 0; i < 11; ++i) zp[i] = zm[i] = z[i];
    zp[k] += h;
    zm[k] -= h;
    flux(hll, zp, fp);
    flux(hll, zm, fm);
    for (int v = 0; v < 4; ++v) fd += Fb[v] * (fp[v] - fm[v]) / (2.0 * h);
    scale = std::fmax(scale, std::fabs(fd));
    if (!(std::fabs(fd - zb[k]) <= dev)) dev = std::fabs(fd - zb[k]);
    if (std::isnan(dev)) break;
  }
  std::printf("%s %.3e\n", name, dev / scale);
}

int main() {
  // p = 0.4 (E - m.m / 2 rho): -0.02 on the left, 0.8 on the right
  const double cold[11] = {0.9, 0.3, -0.2, 0.5 * (0.09 + 0.04) / 0.9 - 0.05, 1.1, 0.2, 0.1,
                           2.0 + 0.5 * 0.05 / 1.1, 0.6, -0.3, 0.1};
  check("rusanov_cold_left", false, cold);
  check("hll_cold_left", true, cold);
  // upwind from a cold left state: the right side moves off faster than sound
  double up[11];
  for (int i = 0; i < 11; ++i) up[i] = cold[i];
  up[10] = 3.0;
  check("hll_cold_left_upwind", true, up);
  // upwind along time alone: no part of the normal in space
  double still[11];
  for (int i = 0; i < 11; ++i) still[i] = cold[i];
  still[3] = 2.0;
  still[8] = still[9] = 0.0;
  still[10] = 1.0;
  const double Fb[4] = {0.7, -0.4, 0.9, 0.3};
  double a[4] = {}, b[4] = {}, n[3] = {}, F[4];
  hll_flux_vjp(still, still + 4, still + 8, 1.4, Fb, a, b, n, F);
  double dev = 0.0;   // F = ql, so the products are Fb and nothing
  for (int v = 0; v < 4; ++v) dev = dev + std::fabs(a[v] - Fb[v]) + std::fabs(b[v]) + std::fabs(F[v] - still[v]);
  std::printf("hll_upwind_in_time %.3e\n", dev + 0.0 * (n[0] + n[1] + n[2]));
}
