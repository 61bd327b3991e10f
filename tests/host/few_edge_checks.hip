// The few-edge tables against the decision tables and the definition, on the
// CPU: the library's host source is included to reach make_binning.
#include "../../paper_1911_08275_amd/csrc/api.hip"

#include <cstdio>

using namespace cp;

// Slot of value s: the number of edges at or below it (an edge at zero always).
static int slot_of(const EdgeD &E, double s) {
  int n = 0;
  for (int k = 0; k < E.size(); k++) n += E[k] == 0.0 || E[k] <= s;
  return n;
}

static long g_certain = 0, g_unsure = 0;

static bool check_value(const Binning &B, float v) {
  const int cell = (int)fbits(v) >> B.shift;
  const double eps = B.bnd.eps;
  if (!(v < B.AB32)) return (double)v - eps >= B.E[B.E.size() - 1] * (1 - 1e-15);
  const uint2 e = B.few.e[std::min(std::max(cell, B.few.lo), B.few.hi) - B.few.lo];
  float t;
  memcpy(&t, &e.x, 4);
  const float d = v - t;
  const bool unsure = std::fabs(d) < B.eps32_3 || (int)e.y < 0;
  unsure ? g_unsure++ : g_certain++;
  if (unsure) return true;
  const int slot = (int)(e.y & 63u) - (d < 0.f ? 1 : 0);
  if (slot < 0 || slot > B.E.size() - 1) return false;
  if (slot != slot_of(B.E, (double)v - eps) || slot != slot_of(B.E, (double)v + eps)) return false;
  // the decision table's slot, where it is certain
  const uint2 g = B.t32.e[std::min(std::max(cell, B.t32.lo), B.t32.hi) - B.t32.lo];
  float lo, hi;
  memcpy(&lo, &g.x, 4);
  memcpy(&hi, &g.y, 4);
  const bool ch = v >= hi, unc = v >= lo && !ch;
  return unc || slot == (int)(g.y & 63u) - 1 + (ch ? 1 : 0);
}

static int check(const Binning &B) {
  uint64_t rng = 88172645463325252ull;
  auto next = [&]() {
    rng ^= rng << 13;
    rng ^= rng >> 7;
    rng ^= rng << 17;
    return rng;
  };
  const double EB = B.E[B.E.size() - 1];
  auto around = [&](double x) {
    float v = (float)x;
    for (int i = 0; i < 3; i++) v = std::nextafter(v, -INFINITY);
    for (int i = 0; i < 7; i++, v = std::nextafter(v, INFINITY))
      if (!check_value(B, v)) {
        printf("value %.9g\n", v);
        return false;
      }
    return true;
  };
  for (int k = 0; k < B.E.size(); k++)
    for (double f = -2.0; f <= 2.0; f += 0.25)
      if (!around(B.E[k] + f * B.bnd.eps) || !around(B.E[k] + f * B.eps32_3)) return 1;
  for (int m = B.few.lo - 1; m <= B.few.hi + 2; m++)
    if (m >= 0 && !around(bitsf((uint32_t)m << B.shift))) return 1;
  for (int i = 0; i < 200000; i++) {
    const double u = (double)(next() >> 11) * 0x1p-53;
    const float v = (float)((i & 1) ? EB * 1.1 * u : EB * std::exp(-18.0 * u));
    if (!check_value(B, v) || !check_value(B, -v * 1e-6f)) {
      printf("value %.9g\n", v);
      return 1;
    }
  }
  return 0;
}

int main() {
  std::vector<std::vector<double>> sets = {
      {0.5, 6.0}, {0.0, 6.0}, {0.0, 1.0, 2.5, 6.0}, {0.5, 2.0, 2.0 + 1e-7, 3.0, 5.75, 5.75 * (1 + 1e-9), 6.0},
      {1e-6, 1e-3, 6.0}, {5.9, 5.95, 6.0}};
  std::vector<double> lin, lg, dense;
  for (int k = 0; k <= 60; k++) lin.push_back(0.1 * k);
  for (int k = 0; k <= 20; k++) lg.push_back(0.1 * std::pow(60.0, k / 20.0));
  for (int k = 0; k <= 60; k++) dense.push_back(5.0 + k / 60.0);
  sets.push_back(lin);
  sets.push_back(lg);
  sets.push_back(dense);
  const double zero[3] = {0, 0, 0};
  int n = 0;
  for (double box : {31.0, 420.0, 3000.0})
    for (size_t q = 0; q < sets.size(); q++)
      for (int mode : {XI, WP}) {
        const double ext[3] = {box, box, box};
        const int refine[3] = {2, 2, 2};
        const std::vector<double> &e = sets[q];
        const Geometry g = choose_geometry(mode, true, box, zero, ext, e.back(), 8.0, refine, 1000000);
        Binning B, X;
        if (make_binning(mode, F32R, e.data(), (int)e.size(), 8.0, 8, g, box, B) != CP_OK) return 2;
        if (check(B)) {
          printf("set %zu mode %d box %g\n", q, mode, box);
          return 1;
        }
        n++;
        if (mode == WP && make_binning_wpxi(e.data(), (int)e.size(), B, X)) {
          if (check(X)) {
            printf("set %zu fused xi box %g\n", q, box);
            return 1;
          }
          n++;
        }
      }
  printf("few-edge checks passed: %d tables, %ld certain, %ld uncertain\n", n, g_certain, g_unsure);
  return g_certain > 10 * g_unsure ? 0 : 3;
}
