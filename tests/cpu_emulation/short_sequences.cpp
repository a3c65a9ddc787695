// The device's element maps on the CPU (the header with its register constraints
// taken out, see the test), with the hardware reciprocal and reciprocal-square-root
// estimates modelled as the exact value times (1 + eps), |eps| up to the bounds
// measured on gfx950 (2^-24.36 and 2^-24.17), at both extremes and inside.
// Namespace xtmm holds the short sequences; namespace generic the same header
// with the IEEE operations in their place.  Prints, for each step, the inputs that
// the short form served and those of them that it served with other bits.
#include <math.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#define __device__
#define __constant__
#define __forceinline__ inline
#define __builtin_amdgcn_rsq est_rsq
#define __builtin_amdgcn_rcp est_rcp
#define __builtin_amdgcn_bitop3_b32(a, b, c, t) ((a) ^ (b) ^ (c))
#define __builtin_amdgcn_alignbit(a, b, n) \
  ((unsigned int)(((unsigned long long)(a) << 32 | (b)) >> (n)))

static uint64_t st = 0x9e3779b97f4a7c15ull;
static uint64_t rnd() { st ^= st << 13; st ^= st >> 7; st ^= st << 17; return st; }
static double urand() { return (double)(rnd() >> 11) * 0x1p-53; }
static double eps(double b) {
  const uint64_t k = rnd() % 4;
  return k == 0 ? b : k == 1 ? -b : (2.0 * urand() - 1.0) * b;
}
static double est_rsq(double x) {
  return (double)(1.0L / sqrtl((long double)x) * (1.0L + eps(0x1.c7p-25)));  // 2^-24.17
}
static double est_rcp(double x) {
  return (double)(1.0L / (long double)x * (1.0L + eps(0x1.8fp-25)));  // 2^-24.36
}

#include "short.h"
#include "generic.h"

static bool same(double a, double b) { return !memcmp(&a, &b, 8) || (a != a && b != b); }
template <class A, class B>
static bool same_state(const A& a, const B& b) {
  return same(a.x, b.x) && same(a.px, b.px) && same(a.y, b.y) && same(a.py, b.py) &&
         same(a.zeta, b.zeta) && same(a.delta, b.delta) && same(a.ptau, b.ptau) &&
         same(a.rpp, b.rpp) && same(a.rvv, b.rvv);
}
static double pow2(int lo, int hi) { return ldexp(1.0, lo + (int)(rnd() % (uint64_t)(hi - lo + 1))); }
// significands: random, next to all ones or to a power of two, both themselves
static double sig() {
  switch (rnd() % 6) {
    case 0: return 1.0;
    case 1: return 2.0 - 0x1p-52;
    case 2: return 1.0 + (double)(rnd() % 8) * 0x1p-52;
    case 3: return 2.0 - (double)(1 + rnd() % 8) * 0x1p-52;
    default: return 1.0 + urand();
  }
}
static double sign() { return rnd() & 1 ? 1.0 : -1.0; }
static void report(const char* what, long served, long wrong) {
  printf("%s served %ld wrong %ld\n", what, served, wrong);
}

int main(int argc, char** argv) {
  const long n = argc > 1 ? atol(argv[1]) : 1000000;
  {  // the quotient with a rounded reciprocal: quotients next to a midpoint of two
    long bad = 0;
    for (long i = 0; i < n; ++i) {
      const double b = sig() * pow2(-100, 100), r = 1.0 / b;
      double a = sig() * pow2(-300, 300) * sign();
      if (i & 1) {
        const double q = a / b, mid = fabs(nextafter(q, HUGE_VAL) - q) * 0.5;
        a = (double)(((long double)q + (long double)mid) * (long double)b);
        for (uint64_t k = rnd() % 3; k; --k) a = nextafter(a, rnd() & 1 ? HUGE_VAL : -HUGE_VAL);
      }
      bad += !same(xtmm::div_known(a, b, r), a / b);
    }
    report("div_known", n, bad);
  }
  {  // logarithm and deviate, next to the all-ones divisor among others
    long bad = 0;
    double c[xtmm::kLogCoefs], d[generic::kLogCoefs];
    xtmm::log_coef<xtmm::kLiteral>(c);
    generic::log_coef<generic::kLiteral>(d);
    for (long i = 0; i < n; ++i) {
      double x = urand() + 0x1p-54;
      if (i % 3 == 0) x = (1.0 + (double)((int)(rnd() % 64) - 32) * 0x1p-53) * pow2(-40, 0);
      bad += !same(xtmm::xlog(x, c), generic::xlog(x, d));
    }
    report("xlog", n, bad);
    bad = 0;
    for (long i = 0; i < n / 8; ++i) {
      const uint64_t seed = rnd();
      bad += !same(xtmm::gauss_at(seed, (long long)i, 3, 5, 0),
                   generic::gauss_at(seed, (long long)i, 3, 5, 0));
    }
    report("gauss_at", n / 8, bad);
  }
  const double beta0 = 1.0 - 6e-11, tob = 2.0 / beta0;
  // a particle whose derived fields are the rounded ones, and steps with operands
  // inside and outside of what they serve
  auto state = [&](xtmm::Pt& q, generic::Pt& g) {
    xtmm::Pt p{};
    const bool wild = rnd() % 4 == 0;
    auto v = [&](double scale) {
      if (wild && rnd() % 6 == 0) return rnd() % 3 ? sig() * pow2(-400, 400) * sign() : 0.0;
      return scale * (2.0 * urand() - 1.0);
    };
    p.x = v(1e-2); p.px = v(1e-3); p.y = v(1e-2); p.py = v(1e-3); p.zeta = v(0.1);
    p.ptau = rnd() % 16 ? v(0.01) : sign() * sig() * pow2(-80, 0);
    generic::Pt r{};
    r.ptau = p.ptau;
    generic::from_ptau(r, beta0, tob);
    p.delta = r.delta; p.rpp = r.rpp; p.rvv = r.rvv;
    p.opd2 = r.opd2; p.u = r.u; p.bpt = r.bpt;
    q = p;
    memcpy(&g, &q, sizeof g);
  };
  for (int run = 0; run < 4; ++run) {
    const int mode = 1 + run % 2;
    const bool no_kick = run >= 2;  // (a square that underflows among them)
    long served = 0, bad = 0;
    for (long i = 0; i < n; ++i) {
      xtmm::Pt q;
      generic::Pt g;
      state(q, g);
      const double scale = rnd() % 3 ? 1e-3 : pow2(-300, 4);
      double kx = scale * sig() * sign(), ky = scale * sig() * sign();
      if (rnd() % 8 == 0) kx = 0.0;
      if (no_kick) kx = rnd() % 8 ? 0.0 : pow2(-900, -600);
      if (rnd() % 8 == 0) ky = rnd() & 1 ? 0.0 : -0.0;
      if (no_kick) ky = rnd() & 1 ? 0.0 : -0.0;
      const double lr = rnd() % 2 ? sig() * pow2(-3, 5) : sig() * pow2(-99, 99);
      const double p0c = sig() * pow2(30, 40), c_mean = sig() * pow2(-40, 0),
                   c_quant = sig() * pow2(-60, -20), gamma0 = sig() * pow2(8, 17);
      const double dev = rnd() % 16 ? 3.0 * (2.0 * urand() - 1.0) : 0.0;
      bool flag = !xtmm::drift_range(q);
      const xtmm::Rad a{gamma0, c_mean, c_quant, p0c};
      const generic::Rad b{gamma0, c_mean, c_quant, p0c};
      if (mode == 1) xtmm::radiate_flag<1>(q, kx, ky, lr, 1.0 / lr, a, 1.0 / p0c, dev, beta0, tob, flag);
      else xtmm::radiate_flag<2>(q, kx, ky, lr, 1.0 / lr, a, 1.0 / p0c, dev, beta0, tob, flag);
      flag |= !(q.x == q.x);
      if (flag) continue;
      generic::radiate(g, kx, ky, lr, b, mode, mode == 2 ? dev : 0.0, beta0, tob);
      ++served;
      bad += !same_state(q, g);
    }
    report(no_kick ? (mode == 1 ? "no kick, mean" : "no kick, quantum")
                   : (mode == 1 ? "radiate mean" : "radiate quantum"), served, bad);
  }
  {
    long served = 0, bad = 0;
    for (long i = 0; i < n; ++i) {
      xtmm::Pt q;
      generic::Pt g;
      state(q, g);
      const double hxl = sig() * pow2(-100, 99) * sign(), lr = sig() * pow2(-100, 99);
      const double k0h = rnd() % 8 ? sig() * pow2(-200, 200) * sign() : 0.0;
      bool flag = !xtmm::drift_range(q);
      xtmm::curvature_flag(q, hxl, k0h, lr, 1.0 / lr, flag);
      flag |= !(q.x == q.x);
      if (flag) continue;
      generic::curvature(g, hxl, k0h, lr);
      ++served;
      bad += !same_state(q, g);
    }
    report("curvature", served, bad);
  }
  for (int cls = 0; cls <= 2; ++cls) {
    long served = 0, bad = 0;
    for (long i = 0; i < n; ++i) {
      xtmm::Pt q;
      generic::Pt g;
      state(q, g);
      double L = cls == 1 ? pow2(-600, 600) : sig() * pow2(-600, 599);
      if (cls == 0 && rnd() % 2) L = 0.1 + 50.0 * urand();
      int e;
      if (cls == 0 && frexp(L, &e) == 0.5) L = 1.5 * L;
      L *= sign();
      bool flag = !xtmm::drift_range(q);
      xtmm::drift_flag<false>(q, L, cls, xtmm::kDriftMin, flag);
      flag |= !(q.x == q.x);
      if (flag) continue;
      const generic::DriftIn d = generic::drift_in(g);
      double lp, dq;
      generic::drift_generic(L, d, lp, dq);
      generic::drift_apply(g, lp, dq);
      ++served;
      bad += !same_state(q, g) || !(d.pz2 > 0.0);
    }
    report(cls == 0 ? "drift" : cls == 1 ? "drift power of two" : "drift other", served, bad);
  }
  return 0;
}
