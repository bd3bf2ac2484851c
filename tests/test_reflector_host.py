"""The scalars of a Householder reflector, made from the hardware's approximate
reciprocals, against sqrt and division: the kernel's own function compiled for
the host, with seeds that are off by up to 2^-22 (the hardware's by 2^-24).
Equal bits while alpha^2 + sigma^2 stays above 2^-960; below, the square root's
residual underflows: beta within 2 ulp, tau and scal equal for that beta."""

import os
import shutil
import subprocess

import pytest

from paper_2301_05844_amd import build

HEAD = """
#include <cmath>
#include <cstdio>
#include <random>
#define __device__
#define __forceinline__ inline
static double dq, dr;
static double rsq_(double x) { return (double)((1.0L / sqrtl((long double)x)) * (1.0L + dq)); }
static double rcp_(double x) { return (double)((1.0L / (long double)x) * (1.0L + dr)); }
#define __builtin_amdgcn_rsq rsq_
#define __builtin_amdgcn_rcp rcp_
using std::fma;
using std::fabs;
"""
# counts per scale: samples, beta unequal, beta beyond 2 ulp, tau or scal unequal
MAIN = r"""
int main() {
  std::mt19937_64 g(1);
  std::uniform_real_distribution<double> u(-1, 1);
  for (int scale : {0, 511, -300, -450, -511, -530}) {
    long n = 0, unequal = 0, far = 0, other = 0;
    for (int i = 0; i < 200000; ++i) {
      dq = 0x1p-22 * u(g);
      dr = 0x1p-22 * u(g);
      const int x = (int)(60 * fabs(u(g)));
      double al = ldexp(u(g), scale), s = fabs(ldexp(u(g), 2 * scale));
      if (i & 1) s = ldexp(s, -x);
      else al = ldexp(al, -x);
      const double s2 = fma(al, al, s);
      if (!(s > 0.0) || (scale > -500 && s2 < 0x1p-960)) continue;
      ++n;
      const Reflector h = make_reflector(al, s);
      const double nrm = sqrt(s2), be = al >= 0 ? -nrm : nrm;
      unequal += h.beta != be;
      far += !(fabs(h.beta - be) <= 2 * (nextafter(nrm, INFINITY) - nrm));
      other += h.tau != (h.beta - al) / h.beta || h.scal != 1.0 / (al - h.beta);
    }
    printf("%d %ld %ld %ld %ld\n", scale, n, unequal, far, other);
  }
  dq = dr = 0x1p-22;
  const Reflector a = make_reflector(0.7, 1e-40), b = make_reflector(-0.7, 1e-40),
                  z = make_reflector(0.3, 0.0);
  printf("exact %d\n", a.tau == 2.0 && a.beta == -0.7 && b.tau == 2.0 && b.beta == 0.7 &&
                          z.tau == 0.0 && z.scal == 0.0 && z.beta == 0.3);
}
"""


def test_reflector_scalars_are_those_of_sqrt_and_division(tmp_path):
    if not shutil.which("g++"):
        pytest.skip("no host compiler")
    with open(os.path.join(build.CSRC, "bbp_kernels.hip")) as f:
        text = f.read()
    start = text.index("struct Reflector {")
    end = text.index("\n}\n", text.index("make_reflector(double", start)) + 3
    src, exe = str(tmp_path / "r.cpp"), str(tmp_path / "r")
    with open(src, "w") as f:
        f.write(HEAD + text[start:end] + MAIN)
    subprocess.run(["g++", "-O2", "-ffp-contract=off", "-o", exe, src], check=True)
    out = subprocess.run([exe], check=True, capture_output=True, text=True).stdout.splitlines()
    print(out)
    for line in out[:-1]:
        scale, n, unequal, far, other = map(int, line.split())
        assert n > 50000 and far == 0 and other == 0
        assert unequal == 0 or scale < -500
    assert len(out) == 7 and out[-1] == "exact 1"
