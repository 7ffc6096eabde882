"""The cosine and sine of the inlet modes' phases (nearer and cos_sin in csrc/stg.hip), compiled for the host from
the kernel's own source, against the 80-bit functions of the phase reduced by fmod.

A phase is omega t + ..., so its size is the caller's choice of time.  Bound: the FP64 reduction and
the polynomials are each good to about an ulp of a value of at most 1, and 2 pi in FP64 differs from
2 pi by 2.5e-16, by which a phase reduced to the other side of zero is off: 5e-16 in all."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

MAIN = r"""
#include <cmath>
#include <cstdio>
#include <cstdlib>
#define __device__
#define __forceinline__ inline
struct double2 { double x, y; };
static double2 make_double2(double x, double y) { return {x, y}; }
using std::fma; using std::trunc; using std::rint; using std::fabs; using std::ldexp; using std::ilogb;
%s
int main() {
  unsigned long long s = 88172645463325252ull;
  auto uniform = [&] { s ^= s << 13; s ^= s >> 7; s ^= s << 17; return (double)(s >> 11) / 9007199254740992.0; };
  for (int e = -20; e <= 1020; ++e) {
    double worst = 0.0;
    for (int k = 0; k < 400; ++k) {
      double ph = std::ldexp(1.0 + uniform(), e);
      if (k & 1) ph = -ph;
      if (k >= 300 && e < 50) ph = TWO_PI * std::rint(ph) * (1.0 + (k %% 3 - 1) * 2.3e-16);  // close to whole turns
      if (k >= 380 && e < 50) ph = TWO_PI / 8 * (2 * std::rint(ph) + 1);  // between quadrants
      const double2 v = cos_sin(far_phase(ph) ? nearer(ph) : ph);
      const long double r = std::fmod(ph, TWO_PI);
      const double d = (double)std::fmax(std::fabs(v.x - cosl(r)), std::fabs(v.y - sinl(r)));
      worst = d > worst || d != d ? d : worst;
    }
    std::printf("%%d %%.3e\n", e, worst);
  }
  const double2 n = cos_sin(nearer(INFINITY)), m = cos_sin(nearer(NAN));
  std::printf("nan %%d\n", n.x != n.x && n.y != n.y && m.x != m.x && m.y != m.y);
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_phases_of_every_size(tmp_path):
    text = open(os.path.join(ROOT, "paper_2304_04214_amd", "csrc", "stg.hip")).read()
    two_pi = re.search(r"^constexpr double TWO_PI = [^;]*;", text, flags=re.M).group(0)
    body = re.search(r"^__device__ __forceinline__ bool far_phase\(.*?^__device__ __forceinline__ double2 cos_sin.*?^}", text, flags=re.M | re.S).group(0)
    src, exe = str(tmp_path / "phases.cpp"), str(tmp_path / "phases")
    with open(src, "w") as f:
        f.write(MAIN % (two_pi + "\n" + body))
    subprocess.run(["g++", "-O2", "-ffp-contract=off", "-std=c++17", "-o", exe, src], check=True)
    lines = subprocess.run([exe], capture_output=True, text=True, check=True, timeout=120).stdout.split("\n")
    got = {int(l.split()[0]): float(l.split()[1]) for l in lines if l and not l.startswith("nan")}
    assert len(got) == 1041
    bad = {e: d for e, d in got.items() if not d <= 5e-16}
    assert not bad, ("phases of 2^e", dict(list(bad.items())[:5]), len(bad))
    assert "nan 1" in lines  # no phase: no plane, which the Mach check then reports
