"""The selection's order-independent sum of squares (csrc/k_fixedsum.h),
compiled for the host and added up as the kernels do: each lane its own terms,
64 lanes by a wave, the waves into one pair of shared counters."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1309_0302_amd", "csrc")

MAIN = r"""
#include <stdio.h>
#include <stdlib.h>
#include "k_fixedsum.h"
using u64 = unsigned long long;
static u64 mix(u64 z) {
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}
// term i of the four kinds: all alike with every low bit set, spread over 30
// binary orders, tiny beside the bound, one large among small ones
static double term(int kind, u64 i) {
  const double u = (double)(mix(i + 1) >> 11) * 0x1p-53 + 0x1p-54;
  if (kind == 0) return 1.0 - 0x1p-53;
  if (kind == 1) return ldexp(u, -(int)(mix(i) % 30));
  if (kind == 2) return u * 0x1p-30;
  return i == 7 ? 1e6 : u * u;
}
int main(int argc, char** argv) {
  const int kind = atoi(argv[1]);
  const u64 waves = strtoull(argv[2], nullptr, 10), per = strtoull(argv[3], nullptr, 10);
  const u64 every = strtoull(argv[4], nullptr, 10);   // terms of a lane between carries
  const u64 n = waves * 64 * per;
  // the same sum in 128-bit fixed point, 2^-96 of the bound per unit
  double bound = 0.0;
  for (u64 i = 0; i < n; ++i) bound += term(kind, i);
  bound *= 1.0 + 1e-9;
  int ex;
  frexp(bound, &ex);
  unsigned __int128 ref = 0;
  const godec::FixedSum fs(bound);
  u64 hi = 0, lo = 0;   // the shared counters
  for (u64 w = 0; w < waves; ++w) {
    u64 whi = 0, wlo = 0;
    for (int l = 0; l < 64; ++l) {
      u64 lhi = 0, llo = 0;
      for (u64 e = 0; e < per; ++e) {
        const double q = term(kind, (w * per + e) * 64 + l);
        fs.add(q, lhi, llo);
        if (e % every == every - 1) godec::FixedSum::carry(lhi, llo);
        ref += (unsigned __int128)ldexp(q, 96 - ex);
      }
      godec::FixedSum::carry(lhi, llo);
      whi += lhi;
      wlo += llo;
    }
    godec::FixedSum::carry(whi, wlo);
    hi += whi;
    lo += wlo;
  }
  const double exact = ldexp((double)ref, ex - 96);
  printf("%.17g %.17g\n", fs.value(hi, lo), exact);
  return 0;
}
"""


@pytest.fixture(scope="module")
def prog(tmp_path_factory):
    d = tmp_path_factory.mktemp("fixedsum")
    src, exe = str(d / "main.hip"), str(d / "main")
    with open(src, "w") as f:
        f.write(MAIN)
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    subprocess.run([hipcc, "-O2", "-std=c++17", "--offload-host-only", "-I", CSRC, src, "-o", exe],
                   check=True, capture_output=True, text=True)
    return exe


# 6.4e7 terms in one wave and in thousands: the low limbs alone add up to
# several times 2^64
@pytest.mark.parametrize("kind", [0, 1, 2, 3])
@pytest.mark.parametrize("waves,per,every", [(1, 1000000, 16), (4000, 250, 1), (1, 1, 1),
                                             (65000, 1, 1), (1, 1000000, 1 << 23)])
def test_many_terms(prog, kind, waves, per, every):
    """What each term loses is below 2^-80 of the bound, and the value rounds
    twice."""
    out = subprocess.run([prog, str(kind), str(waves), str(per), str(every)], check=True,
                         capture_output=True, text=True).stdout.split()
    got, exact = float(out[0]), float(out[1])
    assert abs(got - exact) <= exact * 2.0 ** -51 + 64 * waves * per * 2.0 ** -80 * exact * 2.01
