"""Distance and inverse distance of a pair from an estimate of the inverse root: errors against extended
precision on the host, and the special values the kernels meet."""
import subprocess

from paper_2510_00193_amd import build

SOURCE = r"""
#include "mtp_device.h"
#include <cmath>
#include <cstdio>
#include <random>
int main() {
  std::mt19937_64 rng(5);
  std::uniform_real_distribution<double> expo(-12.0, 12.0), delta(-1.0, 1.0);
  long double er = 0, ei = 0;  // largest errors in ulps of the exact value
  for (int k = 0; k < 400000; ++k) {
    const double dd = std::exp2(expo(rng));
    const double edge[4] = {1.0, -1.0, delta(rng), 0.0};
    const double y0 = (double)(1.0L / sqrtl(dd)) * (1.0 + edge[k % 4] * 0x1p-23);
    double r, rinv;
    mtp::root_from_estimate(dd, y0, r, rinv);
    const long double sr = sqrtl(dd), si = 1.0L / r;  // the inverse of the r that the kernels use
    er = fmaxl(er, fabsl(r - sr) / (nextafter((double)sr, 1e300) - (double)sr));
    ei = fmaxl(ei, fabsl(rinv - si) / (nextafter((double)si, 1e300) - (double)si));
  }
  double r0, i0, rn, in, rt, it;
  mtp::root_from_estimate(0.0, INFINITY, r0, i0);
  mtp::root_from_estimate(NAN, NAN, rn, in);
  mtp::root_from_estimate(1e-280, 1e140, rt, it);
  std::printf("%.6Lf %.6Lf %d %d %d\n", er, ei, r0 == 0.0 && std::isinf(i0) && i0 > 0, std::isnan(rn) && std::isnan(in),
              std::fabs(rt * 1e140 - 1.0) < 1e-15 && std::fabs(it / 1e140 - 1.0) < 1e-15);
  return 0;
}
"""


def test_root_and_inverse_from_an_estimate(tmp_path):
    """Half an ulp of rounding each, and what the estimate's 2^-23 and the reference's own rounding
    (2^-11 ulp) leave."""
    src, exe = tmp_path / "root.hip", tmp_path / "root"
    src.write_text(SOURCE)
    subprocess.run([build.HIPCC, *build.FLAGS, "-mfma", str(src), "-o", str(exe)], check=True, capture_output=True, text=True)
    er, ei, zero, nan, tiny = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split()
    assert float(er) < 0.501, er
    assert float(ei) < 0.501, ei
    assert (zero, nan, tiny) == ("1", "1", "1")
