"""Host (CPU) build of the part functions of the generated level programs (acc_part, pair_part)
against the plain definitions, summed over the parts, with parts cut at several sizes."""
import shutil
import subprocess

import pytest

from paper_2510_00193_amd.codegen import emit

SOURCE = r"""
#include <cmath>
#include <cstdio>
#include <random>
#define __device__
#define __forceinline__ inline
#define __restrict__
#define MTP_BLOCK_FENCE()
using std::fma;
#include MTP_LEVEL_HEADER
using L = MTP_LEVEL_STRUCT;
static std::mt19937_64 rng(7);
static double unif() { return std::uniform_real_distribution<double>(-1.5, 1.5)(rng); }
static double ma = 0, mg = 0;  // largest relative errors
static int seen[L::NMOM];

template <int P>
static void parts(const double* mb, const double* f, const double* h, double x, double y, double z, double* m, double* g) {
  if constexpr (P < L::NPART) {
    double loc[L::PART_MAX] = {0}, c[L::PART_MAX];
    L::template acc_part<P>(loc, f, x, y, z);
    for (int k = 0; k < L::PART_SIZE[P]; ++k) {
      const int e = L::PART_ENTRY[P][k];
      m[e] += loc[k];
      c[k] = mb[e];
      seen[e]++;
    }
    L::template pair_part<P>(c, f, h, x, y, z, g[0], g[1], g[2], g[3]);
    parts<P + 1>(mb, f, h, x, y, z, m, g);
  }
}

int main() {
  for (int rep = 0; rep < 20; ++rep) {
    double x = unif(), y = unif(), z = unif(), f[L::NMU], h[L::NMU], mb[L::NMOM], m[L::NMOM] = {0}, g[4] = {0};
    double want[4] = {0}, mag[4] = {0};
    for (auto& v : f) v = unif();
    for (auto& v : h) v = unif();
    for (auto& v : mb) v = unif();
    for (auto& v : seen) v = 0;
    parts<0>(mb, f, h, x, y, z, m, g);
    for (int e = 0; e < L::NMOM; ++e) {
      const int mu = L::ENTRIES[e][0], a = L::ENTRIES[e][1], b = L::ENTRIES[e][2], c = L::ENTRIES[e][3];
      const double mono = std::pow(x, a) * std::pow(y, b) * std::pow(z, c);
      ma = std::fmax(ma, seen[e] == 1 ? std::fabs(m[e] - f[mu] * mono) / std::fabs(f[mu] * mono) : 1.0);
      const double t[4] = {a ? f[mu] * a * std::pow(x, a - 1) * std::pow(y, b) * std::pow(z, c) : 0.0,
                           b ? f[mu] * b * std::pow(x, a) * std::pow(y, b - 1) * std::pow(z, c) : 0.0,
                           c ? f[mu] * c * std::pow(x, a) * std::pow(y, b) * std::pow(z, c - 1) : 0.0, h[mu] * mono};
      for (int k = 0; k < 4; ++k) { want[k] += mb[e] * t[k]; mag[k] += std::fabs(mb[e] * t[k]); }
    }
    for (int k = 0; k < 4; ++k)
      if (mag[k] > 0) mg = std::fmax(mg, std::fabs(g[k] - want[k]) / mag[k]);
  }
  std::printf("%.3e %.3e %d\n", ma, mg, L::NPART);
  return 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")
@pytest.mark.parametrize("level,cap,n_parts", [(2, 84, 1), (6, 84, 1), (10, 84, 1), (14, 84, 1), (16, 84, 2), (16, 50, 3),
                                               (20, 84, 4)])
def test_parts_match_the_definition(tmp_path, monkeypatch, level, cap, n_parts):
    """Errors: a product of at most 9 factors rounds to 9 x 2^-53 relative; a Horner sum of up to 300
    terms stays within 320 x 2^-53 of the sum of magnitudes."""
    monkeypatch.setattr(emit.moment_parts, "__defaults__", (cap,))
    (tmp_path / "level.inc").write_text(emit.emit_level(level, 1 if level < 18 else 3))
    (tmp_path / "main.cpp").write_text(SOURCE)
    exe = tmp_path / "main"
    subprocess.run(["g++", "-O1", "-std=c++17", f'-DMTP_LEVEL_HEADER="{tmp_path}/level.inc"',
                    f"-DMTP_LEVEL_STRUCT=Lv{level}", str(tmp_path / "main.cpp"), "-o", str(exe)], check=True)
    acc, grad, n = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split()
    assert int(n) == n_parts
    assert float(acc) < 2e-15 * (2 if level == 20 else 1), acc
    assert float(grad) < 320 * 2.0 ** -53, grad
