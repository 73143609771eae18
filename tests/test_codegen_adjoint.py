"""Host (CPU) build of the stages of the adjoint pair pass and of the parts of the moment tangent, called
as the kernels call them (coefficients ebar mb - mbd of the value polynomials, ebar not zero), against the
plain definitions."""
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
static std::mt19937_64 rng(9);
static double unif() { return std::uniform_real_distribution<double>(-1.5, 1.5)(rng); }
static double d[3], t[3];  // displacement and its tangent

template <int B>
static void stages(const double* mb, const double* mbd, double ebar, double* S, double* X) {
  if constexpr (B < L::NASTAGE) {
    double c[L::ADJ_MAX];
    for (int k = 0; k < L::ADJ_SIZE[B]; ++k) {
      const int e = L::ADJ_ENTRY[B][k];
      c[k] = L::ADJ_VALUE[B][k] ? fma(ebar, mb[e], -mbd[e]) : mb[e];
    }
    L::template adj_stage<B>(c, d[0], d[1], d[2], t[0], t[1], t[2], S, X);
    stages<B + 1>(mb, mbd, ebar, S, X);
  }
}
template <int P>
static void tangents(const double* f, const double* fd, double* md, int* seen) {
  if constexpr (P < L::NTPART) {
    double loc[L::TPART_MAX] = {0};
    L::template tan_part<P>(loc, f, fd, d[0], d[1], d[2], t[0], t[1], t[2]);
    for (int k = 0; k < L::TPART_SIZE[P]; ++k) {
      md[L::TPART_ENTRY[P][k]] += loc[k];
      seen[L::TPART_ENTRY[P][k]]++;
    }
    tangents<P + 1>(f, fd, md, seen);
  }
}

int main() {
  double es = 0, ex = 0, et = 0;  // largest errors over the sum of magnitudes
  for (int rep = 0; rep < 20; ++rep) {
    const double ebar = rep % 4 ? unif() : 0.0;
    double mb[L::NMOM], mbd[L::NMOM], f[L::NMU], fd[L::NMU], S[L::NMU] = {0}, X[L::NMU] = {0}, md[L::NMOM] = {0};
    double ws[L::NMU] = {0}, wx[L::NMU] = {0}, ms[L::NMU] = {0}, mx[L::NMU] = {0};
    int seen[L::NMOM] = {0};
    for (int k = 0; k < 3; ++k) { d[k] = unif(); t[k] = unif(); }
    for (auto& v : mb) v = unif();
    for (auto& v : mbd) v = unif();
    for (auto& v : f) v = unif();
    for (auto& v : fd) v = unif();
    stages<0>(mb, mbd, ebar, S, X);
    tangents<0>(f, fd, md, seen);
    for (int e = 0; e < L::NMOM; ++e) {
      const int mu = L::ENTRIES[e][0];
      double mono = 1.0, grad = 0.0, gmag = 0.0;
      for (int k = 0; k < 3; ++k) mono *= std::pow(d[k], L::ENTRIES[e][1 + k]);
      for (int k = 0; k < 3; ++k) {
        double part = L::ENTRIES[e][1 + k];
        for (int q = 0; q < 3; ++q)
          if (part != 0.0) part *= std::pow(d[q], L::ENTRIES[e][1 + q] - (q == k));
        grad += t[k] * part;
        gmag += std::fabs(t[k] * part);
      }
      ws[mu] += mb[e] * mono;
      ms[mu] += std::fabs(mb[e] * mono);
      wx[mu] += (ebar * mb[e] - mbd[e]) * mono - mb[e] * grad;
      mx[mu] += (std::fabs(ebar * mb[e]) + std::fabs(mbd[e])) * std::fabs(mono) + std::fabs(mb[e]) * gmag;
      const double want = fd[mu] * mono + f[mu] * grad;
      et = std::fmax(et, seen[e] == 1 ? std::fabs(md[e] - want) / (std::fabs(fd[mu] * mono) + std::fabs(f[mu]) * gmag) : 1.0);
    }
    for (int mu = 0; mu < L::NMU; ++mu) {
      es = std::fmax(es, std::fabs(S[mu] - ws[mu]) / ms[mu]);
      ex = std::fmax(ex, std::fabs(X[mu] - wx[mu]) / mx[mu]);
    }
  }
  std::printf("%.3e %.3e %.3e %d %d\n", es, ex, et, L::NASTAGE, L::NTPART);
  return 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")
@pytest.mark.parametrize("level,n_stages,n_parts", [(10, 1, 1), (14, 2, 2), (16, 4, 2), (20, 8, 5)])
def test_stages_and_parts_match_the_definitions(tmp_path, level, n_stages, n_parts):
    """Sums of at most 300 terms of at most 12 roundings each: 320 x 2^-53 of the sum of magnitudes; a
    tangent is one term of three products: 40 x 2^-53."""
    prog = emit.build_program(level)
    items = prog.layout.items
    w = emit._W()
    w(f"struct Lv{level} {{")
    w(f"static constexpr int NMOM = {len(items)}, NMU = {max(it[0] for it in items) + 1};")
    w("static constexpr int ENTRIES[NMOM][4] = {" + ", ".join("{%d, %d, %d, %d}" % it for it in items) + "};")
    emit._emit_tangent_moment_parts(w, prog, emit.moment_parts(prog, emit.TANGENT_PART_CAP))
    emit._emit_adj_stages(w, prog, emit.adj_stages(prog))
    w("};")
    (tmp_path / "level.inc").write_text(w.text())
    (tmp_path / "main.cpp").write_text(SOURCE)
    exe = tmp_path / "main"
    subprocess.run(["g++", "-O0", "-std=c++17", f'-DMTP_LEVEL_HEADER="{tmp_path}/level.inc"',
                    f"-DMTP_LEVEL_STRUCT=Lv{level}", str(tmp_path / "main.cpp"), "-o", str(exe)], check=True)
    s, x, t, stages, parts = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split()
    assert (int(stages), int(parts)) == (n_stages, n_parts)
    assert float(s) < 320 * 2.0 ** -53 and float(x) < 320 * 2.0 ** -53, (s, x)
    assert float(t) < 40 * 2.0 ** -53, t
