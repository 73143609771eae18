"""Host (CPU) build of the wave programs (several waves per tile: energies, basis values, contraction
and moment adjoints, and their tangents) against the one-lane programs of the same level."""
import shutil
import subprocess

import pytest

from paper_2510_00193_amd.codegen.emit import emit_level

SOURCE = r"""
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <random>
#include <vector>
#define __device__
#define __forceinline__ inline
#define __restrict__
#define MTP_BLOCK_FENCE()
#define MTP_TILE_FENCE()
#define MTP_PIN(x)
using std::fma;
#include MTP_LEVEL_HEADER
using L = MTP_LEVEL_STRUCT;
using V = std::vector<double>;
static std::mt19937_64 rng(11);
static double unif() { return std::uniform_real_distribution<double>(-1.0, 1.0)(rng); }
static double err(const V& a, const V& b) {
  double num = 0, den = 1e-300;
  for (size_t k = 0; k < a.size(); ++k) { num = std::fmax(num, std::fabs(a[k] - b[k])); den = std::fmax(den, std::fabs(b[k])); }
  return num / den;
}
struct Reg { const double* m; double operator()(int e) const { return m[e]; } };
struct Put { double* p; int* n; void operator()(int k, double v) const { p[k] = v; n[k]++; } };

static V m(L::NMOM), md(L::NMOM), xi(L::NALPHA), crow(L::NGEN * 64), cdrow(L::NGEN * 64), cb(L::NGEN), cbd(L::NGEN);
static V B(L::NALPHA), out(L::NALPHA), mb(L::NMOM), mbd(L::NMOM), sh(64 * std::max(std::max(L::SHARED_ROWS, L::TSHARED_ROWS), 1));
static std::vector<int> hit(std::max(L::NMOM, L::NALPHA));
static double e = 0, c0b = 0, c0bd = 0;
static const double ebar = 0.7;
static double mbs[16][L::NMOM];

template <int W> static void fwd() {
  if constexpr (W < L::NFWAVE) {
    double ew = 0, cw = 0;
    L::fwd_wave<W, true>(Reg{m.data()}, xi.data(), crow.data(), B.data(), 1, ew, cw);
    e += ew; c0b += cw;
    fwd<W + 1>();
  }
}
template <int W> static void core() {
  if constexpr (W < L::NFWAVE) {
    double ew = 0, cw = 0;
    L::core_wave<W, true>(Reg{m.data()}, xi.data(), crow.data(), Put{cb.data(), hit.data()}, B.data(), 1, ew, cw);
    e += ew; c0b += cw;
    core<W + 1>();
  }
}
template <int W> static void rev() {
  if constexpr (W < L::NRWAVE) {
    L::rev_wave<W>(Reg{m.data()}, Reg{cb.data()}, xi.data(), mbs[W], Put{mb.data(), hit.data()});
    rev<W + 1>();
    }
}
template <int W> static void comb() {
  if constexpr (W < L::NRWAVE) { L::rev_combine<W>(mbs[W], sh.data(), Put{mb.data(), hit.data()}); comb<W + 1>(); }
}
template <int W> static void tfwd() {
  if constexpr (W < L::NTFWAVE) {
    L::tfwd_wave<W>(Reg{m.data()}, Reg{md.data()}, xi.data(), ebar, crow.data(), cdrow.data(), out.data(), 1, c0bd);
    tfwd<W + 1>();
  }
}
template <int W> static void tcore() {
  if constexpr (W < L::NTFWAVE) {
    L::tcore_wave<W>(Reg{m.data()}, Reg{md.data()}, xi.data(), ebar, crow.data(), cdrow.data(), Put{cbd.data(), hit.data()}, out.data(), 1, c0bd);
    tcore<W + 1>();
  }
}
template <int W> static void trev() {
  if constexpr (W < L::NTRWAVE) {
    L::trev_wave<W>(Reg{m.data()}, Reg{md.data()}, Reg{cb.data()}, Reg{cbd.data()}, xi.data(), mbs[W], Put{mbd.data(), hit.data()});
    trev<W + 1>();
  }
}
template <int W> static void tcomb() {
  if constexpr (W < L::NTRWAVE) { L::trev_combine<W>(mbs[W], sh.data(), Put{mbd.data(), hit.data()}); tcomb<W + 1>(); }
}
template <int P> static void oldrevtan(const double* Cb, const double* Cbd, double* o) {
  if constexpr (P < L::NRTPART) { L::rev_tan<P, double>(Reg{m.data()}, Reg{md.data()}, Cb, Cbd, o, 1); oldrevtan<P + 1>(Cb, Cbd, o); }
}
template <int G> static void oldrev(const double* Cb, double* o) {
  if constexpr (G < L::NGROUP) { L::rev<G, double>(Reg{m.data()}, Cb, o + L::GROUP_LO[G]); oldrev<G + 1>(Cb, o); }
}
static int once(int n) { int bad = 0; for (int k = 0; k < n; ++k) { bad += hit[k] != 1; hit[k] = 0; } return bad; }

int main() {
  for (auto* v : {&m, &md, &xi}) for (auto& x : *v) x = unif();
  V C(L::NCOMP), Cd(L::NCOMP), Cb(L::NCOMP), Cb2(L::NCOMP), Cbd(L::NCOMP), B0(L::NALPHA), out0(L::NALPHA), mb0(L::NMOM), mbd0(L::NMOM);
  L::fwd<double>(Reg{m.data()}, C.data());
  const double e0 = L::products<true, double>(C.data(), xi.data(), Cb.data(), B0.data(), 1);
  oldrev<0>(Cb.data(), mb0.data());
  L::fwd_tan<double>(Reg{m.data()}, Reg{md.data()}, C.data(), Cd.data());
  L::products_tan<double>(C.data(), Cd.data(), xi.data(), ebar, Cb2.data(), Cbd.data(), out0.data(), 1);
  oldrevtan<0>(Cb.data(), Cbd.data(), mbd0.data());
  fwd<0>();
  core<0>();
  cb[L::GEN0] = c0b;
  hit[L::GEN0]++;
  int bad = once(L::NGEN);
  rev<0>();
  comb<0>();
  bad += once(L::NMOM);
  tfwd<0>();
  tcore<0>();
  cbd[L::GEN0] = c0bd;
  hit[L::GEN0]++;
  bad += once(L::NGEN);
  trev<0>();
  tcomb<0>();
  bad += once(L::NMOM);
  std::printf("%.3e %.3e %.3e %.3e %.3e %d\n", std::fabs(e - e0) / std::fmax(1.0, std::fabs(e0)), err(B, B0), err(mb, mb0), err(out, out0), err(mbd, mbd0), bad);
  return 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")
@pytest.mark.parametrize("level", [12, 14, 16, 20])
def test_wave_programs_match_the_one_lane_programs(tmp_path, level):
    """Every output written exactly once; sums of up to 500 terms of order one: 1e-12 of the largest."""
    (tmp_path / "level.inc").write_text(emit_level(level, 1 if level < 18 else 3))
    (tmp_path / "main.cpp").write_text(SOURCE)
    exe = tmp_path / "main"
    subprocess.run(["g++", "-O0", "-std=c++17", f'-DMTP_LEVEL_HEADER="{tmp_path}/level.inc"',
                    f"-DMTP_LEVEL_STRUCT=Lv{level}", str(tmp_path / "main.cpp"), "-o", str(exe)], check=True)
    got = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split()
    assert int(got[-1]) == 0, got
    assert all(float(x) < 1e-12 for x in got[:-1]), got
