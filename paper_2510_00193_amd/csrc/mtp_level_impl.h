// Level-templated MTP kernels.  A translation unit includes one generated level header
// (struct LvXX with the straight-line program) and then this file, and instantiates the
// launchers with MTP_DEFINE_CHAIN / MTP_DEFINE_ADJ / MTP_DEFINE_ADJ_FWD / MTP_DEFINE_ADJ_REV.
//
// The pair kernels give an atom one lane, or two, four or eight where there are few atoms; levels of many
// entries cut them over waves that each hold a part of the atom's moments or adjoints in registers (with
// compile-time indices) and walk the same CSR row, or hand its pairs on along a pipeline.  The contraction
// programs run one lane per atom up to level 10 and in binary32, above in several waves per 64 atoms with
// the moments in LDS.
#pragma once
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>
#include <utility>

#include "mtp_device.h"
#include "mtp_internal.h"

namespace mtp {

constexpr int kLaneBlock = 64;   // one wave per workgroup for the lane-per-atom kernels
constexpr int kMaxWaves = 8;     // waves a SIMD can hold

// Tiles of kLaneBlock atoms a workgroup of a pair kernel processes: its own block of the grid
// (PERSIST false: the loop body runs once), or, for a persistent launch, tiles pulled from the
// device counter a.queue until none is left, so that workgroups that finish early take the
// remaining tiles.  Every tile writes its own outputs (per-tile partials included), so the
// result does not depend on which workgroup takes which tile.
template <bool PERSIST>
struct TileLoop {
  int nblocks;
  int* slot;  // LDS word that broadcasts a pulled tile to the workgroup
  __device__ __forceinline__ int pull(int* q) const {
    __syncthreads();
    if (threadIdx.x == 0) *slot = atomicAdd(q, 1);
    __syncthreads();
    return *slot;
  }
  __device__ __forceinline__ int first(const SysArgs& a) const {
    if constexpr (PERSIST) return pull(a.queue);
    else return xcd_logical_block(blockIdx.x, gridDim.x);
  }
  __device__ __forceinline__ int next(const SysArgs& a) const {
    if constexpr (PERSIST) return pull(a.queue);
    else return nblocks;
  }
};
// tiles of kLaneBlock / k atoms (k lanes per atom)
__host__ __device__ inline int split_tiles(int n, int k) { return (int)(((long)n * k + kLaneBlock - 1) / kLaneBlock); }
// K lanes per atom, NP workgroups (parts) per tile: b counts tile * NP + part
#define MTP_FOR_TILES_K(a, n, K, NP, b)                                                                \
  __shared__ int tile_slot_[1]; /* no storage unless PERSIST uses it */                                \
  const TileLoop<PERSIST> tiles_{split_tiles(n, K) * (NP), tile_slot_};                                \
  for (int b = tiles_.first(a); b < tiles_.nblocks; b = tiles_.next(a))
#define MTP_FOR_TILES(a, n, b) MTP_FOR_TILES_K(a, n, 1, 1, b)

// Sum over the K consecutive lanes of an atom (K = 1, 2, 4, 8) by DPP lane exchanges inside
// quads and half-rows; every lane of the group ends with the same value (each step adds two
// equal partial sums in either order, which is exact commutativity).
template <int CTRL>
__device__ __forceinline__ double dpp_exchange(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xF, 0xF, true);
  return __hiloint2double(hi, lo);
}
template <int CTRL>
__device__ __forceinline__ float dpp_exchange(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true));
}
template <int K, class R>
__device__ __forceinline__ R group_sum(R v) {
  static_assert(K == 1 || K == 2 || K == 4 || K == 8, "lanes per atom");
  if constexpr (K >= 2) v += dpp_exchange<0xB1>(v);   // quad_perm [1, 0, 3, 2]
  if constexpr (K >= 4) v += dpp_exchange<0x4E>(v);   // quad_perm [2, 3, 0, 1]
  if constexpr (K >= 8) v += dpp_exchange<0x141>(v);  // row_half_mirror
  return v;
}

// Sum over the 64 lanes of a wave in a fixed order (every lane gets it): DPP exchanges inside
// 16-lane rows (quads, half-row mirror, row mirror), two cross-row exchanges.
__device__ __forceinline__ double wave_sum(double v) {
  v += dpp_exchange<0xB1>(v);   // quad_perm [1, 0, 3, 2]
  v += dpp_exchange<0x4E>(v);   // quad_perm [2, 3, 0, 1]
  v += dpp_exchange<0x141>(v);  // row_half_mirror
  v += dpp_exchange<0x140>(v);  // row_mirror
  v += __shfl_xor(v, 16, 64);
  v += __shfl_xor(v, 32, 64);
  return v;
}

// Workgroups of a pair kernel: one per tile (nb), or, persistent, as many of `waves` waves as the SIMDs hold:
// two waves each where a tile is cut into `parts`, else one.  Passes with persistent kernels, workgroups for
// one wave per SIMD -> for two, ms: 540,428 atoms of level 20 16.79 -> 15.96, 272,280 of level 16 2.44 -> 2.33
// (one-shot 15.89, 2.33), but 540,428 of level 10 in sorted order 2.58 -> 2.87.
inline int pair_grid(const SysArgs& a, int nb, int parts, int waves) {
  if (!a.queue || a.split != 1) return nb;
  return std::max(1, std::min(nb, a.simds * (parts > 1 ? 2 : 1) / waves));
}

// Accessors of [row][atom] arrays in global memory.  The address of a row is the same for the
// whole wave (scalar registers) and each lane adds its byte offset, so a load takes the
// scalar-base form: no per-row 64-bit address is kept in vector registers (the compiler
// otherwise precomputes the addresses of every row a program reads and spills them).
// The host caps a chunk (the atoms of one row) at 2^28, so the byte offset fits 32 bits.
__device__ __forceinline__ unsigned lane_bytes(int li, int size) { return (unsigned)li * (unsigned)size; }

// Moment vector of a lane, [entry][atom] layout.
template <class R>
struct GlobalMoments {
  const R* __restrict__ base;
  long ld;
  unsigned off;  // byte offset of the lane's atom in a row
  __device__ __forceinline__ R operator()(int e) const {
    return *reinterpret_cast<const R*>(reinterpret_cast<const char*>(base + (long)e * ld) + off);
  }
};

// The same with a per-lane 64-bit pointer (vector addresses): measured faster for the forward
// program kernels (k_program, k_program_fwd), whose few spills do not come from addresses.
template <class R>
struct LaneMoments {
  const R* __restrict__ p;
  long ld;
  __device__ __forceinline__ R operator()(int e) const { return p[(long)e * ld]; }
};

// Per-lane vector read from a [component][atom] array in global memory, one load per use.
template <class R>
struct GlobalVector {
  const R* __restrict__ base;
  long ld;
  unsigned off;
  __device__ __forceinline__ R operator[](int q) const {
    return *reinterpret_cast<const R*>(reinterpret_cast<const char*>(base + (long)q * ld) + off);
  }
};

// Per-lane element i of a [row][atom] array written in place (i = row * ld).
template <class R>
struct LaneRows {
  R* __restrict__ base;
  unsigned off;
  __device__ __forceinline__ R& operator[](long i) const {
    return *reinterpret_cast<R*>(reinterpret_cast<char*>(base + i) + off);
  }
};

// Contraction-adjoint vectors longer than this are read from memory where a block needs them
// instead of being loaded into registers up front (which spills at the largest levels).
constexpr int kRegComps = 64;

// Per-lane vector held in LDS in [component][lane] layout (conflict-free across a wave).
template <class R>
struct LaneVector {
  const R* p;
  __device__ __forceinline__ R operator[](int q) const { return p[q * kLaneBlock]; }
};

template <class R>
struct RegMoments {
  const R* m;
  __device__ __forceinline__ R operator()(int e) const { return m[e]; }
};

// radial coefficient table staged in LDS (in the arithmetic type of the kernel); dynamic shared
// memory of radial_bytes at the launch, so that a small table leaves room for more waves.  The rows of two
// species are an odd number of values apart: lanes of a wave read the same place of different rows, and
// rows of a multiple of 32 values (8 Chebyshev functions of 4 radial functions) would meet in the same
// banks.  The parts of a tile each read the table: grade of 101,306 atoms at level 16, 16 functions and
// four species, 399 us in one part with rows end to end, 479 in two parts, 278 with odd rows.
template <int NMU, int NC = 0>
__host__ __device__ __forceinline__ int radial_row(int ncheb) { return NMU * (NC > 0 ? NC : ncheb) | 1; }

template <class R, int NMU>
__device__ __forceinline__ R* stage_radial(const SysArgs& a) {
  extern __shared__ __align__(16) double radial_table_[];
  R* sh = reinterpret_cast<R*>(radial_table_);
  const int row = NMU * a.ncheb, n = a.nsp * a.nsp * row;
  if (row & 1 || a.nsp == 1) {
    for (int k = threadIdx.x; k < n; k += blockDim.x) sh[k] = (R)a.radial[k];
  } else {
    for (int k = threadIdx.x; k < n; k += blockDim.x) sh[k + (unsigned)k / (unsigned)row] = (R)a.radial[k];
  }
  __syncthreads();
  return sh;
}
template <class R, int NMU>
inline unsigned radial_bytes(const SysArgs& a) {
  return (unsigned)(a.nsp * a.nsp * radial_row<NMU>(a.ncheb) * (int)sizeof(R));
}

// One lane per atom: the lanes of a wave read 64 different rows of the list, so each 4-byte read
// of a list array touches 64 cache lines, and the lines of the four waves of a CU do not stay in
// its 32 KB L1 until the next pair; the refills bounded the pair loops (the loads issued a whole
// pair ahead were still waited for: with the instructions cut by a quarter the pair-gradient kernel
// stayed at 1.14 ms at a million atoms, staged rows took it to 0.95).  So a lane copies its row,
// kRowStage pairs at a time with 16-byte reads, to a column of its own in LDS (16 KB per wave) and reads
// the pairs from there.  A read of four may pass the end of its row, but not of the list: the waves of
// the last rows read entry by entry, which one test per wave decides.  A stage takes about 130
// instructions; with selects in every read and single entries written it took 740, and the wave's first
// pair waits for it.  Evaluations in binary32, unstaged / that way / now: 33,600 atoms of 42 pairs at
// level 12 122 / 128 / 122 us, 63,488 of 27 at level 16 142 / 148 / 142.
constexpr int kRowStage = 32;
constexpr int kStageInts = 2 * kRowStage * kLaneBlock;  // partners, then shifts: [pair][lane] each
struct ListEntry {
  int j, shift;
};
__device__ __forceinline__ ListEntry staged(const int* col, int k) {
  return ListEntry{col[k * kLaneBlock], col[(kRowStage + k) * kLaneBlock]};
}
__device__ __forceinline__ void stage_entry(int* col, int k, ListEntry e) {
  col[k * kLaneBlock] = e.j;
  col[(kRowStage + k) * kLaneBlock] = e.shift;
}

// Copy pairs [p, p + m) of a row to the lane's LDS column; 1 <= m <= kRowStage.  Up to three entries past
// m are written with them (pairs of other rows, not used).
__device__ __forceinline__ void stage_row(const SysArgs& a, int p, int m, int* __restrict__ col) {
  typedef int v4i __attribute__((ext_vector_type(4), aligned(4)));
  if (__any(p > a.npairs - kRowStage)) {
    for (int k = 0; k < m; ++k) stage_entry(col, k, ListEntry{a.nj[p + k], a.shift[p + k]});
    return;
  }
  v4i j[kRowStage / 4], s[kRowStage / 4];
#pragma unroll
  for (int k = 0; k < kRowStage / 4; ++k)
    if (4 * k < m) {
      j[k] = *reinterpret_cast<const v4i*>(a.nj + p + 4 * k);
      s[k] = *reinterpret_cast<const v4i*>(a.shift + p + 4 * k);
    }
#pragma unroll
  for (int k = 0; k < kRowStage / 4; ++k)
    if (4 * k < m) {
#pragma unroll
      for (int q = 0; q < 4; ++q) stage_entry(col, 4 * k + q, ListEntry{j[k][q], s[k][q]});
    }
}

// Position and species of a pair's partner, and with TAN its force cotangent.
template <bool TAN>
struct Partner {
  double x, y, z, bx, by, bz;
  int s;
  __device__ __forceinline__ void load(const SysArgs& a, const double* __restrict__ fbar, int j) {
    x = a.pos[3 * j];
    y = a.pos[3 * j + 1];
    z = a.pos[3 * j + 2];
    s = a.species[j];
    if constexpr (TAN) {
      bx = fbar[3 * j];
      by = fbar[3 * j + 1];
      bz = fbar[3 * j + 2];
    }
  }
};

// One pair as the bodies of the pair loops see it: species of the partner, displacement, distance and
// its inverse, and with TAN the difference of the force cotangents (partner minus centre).
struct Pair {
  int zj;
  double dx, dy, dz, r, rinv, ex, ey, ez;
};

// Displacement, then prefetch() (the next pair's loads, into the registers this pair's partner just
// left: no copies, which would wait for the loads), then distance and body(p, pair).  own: the centre
// atom.  The barriers keep the scheduler from moving the loads.  R is the arithmetic type of the
// kernel (binary32 kernels round the correctly rounded r).
template <class R, bool TAN, class P, class F>
__device__ __forceinline__ void one_pair(const SysArgs& a, int p, int sh, const double* H, const Partner<TAN>& own,
                                         const Partner<TAN>& q, P&& prefetch, F&& body) {
  Pair t;
  int n1, n2, n3;
  unpack_shift(sh, n1, n2, n3);
  pair_displacement(own.x, own.y, own.z, q.x, q.y, q.z, n1, n2, n3, H, t.dx, t.dy, t.dz);
  if constexpr (TAN) {
    t.ex = q.bx - own.bx;
    t.ey = q.by - own.by;
    t.ez = q.bz - own.bz;
  }
  t.zj = clamp_species(q.s, a.nsp);
  __builtin_amdgcn_sched_barrier(0);
  prefetch();
  __builtin_amdgcn_sched_barrier(0);
  if constexpr (std::is_same_v<R, double>) {
    root_and_inverse(dist2_exact(t.dx, t.dy, t.dz), t.r, t.rinv);
  } else {
    t.r = sqrt(dist2_exact(t.dx, t.dy, t.dz));
    t.rinv = 0.0;  // not used
  }
  body(p, t);
}

// Wait for every outstanding vector memory operation (vmcnt 0; the other counters at their
// maximum).  Before a pair loop: the waits inside it are then counted for the loop's own
// operations alone, not for the path that enters it.
__device__ __forceinline__ void drain_loads() { __builtin_amdgcn_s_waitcnt(0x0F70); }

// Walk the CSR row of atom i with software prefetch: the partner's data are loaded one pair ahead,
// so the gather latency overlaps the arithmetic of the current pair.  The prefetch index is clamped
// to the row instead of guarded: a loop body without branches around its memory operations lets the
// waits count them exactly, so the wait for a pair's loads does not also wait for younger stores
// (guarded loads and stores make every wait a full drain).
// With K lanes per atom, lane sub of the atom takes pairs sub, sub + K, sub + 2K, ... of the row
// (the lanes of an atom read consecutive list entries); with one, lst is the wave's LDS stage.
template <int K, class R, bool TAN, class F>
__device__ __forceinline__ void for_pairs(const SysArgs& a, int* lst, int i, int sub, const double* H,
                                          const Partner<TAN>& own, const double* __restrict__ fbar, F&& body) {
  const int p0 = a.off[i] + sub, p1 = a.off[i + 1];
  Partner<TAN> q;
  if constexpr (K == 1) {
    int* col = lst + (threadIdx.x & (kLaneBlock - 1));
    for (int b = p0; b < p1; b += kRowStage) {
      const int m = min(kRowStage, p1 - b);
      stage_row(a, b, m, col);
      ListEntry cur = staged(col, 0), nxt = staged(col, m > 1);
      q.load(a, fbar, cur.j);
      int k = 0;
      drain_loads();
      do {
        one_pair<R, TAN>(
            a, b + k, cur.shift, H, own, q,
            [&]() {
              cur = nxt;
              q.load(a, fbar, cur.j);
              nxt = staged(col, min(k + 2, m - 1));
            },
            body);
        ++k;
      } while (k < m);
    }
  } else {
    if (p0 >= p1) return;
    const int pB = min(p0 + K, p1 - 1);
    int jA = a.nj[p0], shA = a.shift[p0], jB = a.nj[pB], shB = a.shift[pB];
    q.load(a, fbar, jA);
    int p = p0;
    drain_loads();
    do {
      one_pair<R, TAN>(
          a, p, shA, H, own, q,
          [&]() {
            q.load(a, fbar, jB);
            shA = shB;
            const int pn = min(p + 2 * K, p1 - 1);
            jB = a.nj[pn];
            shB = a.shift[pn];
          },
          body);
      p += K;
    } while (p < p1);
  }
}

// The same with T steps in every lane, for the first wave of a pipeline of waves.  A lane past its len pairs
// repeats its last one, or, without pairs in the present stage of its row, takes atom i itself, at no
// distance; the results of these steps are dropped.
template <int K, bool TAN, class F>
__device__ __forceinline__ void for_steps(const SysArgs& a, int* lst, int i, int lane, int p0, int len, int T,
                                          const double* H, const Partner<TAN>& own, const double* __restrict__ fbar,
                                          F&& body) {
  Partner<TAN> q;
  if constexpr (K == 1) {
    int* col = lst + lane;
    for (int b = 0; b < T; b += kRowStage) {
      const int m = min(kRowStage, len - b), kn = min(kRowStage, T - b);
      if (m > 0) stage_row(a, p0 + b, m, col);
      else stage_entry(col, 0, ListEntry{i, 0});  // a lane past its row
      const int last = max(m - 1, 0);
      ListEntry cur = staged(col, 0), nxt = staged(col, min(1, last));
      q.load(a, fbar, cur.j);
      drain_loads();
      for (int k = 0; k < kn; ++k) {
        one_pair<double, TAN>(
            a, b + k, cur.shift, H, own, q,
            [&]() {
              cur = nxt;
              q.load(a, fbar, cur.j);
              nxt = staged(col, min(k + 2, last));
            },
            body);
      }
    }
  } else if (T > 0) {
    // entry t of the lane; a lane without pairs reads the first entry of the (non-empty) list
    auto at = [&](int t) { return len > 0 ? p0 + min(t, len - 1) * K : 0; };
    int jA = a.nj[at(0)], shA = a.shift[at(0)], jB = a.nj[at(1)], shB = a.shift[at(1)];
    q.load(a, fbar, jA);
    drain_loads();
    for (int t = 0; t < T; ++t) {
      one_pair<double, TAN>(
          a, t, shA, H, own, q,
          [&]() {
            q.load(a, fbar, jB);
            shA = shB;
            jB = a.nj[at(t + 2)];
            shB = a.shift[at(t + 2)];
          },
          body);
    }
  }
}

// Of the pairs p0, p0 + k, ... below p1 (k a power of two): those in [lo, hi).
__device__ __forceinline__ void clip_pairs(int k, int lo, int hi, int& p0, int& p1) {
  p0 += max(lo - p0 + k - 1, 0) & -k;
  p1 = min(p1, hi);
}

// pairs of a lane (every K-th of its atom's row from sub on; with CLIP those in [lo, hi)) and the longest
// such count of the wave
template <int K, bool CLIP = false>
__device__ __forceinline__ int lane_pairs(const SysArgs& a, bool live, int i, int sub, int& p0, int& T, int lo = 0,
                                          int hi = 0) {
  p0 = live ? a.off[i] + sub : 0;
  int p1 = live ? a.off[i + 1] : 0;
  if constexpr (CLIP) clip_pairs(K, lo, hi, p0, p1);
  const int len = p1 > p0 ? (p1 - p0 + K - 1) / K : 0;
  T = len;
#pragma unroll
  for (int s = 32; s > 0; s >>= 1) T = max(T, __shfl_xor(T, s, 64));
  T = __builtin_amdgcn_readfirstlane(T);
  return len;
}

// ---------------------------------------------------------------------------- moments
template <bool BATCH>
__device__ __forceinline__ int sweep_atom(const SysArgs& a, int k) {
  if constexpr (BATCH) return atom_at(a, k);
  else return k;
}
// cell of atom i: the kernel-argument copy (uniform, scalar registers) for one system
template <bool BATCH>
__device__ __forceinline__ void cell_of(const SysArgs& a, int i, double* H) {
  if constexpr (BATCH) {
    load_cell(a, i, H);
  } else {
#pragma unroll
    for (int k = 0; k < 9; ++k) H[k] = a.H[k];
  }
}

// One part of the moments (binary64) or one group of the layout (binary32) of one atom: K lanes
// per atom each accumulate every K-th pair of the row, the partial moments are summed over the atom's
// lanes and its first lane writes them.
template <class L, int P, class R, bool BATCH, int NC, int K>
__device__ __forceinline__ void moments_of_atom(const SysArgs& a, const R* csh, int* lst, int i, int li, int sub,
                                                R* __restrict__ mout, long ld) {
  constexpr bool PARTS = std::is_same_v<R, double>;
  constexpr int LO = PARTS ? 0 : L::GROUP_LO[PARTS ? 0 : P];
  constexpr int NE = PARTS ? L::PART_SIZE[PARTS ? P : 0] : L::GROUP_HI[PARTS ? 0 : P] - LO;
  double H[9];
  cell_of<BATCH>(a, i, H);
  R m[NE];
#pragma unroll
  for (int e = 0; e < NE; ++e) m[e] = R(0);
  Partner<false> own;
  own.load(a, nullptr, i);
  const R* cz = csh + clamp_species(own.s, a.nsp) * a.nsp * radial_row<L::NMU, NC>(a.ncheb);
  for_pairs<K, R, false>(a, lst, i, sub, H, own, nullptr, [&](int, const Pair& t) {
    R f[L::NMU];
    radial_values<R, L::NMU, NC>((R)t.r, (R)a.sa, (R)a.sb, (R)a.rcut, cz + t.zj * radial_row<L::NMU, NC>(a.ncheb), a.ncheb, f);
    if constexpr (PARTS) L::template acc_part<P>(m, f, (R)t.dx, (R)t.dy, (R)t.dz);
    else L::template acc_moments<P>(m, f, (R)t.dx, (R)t.dy, (R)t.dz);
  });
  if constexpr (K > 1) {
#pragma unroll
    for (int e = 0; e < NE; ++e) {
      m[e] = group_sum<K>(m[e]);
      asm volatile("" : "+v"(m[e]));  // finished here: the last addition is not moved to the store (spills)
    }
  }
  if (sub == 0) {
#pragma unroll
    for (int e = 0; e < NE; ++e) mout[(long)(PARTS ? L::PART_ENTRY[PARTS ? P : 0][PARTS ? e : 0] : LO + e) * ld + li] = m[e];
  }
}

// Moments of 64 / K atoms per workgroup (one wave).  In binary64 the entries are cut into NPART
// parts of at most 84 that different waves accumulate over the same pairs: one wave with all 130
// entries of level 16 filled the registers of a SIMD by itself, moved a third of its accumulators
// through accumulation registers for every pair and stood waiting on its loads a quarter of the
// time.  The parts repeat a pair's geometry and radial functions, but two waves share a SIMD:
// 0.73 -> 0.57 ms at 1,024,000 atoms of level 16 (the vector unit is busy about 0.6 of it),
// 1.93 -> 1.17 ms at level 20 (545,505 atoms; it took three passes before).
// Binary32: group G of the layout.
// ALONE: one wave per SIMD (launch_moments_g).
template <class L, int G, class R, bool BATCH, int NC, bool PERSIST = false, int K = 1, bool ALONE = false>
__global__ __launch_bounds__(kLaneBlock)
__attribute__((amdgpu_waves_per_eu(std::is_same_v<R, double> && !ALONE ? 2 : 1, ALONE ? 1 : kMaxWaves)))
void k_moments(SysArgs a, int i0, int n, R* __restrict__ mout, long ld) {
  constexpr int NP = std::is_same_v<R, double> ? L::NPART : 1;
  __shared__ int lst[K == 1 ? kStageInts : 1];
  const R* csh = stage_radial<R, L::NMU>(a);
  MTP_FOR_TILES_K(a, n, K, NP, b) {
  // parts of a tile in consecutive workgroups: they read the same rows
  const int li = (b / NP) * (kLaneBlock / K) + (int)threadIdx.x / K, sub = (int)threadIdx.x % K;
  if (li >= n) continue;
  const int i = sweep_atom<BATCH>(a, i0 + li);
  if constexpr (NP == 1) {
    moments_of_atom<L, G, R, BATCH, NC, K>(a, csh, lst, i, li, sub, mout, ld);
  } else {
    static_assert(NP <= 4, "moment parts");
    const int part = b % NP;
    if (part == 0) moments_of_atom<L, 0, R, BATCH, NC, K>(a, csh, lst, i, li, sub, mout, ld);
    else if (part == 1) moments_of_atom<L, 1, R, BATCH, NC, K>(a, csh, lst, i, li, sub, mout, ld);
    else if (NP > 2 && part == 2) moments_of_atom<L, (NP > 2 ? 2 : 0), R, BATCH, NC, K>(a, csh, lst, i, li, sub, mout, ld);
    else if (NP > 3) moments_of_atom<L, (NP > 3 ? 3 : 0), R, BATCH, NC, K>(a, csh, lst, i, li, sub, mout, ld);
  }
  }
}

// ---------------------------------------------------------------------------- program forward
template <class L, class R>
__global__ __launch_bounds__(kLaneBlock) void k_program_fwd(const R* __restrict__ mom, long ld,
                                                            int i0, int n, const int* __restrict__ perm,
                                                            const int* __restrict__ species,
                                                            const double* __restrict__ xi,
                                                            const double* __restrict__ shift, int nsp,
                                                            double* __restrict__ e_atom,
                                                            R* __restrict__ cbar,
                                                            double* __restrict__ bout) {
  const int b = xcd_logical_block(blockIdx.x, gridDim.x);
  const int li = b * kLaneBlock + threadIdx.x;
  if (li >= n) return;
  LaneMoments<R> M{mom + li, ld};
  R C[L::NCOMP];
  L::template fwd<R>(M, C);
  R Cb[L::NCOMP];
  const double e = bout ? L::template products<true, R>(C, xi, Cb, bout + li, ld)
                        : L::template products<false, R>(C, xi, Cb, nullptr, ld);
  const int i = perm ? perm[i0 + li] : i0 + li;
  e_atom[i] = e + shift[clamp_species(species[i], nsp)];
#pragma unroll
  for (int q = 0; q < L::NCOMP; ++q) cbar[(long)q * ld + li] = Cb[q];
}

// ---------------------------------------------------------------------------- program reverse
template <class L, int G, class R>
__global__ __launch_bounds__(kLaneBlock) void k_program_rev(const R* __restrict__ mom, long ld,
                                                            int n, const R* __restrict__ cbar,
                                                            R* __restrict__ mbar) {
  const int b = xcd_logical_block(blockIdx.x, gridDim.x);
  const int li = b * kLaneBlock + threadIdx.x;
  if (li >= n) return;
  constexpr int LO = L::GROUP_LO[G], HI = L::GROUP_HI[G], NG = HI - LO;
  GlobalMoments<R> M{mom, ld, lane_bytes(li, sizeof(R))};
  R mb[NG];
#pragma unroll
  for (int e = 0; e < NG; ++e) mb[e] = R(0);
  if constexpr (L::NCOMP > kRegComps) {
    L::template rev<G>(M, GlobalVector<R>{cbar, ld, lane_bytes(li, sizeof(R))}, mb);
  } else {
    R Cb[L::NCOMP];
#pragma unroll
    for (int q = 0; q < L::NCOMP; ++q) Cb[q] = cbar[(long)q * ld + li];
    L::template rev<G>(M, Cb, mb);
  }
#pragma unroll
  for (int e = 0; e < NG; ++e) mbar[(long)(LO + e) * ld + li] = mb[e];
}

// ---------------------------------------------------------------------------- fused program
// Forward program, energy and basis products, then the reverse program, in one pass over an
// atom's moments (single-group levels): the contraction adjoints stay in registers instead of
// taking a round trip through memory, and the moments are read by one kernel instead of two.
template <class L, class R>
__global__ __launch_bounds__(kLaneBlock) void k_program(const R* __restrict__ mom, long ld, int i0, int n,
                                                        const int* __restrict__ species,
                                                        const double* __restrict__ xi,
                                                        const double* __restrict__ shift, int nsp,
                                                        double* __restrict__ e_atom, R* __restrict__ mbar) {
  static_assert(L::NGROUP == 1, "the fused program needs all moment entries in one group");
  // contraction adjoints parked in LDS between the two programs (registers are the limit)
  __shared__ R cbs[L::NCOMP * kLaneBlock];
  const int b = xcd_logical_block(blockIdx.x, gridDim.x);
  const int li = b * kLaneBlock + threadIdx.x;
  if (li >= n) return;
  LaneMoments<R> M{mom + li, ld};
  {
    R C[L::NCOMP], Cb[L::NCOMP];
    L::template fwd<R>(M, C);
    const double e = L::template products<false, R>(C, xi, Cb, nullptr, ld);
    const int i = i0 + li;
    e_atom[i] = e + shift[clamp_species(species[i], nsp)];
#pragma unroll
    for (int q = 0; q < L::NCOMP; ++q) cbs[q * kLaneBlock + threadIdx.x] = Cb[q];
  }
  // the reverse program re-reads the moments it needs: no loaded value stays live across
  asm volatile("" ::: "memory");
  R mb[L::NMOM];
#pragma unroll
  for (int e = 0; e < L::NMOM; ++e) mb[e] = R(0);
  L::template rev<0>(M, LaneVector<R>{cbs + threadIdx.x}, mb);
#pragma unroll
  for (int e = 0; e < L::NMOM; ++e) mbar[(long)e * ld + li] = mb[e];
}

// ---------------------------------------------------------------------------- wave programs
// Levels from 12 on in binary64: a workgroup runs the contraction program of one tile of 64 atoms on
// several waves, each a part of the contraction blocks.  The moments (at level 20 those that two blocks
// or more read) are staged in LDS once ([row][atom]).  With one lane running the whole program the re-reads of shared
// moments missed L2 (twice the moments fetched at level 16, 5 times at level 20) and the single wave
// of a SIMD stood waiting for them four fifths of its time at level 20, where the contraction values
// and adjoints of 160 components also went to scratch (up to 8.9 KB per lane).  Now the
// vector unit is busy 0.27 of the time at level 16, where 2.1 GB at a million atoms and waits for LDS take
// the rest.  Measured before -> after, us:
//   level 16: 1008 atoms 20 -> 12.9 (both programs); 1,024,000 atoms 742 -> 588 (2.1 GB moved: 3.6 TB/s)
//   level 20: 31,416 atoms 385 -> 130 (forward 42, reverse 88)
//   level 20, 540,480 atoms in a batch: forward 2200 -> 650, reverse 2460 -> 1500, tangent of the forward
//   6200 -> 1510, of the reverse 8100 -> 4870
// Two waves (level 12) and four (14, 16) keep two workgroups or more on a compute unit; at level 20 the
// rows fill its LDS, so eight waves run the forward programs, and four of 512 registers the reverse ones,
// whose accumulators eight of 256 would spill.

// Moment of the lane's atom: LDS row or, for a moment that one block reads, memory.
template <class L, bool TANGENT>
struct TileMoments {
  const double* lds;  // row 0 of the lane
  const double* __restrict__ base;
  long ld;
  unsigned off;
  __device__ __forceinline__ double operator()(int e) const {
    const int row = TANGENT ? L::THOT_ROW[e] : L::HOT_ROW[e];
    if (row >= 0) return lds[row * kLaneBlock];
    return *reinterpret_cast<const double*>(reinterpret_cast<const char*>(base + (long)e * ld) + off);
  }
};
// Row e of a [row][atom] array: stores, loads.
struct RowStore {
  double* __restrict__ base;
  long ld;
  unsigned off;
  __device__ __forceinline__ void operator()(int e, double v) const {
    *reinterpret_cast<double*>(reinterpret_cast<char*>(base + (long)e * ld) + off) = v;
  }
};
struct RowLoad {
  const double* __restrict__ base;
  long ld;
  unsigned off;
  __device__ __forceinline__ double operator()(int e) const {
    return *reinterpret_cast<const double*>(reinterpret_cast<const char*>(base + (long)e * ld) + off);
  }
};
struct LdsRows {
  double* p;
  __device__ __forceinline__ double operator()(int g) const { return p[g * kLaneBlock]; }
  __device__ __forceinline__ void operator()(int g, double v) const { p[g * kLaneBlock] = v; }
};
// both an LDS row (for the reverse program of the same launch) and a row in memory (for the adjoint)
struct LdsAndRow {
  LdsRows lds;
  RowStore row;
  bool keep;
  __device__ __forceinline__ void operator()(int g, double v) const {
    lds(g, v);
    if (keep) row(g, v);
  }
};

// Tile of the workgroup; lane: bytes of the lane's atom in a row, of LDS as of an array from the tile's
// first atom on (one register for both).  Lanes past the last atom repeat it: they read, compute and
// store what its own lane does.
struct Tile {
  int wave, first;
  unsigned lane;
};
__device__ __forceinline__ Tile tile_of(int n) {
  Tile t;
  t.wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kLaneBlock);
  t.first = xcd_logical_block(blockIdx.x, gridDim.x) * kLaneBlock;
  t.lane = lane_bytes(min((int)threadIdx.x & (kLaneBlock - 1), n - 1 - t.first), sizeof(double));
  return t;
}
__device__ __forceinline__ double* lane_ptr(double* p, unsigned lane) {
  return reinterpret_cast<double*>(reinterpret_cast<char*>(p) + lane);
}

// f(constant<W>, LDS pointer of the lane, lane) for the wave's number.  The lane's offset is made anew
// for each part: known from before it, its 64-bit form was what the register allocator kept, spilled and read
// back for every row (reverse tangent of level 20, 540480 atoms: 8.9 -> 4.9 ms, with its loads one
// block ahead instead of at the start).
template <int N, int W = 0, class F>
__device__ __forceinline__ void for_wave(const Tile& t, double* sm, F&& f) {
  if constexpr (W < N) {
    if (t.wave == W) {
      unsigned lane = t.lane;
      MTP_PIN(lane);
      f(std::integral_constant<int, W>{}, lane_ptr(sm, lane), lane);
    } else {
      for_wave<N, W + 1>(t, sm, f);
    }
  }
}

// Rows entry[0..COUNT) of src for the lane's atom to LDS rows 0, 1, ..., the waves in turn.  Where that is
// every row (ALL: levels up to 16) the addresses follow from one another and all loads of a wave are in
// flight at once: 1,024,000 atoms at level 16 693 -> 588 us, with the moments of one contraction staged
// too.  Rows from the table go eight at a time.
template <int COUNT, int NW, bool ALL>
__device__ __forceinline__ void stage_moments(const int (&entry)[COUNT], const Tile& t, const double* __restrict__ src,
                                              long ld, double* lds) {
  const RowLoad rows{src + t.first, ld, t.lane};
  if constexpr (ALL) {
    constexpr int N = COUNT / NW, REST = COUNT % NW;
    double v[N];
#pragma unroll
    for (int k = 0; k < N; ++k) v[k] = rows(t.wave + k * NW);
    if (t.wave < REST) lds[(N * NW + t.wave) * kLaneBlock] = rows(N * NW + t.wave);
#pragma unroll
    for (int k = 0; k < N; ++k) lds[(t.wave + k * NW) * kLaneBlock] = v[k];
  } else {
#pragma unroll 8
    for (int r = t.wave; r < COUNT; r += NW) lds[r * kLaneBlock] = rows(entry[r]);
  }
}

// between two phases of a tile (the waves of a workgroup exchange data through LDS only)
__device__ __forceinline__ void step_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt 0; vector memory operations stay in flight
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// Reverse phase: the blocks of the wave, then the entries that several waves touch added in wave order
// through the LDS rows the moments no longer need.
template <class L, int W, class MA, class CB>
__device__ __forceinline__ void reverse_wave(const MA& M, const CB& cb, const double* __restrict__ xi, double* lds,
                                             const RowStore& out) {
  double mbs[L::SHARED[W] > 0 ? L::SHARED[W] : 1];
  L::template rev_wave<W>(M, cb, xi, mbs, out);
  step_barrier();
#pragma unroll
  for (int k = 0; k < W; ++k) step_barrier();
  L::template rev_combine<W>(mbs, lds, out);
#pragma unroll
  for (int k = W + 1; k < L::NRWAVE; ++k) step_barrier();
}

// Four waves hold the accumulators of level 20 in 512 registers each; otherwise two waves per SIMD.
template <class L>
constexpr int wave_occupancy(int waves) { return waves == 4 && L::NMOM > 200 ? 1 : 2; }

template <class L, bool WB>
__global__ __launch_bounds__(kLaneBlock * L::NFWAVE) __attribute__((amdgpu_waves_per_eu(2)))
void k_wave_forward(const double* __restrict__ mom, long ld, int i0, int n, const int* __restrict__ perm,
                    const int* __restrict__ species, const double* __restrict__ xi, const double* __restrict__ shift,
                    int nsp, double* __restrict__ e_atom, double* __restrict__ cbar, double* __restrict__ bout) {
  constexpr int NW = L::NFWAVE, CROW = L::NHOT, PROW = CROW + L::NGEN;
  __shared__ double sm[(PROW + 2 * NW) * kLaneBlock];
  const Tile t = tile_of(n);
  double* lds = lane_ptr(sm, t.lane);
  stage_moments<L::NHOT, NW, L::NHOT == L::NMOM>(L::HOT_ENTRY, t, mom, ld, lds);
  double e = 0.0, c0b = 0.0;
  step_barrier();
  for_wave<NW>(t, sm, [&](auto w, double* p, unsigned lane) {
    L::template fwd_wave<decltype(w)::value, WB>(TileMoments<L, false>{p, mom + t.first, ld, lane}, xi,
                                                 p + CROW * kLaneBlock, WB ? lane_ptr(bout + t.first, lane) : nullptr,
                                                 ld, e, c0b);
  });
  step_barrier();
  for_wave<NW>(t, sm, [&](auto w, double* p, unsigned lane) {
    L::template core_wave<decltype(w)::value, WB>(TileMoments<L, false>{p, mom + t.first, ld, lane}, xi,
                                                  p + CROW * kLaneBlock, RowStore{cbar + t.first, ld, lane},
                                                  WB ? lane_ptr(bout + t.first, lane) : nullptr, ld, e, c0b);
  });
  lds[(PROW + t.wave) * kLaneBlock] = e;
  lds[(PROW + NW + t.wave) * kLaneBlock] = c0b;
  step_barrier();
  if (t.wave == 0) {
#pragma unroll
    for (int k = 1; k < NW; ++k) {
      e += lds[(PROW + k) * kLaneBlock];
      c0b += lds[(PROW + NW + k) * kLaneBlock];
    }
    const int li = t.first + (int)(t.lane / sizeof(double)), i = perm ? perm[i0 + li] : i0 + li;
    e_atom[i] = e + shift[clamp_species(species[i], nsp)];
    RowStore{cbar + t.first, ld, t.lane}(L::GEN0, c0b);
  }
}

template <class L>
__global__ __launch_bounds__(kLaneBlock * L::NRWAVE)
__attribute__((amdgpu_waves_per_eu(wave_occupancy<L>(L::NRWAVE))))
void k_wave_reverse(const double* __restrict__ mom, long ld, int n, const double* __restrict__ xi,
                    const double* __restrict__ cbar, double* __restrict__ mbar) {
  constexpr int ROWS = L::NHOT > L::SHARED_ROWS ? L::NHOT : L::SHARED_ROWS;
  __shared__ double sm[ROWS * kLaneBlock];
  const Tile t = tile_of(n);
  double* lds = lane_ptr(sm, t.lane);
  stage_moments<L::NHOT, L::NRWAVE, L::NHOT == L::NMOM>(L::HOT_ENTRY, t, mom, ld, lds);
  step_barrier();
  for_wave<L::NRWAVE>(t, sm, [&](auto w, double* p, unsigned lane) {
    reverse_wave<L, decltype(w)::value>(TileMoments<L, false>{p, mom + t.first, ld, lane},
                                        RowLoad{cbar + t.first, ld, lane}, xi, p, RowStore{mbar + t.first, ld, lane});
  });
}

// Forward and reverse of a tile in one launch (levels whose forward and reverse programs take the same
// number of waves): the moments stay in LDS between the two, and so do the general contractions'
// adjoints (also stored to cbar when given).
template <class L>
__global__ __launch_bounds__(kLaneBlock * L::NFWAVE) __attribute__((amdgpu_waves_per_eu(2)))
void k_wave_program(const double* __restrict__ mom, long ld, int i0, int n, const int* __restrict__ perm,
                    const int* __restrict__ species, const double* __restrict__ xi, const double* __restrict__ shift,
                    int nsp, double* __restrict__ e_atom, double* __restrict__ cbar, double* __restrict__ mbar) {
  constexpr int NW = L::NFWAVE, CROW = L::NHOT, BROW = CROW + L::NGEN, PROW = BROW + L::NGEN;
  static_assert(L::NFWAVE == L::NRWAVE && L::SHARED_ROWS <= PROW, "one launch for both programs");
  __shared__ double sm[(PROW + 2 * NW) * kLaneBlock];
  const Tile t = tile_of(n);
  double* lds = lane_ptr(sm, t.lane);
  stage_moments<L::NHOT, NW, L::NHOT == L::NMOM>(L::HOT_ENTRY, t, mom, ld, lds);
  const long first = cbar ? t.first : 0;  // no offset to a null pointer
  double e = 0.0, c0b = 0.0;
  step_barrier();
  for_wave<NW>(t, sm, [&](auto w, double* p, unsigned lane) {
    L::template fwd_wave<decltype(w)::value, false>(TileMoments<L, false>{p, mom + t.first, ld, lane}, xi,
                                                    p + CROW * kLaneBlock, nullptr, ld, e, c0b);
  });
  step_barrier();
  for_wave<NW>(t, sm, [&](auto w, double* p, unsigned lane) {
    const LdsAndRow cb{LdsRows{p + BROW * kLaneBlock}, RowStore{cbar + first, ld, lane}, cbar != nullptr};
    L::template core_wave<decltype(w)::value, false>(TileMoments<L, false>{p, mom + t.first, ld, lane}, xi,
                                                     p + CROW * kLaneBlock, cb, nullptr, ld, e, c0b);
  });
  lds[(PROW + t.wave) * kLaneBlock] = e;
  lds[(PROW + NW + t.wave) * kLaneBlock] = c0b;
  step_barrier();
  if (t.wave == 0) {
#pragma unroll
    for (int k = 1; k < NW; ++k) {
      e += lds[(PROW + k) * kLaneBlock];
      c0b += lds[(PROW + NW + k) * kLaneBlock];
    }
    const int li = t.first + (int)(t.lane / sizeof(double)), i = perm ? perm[i0 + li] : i0 + li;
    e_atom[i] = e + shift[clamp_species(species[i], nsp)];
    LdsAndRow{LdsRows{lds + BROW * kLaneBlock}, RowStore{cbar + first, ld, t.lane}, cbar != nullptr}(L::GEN0, c0b);
  }
  step_barrier();
  for_wave<NW>(t, sm, [&](auto w, double* p, unsigned lane) {
    reverse_wave<L, decltype(w)::value>(TileMoments<L, false>{p, mom + t.first, ld, lane}, LdsRows{p + BROW * kLaneBlock},
                                        xi, p, RowStore{mbar + t.first, ld, lane});
  });
}

// ---------------------------------------------------------------------------- backward pairs
// The end of a pair-gradient tile: per-atom virials (batches), the atoms' own gradient sums and the
// workgroup's virial partial.  With ADD (a later pass over the pairs) everything is added to.
template <bool BATCH, int K, bool ADD>
__device__ __forceinline__ void finish_gradients(bool live, int i, int sub, int tile, double* w, double* fo,
                                                 double* __restrict__ wpart, double* __restrict__ watom,
                                                 double* __restrict__ fown) {
  if (live) {
    if constexpr (BATCH) {
#pragma unroll
      for (int k = 0; k < 6; ++k) {
        const double v = group_sum<K>(w[k]);
        if (sub == 0) watom[6L * i + k] = ADD ? watom[6L * i + k] + v : v;
      }
    }
    if constexpr (K > 1) {
#pragma unroll
      for (int k = 0; k < 3; ++k) fo[k] = group_sum<K>(fo[k]);
    }
    if (fown && sub == 0) {
#pragma unroll
      for (int k = 0; k < 3; ++k) fown[3L * i + k] = ADD ? fown[3L * i + k] + fo[k] : fo[k];
    }
  }
  // one wave holds the tile's sums: register butterflies (fixed order)
#pragma unroll
  for (int k = 0; k < 6; ++k) w[k] = wave_sum(w[k]);
  if ((threadIdx.x & (kLaneBlock - 1)) == 0) {
#pragma unroll
    for (int k = 0; k < 6; ++k) wpart[6L * tile + k] = ADD ? wpart[6L * tile + k] + w[k] : w[k];
  }
}

// own sum and virial of one pair gradient
__device__ __forceinline__ void add_gradient(double dx, double dy, double dz, double gx, double gy, double gz,
                                             double* fo, double* w) {
  fo[0] += gx;
  fo[1] += gy;
  fo[2] += gz;
  w[0] -= dx * gx;
  w[1] -= dy * gy;
  w[2] -= dz * gz;
  w[3] -= dx * gy;
  w[4] -= dx * gz;
  w[5] -= dy * gz;
}

// Waves per SIMD of the binary64 kernel of one part: two up to 64 entries (46 at level 12 take 198 to 250
// registers).  The 81 of level 14, next to six own sums and a pair's values, spill 40 to 180 bytes per lane
// in the 256 registers of two waves and take 266 to 278 of one: 1.47 -> 0.72 ms at 998,560 atoms, 99 -> 55 us
// at 63,488.
constexpr int gradient_occupancy(int entries) { return entries > 64 ? 1 : 2; }

// g[p] (+)= dE_i/dd_ij restricted to the entries of group G (binary32; binary64 levels of one part
// take the whole adjoint by pair_part); per-workgroup virial partials;
// fown[i] (+)= sum of the atom's own g over its row (the first half of its force), when given.
// K lanes per atom: each takes every K-th pair of the row; the own sums are
// combined over the atom's lanes, the virial partial over the workgroup as before.
template <class L, int G, class R, bool BATCH, int NC, bool PERSIST = false, int K = 1, bool ALONE = false>
__global__ __launch_bounds__(kLaneBlock)
__attribute__((amdgpu_waves_per_eu(std::is_same_v<R, double> && !ALONE ? gradient_occupancy(L::NMOM) : 1,
                                   ALONE ? 1 : kMaxWaves)))
void k_backward(SysArgs a, int i0, int n, const R* __restrict__ mbar, long ld, double* __restrict__ g,
                double* __restrict__ wpart, double* __restrict__ watom, double* __restrict__ fown) {
  constexpr bool PARTS = std::is_same_v<R, double>;
  constexpr bool accumulate = G > 0;  // the first pass stores, later ones add
  constexpr int LO = PARTS ? 0 : L::GROUP_LO[PARTS ? 0 : G];
  constexpr int NG = PARTS ? L::NMOM : L::GROUP_HI[PARTS ? 0 : G] - LO;
  static_assert(!PARTS || L::NPART == 1, "levels of several parts take k_backward_stages");
  __shared__ int lst[K == 1 ? kStageInts : 1];
  const R* csh = stage_radial<R, L::NMU>(a);
  MTP_FOR_TILES_K(a, n, K, 1, b) {
  const int li = b * (kLaneBlock / K) + (int)threadIdx.x / K, sub = (int)threadIdx.x % K;
  double w[6] = {0, 0, 0, 0, 0, 0};
  double fo[3] = {0, 0, 0};  // sum of the atom's own pair gradients
  int i = 0;
  if (li < n) {
    i = sweep_atom<BATCH>(a, i0 + li);
    double H[9];
    cell_of<BATCH>(a, i, H);
    R mb[NG];
    // binary32: adjoints scaled by a! b! c! for the scaled monomials of pair_grad
#pragma unroll
    for (int e = 0; e < NG; ++e) {
      mb[e] = mbar[(long)(PARTS ? L::PART_ENTRY[0][PARTS ? e : 0] : LO + e) * ld + li];
      if constexpr (!PARTS) mb[e] *= R(L::MFACT[LO + e]);
    }
    Partner<false> own;
    own.load(a, nullptr, i);
    const R* cz = csh + clamp_species(own.s, a.nsp) * a.nsp * radial_row<L::NMU, NC>(a.ncheb);
    for_pairs<K, R, false>(a, lst, i, sub, H, own, nullptr, [&](int p, const Pair& t) {
      const double dx = t.dx, dy = t.dy, dz = t.dz;
      double old[3] = {0.0, 0.0, 0.0};  // loaded ahead of the arithmetic
      if constexpr (accumulate) {
#pragma unroll
        for (int k = 0; k < 3; ++k) old[k] = g[3L * p + k];
        __builtin_amdgcn_sched_barrier(0);
      }
      R f[L::NMU], fp[L::NMU];
      radial<R, L::NMU, NC>((R)t.r, (R)a.sa, (R)a.sb, (R)a.rcut, cz + t.zj * radial_row<L::NMU, NC>(a.ncheb), a.ncheb, f, fp);
      R rgx = R(0), rgy = R(0), rgz = R(0), ru = R(0);
      double ur;
      if constexpr (PARTS) {
        L::template pair_part<0>(mb, f, fp, dx, dy, dz, rgx, rgy, rgz, ru);
        ur = ru * t.rinv;
      } else {
        L::template pair_grad<G>(mb, f, fp, (R)dx, (R)dy, (R)dz, rgx, rgy, rgz, ru);
        ur = (double)ru / t.r;
      }
      const double gx = fma(ur, dx, (double)rgx);
      const double gy = fma(ur, dy, (double)rgy);
      const double gz = fma(ur, dz, (double)rgz);
      // stored after the next pair's loads were issued, so that no wait for a load covers it
      g[3L * p] = accumulate ? old[0] + gx : gx;
      g[3L * p + 1] = accumulate ? old[1] + gy : gy;
      g[3L * p + 2] = accumulate ? old[2] + gz : gz;
      add_gradient(dx, dy, dz, gx, gy, gz, fo, w);
    });
  }
  finish_gradients<BATCH, K, accumulate>(li < n, i, sub, b, w, fo, wpart, watom, fown);
  }
}

// Levels whose adjoints do not fit the 256 registers that two waves per SIMD leave a lane (above
// 84 entries): the entries stay cut into the parts of the moment kernel, and the NPART waves of a
// workgroup pass the pairs of the same 64 / K atoms along a pipeline.  The wave of the last
// (smallest) part forms a pair's geometry and all radial functions, evaluates its own part and
// leaves displacement, gradient so far and the radial factors of the other parts in an LDS slot;
// each further wave adds its part one step later, the wave of part 0 stores the gradient and
// takes the sums.  One barrier per step; a ring of NPART slots keeps the stages apart.  All lanes
// run the same number of steps (the longest row of the tile); what a lane does past its
// row is dropped.
// One wave holding all 130 adjoints of level 16 filled a SIMD, read 100 accumulation registers per
// pair and stood waiting a quarter of its time: 1.27 ms at 1,024,000 atoms with the monomial form and
// list reads pair by pair, 0.95 with Horner's scheme and staged rows, 0.85 as a pipeline; at level 20
// (545,505 atoms) 4.7 ms in three passes, 2.4 in two, 1.27 here.  The first stage bounds a step
// (250 vector instructions against 195 of the second at level 16).
template <class L>
struct StageSlots {
  static constexpr int WIDTH = 3 + L::NMU_SHARED;  // 16-byte fields: (dx, dy) (dz, gx) (gy, gz) (f, h) ...
  double2 v[L::NPART][WIDTH][kLaneBlock];
};

// First stage (part NPART - 1): T steps.
template <class L, bool BATCH, int NC, int K>
__device__ __forceinline__ void gradient_stage_first(const SysArgs& a, const double* csh, int* lst,
                                                     StageSlots<L>& slots, int i, int li, int sub, int lane, int p0,
                                                     int len, int T, const double* __restrict__ mbar, long ld) {
  constexpr int P = L::NPART - 1, NE = L::PART_SIZE[P];
  double H[9];
  cell_of<BATCH>(a, i, H);
  double mb[NE];
#pragma unroll
  for (int e = 0; e < NE; ++e) mb[e] = mbar[(long)L::PART_ENTRY[P][e] * ld + li];
  Partner<false> own;
  own.load(a, nullptr, i);
  const double* cz = csh + clamp_species(own.s, a.nsp) * a.nsp * radial_row<L::NMU, NC>(a.ncheb);
  int slot = 0;
  for_steps<K, false>(a, lst, i, lane, p0, len, T, H, own, nullptr, [&](int, const Pair& t) {
    double f[L::NMU], h[L::NMU];
    radial<double, L::NMU, NC>(t.r, a.sa, a.sb, a.rcut, cz + t.zj * radial_row<L::NMU, NC>(a.ncheb), a.ncheb, f, h);
#pragma unroll
    for (int mu = 0; mu < L::NMU; ++mu) h[mu] *= t.rinv;
    double gx = 0.0, gy = 0.0, gz = 0.0, u = 0.0;
    L::template pair_part<P>(mb, f, h, t.dx, t.dy, t.dz, gx, gy, gz, u);
    auto& v = slots.v[slot];
    v[0][lane] = double2{t.dx, t.dy};
    v[1][lane] = double2{t.dz, fma(u, t.dx, gx)};
    v[2][lane] = double2{fma(u, t.dy, gy), fma(u, t.dz, gz)};
#pragma unroll
    for (int mu = 0; mu < L::NMU_SHARED; ++mu) v[3 + mu][lane] = double2{f[mu], h[mu]};
    slot = slot + 1 < L::NPART ? slot + 1 : 0;
    step_barrier();
  });
#pragma unroll
  for (int k = 1; k < L::NPART; ++k) step_barrier();
}

// Stage S > 0 (part NPART - 1 - S).
template <class L, int S, bool BATCH, int K>
__device__ __forceinline__ void gradient_stage(StageSlots<L>& slots, bool live, int i, int li, int sub, int lane, int tile,
                                               int p0, int len, int T, const double* __restrict__ mbar, long ld,
                                               double* __restrict__ g, double* __restrict__ wpart,
                                               double* __restrict__ watom, double* __restrict__ fown) {
  constexpr int P = L::NPART - 1 - S, NE = L::PART_SIZE[P];
  double mb[NE];
#pragma unroll
  for (int e = 0; e < NE; ++e) mb[e] = mbar[(long)L::PART_ENTRY[P][e] * ld + li];
  double w[6] = {0, 0, 0, 0, 0, 0}, fo[3] = {0, 0, 0};
#pragma unroll
  for (int k = 0; k < S; ++k) step_barrier();
  int slot = 0;
  for (int t = 0; t < T; ++t) {
    auto& v = slots.v[slot];
    const double2 v0 = v[0][lane], v1 = v[1][lane], v2 = v[2][lane];
    double f[L::NMU_SHARED], h[L::NMU_SHARED];
#pragma unroll
    for (int mu = 0; mu < L::NMU_SHARED; ++mu) {
      const double2 fh = v[3 + mu][lane];
      f[mu] = fh.x;
      h[mu] = fh.y;
    }
    const double dx = v0.x, dy = v0.y, dz = v1.x;
    double gx = v1.y, gy = v2.x, gz = v2.y, u = 0.0;
    L::template pair_part<P>(mb, f, h, dx, dy, dz, gx, gy, gz, u);
    gx = fma(u, dx, gx);
    gy = fma(u, dy, gy);
    gz = fma(u, dz, gz);
    if constexpr (P > 0) {
      v[1][lane].y = gx;
      v[2][lane] = double2{gy, gz};
    } else if (t < len) {
      const long p = p0 + t * K;
      g[3 * p] = gx;
      g[3 * p + 1] = gy;
      g[3 * p + 2] = gz;
      add_gradient(dx, dy, dz, gx, gy, gz, fo, w);
    }
    slot = slot + 1 < L::NPART ? slot + 1 : 0;
    step_barrier();
  }
#pragma unroll
  for (int k = S + 1; k < L::NPART; ++k) step_barrier();
  if constexpr (P == 0) finish_gradients<BATCH, K, false>(live, i, sub, tile, w, fo, wpart, watom, fown);
}

template <class L, bool BATCH, int NC, bool PERSIST = false, int K = 1>
__global__ __launch_bounds__(kLaneBlock * L::NPART) __attribute__((amdgpu_waves_per_eu(2)))
void k_backward_stages(SysArgs a, int i0, int n, const double* __restrict__ mbar, long ld, double* __restrict__ g,
                       double* __restrict__ wpart, double* __restrict__ watom, double* __restrict__ fown) {
  static_assert(L::NPART <= 4, "pair-gradient stages");
  __shared__ int lst[K == 1 ? kStageInts : 1];
  __shared__ StageSlots<L> slots;
  const double* csh = stage_radial<double, L::NMU>(a);
  const int lane = (int)threadIdx.x & (kLaneBlock - 1);
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kLaneBlock);
  MTP_FOR_TILES_K(a, n, K, 1, b) {
    const int li = b * (kLaneBlock / K) + lane / K, sub = lane % K;
    const bool live = li < n;
    const int ls = live ? li : 0;  // lanes past the last atom read the first one's data
    const int i = sweep_atom<BATCH>(a, i0 + ls);
    int p0, T;
    const int len = lane_pairs<K>(a, live, i, sub, p0, T);
    // the stages alternate over the workgroup's waves from tile to tile (they differ in work, and
    // a wave's SIMD follows from its number)
    const int stage = (wave + b) % L::NPART;
    if (stage == 0)
      gradient_stage_first<L, BATCH, NC, K>(a, csh, lst, slots, i, ls, sub, lane, p0, len, T, mbar, ld);
    else if (stage == 1)
      gradient_stage<L, 1, BATCH, K>(slots, live, i, ls, sub, lane, b, p0, len, T, mbar, ld, g, wpart, watom, fown);
    else if (L::NPART > 2 && stage == 2)
      gradient_stage<L, (L::NPART > 2 ? 2 : 1), BATCH, K>(slots, live, i, ls, sub, lane, b, p0, len, T, mbar, ld, g, wpart,
                                                          watom, fown);
    else if (L::NPART > 3)
      gradient_stage<L, (L::NPART > 3 ? 3 : 1), BATCH, K>(slots, live, i, ls, sub, lane, b, p0, len, T, mbar, ld, g, wpart,
                                                          watom, fown);
    if constexpr (PERSIST) __syncthreads();
  }
}

// ---------------------------------------------------------------------------- parameter adjoint
// Tangent of the moments along delta_ij = fbar_j - fbar_i (the direction in which the force-weighted
// loss term differentiates the energy), in parts of at most 66 entries as in the moment kernel: 1.8 ms
// for 545,505 atoms at level 20 (4.3 in four passes of one wave per SIMD), 25 us for 16,000 at level 16
// with four lanes per atom (139 in three passes of one lane per atom).
template <class L, int P, int NC, int K>
__device__ __forceinline__ void tangents_of_atom(const SysArgs& a, const double* csh, int* lst, int i, int li,
                                                 int sub, const double* __restrict__ fbar,
                                                 double* __restrict__ mdot, long ld) {
  constexpr int NE = L::TPART_SIZE[P];
  double H[9];
  load_cell(a, i, H);
  double md[NE];
#pragma unroll
  for (int e = 0; e < NE; ++e) md[e] = 0.0;
  Partner<true> own;
  own.load(a, fbar, i);
  const double* cz = csh + clamp_species(own.s, a.nsp) * a.nsp * radial_row<L::NMU, NC>(a.ncheb);
  for_pairs<K, double, true>(a, lst, i, sub, H, own, fbar, [&](int, const Pair& t) {
    double f[L::NMU], fd[L::NMU];
    radial<double, L::NMU, NC>(t.r, a.sa, a.sb, a.rcut, cz + t.zj * radial_row<L::NMU, NC>(a.ncheb), a.ncheb, f, fd);
    const double rdot = (t.dx * t.ex + t.dy * t.ey + t.dz * t.ez) * t.rinv;
#pragma unroll
    for (int mu = 0; mu < L::NMU; ++mu) fd[mu] *= rdot;
    L::template tan_part<P>(md, f, fd, t.dx, t.dy, t.dz, t.ex, t.ey, t.ez);
  });
  if constexpr (K > 1) {
#pragma unroll
    for (int e = 0; e < NE; ++e) {
      md[e] = group_sum<K>(md[e]);
      asm volatile("" : "+v"(md[e]));
    }
  }
  if (sub == 0) {
#pragma unroll
    for (int e = 0; e < NE; ++e) mdot[(long)L::TPART_ENTRY[P][e] * ld + li] = md[e];
  }
}

template <class L, int NC, bool PERSIST = false, int K = 1>
__global__ __launch_bounds__(kLaneBlock) __attribute__((amdgpu_waves_per_eu(2)))
void k_tan_moments(SysArgs a, const double* __restrict__ fbar, int i0, int n, double* __restrict__ mdot, long ld) {
  constexpr int NP = L::NTPART;
  static_assert(NP <= 5, "moment-tangent parts");
  __shared__ int lst[K == 1 ? kStageInts : 1];
  const double* csh = stage_radial<double, L::NMU>(a);
  MTP_FOR_TILES_K(a, n, K, NP, b) {
  const int li = (b / NP) * (kLaneBlock / K) + (int)threadIdx.x / K, sub = (int)threadIdx.x % K;
  if (li >= n) continue;
  const int i = atom_at(a, i0 + li);
  const int part = b % NP;
  if (part == 0) tangents_of_atom<L, 0, NC, K>(a, csh, lst, i, li, sub, fbar, mdot, ld);
  else if (NP > 1 && part == 1) tangents_of_atom<L, (NP > 1 ? 1 : 0), NC, K>(a, csh, lst, i, li, sub, fbar, mdot, ld);
  else if (NP > 2 && part == 2) tangents_of_atom<L, (NP > 2 ? 2 : 0), NC, K>(a, csh, lst, i, li, sub, fbar, mdot, ld);
  else if (NP > 3 && part == 3) tangents_of_atom<L, (NP > 3 ? 3 : 0), NC, K>(a, csh, lst, i, li, sub, fbar, mdot, ld);
  else if (NP > 4) tangents_of_atom<L, (NP > 4 ? 4 : 0), NC, K>(a, csh, lst, i, li, sub, fbar, mdot, ld);
  }
}

// Tangents of contractions and basis: out[alpha] = ebar B_alpha - dB_alpha, and dCbar.
template <class L>
__global__ __launch_bounds__(kLaneBlock) void k_tan_forward(const double* __restrict__ mom,
                                                            const double* __restrict__ mdot, long ld,
                                                            int i0, int n, const int* __restrict__ perm,
                                                            const int* __restrict__ cfg,
                                                            const double* __restrict__ ebar_cfg,
                                                            const double* __restrict__ xi,
                                                            double ebar, double* __restrict__ out,
                                                            double* __restrict__ cbard) {
  const int b = xcd_logical_block(blockIdx.x, gridDim.x);
  const int li = b * kLaneBlock + threadIdx.x;
  if (li >= n) return;
  if (ebar_cfg) {
    const int i = perm ? perm[i0 + li] : i0 + li;
    ebar = ebar_cfg[cfg ? cfg[i] : 0];
  }
  const unsigned lo = lane_bytes(li, sizeof(double));
  GlobalMoments<double> M{mom, ld, lo}, Md{mdot, ld, lo};
  double C[L::NCOMP], Cd[L::NCOMP];
  L::template fwd_tan<double>(M, Md, C, Cd);
  double Cb[L::NCOMP], Cbd[L::NCOMP];
  L::template products_tan<double>(C, Cd, xi, ebar, Cb, Cbd, out + li, ld);
#pragma unroll
  for (int q = 0; q < L::NCOMP; ++q) cbard[(long)q * ld + li] = Cbd[q];
}

// Tangent of the moment adjoint: mbd = d(mbar) along the moment tangent.  The reverse program
// is cut into parts of contraction blocks sized for the registers; part P stores or adds the
// entries it touches, so the parts run in order 0, 1, ... on one stream.
template <class L, int P>
__global__ __launch_bounds__(kLaneBlock) void k_tan_reverse(const double* __restrict__ mom,
                                                            const double* __restrict__ mdot, long ld,
                                                            int n, const double* __restrict__ cbar,
                                                            const double* __restrict__ cbard,
                                                            double* __restrict__ mbard) {
  const int b = xcd_logical_block(blockIdx.x, gridDim.x);
  const int li = b * kLaneBlock + threadIdx.x;
  if (li >= n) return;
  const unsigned lo = lane_bytes(li, sizeof(double));
  GlobalMoments<double> M{mom, ld, lo}, Md{mdot, ld, lo};
  if constexpr (L::NCOMP > kRegComps) {
    L::template rev_tan<P, double>(M, Md, GlobalVector<double>{cbar, ld, lo}, GlobalVector<double>{cbard, ld, lo},
                                   LaneRows<double>{mbard, lo}, ld);
  } else {
    double Cb[L::NCOMP], Cbd[L::NCOMP];
#pragma unroll
    for (int q = 0; q < L::NCOMP; ++q) {
      Cb[q] = cbar[(long)q * ld + li];
      Cbd[q] = cbard[(long)q * ld + li];
    }
    L::template rev_tan<P, double>(M, Md, Cb, Cbd, LaneRows<double>{mbard, lo}, ld);
  }
}

// The same by several waves per tile (see the wave programs above): moments and tangents of the entries
// most blocks read in LDS.  out[alpha] = ebar B_alpha - dB_alpha; cbard: rows of the general
// contractions.
template <class L>
__global__ __launch_bounds__(kLaneBlock * L::NTFWAVE) __attribute__((amdgpu_waves_per_eu(2)))
void k_wave_tan_forward(const double* __restrict__ mom, const double* __restrict__ mdot, long ld, int i0, int n,
                        const int* __restrict__ perm, const int* __restrict__ cfg,
                        const double* __restrict__ ebar_cfg, const double* __restrict__ xi, double ebar,
                        double* __restrict__ out, double* __restrict__ cbard) {
  constexpr int NW = L::NTFWAVE, DROW = L::NTHOT, CROW = 2 * L::NTHOT, PROW = CROW + 2 * L::NGEN;
  __shared__ double sm[(PROW + NW) * kLaneBlock];
  const Tile t = tile_of(n);
  double* lds = lane_ptr(sm, t.lane);
  stage_moments<L::NTHOT, NW, L::NTHOT == L::NMOM>(L::THOT_ENTRY, t, mom, ld, lds);
  stage_moments<L::NTHOT, NW, L::NTHOT == L::NMOM>(L::THOT_ENTRY, t, mdot, ld, lds + DROW * kLaneBlock);
  if (ebar_cfg) {
    const int li = t.first + (int)(t.lane / sizeof(double)), i = perm ? perm[i0 + li] : i0 + li;
    ebar = ebar_cfg[cfg ? cfg[i] : 0];
  }
  double c0bd = 0.0;
  step_barrier();
  for_wave<NW>(t, sm, [&](auto w, double* p, unsigned lane) {
    double* crow = p + CROW * kLaneBlock;
    L::template tfwd_wave<decltype(w)::value>(
        TileMoments<L, true>{p, mom + t.first, ld, lane},
        TileMoments<L, true>{p + DROW * kLaneBlock, mdot + t.first, ld, lane}, xi, ebar, crow,
        crow + L::NGEN * kLaneBlock, LaneRows<double>{out + t.first, lane}, ld, c0bd);
  });
  step_barrier();
  for_wave<NW>(t, sm, [&](auto w, double* p, unsigned lane) {
    double* crow = p + CROW * kLaneBlock;
    L::template tcore_wave<decltype(w)::value>(
        TileMoments<L, true>{p, mom + t.first, ld, lane},
        TileMoments<L, true>{p + DROW * kLaneBlock, mdot + t.first, ld, lane}, xi, ebar, crow,
        crow + L::NGEN * kLaneBlock, RowStore{cbard + t.first, ld, lane}, LaneRows<double>{out + t.first, lane}, ld,
        c0bd);
  });
  lds[(PROW + t.wave) * kLaneBlock] = c0bd;
  step_barrier();
  if (t.wave == 0) {
#pragma unroll
    for (int k = 1; k < NW; ++k) c0bd += lds[(PROW + k) * kLaneBlock];
    RowStore{cbard + t.first, ld, t.lane}(L::GEN0, c0bd);
  }
}

template <class L, int W, class MA>
__device__ __forceinline__ void tangent_reverse_wave(const MA& M, const MA& Md, const RowLoad& cb, const RowLoad& cbd,
                                                     const double* __restrict__ xi, double* lds, const RowStore& out) {
  double mbs[L::TSHARED[W] > 0 ? L::TSHARED[W] : 1];
  L::template trev_wave<W>(M, Md, cb, cbd, xi, mbs, out);
  step_barrier();
#pragma unroll
  for (int k = 0; k < W; ++k) step_barrier();
  L::template trev_combine<W>(mbs, lds, out);
#pragma unroll
  for (int k = W + 1; k < L::NTRWAVE; ++k) step_barrier();
}

template <class L>
__global__ __launch_bounds__(kLaneBlock * L::NTRWAVE)
__attribute__((amdgpu_waves_per_eu(wave_occupancy<L>(L::NTRWAVE))))
void k_wave_tan_reverse(const double* __restrict__ mom, const double* __restrict__ mdot, long ld, int n,
                        const double* __restrict__ xi, const double* __restrict__ cbar,
                        const double* __restrict__ cbard, double* __restrict__ mbard) {
  constexpr int NW = L::NTRWAVE, DROW = L::NTHOT;
  constexpr int ROWS = 2 * L::NTHOT > L::TSHARED_ROWS ? 2 * L::NTHOT : L::TSHARED_ROWS;
  __shared__ double sm[ROWS * kLaneBlock];
  const Tile t = tile_of(n);
  double* lds = lane_ptr(sm, t.lane);
  stage_moments<L::NTHOT, NW, L::NTHOT == L::NMOM>(L::THOT_ENTRY, t, mom, ld, lds);
  stage_moments<L::NTHOT, NW, L::NTHOT == L::NMOM>(L::THOT_ENTRY, t, mdot, ld, lds + DROW * kLaneBlock);
  step_barrier();
  for_wave<NW>(t, sm, [&](auto w, double* p, unsigned lane) {
    tangent_reverse_wave<L, decltype(w)::value>(TileMoments<L, true>{p, mom + t.first, ld, lane},
                                                TileMoments<L, true>{p + DROW * kLaneBlock, mdot + t.first, ld, lane},
                                                RowLoad{cbar + t.first, ld, lane}, RowLoad{cbard + t.first, ld, lane},
                                                xi, p, RowStore{mbard + t.first, ld, lane});
  });
}

// Radial-coefficient gradient: per pair (i, j) with species (s, t),
//   dc[s][t][mu][b] += Q_b X_mu + Q'_b Y_mu,  X_mu = ebar S_mu - A_mu,  Y_mu = -(rhat . delta) S_mu,
// with S_mu = sum_e mb_e mono_e and A_mu its tangent (adjoint tangents mbd, displacement tangent
// delta).  Two kernels: k_adj_stages evaluates X and Y of every pair and leaves a record
// [r, t, X_0, Y_0, X_1, Y_1, ...] per pair, k_adj_radial sums them against the radial basis.
// Adjoints and tangents of every entry (260 values at level 16, 590 at level 20) do not fit a lane,
// and one kernel over ranges of 64 entries walked the pairs three to six times, species by species,
// forming geometry, monomials, tangents and the radial sums each time: 10.2 ms for 545,505 atoms at
// level 20 and 213 us for 16,000 at level 16 (one lane per atom).  Together the two take 3.3 ms (2.3
// and 1.0) and 61 us (four lanes per atom).

// NASTAGE waves per tile pass the pairs along as in k_backward_stages (at most 90 coefficients each);
// the first forms the geometry, the last writes the records.
template <class L>
struct AdjSlots {
  double2 v[L::NASTAGE][4 + L::NMU][kLaneBlock];  // (dx, dy) (dz, ex) (ey, ez) (r, rdot) (X, S) ...
  int zj[L::NASTAGE][kLaneBlock];
};
template <int NMU>
constexpr int adj_record() { return 2 * NMU + 2; }

template <int NMU>
__device__ __forceinline__ void write_record(double* __restrict__ rec, long p, double r, double rdot, int zj,
                                             const double* S, const double* X) {
  double2* q = reinterpret_cast<double2*>(rec + p * adj_record<NMU>());
  q[0] = double2{r, (double)zj};
#pragma unroll
  for (int mu = 0; mu < NMU; ++mu) q[1 + mu] = double2{X[mu], -rdot * S[mu]};
}

template <class L, int B>
__device__ __forceinline__ void adj_coefficients(const double* __restrict__ mbar, const double* __restrict__ mbard,
                                                 long ld, int li, double ebar, double* c) {
#pragma unroll
  for (int k = 0; k < L::ADJ_SIZE[B]; ++k) {
    const long at = (long)L::ADJ_ENTRY[B][k] * ld + li;
    c[k] = L::ADJ_VALUE[B][k] ? fma(ebar, mbar[at], -mbard[at]) : mbar[at];
  }
}

template <class L, int K>
__device__ __forceinline__ void adj_stage_first(const SysArgs& a, int* lst, AdjSlots<L>& slots, int i, int li,
                                                int lane, int p0, int len, int T, const double* __restrict__ fbar,
                                                const double* __restrict__ mbar, const double* __restrict__ mbard,
                                                long ld, double ebar, double* __restrict__ rec, int first) {
  double H[9];
  load_cell(a, i, H);
  double c[L::ADJ_SIZE[0]];
  adj_coefficients<L, 0>(mbar, mbard, ld, li, ebar, c);
  Partner<true> own;
  own.load(a, fbar, i);
  int slot = 0;
  for_steps<K, true>(a, lst, i, lane, p0, len, T, H, own, fbar, [&](int t, const Pair& q) {
    const double rdot = (q.dx * q.ex + q.dy * q.ey + q.dz * q.ez) * q.rinv;
    double S[L::NMU], X[L::NMU];
#pragma unroll
    for (int mu = 0; mu < L::NMU; ++mu) S[mu] = X[mu] = 0.0;
    L::template adj_stage<0>(c, q.dx, q.dy, q.dz, q.ex, q.ey, q.ez, S, X);
    if constexpr (L::NASTAGE == 1) {
      if (t < len) write_record<L::NMU>(rec, first + (long)t * K, q.r, rdot, q.zj, S, X);
    } else {
      auto& v = slots.v[slot];
      v[0][lane] = double2{q.dx, q.dy};
      v[1][lane] = double2{q.dz, q.ex};
      v[2][lane] = double2{q.ey, q.ez};
      v[3][lane] = double2{q.r, rdot};
#pragma unroll
      for (int mu = 0; mu < L::NMU; ++mu) v[4 + mu][lane] = double2{X[mu], S[mu]};
      slots.zj[slot][lane] = q.zj;
      slot = slot + 1 < L::NASTAGE ? slot + 1 : 0;
      step_barrier();
    }
  });
#pragma unroll
  for (int k = 1; k < L::NASTAGE; ++k) step_barrier();
}

template <class L, int B, int K>
__device__ __forceinline__ void adj_stage(AdjSlots<L>& slots, int li, int lane, int first, int len, int T,
                                          const double* __restrict__ mbar, const double* __restrict__ mbard, long ld,
                                          double ebar, double* __restrict__ rec) {
  double c[L::ADJ_SIZE[B]];
  adj_coefficients<L, B>(mbar, mbard, ld, li, ebar, c);
#pragma unroll
  for (int k = 0; k < B; ++k) step_barrier();
  int slot = 0;
  for (int t = 0; t < T; ++t) {
    auto& v = slots.v[slot];
    const double2 v0 = v[0][lane], v1 = v[1][lane], v2 = v[2][lane];
    constexpr bool LAST = B == L::NASTAGE - 1;
    double S[L::NMU], X[L::NMU];
#pragma unroll
    for (int mu = 0; mu < L::NMU; ++mu) {
      if (LAST || (mu >= L::ADJ_MU_LO[B] && mu <= L::ADJ_MU_HI[B])) {
        const double2 xs = v[4 + mu][lane];
        X[mu] = xs.x;
        S[mu] = xs.y;
      } else {
        X[mu] = S[mu] = 0.0;
      }
    }
    L::template adj_stage<B>(c, v0.x, v0.y, v1.x, v1.y, v2.x, v2.y, S, X);
    if constexpr (LAST) {
      const double2 v3 = v[3][lane];
      const int zj = slots.zj[slot][lane];
      if (t < len) write_record<L::NMU>(rec, first + (long)t * K, v3.x, v3.y, zj, S, X);
    } else {
#pragma unroll
      for (int mu = L::ADJ_MU_LO[B]; mu <= L::ADJ_MU_HI[B]; ++mu) v[4 + mu][lane] = double2{X[mu], S[mu]};
    }
    slot = slot + 1 < L::NASTAGE ? slot + 1 : 0;
    step_barrier();
  }
#pragma unroll
  for (int k = B + 1; k < L::NASTAGE; ++k) step_barrier();
}

// WINDOW: of the pairs lo .. hi - 1 alone.
template <class L, bool PERSIST = false, int K = 1, bool WINDOW = false>
__global__ __launch_bounds__(kLaneBlock * L::NASTAGE) __attribute__((amdgpu_waves_per_eu(2)))
void k_adj_stages(SysArgs a, const double* __restrict__ fbar, int i0, int n, const double* __restrict__ mbar,
                  const double* __restrict__ mbard, long ld, double ebar0, double* __restrict__ rec, int lo, int hi) {
  static_assert(L::NASTAGE <= 8, "adjoint stages");
  __shared__ int lst[K == 1 ? kStageInts : 1];
  __shared__ AdjSlots<L> slots;
  const int lane = (int)threadIdx.x & (kLaneBlock - 1);
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kLaneBlock);
  MTP_FOR_TILES_K(a, n, K, 1, b) {
    const int li = b * (kLaneBlock / K) + lane / K, sub = lane % K;
    const bool live = li < n;
    const int ls = live ? li : 0;  // lanes past the last atom read the first one's data
    const int i = atom_at(a, i0 + ls);
    int p0, T;
    const int len = lane_pairs<K, WINDOW>(a, live, i, sub, p0, T, lo, hi);
    if (WINDOW && T == 0) continue;  // the same in every wave of the workgroup
    const int first = WINDOW ? p0 - lo : p0;  // record of the lane's first pair
    const double ebar = a.ebar ? a.ebar[a.cfg ? a.cfg[i] : 0] : ebar0;
    const int stage = (wave + b) % L::NASTAGE;
    if (stage == 0)
      adj_stage_first<L, K>(a, lst, slots, i, ls, lane, p0, len, T, fbar, mbar, mbard, ld, ebar, rec, first);
#define MTP_ADJ_STAGE(S)                                                                                     \
  else if (L::NASTAGE > S && stage == S)                                                                     \
      adj_stage<L, (L::NASTAGE > S ? S : 0), K>(slots, ls, lane, first, len, T, mbar, mbard, ld, ebar, rec);
    MTP_ADJ_STAGE(1) MTP_ADJ_STAGE(2) MTP_ADJ_STAGE(3) MTP_ADJ_STAGE(4) MTP_ADJ_STAGE(5) MTP_ADJ_STAGE(6)
    MTP_ADJ_STAGE(7)
#undef MTP_ADJ_STAGE
    if constexpr (PERSIST) __syncthreads();
  }
}

// Sums of the pair records against the radial basis.  A lane orders its pairs by neighbour species in
// LDS (kOrderStage at a time) and the wave takes one species after the other, accumulating
// NMU x n_cheb sums in registers; they are transposed through LDS and each lane adds one sum over
// the wave's atoms of each centre species (in lane order).  One partial per (tile, s, t) in cpart.
// The record reads (96 bytes per pair at level 20, the species a second time) and about 180 vector
// instructions per pair bound it.
// WINDOW: the pairs lo .. hi - 1 of atoms from i0 on, onto cpart if add; else atoms from 0 on with all their
// pairs (which that form sums in 24.3 us for 23.3 at 4,000 atoms of level 10).
constexpr int kOrderStage = 64;
template <int NMU, int NC, bool WINDOW>
__global__ __launch_bounds__(kLaneBlock)
void k_adj_radial(SysArgs a, int i0, int n, const double* __restrict__ rec, int lo, int hi, bool add,
                  double* __restrict__ cpart) {
  constexpr int NQ = NC > 0 ? NC : kMaxCheb, NV = NMU * NQ, RW = adj_record<NMU>();
  __shared__ unsigned char zp[kOrderStage][kLaneBlock], ord[kOrderStage][kLaneBlock];
  __shared__ unsigned char first[kMaxSpecies + 1][kLaneBlock], cnt[kMaxSpecies][kLaneBlock];
  constexpr int PASSES = (NV + 31) / 32, NR = (NV + PASSES - 1) / PASSES;  // sums transposed at a time
  __shared__ double red[NR * (kLaneBlock + 1)];  // padded rows: a lane reads along its own row
  const int nq = NC > 0 ? NC : a.ncheb, K = a.split;
  const int lane = threadIdx.x;
  const int b = xcd_logical_block(blockIdx.x, gridDim.x);
  const int li = b * (kLaneBlock / K) + lane / K;
  const bool live = li < n;
  const int i = atom_at(a, WINDOW ? i0 + (live ? li : 0) : live ? li : 0);
  const int zi = live ? clamp_species(a.species[i], a.nsp) : -1;
  int p0 = live ? a.off[i] + lane % K : 0, p1 = live ? a.off[i + 1] : 0;
  if constexpr (WINDOW) clip_pairs(K, lo, hi, p0, p1);
  const int len = p1 > p0 ? (p1 - p0 + K - 1) / K : 0;
  if constexpr (WINDOW) {
    if (add && !__any(len > 0)) return;
    p0 -= lo;  // from here on the first record
  }
  // order of pairs [base, base + m) of the lane by species
  auto arrange = [&](int base, int m) {
    for (int t = 0; t < a.nsp; ++t) cnt[t][lane] = 0;
#pragma unroll 8
    for (int k = 0; k < m; ++k) {
      const int t = (int)rec[(p0 + (long)(base + k) * K) * RW + 1];
      zp[k][lane] = (unsigned char)t;
      cnt[t][lane]++;
    }
    int at = 0;
    for (int t = 0; t < a.nsp; ++t) {
      first[t][lane] = (unsigned char)at;
      at += cnt[t][lane];
      cnt[t][lane] = first[t][lane];
    }
    first[a.nsp][lane] = (unsigned char)at;
    for (int k = 0; k < m; ++k) {
      const int t = zp[k][lane];
      ord[cnt[t][lane]++][lane] = (unsigned char)k;
    }
  };
  const bool once = !__any(len > kOrderStage);  // every row of the wave fits one arrangement
  if (once) arrange(0, len);
  for (int t = 0; t < a.nsp; ++t) {
    double acc[NV];
#pragma unroll
    for (int k = 0; k < NV; ++k) acc[k] = 0.0;
    for (int base = 0; base < len; base += kOrderStage) {
      if (!once) arrange(base, min(kOrderStage, len - base));
      const int k0 = first[t][lane], k1 = first[t + 1][lane];
      if (k0 >= k1) continue;
      auto row = [&](int k) {
        return reinterpret_cast<const double2*>(rec + (p0 + (long)(base + ord[k][lane]) * K) * RW);
      };
      const double2* q = row(k0);
      double2 v[NMU + 1];
#pragma unroll
      for (int m = 0; m <= NMU; ++m) v[m] = q[m];
      int k = k0;
      do {
        double X[NMU], Y[NMU];
        const double r = v[0].x;
#pragma unroll
        for (int m = 0; m < NMU; ++m) {
          X[m] = v[1 + m].x;
          Y[m] = v[1 + m].y;
        }
        const double u = fma(a.sa, r, a.sb), w = a.rcut - r, w2 = w * w;
        q = row(min(k + 1, k1 - 1));
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int m = 0; m <= NMU; ++m) v[m] = q[m];
        __builtin_amdgcn_sched_barrier(0);
        // Q_b = T_b(u) w^2, Q'_b = sa T'_b(u) w^2 - 2 T_b(u) w
        double t2 = 1.0, t1 = u, d2 = 0.0, d1 = 1.0;
#pragma unroll
        for (int bq = 0; bq < NQ; ++bq) {
          if (NC == 0 && bq >= nq) continue;
          double T, D;
          if (bq == 0) {
            T = 1.0;
            D = 0.0;
          } else if (bq == 1) {
            T = u;
            D = 1.0;
          } else {
            T = fma(2.0 * u, t1, -t2);
            D = fma(2.0 * u, d1, fma(2.0, t1, -d2));
            t2 = t1;
            t1 = T;
            d2 = d1;
            d1 = D;
          }
          const double qb = T * w2, qp = fma(a.sa * w2, D, -2.0 * w * T);
#pragma unroll
          for (int m = 0; m < NMU; ++m) acc[m * NQ + bq] = fma(qb, X[m], fma(qp, Y[m], acc[m * NQ + bq]));
        }
        ++k;
      } while (k < k1);
    }
#pragma unroll
    for (int v0 = 0; v0 < NV; v0 += NR) {
      __syncthreads();  // the sums transposed before are read
#pragma unroll
      for (int k = 0; k < NR; ++k)
        if (v0 + k < NV) red[k * (kLaneBlock + 1) + lane] = acc[v0 + k];
      __syncthreads();
      const int v = v0 + lane;
      const double* row = red + (lane < NR ? lane : 0) * (kLaneBlock + 1);
      for (int sp = 0; sp < a.nsp; ++sp) {
        double* dst = cpart + (long)b * a.nsp * a.nsp * NMU * nq + (long)(sp * a.nsp + t) * NMU * nq;
        const unsigned long long mask = __ballot(zi == sp);
        double sum = 0.0;
        if (mask == ~0ull) {
#pragma unroll 16
          for (int l = 0; l < kLaneBlock; ++l) sum += row[l];
        } else {
          for (unsigned long long mk = mask; mk; mk &= mk - 1) sum += row[__ffsll(mk) - 1];
        }
        if (lane < NR && v < NV && v % NQ < nq) {
          if (WINDOW && add) sum += dst[(v / NQ) * nq + v % NQ];
          dst[(v / NQ) * nq + v % NQ] = sum;
        }
      }
    }
  }
}

// ---------------------------------------------------------------------------- launchers
// The pair kernels come in Chebyshev-count specialisations for the common sizes 8 and 10 and a
// runtime-count form for the rest.
template <class L, int G, class R, bool BATCH, bool PERSIST, int K, bool ALONE>
void launch_moments_nc(const SysArgs& a, int nb, int i0, int n, void* m, long ld, hipStream_t s) {
  const unsigned sh = radial_bytes<R, L::NMU>(a);
  if (a.ncheb == 8)
    hipLaunchKernelGGL((k_moments<L, G, R, BATCH, 8, PERSIST, K, ALONE>), dim3(nb), dim3(kLaneBlock), sh, s, a, i0, n, (R*)m, ld);
  else if (a.ncheb == 10)
    hipLaunchKernelGGL((k_moments<L, G, R, BATCH, 10, PERSIST, K, ALONE>), dim3(nb), dim3(kLaneBlock), sh, s, a, i0, n, (R*)m, ld);
  else
    hipLaunchKernelGGL((k_moments<L, G, R, BATCH, 0, PERSIST, K, ALONE>), dim3(nb), dim3(kLaneBlock), sh, s, a, i0, n, (R*)m, ld);
}
// Single systems, levels of one part: while there is a SIMD for every wave of a launch, the form that
// takes a SIMD's registers whole, so that no two waves share one with others idle.  The hardware deals
// single waves so in some sequences of launches and not in others: moments of 35,280 atoms at level 12 44
// or 57 us (after a force reduction, after a grade) where two fit a SIMD, 42 always with this form.
// Levels of several parts have two waves per SIMD to deal out from half that size on.
template <class L, class R, bool BATCH>
constexpr bool may_run_alone() { return std::is_same_v<R, double> && !BATCH && L::NPART == 1; }

template <class L, int G, class R, bool BATCH, bool PERSIST, int K = 1>
void launch_moments_gp(const SysArgs& a, int i0, int n, void* m, long ld, hipStream_t s) {
  const int nb = pair_grid(a, split_tiles(n, K) * (std::is_same_v<R, double> ? L::NPART : 1), L::NPART, 1);
  if constexpr (may_run_alone<L, R, BATCH>()) {
    if (nb <= a.simds) return launch_moments_nc<L, G, R, BATCH, PERSIST, K, true>(a, nb, i0, n, m, ld, s);
  }
  launch_moments_nc<L, G, R, BATCH, PERSIST, K, false>(a, nb, i0, n, m, ld, s);
}
// split lanes in binary64 only; persistent variants exist for batches of one lane per atom (a
// system small enough for split lanes is one round of workgroups)
template <class L, int G, class R, bool BATCH>
void launch_moments_g(const SysArgs& a, int i0, int n, void* m, long ld, hipStream_t s) {
  if constexpr (std::is_same_v<R, double>) {
    if (a.split == 2) return launch_moments_gp<L, G, R, BATCH, false, 2>(a, i0, n, m, ld, s);
    if (a.split == 4) return launch_moments_gp<L, G, R, BATCH, false, 4>(a, i0, n, m, ld, s);
    if (a.split == 8) return launch_moments_gp<L, G, R, BATCH, false, 8>(a, i0, n, m, ld, s);
  }
  if constexpr (BATCH) {
    if (a.queue) return launch_moments_gp<L, G, R, BATCH, true>(a, i0, n, m, ld, s);
  }
  launch_moments_gp<L, G, R, BATCH, false>(a, i0, n, m, ld, s);
}
template <class L, int G, class R>
void launch_rev_g(const void* m, long ld, int n, const void* cb, void* mb, hipStream_t s) {
  const int nb = (n + kLaneBlock - 1) / kLaneBlock;
  hipLaunchKernelGGL((k_program_rev<L, G, R>), dim3(nb), dim3(kLaneBlock), 0, s, (const R*)m, ld, n,
                     (const R*)cb, (R*)mb);
}
template <class L, int G, class R, bool BATCH, bool PERSIST, int K, int NC>
void launch_backward_nc(const SysArgs& a, int i0, int n, const void* mb, long ld, double* g, double* wpart,
                        double* watom, double* fown, hipStream_t s) {
  const int nb = pair_grid(a, split_tiles(n, K), L::NPART, L::NPART);
  const unsigned sh = radial_bytes<R, L::NMU>(a);
  if constexpr (std::is_same_v<R, double> && L::NPART > 1) {
    hipLaunchKernelGGL((k_backward_stages<L, BATCH, NC, PERSIST, K>), dim3(nb), dim3(kLaneBlock * L::NPART), sh, s, a,
                       i0, n, (const double*)mb, ld, g, wpart, watom, fown);
  } else {
    // as for the moments (a kernel for one wave per SIMD runs so by itself)
    constexpr bool ALONE = may_run_alone<L, R, BATCH>() && gradient_occupancy(L::NMOM) > 1;
    if (ALONE && nb <= a.simds)
      hipLaunchKernelGGL((k_backward<L, G, R, BATCH, NC, PERSIST, K, ALONE>), dim3(nb), dim3(kLaneBlock), sh, s, a, i0, n,
                         (const R*)mb, ld, g, wpart, watom, fown);
    else
      hipLaunchKernelGGL((k_backward<L, G, R, BATCH, NC, PERSIST, K, false>), dim3(nb), dim3(kLaneBlock), sh, s, a, i0, n,
                         (const R*)mb, ld, g, wpart, watom, fown);
  }
}
template <class L, int G, class R, bool BATCH, bool PERSIST, int K = 1>
void launch_backward_gp(const SysArgs& a, int i0, int n, const void* mb, long ld, double* g, double* wpart,
                        double* watom, double* fown, hipStream_t s) {
  if (a.ncheb == 8) launch_backward_nc<L, G, R, BATCH, PERSIST, K, 8>(a, i0, n, mb, ld, g, wpart, watom, fown, s);
  else if (a.ncheb == 10) launch_backward_nc<L, G, R, BATCH, PERSIST, K, 10>(a, i0, n, mb, ld, g, wpart, watom, fown, s);
  else launch_backward_nc<L, G, R, BATCH, PERSIST, K, 0>(a, i0, n, mb, ld, g, wpart, watom, fown, s);
}
// the virial partials: one per tile, split_tiles(n, a.split) of them
template <class L, int G, class R, bool BATCH>
void launch_backward_g(const SysArgs& a, int i0, int n, const void* mb, long ld, double* g,
                       double* wpart, double* watom, double* fown, hipStream_t s) {
  if constexpr (std::is_same_v<R, double>) {
    if (a.split == 2) return launch_backward_gp<L, G, R, BATCH, false, 2>(a, i0, n, mb, ld, g, wpart, watom, fown, s);
    if (a.split == 4) return launch_backward_gp<L, G, R, BATCH, false, 4>(a, i0, n, mb, ld, g, wpart, watom, fown, s);
    if (a.split == 8) return launch_backward_gp<L, G, R, BATCH, false, 8>(a, i0, n, mb, ld, g, wpart, watom, fown, s);
  }
  if constexpr (BATCH) {
    if (a.queue) return launch_backward_gp<L, G, R, BATCH, true>(a, i0, n, mb, ld, g, wpart, watom, fown, s);
  }
  launch_backward_gp<L, G, R, BATCH, false>(a, i0, n, mb, ld, g, wpart, watom, fown, s);
}

template <class L, class R, bool BATCH, size_t... Gs>
void dispatch_moments(int g, const SysArgs& a, int i0, int n, void* m, long ld, hipStream_t s,
                      std::index_sequence<Gs...>) {
  ((g == (int)Gs ? launch_moments_g<L, (int)Gs, R, BATCH>(a, i0, n, m, ld, s) : void()), ...);
}
template <class L, class R, size_t... Gs>
void dispatch_rev(int g, const void* m, long ld, int n, const void* cb, void* mb, hipStream_t s,
                  std::index_sequence<Gs...>) {
  ((g == (int)Gs ? launch_rev_g<L, (int)Gs, R>(m, ld, n, cb, mb, s) : void()), ...);
}
template <class L, class R, bool BATCH, size_t... Gs>
void dispatch_backward(int g, const SysArgs& a, int i0, int n, const void* mb, long ld,
                       double* gout, double* wpart, double* watom, double* fown, hipStream_t s,
                       std::index_sequence<Gs...>) {
  ((g == (int)Gs ? launch_backward_g<L, (int)Gs, R, BATCH>(a, i0, n, mb, ld, gout, wpart, watom, fown, s)
                 : void()),
   ...);
}

template <class L, class R, bool BATCH>
struct EnergyChain {
  static void moments(int g, const SysArgs& a, int i0, int n, void* m, long ld, hipStream_t s) {
    dispatch_moments<L, R, BATCH>(g, a, i0, n, m, ld, s, std::make_index_sequence<nmgroup()>{});
  }
  static constexpr bool waves() { return std::is_same_v<R, double> && L::WAVES; }
  static constexpr bool one_launch() { return waves() ? L::NFWAVE == L::NRWAVE : L::NGROUP == 1 && !BATCH; }
  static void prog_fwd(const void* m, long ld, int i0, int n, const int* perm, const int* species,
                       const double* xi, const double* shift, int nsp, double* e_atom, void* cbar,
                       double* bout, hipStream_t s) {
    const int nb = (n + kLaneBlock - 1) / kLaneBlock;
    if constexpr (waves()) {
      const dim3 nt(kLaneBlock * L::NFWAVE);
      if (bout)
        hipLaunchKernelGGL((k_wave_forward<L, true>), dim3(nb), nt, 0, s, (const double*)m, ld, i0, n, perm, species, xi,
                           shift, nsp, e_atom, (double*)cbar, bout);
      else
        hipLaunchKernelGGL((k_wave_forward<L, false>), dim3(nb), nt, 0, s, (const double*)m, ld, i0, n, perm, species, xi,
                           shift, nsp, e_atom, (double*)cbar, bout);
    } else {
      hipLaunchKernelGGL((k_program_fwd<L, R>), dim3(nb), dim3(kLaneBlock), 0, s, (const R*)m, ld, i0, n,
                         perm, species, xi, shift, nsp, e_atom, (R*)cbar, bout);
    }
  }
  static void prog_rev(int g, const void* m, long ld, int n, const double* xi, const void* cb, void* mb, hipStream_t s) {
    if constexpr (waves())
      hipLaunchKernelGGL((k_wave_reverse<L>), dim3((n + kLaneBlock - 1) / kLaneBlock), dim3(kLaneBlock * L::NRWAVE), 0, s,
                         (const double*)m, ld, n, xi, (const double*)cb, (double*)mb);
    else
      dispatch_rev<L, R>(g, m, ld, n, cb, mb, s, std::make_index_sequence<L::NGROUP>{});
  }
  static void backward(int grp, const SysArgs& a, int i0, int n, const void* mb, long ld, double* gout,
                       double* wpart, double* watom, double* fown, hipStream_t s) {
    dispatch_backward<L, R, BATCH>(grp, a, i0, n, mb, ld, gout, wpart, watom, fown, s,
                                   std::make_index_sequence<nbgroup()>{});
  }
  // launches of the moment kernel (in binary64 one covers all its parts)
  static constexpr int nmgroup() { return std::is_same_v<R, double> ? 1 : L::NGROUP; }
  // passes of the pair-gradient kernel over the pairs
  static constexpr int nbgroup() { return std::is_same_v<R, double> ? 1 : L::NGROUP; }
  static void program(const void* m, long ld, int i0, int n, const int* perm, const int* species, const double* xi,
                      const double* shift, int nsp, double* e_atom, void* cbar, void* mb, hipStream_t s) {
    const int nb = (n + kLaneBlock - 1) / kLaneBlock;
    if constexpr (one_launch() && waves())
      hipLaunchKernelGGL((k_wave_program<L>), dim3(nb), dim3(kLaneBlock * L::NFWAVE), 0, s, (const double*)m, ld, i0, n,
                         perm, species, xi, shift, nsp, e_atom, (double*)cbar, (double*)mb);
    else if constexpr (one_launch())
      hipLaunchKernelGGL((k_program<L, R>), dim3(nb), dim3(kLaneBlock), 0, s, (const R*)m, ld, i0, n, species, xi,
                         shift, nsp, e_atom, (R*)mb);
  }
  static ChainOps ops() {
    return ChainOps{&moments, &prog_fwd, &prog_rev, &backward, one_launch() ? &program : nullptr, waves(), nmgroup(),
                    nbgroup(), waves() ? 1 : L::NGROUP, std::is_same_v<R, double> ? L::NPART : 1};
  }
};

template <class L>
struct AdjImpl {
  template <int NC, bool PERSIST, int K>
  static void tan_moments_k(const SysArgs& a, const double* fbar, int i0, int n, double* md, long ld, hipStream_t s) {
    const int nb = pair_grid(a, split_tiles(n, K) * L::NTPART, L::NTPART, 1);
    const unsigned sh = radial_bytes<double, L::NMU>(a);
    hipLaunchKernelGGL((k_tan_moments<L, NC, PERSIST, K>), dim3(nb), dim3(kLaneBlock), sh, s, a,
                       fbar, i0, n, md, ld);
  }
  template <int NC>
  static void tan_moments_nc(const SysArgs& a, const double* fbar, int i0, int n, double* md, long ld, hipStream_t s) {
    if (a.split == 2) tan_moments_k<NC, false, 2>(a, fbar, i0, n, md, ld, s);
    else if (a.split == 4) tan_moments_k<NC, false, 4>(a, fbar, i0, n, md, ld, s);
    else if (a.split == 8) tan_moments_k<NC, false, 8>(a, fbar, i0, n, md, ld, s);
    else if (a.queue) tan_moments_k<NC, true, 1>(a, fbar, i0, n, md, ld, s);
    else tan_moments_k<NC, false, 1>(a, fbar, i0, n, md, ld, s);
  }
  static void tan_moments(const SysArgs& a, const double* fbar, int i0, int n, double* md, long ld, hipStream_t s) {
    if (a.ncheb == 8) tan_moments_nc<8>(a, fbar, i0, n, md, ld, s);
    else if (a.ncheb == 10) tan_moments_nc<10>(a, fbar, i0, n, md, ld, s);
    else tan_moments_nc<0>(a, fbar, i0, n, md, ld, s);
  }
  static void tan_forward(const SysArgs& a, const double* m, const double* md, long ld, int i0, int n,
                          const double* xi, double ebar, double* out, double* cbard, hipStream_t s) {
    const int nb = (n + kLaneBlock - 1) / kLaneBlock;
    if constexpr (L::WAVES)
      hipLaunchKernelGGL((k_wave_tan_forward<L>), dim3(nb), dim3(kLaneBlock * L::NTFWAVE), 0, s, m, md, ld, i0, n, a.perm,
                         a.cfg, a.ebar, xi, ebar, out, cbard);
    else
      hipLaunchKernelGGL((k_tan_forward<L>), dim3(nb), dim3(kLaneBlock), 0, s, m, md, ld, i0, n, a.perm, a.cfg,
                         a.ebar, xi, ebar, out, cbard);
  }
  template <int P>
  static void tan_reverse_g(const double* m, const double* md, long ld, int n, const double* xi, const double* cb,
                            const double* cbd, double* mbd, hipStream_t s) {
    const int nb = (n + kLaneBlock - 1) / kLaneBlock;
    if constexpr (L::WAVES)
      hipLaunchKernelGGL((k_wave_tan_reverse<L>), dim3(nb), dim3(kLaneBlock * L::NTRWAVE), 0, s, m, md, ld, n, xi, cb, cbd,
                         mbd);
    else
      hipLaunchKernelGGL((k_tan_reverse<L, P>), dim3(nb), dim3(kLaneBlock), 0, s, m, md, ld, n, cb, cbd, mbd);
  }
  template <bool PERSIST, int K>
  static void adj_pairs_k(const SysArgs& a, const double* fbar, int i0, int n, const double* mb, const double* mbd,
                          long ld, double ebar, double* rec, int lo, int hi, hipStream_t s) {
    const int nb = pair_grid(a, split_tiles(n, K), L::NASTAGE, L::NASTAGE);
    if (PERSIST || (lo == 0 && hi == a.npairs))
      hipLaunchKernelGGL((k_adj_stages<L, PERSIST, K>), dim3(nb), dim3(kLaneBlock * L::NASTAGE), 0, s, a, fbar, i0, n, mb,
                         mbd, ld, ebar, rec, lo, hi);
    else
      hipLaunchKernelGGL((k_adj_stages<L, false, K, true>), dim3(nb), dim3(kLaneBlock * L::NASTAGE), 0, s, a, fbar, i0, n,
                         mb, mbd, ld, ebar, rec, lo, hi);
  }
  static void adj_pairs(const SysArgs& a, const double* fbar, int i0, int n, const double* mb, const double* mbd,
                        long ld, double ebar, double* rec, int lo, int hi, hipStream_t s) {
    if (a.split == 2) adj_pairs_k<false, 2>(a, fbar, i0, n, mb, mbd, ld, ebar, rec, lo, hi, s);
    else if (a.split == 4) adj_pairs_k<false, 4>(a, fbar, i0, n, mb, mbd, ld, ebar, rec, lo, hi, s);
    else if (a.split == 8) adj_pairs_k<false, 8>(a, fbar, i0, n, mb, mbd, ld, ebar, rec, lo, hi, s);
    else if (a.queue) adj_pairs_k<true, 1>(a, fbar, i0, n, mb, mbd, ld, ebar, rec, lo, hi, s);
    else adj_pairs_k<false, 1>(a, fbar, i0, n, mb, mbd, ld, ebar, rec, lo, hi, s);
  }
  template <bool WINDOW>
  static void adj_radial_w(const SysArgs& a, int i0, int n, const double* rec, int lo, int hi, bool add, double* cpart,
                           hipStream_t s) {
    const dim3 nb(split_tiles(n, a.split)), nt(kLaneBlock);
    if (a.ncheb == 8)
      hipLaunchKernelGGL((k_adj_radial<L::NMU, 8, WINDOW>), nb, nt, 0, s, a, i0, n, rec, lo, hi, add, cpart);
    else if (a.ncheb == 10)
      hipLaunchKernelGGL((k_adj_radial<L::NMU, 10, WINDOW>), nb, nt, 0, s, a, i0, n, rec, lo, hi, add, cpart);
    else
      hipLaunchKernelGGL((k_adj_radial<L::NMU, 0, WINDOW>), nb, nt, 0, s, a, i0, n, rec, lo, hi, add, cpart);
  }
  static void adj_radial(const SysArgs& a, int i0, int n, const double* rec, int lo, int hi, bool add, double* cpart,
                         hipStream_t s) {
    if (lo == 0 && hi == a.npairs) adj_radial_w<false>(a, i0, n, rec, lo, hi, add, cpart, s);
    else adj_radial_w<true>(a, i0, n, rec, lo, hi, add, cpart, s);
  }
  static AdjOps ops() {
    AdjOps o{};
    o.tan_moments = &tan_moments;
    o.adj_pairs = &adj_pairs;
    o.adj_radial = &adj_radial;
    o.record = adj_record<L::NMU>();
    o.nrtpart = L::WAVES ? 1 : L::NRTPART;
    static_assert(L::WAVES || L::NRTPART <= kMaxRevParts, "reverse-tangent parts");
    return o;
  }
};

}  // namespace mtp

// One level is compiled as several translation units (binary64 chain, binary32 chain,
// adjoint, assembly) so that large levels build in parallel.
#define MTP_DEFINE_CHAIN(LV, NUM, TYPE, BATCH, TAG) \
  namespace mtp {                                   \
  ChainOps chain_ops_##NUM##_##TAG() { return EnergyChain<LV, TYPE, BATCH>::ops(); } \
  }
#define MTP_DEFINE_ADJ(LV, NUM) \
  namespace mtp {               \
  AdjOps adj_ops_##NUM() { return AdjImpl<LV>::ops(); } \
  }
#define MTP_DEFINE_ADJ_FWD(LV, NUM) \
  namespace mtp {                   \
  void adj_fwd_##NUM(const SysArgs& a, const double* m, const double* md, long ld, int i0, int n, \
                     const double* xi, double ebar, double* out, double* cbard, hipStream_t s) { \
    AdjImpl<LV>::tan_forward(a, m, md, ld, i0, n, xi, ebar, out, cbard, s);                     \
  }                                                                                             \
  }
#define MTP_DEFINE_ADJ_REV(LV, NUM, G) \
  namespace mtp {                      \
  void adj_rev_##NUM##_##G(const double* m, const double* md, long ld, int n, const double* xi, \
                           const double* cb, const double* cbd, double* mbd, hipStream_t s) {   \
    AdjImpl<LV>::tan_reverse_g<G>(m, md, ld, n, xi, cb, cbd, mbd, s);                         \
  }                                                                                          \
  }
