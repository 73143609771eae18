"""Emit the per-level device code of the MTP evaluation as a HIP header.

For one level the header defines a traits struct ``Lv<L>`` with static
device functions, all straight-line code with compile-time indices so that
per-atom state stays in registers:

  acc_moments<G>(m, f, x, y, z)        m[e] += f[mu_e] x^a y^b z^c   (entry group G; binary32)
  acc_part<P>(m, f, x, y, z)           the same for the entries of part P (binary64)
  pair_grad<G>(mb, f, fp, x, y, z, ...) gradient of sum_e mb[e] f_mu x^a y^b z^c w.r.t. d (binary32)
  pair_part<P>(mb, f, h, x, y, z, ...)  the same for part P by nested Horner schemes (binary64)
  fwd(M, C)                             connected contractions C_q from moments
  products(C, xi, Cb, B)                basis values, site energy, adjoints of C_q
  rev<G>(M, Cb, mb)                     mb[e] += sum_q Cb_q dC_q/dm_e   (entries of group G)
  tan(M, Md, C, Cd)                     forward-mode tangent of the contractions
  ...

The host-side tables (moment layout, product trie, basis order) are
emitted too, for argument checking and tests.
"""
from __future__ import annotations

import math
import os
from collections import defaultdict
from fractions import Fraction

from .program import Program, build_program
from .waves import emit_waves


def _lit(w) -> str:
    v = float(w)
    if v == int(v) and abs(v) < 1e15:
        return f"R({int(v)})"
    return f"R({v!r})"


class _W:
    def __init__(self):
        self.lines = []
        self.ind = 0

    def __call__(self, s=""):
        self.lines.append("  " * self.ind + s)

    def push(self):
        self.ind += 1

    def pop(self):
        self.ind -= 1

    def text(self):
        return "\n".join(self.lines) + "\n"


def entry_groups(prog: Program, n_groups):
    """Split the flat moment layout into contiguous ranges: n_groups ranges of similar size,
    or, given a tuple, the interior boundaries themselves (e.g. (84,) at level 16 separates the
    mu = 0 components from the rest)."""
    n = prog.n_mom
    if isinstance(n_groups, (tuple, list)):
        bounds = [0] + [int(b) for b in n_groups] + [n]
        assert all(bounds[k] < bounds[k + 1] for k in range(len(bounds) - 1))
    else:
        bounds = [round(k * n / n_groups) for k in range(n_groups + 1)]
    return [(bounds[k], bounds[k + 1]) for k in range(len(bounds) - 1)]


def _ref(r, mvar="me"):
    kind, k = r
    if kind == "m":
        return f"{mvar}{k}"
    if kind == "t":
        return f"t{k}"
    return f"C[{k}]"


def _emit_pair_functions(w: _W, prog: Program, groups):
    """Moment accumulation and pair gradient, emitted degree by degree: the monomials of
    degree nu are formed from those of degree nu - 1 and consumed right away, so only two
    degrees of monomials are live at once."""
    items = prog.layout.items
    for gi, (lo, hi) in enumerate(groups):
        ents = list(range(lo, hi))
        by_mono = defaultdict(list)
        for e in ents:
            mu, a, b, c = items[e]
            by_mono[(a, b, c)].append((e, mu))
        gnu = max(a + b + c for (a, b, c) in by_mono)
        # ---------------- moment accumulation
        w(f"// entries [{lo}, {hi}) of the moment layout")
        w("template <class R>")
        w(f"static __device__ __forceinline__ void acc_moments_g{gi}(R* __restrict__ m, const R* __restrict__ f, R x, R y, R z) {{")
        w.push()
        # degree by degree: the monomials of one degree are independent products, formed
        # together (measured faster here than forming each right before its accumulations)
        need = _monomial_closure(by_mono.keys())
        for nu in range(gnu + 1):
            for abc in _degree(need, nu):
                _emit_one_monomial(w, abc)
            for abc in _degree(by_mono.keys(), nu):
                for e, mu in by_mono[abc]:
                    w(f"m[{e - lo}] = fma(f[{mu}], {_mono_name(abc)}, m[{e - lo}]);")
        w.pop()
        w("}")
        # ---------------- gradient of sum_e mb_e f_mu_e mono_e, and u = sum_mu fp_mu S_mu
        # In scaled monomials q_abc = x^a y^b z^c / (a! b! c!) the gradient of q_abc is
        # (q_(a-1)bc, q_a(b-1)c, q_ab(c-1)) without factors, so the caller passes the adjoints
        # multiplied by a! b! c! (MFACT): mb_e mono_e = (mb_e a!b!c!) q_e.
        w("template <class R>")
        w(f"static __device__ __forceinline__ void pair_grad_g{gi}(const R* __restrict__ mb, const R* __restrict__ f,")
        w("    const R* __restrict__ fp, R x, R y, R z, R& gx, R& gy, R& gz, R& u) {")
        w.push()
        mus = sorted({items[e][0] for e in ents})
        for mu in mus:
            w(f"R s{mu} = R(0);")
        # gradient sums of the monomials with a single radial function, per radial function
        # and degree
        single = set()
        for mu in mus:
            for n in range(1, gnu + 1):
                w(f"R hx{mu}_{n} = R(0), hy{mu}_{n} = R(0), hz{mu}_{n} = R(0);")
        top = max(max(k) for k in by_mono)
        for var in "xyz":
            for k in range(2, top + 1):
                w(f"const R {var}_{k} = {var} * {_lit(Fraction(1, k))};")
        made = set()

        def make(abc):
            # a scaled monomial is formed right before its first use (its chain parent first),
            # so that few monomials of the current degree are live at once
            if abc in made:
                return
            a, b, c = abc
            name = _mono_name(abc)
            if a + b + c == 0:
                w(f"const R {name} = R(1);")
            else:
                parent, var, k = ((a, b, c - 1), "z", c) if c else ((a, b - 1, 0), "y", b) if b else ((a - 1, 0, 0), "x", a)
                make(parent)
                fac = var if k == 1 else f"{var}_{k}"
                w(f"const R {name} = {_mono_name(parent)} * {fac};")
            made.add(abc)

        for nu in range(gnu + 1):
            for abc in _degree(by_mono.keys(), nu):
                make(abc)
                for low in ((abc[0] - 1, abc[1], abc[2]), (abc[0], abc[1] - 1, abc[2]), (abc[0], abc[1], abc[2] - 1)):
                    if min(low) >= 0:
                        make(low)
                lst = by_mono[abc]
                a, b, c = abc
                if len(lst) == 1 and a + b + c > 0:
                    # one radial function: accumulate mb_e grad q_e per degree nu, without the
                    # radial factor (applied once per pair); the value sum of these terms follows
                    # from Euler's relation d . grad P = nu P for a homogeneous P of degree nu
                    e, mu = lst[0]
                    single.add((mu, nu))
                    for d, k, low in (("x", a, (a - 1, b, c)), ("y", b, (a, b - 1, c)), ("z", c, (a, b, c - 1))):
                        if k:
                            w(f"h{d}{mu}_{nu} = fma(mb[{e - lo}], {_mono_name(low)}, h{d}{mu}_{nu});")
                    continue
                for e, mu in lst:
                    w(f"s{mu} = fma(mb[{e - lo}], {_mono_name(abc)}, s{mu});")
                if a + b + c == 0:
                    continue
                dirs = [(d, low) for d, k, low in (("x", a, (a - 1, b, c)), ("y", b, (a, b - 1, c)),
                                                   ("z", c, (a, b, c - 1))) if k]
                first = True
                for e, mu in lst:
                    if first:
                        w(f"{{ R t = f[{mu}] * mb[{e - lo}];")
                        first = False
                    else:
                        w(f"  t = fma(f[{mu}], mb[{e - lo}], t);")
                for d, low in dirs:
                    w(f"  g{d} = fma(t, {_mono_name(low)}, g{d});")
                w("}")
        for mu in sorted({m for m, _ in single}):
            nus = sorted(n for m, n in single if m == mu)
            for d in "xyz":
                terms = " + ".join(f"h{d}{mu}_{n}" for n in nus)
                w(f"g{d} = fma(f[{mu}], {terms}, g{d});")
            for n in nus:
                w(f"s{mu} = fma(fma(z, hz{mu}_{n}, fma(y, hy{mu}_{n}, x * hx{mu}_{n})), {_lit(Fraction(1, n))}, s{mu});")
        for mu in mus:
            w(f"u = fma(fp[{mu}], s{mu}, u);")
        w.pop()
        w("}")


# Most moment entries one wave of the binary64 moment kernel accumulates: two registers each, with
# the pair's own values within the 256 that two waves per SIMD leave a lane (no copies to and from
# accumulation registers).
MOMENT_PART_CAP = 84


def moment_parts(prog: Program, cap=MOMENT_PART_CAP):
    """The moment entries cut into parts of at most cap entries, each a list of (mu, a) slices (all
    entries of one radial function and x exponent), in order.  Level 16: mu = 0 (84) and the rest
    (46); level 20: 81, 84, 84, 46."""
    size = defaultdict(int)
    for mu, a, _, _ in prog.layout.items:
        size[mu, a] += 1
    parts, fill = [], 0
    for key in sorted(size):
        if not parts or fill + size[key] > cap:
            parts.append([])
            fill = 0
        parts[-1].append(key)
        fill += size[key]
    return parts


def part_entries(prog: Program, parts):
    """Moment entries of each part, in the order (mu, a, b, c)."""
    at = {it: e for e, it in enumerate(prog.layout.items)}
    return [[at[it] for it in sorted(at) if it[:2] in part] for part in (set(p) for p in parts)]


def _emit_part_tables(w: _W, pre, order):
    """Number, sizes and entries of parts: N{pre}PART, {pre}PART_SIZE, {pre}PART_ENTRY (-1 past a part's end)."""
    width = max(len(o) for o in order)
    rows = ["{" + ", ".join(str(e) for e in o + [-1] * (width - len(o))) + "}" for o in order]
    w(f"static constexpr int N{pre}PART = {len(order)}, {pre}PART_MAX = {width};")
    w(f"static constexpr int {pre}PART_SIZE[N{pre}PART] = {{{', '.join(str(len(o)) for o in order)}}};")
    w(f"static constexpr int {pre}PART_ENTRY[N{pre}PART][{pre}PART_MAX] = {{{', '.join(rows)}}};")


def _emit_moment_parts(w: _W, prog: Program, parts):
    """acc_part<P>(m, f, x, y, z): m[k] += f_mu x^a y^b z^c for the entries PART_ENTRY[P][k].  For
    each (mu, a, b) the run over c multiplies the weighted monomial f_mu x^a y^b z^c by z and adds
    it; the last entry of a run takes its factor z in the addition.  Three running products are
    live, one multiplication less per run than forming every monomial."""
    ents = {}
    for e, (mu, a, b, c) in enumerate(prog.layout.items):
        ents.setdefault((mu, a), {}).setdefault(b, {})[c] = e
    order = part_entries(prog, parts)
    _emit_part_tables(w, "", order)
    # radial functions of every part but the last (what the last part's wave hands to the others
    # in the pair-gradient kernel)
    w(f"static constexpr int NMU_SHARED = {max([mu for p in parts[:-1] for mu, _ in p], default=-1) + 1};")
    for pi, part in enumerate(parts):
        slot = {e: k for k, e in enumerate(order[pi])}
        w("template <class R>")
        w(f"static __device__ __forceinline__ void acc_part_p{pi}(R* __restrict__ m, const R* __restrict__ f, R x, R y, R z) {{")
        w.push()
        for mu in sorted({k[0] for k in part}):
            avals = sorted(a for m2, a in part if m2 == mu)
            w(f"{{  // mu = {mu}")
            w.push()
            w(f"R wx = f[{mu}];")
            at = 0
            for a in avals:
                while at < a:
                    w("wx *= x;")
                    at += 1
                bs = sorted(ents[mu, a])
                assert bs == list(range(len(bs)))
                w("{")
                w.push()
                w("R wy = wx;")
                for b in bs:
                    if b:
                        w("wy *= y;")
                    cs = sorted(ents[mu, a][b])
                    assert cs == list(range(len(cs)))
                    k = [slot[ents[mu, a][b][c]] for c in cs]
                    w(f"m[{k[0]}] += wy;")
                    if len(cs) > 1:
                        w("{")
                        w.push()
                        cur = "wy"
                        if len(cs) > 2:
                            w("R wz = wy * z;")
                            for c in cs[1:-1]:
                                if c > 1:
                                    w("wz *= z;")
                                w(f"m[{k[c]}] += wz;")
                            cur = "wz"
                        w(f"m[{k[-1]}] = fma({cur}, z, m[{k[-1]}]);")
                        w.pop()
                        w("}")
                w.pop()
                w("}")
            w.pop()
            w("}")
        w.pop()
        w("}")
    w("template <int P, class R>")
    w("static __device__ __forceinline__ void acc_part(R* __restrict__ m, const R* __restrict__ f, R x, R y, R z) {")
    w.push()
    for p in range(len(parts)):
        w(f"{'if' if p == 0 else 'else if'} constexpr (P == {p}) acc_part_p{p}<R>(m, f, x, y, z);")
    w.pop()
    w("}")


def _emit_horner(w: _W, coef, pre, gradient=True):
    """Value and gradient of sum coef[a, b, c] x^a y^b z^c in {pre}v, {pre}x, {pre}y, {pre}z by
    Horner's scheme nested over x, y and z, each step carrying the derivative (d <- d t + v before
    v <- v t + c).  A coefficient is read once and enters one multiply-add; about two multiply-adds
    per coefficient in all.  Depth first, so that nine partial values are live at most.  Missing
    coefficients are zero; the names of derivatives that vanish are not declared (returned: the
    names declared, by direction).  Without gradient only the value (one multiply-add per
    coefficient)."""
    top = max(a for a, _, _ in coef)
    P = {}

    def step(state, key, var, add):
        """state[key] <- state[key] var + add (add may be None)."""
        cur = state.get(key)
        if cur is None:
            if add is not None:
                state[key] = f"{pre}{key}"
                w(f"R {pre}{key} = {add};")
        elif add is None:
            w(f"{cur} = {cur} * {var};")
        else:
            w(f"{cur} = fma({cur}, {var}, {add});")

    for a in range(top, -1, -1):
        bs = [b for (a2, b, _) in coef if a2 == a]
        M = {}
        if bs:
            w(f"R {pre}mv{a}" + (f", {pre}my{a}, {pre}mz{a};" if gradient else ";"))
        for b in range(max(bs) if bs else -1, -1, -1):
            cs = [c for (a2, b2, c) in coef if (a2, b2) == (a, b)]
            I = {}
            tag = f"{a}_{b}"
            for c in range(max(cs) if cs else -1, -1, -1):
                k = coef.get((a, b, c))
                v = I.get("v")
                if v is not None:
                    if not gradient:
                        pass
                    elif "d" in I:
                        w(f"{pre}id{tag} = fma({pre}id{tag}, z, {v});")
                    else:
                        w(f"R {pre}id{tag} = {v};")
                        I["d"] = f"{pre}id{tag}"
                    w(f"{v} = {f'fma({v}, z, {k})' if k else f'{v} * z'};")
                elif k:
                    I["v"] = f"{pre}iv{tag}"
                    w(f"R {pre}iv{tag} = {k};")
            for key, var, add in (("my", "y", M.get("mv")), ("mv", "y", I.get("v")), ("mz", "y", I.get("d"))):
                if key != "mv" and not gradient:
                    continue
                cur, name = M.get(key), f"{pre}{key}{a}"
                if cur is None:
                    if add is not None:
                        w(f"{name} = {add};")
                        M[key] = name
                elif add is None:
                    w(f"{name} = {name} * {var};")
                else:
                    w(f"{name} = fma({name}, {var}, {add});")
        if gradient:
            step(P, "x", "x", P.get("v"))
        step(P, "v", "x", M.get("mv"))
        if gradient:
            step(P, "y", "x", M.get("my"))
            step(P, "z", "x", M.get("mz"))
    return P


def _emit_part_gradients(w: _W, prog: Program, parts):
    """pair_part<P>: with the adjoints mb of part P's entries (in PART_ENTRY order), per radial
    function g += f_mu grad P_mu and u += h_mu P_mu, P_mu = sum_e mb_e x^a y^b z^c."""
    items = prog.layout.items
    order = part_entries(prog, parts)
    for pi, ents in enumerate(order):
        w("template <class R>")
        w(f"static __device__ __forceinline__ void pair_part_p{pi}(const R* __restrict__ mb, const R* __restrict__ f,")
        w("    const R* __restrict__ h, R x, R y, R z, R& gx, R& gy, R& gz, R& u) {")
        w.push()
        for mu in sorted({items[e][0] for e in ents}):
            coef = {items[e][1:]: f"mb[{k}]" for k, e in enumerate(ents) if items[e][0] == mu}
            w("{")
            w.push()
            names = _emit_horner(w, coef, "p")
            for d in "xyz":
                if d in names:
                    w(f"g{d} = fma(f[{mu}], {names[d]}, g{d});")
            w(f"u = fma(h[{mu}], {names['v']}, u);")
            w.pop()
            w("}")
        w.pop()
        w("}")
    w("template <int P, class R>")
    w("static __device__ __forceinline__ void pair_part(const R* __restrict__ mb, const R* __restrict__ f,")
    w("    const R* __restrict__ h, R x, R y, R z, R& gx, R& gy, R& gz, R& u) {")
    w.push()
    for p in range(len(parts)):
        w(f"{'if' if p == 0 else 'else if'} constexpr (P == {p}) pair_part_p{p}<R>(mb, f, h, x, y, z, gx, gy, gz, u);")
    w.pop()
    w("}")


def _degree(keys, nu):
    return sorted((k for k in keys if k[0] + k[1] + k[2] == nu), key=lambda t: (-t[0], -t[1]))


def _monomial_closure(keys):
    """Every monomial on the construction chain of the given ones (z, then y, then x factors)."""
    need = set()
    for a, b, c in keys:
        for k in range(c + 1):
            need.add((a, b, k))
        for k in range(b + 1):
            need.add((a, k, 0))
        for k in range(a + 1):
            need.add((k, 0, 0))
    return need


def _emit_one_monomial(w, abc):
    """mono_a_b_c from the monomial one factor lower on its chain (z, then y, then x)."""
    a, b, c = abc
    name = _mono_name(abc)
    if a + b + c == 0:
        w(f"const R {name} = R(1);")
    elif c > 0:
        w(f"const R {name} = {_mono_name((a, b, c - 1))} * z;")
    elif b > 0:
        w(f"const R {name} = {_mono_name((a, b - 1, 0))} * y;")
    else:
        w(f"const R {name} = {_mono_name((a - 1, 0, 0))} * x;")


def _mono_name(abc):
    a, b, c = abc
    return f"mono_{a}_{b}_{c}"


def _group_ops(ops):
    """Group a block's ops by (dst, x): {(dst, x): [(y, w), ...]} preserving first-seen order."""
    groups = {}
    for dst, x, y, wgt in ops:
        groups.setdefault((dst, x), []).append((y, wgt))
    return groups


def _emit_block_forward(w: _W, blk, with_output=True):
    for k in range(blk.n_temp):
        w(f"R t{k} = R(0);")
    for (dst, x), lst in _group_ops(blk.ops).items():
        if dst[0] == "c" and not with_output:
            continue
        if lst[0][0] is None:
            w(f"{_ref(dst)} = {_ref(x)};")
            continue
        _emit_inner(w, lst, "s")
        w(f"{_ref(dst)} = fma({_ref(x)}, s, {_ref(dst)}); }}")


def _emit_inner(w, lst, var):
    (y0, w0) = lst[0]
    if w0 == 1:
        w(f"{{ R {var} = {_ref(y0)};")
    else:
        w(f"{{ R {var} = {_lit(w0)} * {_ref(y0)};")
    for y, wgt in lst[1:]:
        if wgt == 1:
            w(f"  {var} += {_ref(y)};")
        else:
            w(f"  {var} = fma({_lit(wgt)}, {_ref(y)}, {var});")


# Moment loads kept in flight by the reverse program (whose blocks are fenced to bound register
# pressure): each contraction block takes its entries from a ring of prefetched values and
# issues the load that many positions ahead, so the global-memory latency of one block is
# covered by the arithmetic of the blocks before it.
PREFETCH_DEPTH = int(os.environ.get("MTP_PREFETCH_DEPTH", "24"))
# the same for the tangent of the reverse program (which loads moments, their tangents and
# the contraction adjoints with their tangents)
TAN_PREFETCH_DEPTH = int(os.environ.get("MTP_TAN_PREFETCH_DEPTH", "24"))

# Register estimate (VGPRs) of the reverse tangent of one block: values, tangents, adjoints and
# adjoint tangents of its temporaries, the values and tangents of the entries it reads, and the
# prefetched loads.  A part of the reverse-tangent program adds the accumulators live at each of
# its blocks (two VGPRs each); parts are cut so that this stays within RTAN_REG_BUDGET (the 512
# VGPR + AGPR of one wave per SIMD).  The estimate is rough (some parts spill, some blocks over
# it do not).  On the device one lane runs it up to level 10, in a single part; levels from 12 on run by
# several waves per tile (at level 20 4.9 ms, where the parts took 8.1) and keep these parts for the
# host's tests.
RTAN_REG_BUDGET = int(os.environ.get("MTP_RTAN_BUDGET", "512"))
# blocks tried for each addition to a part (those adding the fewest new entries)
RTAN_CANDIDATES = 12


def _locality_order(blocks):
    """Contraction blocks reordered so that consecutive blocks share moment entries (each next
    block has the largest overlap with the entries of the last three): re-reads of an entry
    come soon after its first read and hit the cache.  The blocks are independent sums, so the
    order is free."""
    rem = list(blocks)
    if not rem:
        return rem
    order = [max(rem, key=lambda b: (len(b.entries), -b.q))]
    rem.remove(order[0])
    while rem:
        recent = set(e for b in order[-3:] for e in b.entries)
        nxt = max(rem, key=lambda b: (len(set(b.entries) & recent), -len(b.entries), -b.q))
        order.append(nxt)
        rem.remove(nxt)
    return order


def _emit_components_forward(w: _W, prog: Program):
    """Connected contractions.  No block fences here: the blocks are independent and the
    scheduler interleaves them freely (their loads overlap the arithmetic of other blocks)."""
    w("template <class R, class MA>")
    w("static __device__ __forceinline__ void fwd(const MA& M, R* __restrict__ C) {")
    w.push()
    for blk in _locality_order(prog.blocks):
        w(f"{{  // contraction {blk.q}")
        w.push()
        for e in blk.entries:
            w(f"const R me{e} = M({e});")
        w(f"C[{blk.q}] = R(0);")
        _emit_block_forward(w, blk)
        w.pop()
        w("}")
    w.pop()
    w("}")


def _emit_components_reverse(w: _W, prog: Program, groups):
    for gi, (lo, hi) in enumerate(groups):
        # Cb: anything indexable by component (a pointer, or a strided accessor of LDS)
        w("template <class R, class MA, class CB>")
        w(f"static __device__ __forceinline__ void rev_g{gi}(const MA& M, const CB& Cb, R* __restrict__ mb) {{")
        w.push()
        blocks = _locality_order([blk for blk in prog.blocks if any(lo <= e < hi for e in blk.entries)])
        seq = [e for blk in blocks for e in blk.entries]   # every moment load, in program order
        depth = max(1, min(PREFETCH_DEPTH, len(seq)))
        for k in range(depth):
            w(f"R pf{k} = M({seq[k]});")
        pos = 0
        for blk in blocks:
            w(f"{{  // contraction {blk.q}")
            w.push()
            w("MTP_BLOCK_FENCE();")
            for e in blk.entries:
                slot = pos % depth
                w(f"const R me{e} = pf{slot};")
                if pos + depth < len(seq):
                    w(f"pf{slot} = M({seq[pos + depth]});")
                pos += 1
            w(f"const R cb = Cb[{blk.q}];")
            _emit_block_forward(w, blk, with_output=False)
            for k in range(blk.n_temp):
                w(f"R tb{k} = R(0);")
            _emit_block_reverse(w, blk, lambda ref: _adj(ref, lo, hi))
            w.pop()
            w("}")
        w.pop()
        w("}")


def _adj(ref, lo, hi):
    kind, k = ref
    if kind == "t":
        return f"tb{k}"
    if kind == "m":
        return f"mb[{k - lo}]" if lo <= k < hi else None
    return "cb"


def _emit_block_reverse(w: _W, blk, adj):
    """The block read backwards; adj names the adjoint of a reference (None: not accumulated)."""
    # walk steps backwards: ops were appended step by step
    rev_ops = list(reversed(blk.ops))
    # group by (dst, x) for x-adjoints and by (dst, y) for y-adjoints, in reverse step order
    seen_dst = []
    by_dst = defaultdict(list)
    for dst, x, y, wgt in rev_ops:
        if dst not in by_dst:
            seen_dst.append(dst)
        by_dst[dst].append((x, y, wgt))
    for dst in seen_dst:
        lst = by_dst[dst]
        db = adj(dst)
        if lst[0][1] is None:
            (x, _, _), = lst
            tgt = adj(x)
            if tgt:
                w(f"{tgt} += {db};")
            continue
        xs = {}
        ys = {}
        for x, y, wgt in lst:
            xs.setdefault(x, []).append((y, wgt))
            ys.setdefault(y, []).append((x, wgt))
        for x, l2 in xs.items():
            tgt = adj(x)
            if not tgt:
                continue
            _emit_inner(w, l2, "s")
            w(f"{tgt} = fma({db}, s, {tgt}); }}")
        for y, l2 in ys.items():
            tgt = adj(y)
            if not tgt:
                continue
            _emit_inner(w, l2, "s")
            w(f"{tgt} = fma({db}, s, {tgt}); }}")


def _emit_products(w: _W, prog: Program):
    children = defaultdict(list)
    roots = []
    for a, (parent, comp) in enumerate(prog.trie):
        if parent < 0:
            roots.append(a)
        else:
            children[parent].append(a)
    w("// E_i contribution sum_alpha xi_alpha B_alpha; Cb_q = dE_i/dC_q; B written when Bo != nullptr")
    w("template <bool WB, class R>")
    w("static __device__ __forceinline__ double products(const R* __restrict__ C, const double* __restrict__ xi,")
    w("    R* __restrict__ Cb, double* __restrict__ Bo, long ldb) {")
    w.push()
    w("double e = 0.0;")
    for q in range(prog.n_comp):
        w(f"Cb[{q}] = R(0);")

    def node2(a, parent_var):
        # variant that leaves bb{a} declared in the enclosing scope
        parent, comp = prog.trie[a]
        w(f"R bb{a};")
        w("{")
        w.push()
        if parent_var is None:
            w(f"const R b = C[{comp}];")
        else:
            w(f"const R b = {parent_var} * C[{comp}];")
        w(f"e = fma(xi[{a}], double(b), e);")
        w(f"if constexpr (WB) Bo[{a} * ldb] = double(b);")
        w(f"bb{a} = R(xi[{a}]);")
        if children[a]:
            w(f"const R p{a} = b;")
            for ch in children[a]:
                node2(ch, f"p{a}")
                _, ccomp = prog.trie[ch]
                w(f"bb{a} = fma(bb{ch}, C[{ccomp}], bb{a});")
        w.pop()
        w("}")
        if parent_var is None:
            w(f"Cb[{comp}] += bb{a};")
        else:
            w(f"Cb[{comp}] = fma(bb{a}, {parent_var}, Cb[{comp}]);")

    for a in roots:
        node2(a, None)
    w("return e;")
    w.pop()
    w("}")


def _emit_dispatchers(w: _W, n_groups: int):
    sigs = (
        ("acc_moments", "R* __restrict__ m, const R* __restrict__ f, R x, R y, R z", "m, f, x, y, z", "class R"),
        ("pair_grad", "const R* __restrict__ mb, const R* __restrict__ f, const R* __restrict__ fp, R x, R y, R z, "
                      "R& gx, R& gy, R& gz, R& u", "mb, f, fp, x, y, z, gx, gy, gz, u", "class R"),
        ("rev", "const MA& M, const CB& Cb, R* __restrict__ mb", "M, Cb, mb", "class R, class MA, class CB"),
    )
    for name, params, args, tparams in sigs:
        w(f"template <int G, {tparams}>")
        w(f"static __device__ __forceinline__ void {name}({params}) {{")
        w.push()
        for g in range(n_groups):
            kw = "if constexpr" if g == 0 else "else if constexpr"
            targs = "<R>" if name != "rev" else "<R, MA, CB>"
            w(f"{kw} (G == {g}) {name}_g{g}{targs}({args});")
        w.pop()
        w("}")


def emit_level(level: int, n_groups: int = 1, rtan_budget: int = RTAN_REG_BUDGET) -> str:
    prog = build_program(level)
    groups = entry_groups(prog, n_groups)
    w = _W()
    w(f"// Generated MTP level-{level} program.  Do not edit; produced by codegen/emit.py.")
    w("#pragma once")
    w("#ifndef MTP_TILE_FENCE  // compiled for the host, where the order of the code is the compiler's")
    w("#define MTP_TILE_FENCE()")
    w("#define MTP_PIN(x)")
    w("#endif")
    w(f"struct Lv{level} {{")
    w.push()
    w(f"static constexpr int LEVEL = {level};")
    w(f"static constexpr int NMOM = {prog.n_mom};")
    w(f"static constexpr int NCOMP = {prog.n_comp};")
    w(f"static constexpr int NALPHA = {prog.n_alpha};")
    w(f"static constexpr int NMU = {prog.n_mu};")
    w(f"static constexpr int MAXNU = {prog.max_nu};")
    w(f"static constexpr int NGROUP = {len(groups)};")
    w(f"static constexpr int TRIPLES = {prog.triple_count()};")
    w("static constexpr int GROUP_LO[NGROUP] = {" + ", ".join(str(g[0]) for g in groups) + "};")
    w("static constexpr int GROUP_HI[NGROUP] = {" + ", ".join(str(g[1]) for g in groups) + "};")
    rparts = rev_tan_parts(prog, rtan_budget)
    # parts of the reverse-tangent program, run in order (one kernel each)
    w(f"static constexpr int NRTPART = {len(rparts)};")
    w("// flat moment layout: (mu, a, b, c) of component e")
    w("static constexpr int ENTRIES[NMOM][4] = {" + ", ".join("{%d, %d, %d, %d}" % it for it in prog.layout.items) + "};")
    # a! b! c! of each entry: pair_grad takes the moment adjoints scaled by it
    w("static constexpr double MFACT[NMOM] = {" + ", ".join(
        "%d." % (math.factorial(a) * math.factorial(b) * math.factorial(c)) for (_, a, b, c) in prog.layout.items) + "};")
    _emit_pair_functions(w, prog, groups)
    parts = moment_parts(prog)
    _emit_moment_parts(w, prog, parts)
    _emit_part_gradients(w, prog, parts)
    _emit_components_forward(w, prog)
    _emit_components_reverse(w, prog, groups)
    _emit_products(w, prog)
    _emit_dispatchers(w, len(groups))
    emit_tangent_parts(w, prog, rparts)
    emit_waves(w, prog)
    w.pop()
    w("};")
    return w.text()


def write_level(level: int, out_dir: str, n_groups: int = 1) -> str:
    os.makedirs(out_dir, exist_ok=True)
    path = os.path.join(out_dir, f"mtp_L{level}.inc")
    text = emit_level(level, n_groups)
    old = None
    if os.path.exists(path):
        with open(path) as fh:
            old = fh.read()
    if old != text:
        with open(path, "w") as fh:
            fh.write(text)
    return path


# ======================================================================================
# tangent (forward-mode) code for the parameter adjoint
#
# The parameter gradient needs, per atom, the directional derivative of every quantity
# along the per-pair displacement change delta_ij = fbar_j - fbar_i:
#   md   = sum_j d/dd [f_mu(r) mono_e(d)] . delta          (tangent of the moments)
#   Cd, Bd                                                  (tangents of contractions/basis)
#   Cbd, mbd                                                (tangents of the adjoints)
# Each generated function mirrors its value counterpart and carries a tangent next to
# every value (forward-over-reverse).


# Most entries one wave of the moment-tangent kernel accumulates (84, as in the moment kernel, spills
# up to 184 bytes per lane next to the tangents of the running products; 66 gives two parts at
# level 16 and five at level 20).
TANGENT_PART_CAP = 66


def _emit_tangent_moment_parts(w: _W, prog: Program, parts):
    """tan_part<P>(md, f, fd, x, y, z, ex, ey, ez): md[k] += the tangent of f_mu x^a y^b z^c along
    (ex, ey, ez) for the entries TPART_ENTRY[P][k], fd_mu the tangent of f_mu.  Runs as in acc_part,
    each running product (value, tangent): (w, wd) x = (w x, wd x + w ex)."""
    ents = {}
    for e, (mu, a, b, c) in enumerate(prog.layout.items):
        ents.setdefault((mu, a), {}).setdefault(b, {})[c] = e
    order = part_entries(prog, parts)
    _emit_part_tables(w, "T", order)

    def times(dst, src, var):
        w(f"{dst}d = fma({src}d, {var}, {src} * e{var});")
        w(f"{dst} = {src} * {var};")

    for pi, part in enumerate(parts):
        slot = {e: k for k, e in enumerate(order[pi])}
        w("template <class R>")
        w(f"static __device__ __forceinline__ void tan_part_p{pi}(R* __restrict__ md, const R* __restrict__ f,")
        w("    const R* __restrict__ fd, R x, R y, R z, R ex, R ey, R ez) {")
        w.push()
        for mu in sorted({k[0] for k in part}):
            w(f"{{  // mu = {mu}")
            w.push()
            w(f"R wx = f[{mu}], wxd = fd[{mu}];")
            at = 0
            for a in sorted(a for m2, a in part if m2 == mu):
                while at < a:
                    times("wx", "wx", "x")
                    at += 1
                w("{")
                w.push()
                w("R wy = wx, wyd = wxd;")
                for b in sorted(ents[mu, a]):
                    if b:
                        times("wy", "wy", "y")
                    k = [slot[ents[mu, a][b][c]] for c in sorted(ents[mu, a][b])]
                    w(f"md[{k[0]}] += wyd;")
                    if len(k) > 1:
                        w("{")
                        w.push()
                        cur = "wy"
                        if len(k) > 2:
                            w("R wz, wzd;")
                            for c in range(1, len(k) - 1):
                                times("wz", cur, "z")
                                cur = "wz"
                                w(f"md[{k[c]}] += wzd;")
                        w(f"md[{k[-1]}] = fma({cur}d, z, fma({cur}, ez, md[{k[-1]}]));")
                        w.pop()
                        w("}")
                w.pop()
                w("}")
            w.pop()
            w("}")
        w.pop()
        w("}")
    w("template <int P, class R>")
    w("static __device__ __forceinline__ void tan_part(R* __restrict__ md, const R* __restrict__ f, const R* __restrict__ fd,")
    w("    R x, R y, R z, R ex, R ey, R ez) {")
    w.push()
    for p in range(len(parts)):
        w(f"{'if' if p == 0 else 'else if'} constexpr (P == {p}) tan_part_p{p}<R>(md, f, fd, x, y, z, ex, ey, ez);")
    w.pop()
    w("}")


# The adjoint pair pass evaluates, per pair and radial function, S_mu = P_mu (coefficients mb), its
# derivative along (ex, ey, ez), and V_mu = the polynomial of coefficients ebar mb - mbd.  A slice
# (mu, a) of a gradient polynomial costs about two multiply-adds per entry, of a value polynomial
# one; forming a pair's geometry about ADJ_GEOMETRY.
ADJ_STAGE_CAP = 90     # coefficients a wave holds (two registers each, of 256)
ADJ_GEOMETRY = 75


def adj_stages(prog: Program, cap=ADJ_STAGE_CAP):
    """The slices (kind, mu, a), kind 0 gradient or 1 value, cut into stages of one wave each: in
    order, at most cap coefficients per stage, as few stages as the cap allows and the largest cost
    (the first stage also forms the geometry) as small as the order allows."""
    size = defaultdict(int)
    for mu, a, _, _ in prog.layout.items:
        size[mu, a] += 1
    seq = []
    for mu in sorted({k[0] for k in size}, reverse=True):
        for a in sorted((k[1] for k in size if k[0] == mu), reverse=True):
            seq += [(0, mu, a), (1, mu, a)]

    def fill(limit):
        out, regs, cost = [[]], 0, ADJ_GEOMETRY
        for kind, mu, a in seq:
            n = size[mu, a]
            c = n if kind else 2 * n
            if out[-1] and (regs + n > cap or cost + c > limit):
                out.append([])
                regs = cost = 0
            out[-1].append((kind, mu, a))
            regs += n
            cost += c
        return out

    costs = range(ADJ_GEOMETRY, ADJ_GEOMETRY + 3 * prog.n_mom + 1)
    fewest = len(fill(costs[-1]))
    return next(f for f in map(fill, costs) if len(f) == fewest)


def _emit_adj_stages(w: _W, prog: Program, stages):
    """adj_stage<B>(c, x, y, z, ex, ey, ez, S, X): with the coefficients c of stage B (entry
    ADJ_ENTRY[B][k], ADJ_VALUE[B][k] = 1 for those of a value polynomial), S_mu += P_mu and
    X_mu += V_mu - (ex, ey, ez) . grad P_mu over its slices."""
    at = {it: e for e, it in enumerate(prog.layout.items)}
    lists = []
    for st in stages:
        keys = [(kind, it) for kind in (0, 1) for it in sorted(at) if (kind, it[0], it[1]) in set(st)]
        lists.append(keys)
    width = max(len(k) for k in lists)
    w(f"static constexpr int NASTAGE = {len(stages)};")
    w(f"static constexpr int ADJ_MAX = {width};")
    w(f"static constexpr int ADJ_SIZE[NASTAGE] = {{{', '.join(str(len(k)) for k in lists)}}};")
    for name, val in (("ADJ_ENTRY", lambda kind, it: at[it]), ("ADJ_VALUE", lambda kind, it: kind)):
        rows = ["{" + ", ".join([str(val(*k)) for k in keys] + ["-1"] * (width - len(keys))) + "}" for keys in lists]
        w(f"static constexpr int {name}[NASTAGE][ADJ_MAX] = {{{', '.join(rows)}}};")
    for name, fn in (("ADJ_MU_LO", min), ("ADJ_MU_HI", max)):
        w(f"static constexpr int {name}[NASTAGE] = {{{', '.join(str(fn(k[1] for k in st)) for st in stages)}}};")
    for bi, keys in enumerate(lists):
        w("template <class R>")
        w(f"static __device__ __forceinline__ void adj_stage_s{bi}(const R* __restrict__ c, R x, R y, R z, R ex, R ey, R ez,")
        w("    R* __restrict__ S, R* __restrict__ X) {")
        w.push()
        for mu in sorted({it[0] for _, it in keys}):
            for kind in (0, 1):
                coef = {it[1:]: f"c[{k}]" for k, (kd, it) in enumerate(keys) if kd == kind and it[0] == mu}
                if not coef:
                    continue
                w("{")
                w.push()
                names = _emit_horner(w, coef, "p", gradient=kind == 0)
                if kind == 0:
                    w(f"S[{mu}] += {names['v']};")
                    for d in "xyz":
                        if d in names:
                            w(f"X[{mu}] = fma(-e{d}, {names[d]}, X[{mu}]);")
                else:
                    w(f"X[{mu}] += {names['v']};")
                w.pop()
                w("}")
        w.pop()
        w("}")
    w("template <int B, class R>")
    w("static __device__ __forceinline__ void adj_stage(const R* __restrict__ c, R x, R y, R z, R ex, R ey, R ez,")
    w("    R* __restrict__ S, R* __restrict__ X) {")
    w.push()
    for b in range(len(stages)):
        w(f"{'if' if b == 0 else 'else if'} constexpr (B == {b}) adj_stage_s{b}<R>(c, x, y, z, ex, ey, ez, S, X);")
    w.pop()
    w("}")


def _emit_whole_tangents(w: _W, prog: Program, parts, stages):
    """tan_moments<0> and adj_pair<0>: every part of the moment tangent, and every stage of the
    adjoint pair sums, over the whole layout (one range) with A_mu = sum_e (mbd_e mono_e +
    mb_e dmono_e) in place of X_mu (ebar = 0)."""
    w(f"static constexpr int NTGROUP = 1, TGROUP_LO[1] = {{0}}, TGROUP_HI[1] = {{{prog.n_mom}}};")
    w(f"static constexpr int NAGROUP = 1, AGROUP_LO[1] = {{0}}, AGROUP_HI[1] = {{{prog.n_mom}}};")
    w("template <int G, class R>")
    w("static __device__ __forceinline__ void tan_moments(R* __restrict__ md, const R* __restrict__ f, const R* __restrict__ fp,")
    w("    R x, R y, R z, R ex, R ey, R ez, R rdot) {")
    w.push()
    w("R fd[NMU];")
    w("for (int mu = 0; mu < NMU; ++mu) fd[mu] = fp[mu] * rdot;")
    for p in range(len(parts)):
        w(f"{{ R loc[TPART_MAX] = {{}}; tan_part_p{p}<R>(loc, f, fd, x, y, z, ex, ey, ez);")
        w(f"  for (int k = 0; k < TPART_SIZE[{p}]; ++k) md[TPART_ENTRY[{p}][k]] += loc[k]; }}")
    w.pop()
    w("}")
    w("template <int G, class R>")
    w("static __device__ __forceinline__ void adj_pair(const R* __restrict__ mb, const R* __restrict__ mbd, R x, R y, R z,")
    w("    R ex, R ey, R ez, R* __restrict__ S, R* __restrict__ A) {")
    w.push()
    w("R X[NMU] = {};")
    for b in range(len(stages)):
        w(f"{{ R c[ADJ_MAX]; for (int k = 0; k < ADJ_SIZE[{b}]; ++k) c[k] = ADJ_VALUE[{b}][k] ? -mbd[ADJ_ENTRY[{b}][k]] : mb[ADJ_ENTRY[{b}][k]];")
        w(f"  adj_stage_s{b}<R>(c, x, y, z, ex, ey, ez, S, X); }}")
    w("for (int mu = 0; mu < NMU; ++mu) A[mu] -= X[mu];")
    w.pop()
    w("}")


def _tref(r):
    kind, k = r
    if kind == "m":
        return f"mde{k}"
    if kind == "t":
        return f"td{k}"
    return f"Cd[{k}]"


def _emit_block_forward_tangent(w: _W, blk, with_output=True):
    for k in range(blk.n_temp):
        w(f"R t{k} = R(0), td{k} = R(0);")
    for (dst, x), lst in _group_ops(blk.ops).items():
        if dst[0] == "c" and not with_output:
            continue
        if lst[0][0] is None:
            w(f"{_ref(dst)} = {_ref(x)};")
            w(f"{_tref(dst)} = {_tref(x)};")
            continue
        _emit_inner2(w, lst)
        w(f"  {_tref(dst)} = fma({_tref(x)}, s, fma({_ref(x)}, sd, {_tref(dst)}));")
        w(f"  {_ref(dst)} = fma({_ref(x)}, s, {_ref(dst)}); }}")


def _emit_inner2(w, lst):
    """s = sum w y and sd = sum w yd over a group."""
    (y0, w0) = lst[0]
    if w0 == 1:
        w(f"{{ R s = {_ref(y0)}, sd = {_tref(y0)};")
    else:
        w(f"{{ R s = {_lit(w0)} * {_ref(y0)}, sd = {_lit(w0)} * {_tref(y0)};")
    for y, wgt in lst[1:]:
        if wgt == 1:
            w(f"  s += {_ref(y)}; sd += {_tref(y)};")
        else:
            w(f"  s = fma({_lit(wgt)}, {_ref(y)}, s); sd = fma({_lit(wgt)}, {_tref(y)}, sd);")


def _emit_components_forward_tangent(w: _W, prog: Program):
    w("template <class R, class MA>")
    w("static __device__ __forceinline__ void fwd_tan(const MA& M, const MA& Md, R* __restrict__ C, R* __restrict__ Cd) {")
    w.push()
    for blk in _locality_order(prog.blocks):
        w(f"{{  // contraction {blk.q}")
        w.push()
        for e in blk.entries:
            w(f"const R me{e} = M({e}), mde{e} = Md({e});")
        w(f"C[{blk.q}] = R(0); Cd[{blk.q}] = R(0);")
        _emit_block_forward_tangent(w, blk)
        w.pop()
        w("}")
    w.pop()
    w("}")


def _adj2(ref, slot):
    """(adjoint, adjoint tangent) names of a reference inside a reverse-tangent block; slot maps
    the moment entries accumulated by the part to their register index."""
    kind, k = ref
    if kind == "t":
        return f"tb{k}", f"tbd{k}"
    if kind == "m":
        return (None, f"mbd[{slot[k]}]") if k in slot else (None, None)
    return "cb", "cbd"


def _emit_block_reverse_tangent(w: _W, blk, slot, flush=None):
    """The block read backwards.  flush maps moment entries to the line that stores their
    accumulated adjoint tangent; each such line is emitted right after the entry's last update
    in the block, so its register is free for the rest of the block."""
    rev_ops = list(reversed(blk.ops))
    seen_dst = []
    by_dst = defaultdict(list)
    for dst, x, y, wgt in rev_ops:
        if dst not in by_dst:
            seen_dst.append(dst)
        by_dst[dst].append((x, y, wgt))
    items = []  # (lines, moment entry updated or None)
    for dst in seen_dst:
        lst = by_dst[dst]
        db, dbd = _adj2(dst, slot)
        if lst[0][1] is None:
            (x, _, _), = lst
            xb, xbd = _adj2(x, slot)
            lines = []
            if xb:
                lines.append(f"{xb} += {db};")
            if xbd:
                lines.append(f"{xbd} += {dbd};")
            items.append((lines, x[1] if x[0] == "m" and xbd else None))
            continue
        xs, ys = {}, {}
        for x, y, wgt in lst:
            xs.setdefault(x, []).append((y, wgt))
            ys.setdefault(y, []).append((x, wgt))
        for x, l2 in xs.items():
            xb, xbd = _adj2(x, slot)
            if not xb and not xbd:
                continue
            sub = _W()
            _emit_inner2(sub, l2)
            if xb:
                sub(f"  {xb} = fma({db}, s, {xb});")
            sub(f"  {xbd} = fma({dbd}, s, fma({db}, sd, {xbd})); }}")
            items.append((sub.lines, x[1] if x[0] == "m" else None))
        for y, l2 in ys.items():
            yb, ybd = _adj2(y, slot)
            if not ybd:
                continue
            sub = _W()
            _emit_inner2(sub, l2)
            sub(f"  {ybd} = fma({dbd}, s, fma({db}, sd, {ybd})); }}")
            items.append((sub.lines, y[1] if y[0] == "m" else None))
    flush = dict(flush or {})
    last = {e: i for i, (_, e) in enumerate(items) if e is not None}
    for i, (lines, e) in enumerate(items):
        for line in lines:
            w(line)
        if e is not None and last[e] == i and e in flush:
            w(flush.pop(e))
    for line in flush.values():
        w(line)


def _rtan_peak(blk):
    return 8 * blk.n_temp + 4 * len(blk.entries) + 48


def _rtan_live(order):
    """Register estimate of a part whose blocks run in the given order: an entry's accumulator
    lives from the first block of the part that touches it to the last one (where it is stored
    after its last update), next to the block's own need."""
    first, last = {}, {}
    for i, b in enumerate(order):
        for e in b.entries:
            first.setdefault(e, i)
            last[e] = i
    starts, ends = defaultdict(int), defaultdict(int)
    for e in first:
        starts[first[e]] += 1
        ends[last[e]] += 1
    live = worst = 0
    for i, b in enumerate(order):
        live += starts[i]
        worst = max(worst, 2 * live + _rtan_peak(b))
        live -= ends[i]
    return worst


def rev_tan_parts(prog: Program, budget=RTAN_REG_BUDGET):
    """Contraction blocks of the reverse-tangent program cut into parts (one kernel each).  A
    part starts from the remaining block with the largest register need and takes, while the
    estimate of the part in locality order fits the budget, the block that adds the fewest new
    moment entries (among the closest few candidates).  Returns the parts as lists of blocks
    in locality order."""
    rem = sorted(prog.blocks, key=lambda b: b.q)
    parts = []
    while rem:
        b0 = max(rem, key=lambda b: (_rtan_peak(b), len(b.ops), -b.q))
        rem.remove(b0)
        cur, es = [b0], set(b0.entries)
        while rem:
            cand = sorted(rem, key=lambda b: (len(set(b.entries) - es), -len(b.ops), b.q))[:RTAN_CANDIDATES]
            nb = next((b for b in cand if _rtan_live(_locality_order(cur + [b])) <= budget), None)
            if nb is None:
                break
            cur.append(nb)
            rem.remove(nb)
            es |= set(nb.entries)
        parts.append(_locality_order(cur))
    return parts


def _emit_components_reverse_tangent(w: _W, prog: Program, parts):
    """One function per part: the forward tangent of each of its blocks again, then the block
    read backwards, accumulating the tangents of the moment adjoints of the entries the part
    touches.  The part that touches an entry first stores it, later parts add to it, and the
    first part stores zero for entries no block reads, so running the parts in order leaves
    out[e * ld] = d(mbar_e) for every entry."""
    first = {}
    for pi, part in enumerate(parts):
        for blk in part:
            for e in blk.entries:
                first.setdefault(e, pi)
    for pi, part in enumerate(parts):
        entries = sorted(set(e for b in part for e in b.entries))
        slot = {e: k for k, e in enumerate(entries)}
        w("template <class R, class MA, class CB, class OUT>")
        w(f"static __device__ __forceinline__ void rev_tan_p{pi}(const MA& M, const MA& Md, const CB& Cb,")
        w("    const CB& Cbd, const OUT& out, long ld) {")
        w.push()
        last = {}
        for bi, blk in enumerate(part):
            for e in blk.entries:
                last[e] = bi
        started = set()
        w(f"R mbd[{len(entries)}];")
        # every load of the program in order (moments, their tangents, then the block's adjoint
        # pair), kept TAN_PREFETCH_DEPTH ahead across the fenced blocks
        seq = []
        for blk in part:
            seq += [(f"me{e}", f"M({e})") for e in blk.entries] + [(f"mde{e}", f"Md({e})") for e in blk.entries]
            seq += [("cb", f"Cb[{blk.q}]"), ("cbd", f"Cbd[{blk.q}]")]
        depth = max(1, min(TAN_PREFETCH_DEPTH, len(seq)))
        for k in range(depth):
            w(f"R pf{k} = {seq[k][1]};")
        pos = 0
        for bi, blk in enumerate(part):
            w(f"{{  // contraction {blk.q}")
            w.push()
            w("MTP_BLOCK_FENCE();")
            for _ in range(2 * len(blk.entries) + 2):
                sl = pos % depth
                w(f"const R {seq[pos][0]} = pf{sl};")
                if pos + depth < len(seq):
                    w(f"pf{sl} = {seq[pos + depth][1]};")
                pos += 1
            for e in blk.entries:
                if e not in started:
                    started.add(e)
                    w(f"mbd[{slot[e]}] = R(0);")
            _emit_block_forward_tangent(w, blk, with_output=False)
            for k in range(blk.n_temp):
                w(f"R tb{k} = R(0), tbd{k} = R(0);")
            # entries the part touches for the last time here are stored after their last update
            flush = {e: f"out[{e} * ld] {'=' if first[e] == pi else '+='} double(mbd[{slot[e]}]);"
                     for e in blk.entries if last[e] == bi}
            _emit_block_reverse_tangent(w, blk, slot, flush)
            w.pop()
            w("}")
        if pi == 0:
            for e in range(prog.n_mom):
                if e not in first:
                    w(f"out[{e} * ld] = 0.0;")
        w.pop()
        w("}")


def _emit_products_tangent(w: _W, prog: Program):
    children = defaultdict(list)
    roots = []
    for a, (parent, comp) in enumerate(prog.trie):
        if parent < 0:
            roots.append(a)
        else:
            children[parent].append(a)
    w("// Basis values and tangents; writes out[alpha * ld] = ebar B_alpha - dB_alpha, and the")
    w("// adjoints Cb_q = dE_i/dC_q with their tangents Cbd_q.")
    w("template <class R>")
    w("static __device__ __forceinline__ void products_tan(const R* __restrict__ C, const R* __restrict__ Cd,")
    w("    const double* __restrict__ xi, double ebar, R* __restrict__ Cb, R* __restrict__ Cbd,")
    w("    double* __restrict__ out, long ld) {")
    w.push()
    for q in range(prog.n_comp):
        w(f"Cb[{q}] = R(0); Cbd[{q}] = R(0);")

    def node(a, pv, pdv):
        parent, comp = prog.trie[a]
        w(f"R bb{a}, bbd{a};")
        w("{")
        w.push()
        if pv is None:
            w(f"const R b = C[{comp}], bd = Cd[{comp}];")
        else:
            w(f"const R b = {pv} * C[{comp}];")
            w(f"const R bd = fma({pdv}, C[{comp}], {pv} * Cd[{comp}]);")
        w(f"out[{a} * ld] = fma(ebar, double(b), -double(bd));")
        w(f"bb{a} = R(xi[{a}]); bbd{a} = R(0);")
        if children[a]:
            w(f"const R p{a} = b, pd{a} = bd;")
            for ch in children[a]:
                node(ch, f"p{a}", f"pd{a}")
                _, cc = prog.trie[ch]
                w(f"bbd{a} = fma(bbd{ch}, C[{cc}], fma(bb{ch}, Cd[{cc}], bbd{a}));")
                w(f"bb{a} = fma(bb{ch}, C[{cc}], bb{a});")
        w.pop()
        w("}")
        if pv is None:
            w(f"Cb[{comp}] += bb{a}; Cbd[{comp}] += bbd{a};")
        else:
            w(f"Cbd[{comp}] = fma(bbd{a}, {pv}, fma(bb{a}, {pdv}, Cbd[{comp}]));")
            w(f"Cb[{comp}] = fma(bb{a}, {pv}, Cb[{comp}]);")

    for a in roots:
        node(a, None, None)
    w.pop()
    w("}")


def _emit_tangent_dispatchers(w: _W, n_rtparts: int):
    w("template <int G, class R, class MA, class CB, class OUT>")
    w("static __device__ __forceinline__ void rev_tan(const MA& M, const MA& Md, const CB& Cb, const CB& Cbd, const OUT& out, long ld) {")
    w.push()
    for g in range(n_rtparts):
        w(f"{'if' if g == 0 else 'else if'} constexpr (G == {g}) rev_tan_p{g}<R, MA, CB>(M, Md, Cb, Cbd, out, ld);")
    w.pop()
    w("}")


def emit_tangent_parts(w: _W, prog: Program, rparts):
    stages = adj_stages(prog)
    parts = moment_parts(prog, TANGENT_PART_CAP)
    _emit_tangent_moment_parts(w, prog, parts)
    _emit_adj_stages(w, prog, stages)
    _emit_whole_tangents(w, prog, parts, stages)
    _emit_components_forward_tangent(w, prog)
    _emit_components_reverse_tangent(w, prog, rparts)
    _emit_products_tangent(w, prog)
    _emit_tangent_dispatchers(w, len(rparts))
