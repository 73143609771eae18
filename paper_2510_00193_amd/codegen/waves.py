"""Device code of the contraction program for several waves per tile of 64 atoms.

A workgroup keeps the moments its waves share in LDS ([row][atom]) and each wave runs its own part of
the contraction blocks, the same atoms in its lanes:

  fwd_wave<w>      contractions; energies (and basis values) of those that only meet powers of C_0
  core_wave<w>     products of the remaining ("general") contractions and the adjoints of those
  rev_wave<w>      the blocks backwards, moment adjoints accumulated per wave
  rev_combine<w>   sums of the entries that several waves touch, in wave order
  tfwd_wave<w>, tcore_wave<w>, trev_wave<w>, trev_combine<w>   the same for the tangents

C_0 = M_(0,0) is the only contraction of level 2 and every other has level 6 at least, so a basis
function is a core (a multiset of contractions other than C_0) times a power of C_0: with
P_core(C_0) = sum_j xi_(core, j) C_0^j the energy is sum_core B_core P_core, the adjoint of a
contraction q that only occurs alone is P_q (uniform coefficients, formed where it is needed), and
only the general contractions (level <= L - 6) need their values and adjoints passed between waves.
"""
from __future__ import annotations

from collections import Counter, defaultdict

from .program import Block, Program


# Blocks with more inner sums than this form them twice (see _pin), in the tangents and where a wave
# holds more accumulators than PIN_SHARED: without it the reverse of level 20 spills 332 bytes, its
# tangent that of level 16 532 (324 with it); where nothing spills the sums are kept (8 % fewer
# operations at level 16).
PIN_GROUPS, PIN_SHARED = 16, 64
PIECE = 12
AHEAD = 24  # values from memory held for the next block
LDS_ROWS = 318  # rows of 64 doubles in the 160 KB of a compute unit, less the static variables

# Waves per tile by level: forward, reverse, forward tangent, reverse tangent.  From level 18 on four waves
# of 512 registers hold the accumulators of the reverse programs (no spills; eight of 256 would spill).
# Up to level 10 one lane runs the whole program, which holds all of it in registers: two waves gave
# 0.5 % less at 250,000 atoms, 1 % more in a fit of 2048 configurations and 4 % less in a coefficient
# gradient of 50,000 atoms.  Both programs (for grades the forward alone), one lane -> waves, us:
#   level 12:   9,000 atoms 7.3 -> 7.2, 20,000 8.0 -> 8.2, 51,000 11.5 -> 11.9, 119,000 21.8 -> 21.9,
#               250,000 44.5 -> 36.7 (forward 6.4 -> 6.3, 6.8 -> 6.7, 10.7 -> 10.9, 16.0 -> 16.7, 34.8 -> 29.3);
#               a minibatch of 64 configurations as a whole 340 -> 344, a fit of 2048 1729 -> 1692: even up to
#               100,000 atoms, and kept for what is larger
#   level 14:   9,000 atoms 12.5 -> 9.4, 63,000 23.1 -> 22.0, 250,000 86.8 -> 70.3 (forward 62.9 -> 60.2)
#   level 16:   1008 atoms 20 -> 12.9, 1,024,000 742 -> 588
#   level 18:   1024 atoms 70 -> 30, 250,000 625 -> 550 (forward 190 -> 149)
#   level 20:   31,416 atoms 385 -> 130
WAVES = {12: (2, 2, 2, 2), 14: (4, 4, 4, 4), 16: (4, 4, 4, 4), 18: (8, 4, 8, 4), 20: (8, 4, 8, 4)}


def _operations(blk, which):
    """Binary64 operations of a block (entries count as one each), which as in WAVES."""
    from .emit import (_W, _emit_block_forward, _emit_block_forward_tangent, _emit_block_reverse,
                       _emit_block_reverse_tangent)
    w = _W()
    (_emit_block_forward_tangent if which > 1 else _emit_block_forward)(w, blk, with_output=which % 2 == 0)
    if which == 1:
        _emit_block_reverse(w, blk, lambda r: f"{r[0]}b{r[1]}")
    elif which == 3:
        _emit_block_reverse_tangent(w, blk, {e: e for e in blk.entries})
    text = "\n".join(w.lines)
    return text.count("fma(") + text.count("+=") + text.count(" * ") + len(blk.entries)


class Layout:
    """Cores, general contractions, shared rows and the parts of the waves of one level."""

    def __init__(self, prog: Program, waves):
        self.prog = prog
        self.waves = waves
        lev = [sum(2 + 4 * mu + nu for mu, nu in g.labels) for g in prog.basis.components]
        self.q0 = lev.index(2)
        assert lev.count(2) == 1 and min(v for q, v in enumerate(lev) if q != self.q0) >= 6
        self.general = [q for q in range(prog.n_comp) if q == self.q0 or lev[q] <= prog.level - 6]
        self.ahead = set()  # coefficients of the current block that are in registers
        self.grow = {q: g for g, q in enumerate(self.general)}
        # basis functions by core: alpha[core][j]
        self.alpha = defaultdict(dict)
        for a in range(prog.n_alpha):
            path, k = [], a
            while k >= 0:
                k, comp = prog.trie[k]
                path.append(comp)
            core = tuple(sorted(q for q in path if q != self.q0))
            self.alpha[core][path.count(self.q0)] = a
        for core, js in self.alpha.items():
            assert sorted(js) == list(range(0 if core else 1, len(js) + (0 if core else 1)))
        self.cores = sorted(c for c in self.alpha if len(c) > 1)
        assert all(q in self.grow for c in self.cores for q in c)
        use = Counter(e for b in prog.blocks for e in b.entries)
        order = sorted((e for e in range(prog.n_mom) if use[e] > 1), key=lambda e: (-use[e], e))
        self.hot = order  # most used first: the first 128 rows are in reach of an instruction's offset
        # all the moments where two workgroups still share a compute unit (a moment of one block would be
        # read by the forward and by the reverse program, each time with the wave waiting)
        if prog.n_mom + 2 * len(self.general) + 2 * max(waves) <= LDS_ROWS // 2:
            self.hot = list(range(prog.n_mom))
        assert len(self.hot) + 2 * len(self.general) + 2 * max(waves) <= LDS_ROWS
        # the tangents hold two rows per entry; two workgroups share a compute unit if that leaves out
        # a tenth of the entries at most (level 16)
        room, half = ((rows - 2 * len(self.general) - waves[2]) // 2 for rows in (LDS_ROWS, LDS_ROWS // 2))
        room = half if half >= 0.9 * len(order) else room
        self.thot = order[:room]
        (self.e0,) = prog.blocks[self.q0].entries
        self.parts = [self._cut(w, k) for k, w in enumerate(waves)]

    def _cut(self, n, which):
        """Blocks for n waves: largest first, each to the wave (below 1.1 of the mean load) that
        already touches most of its entries.  The load is the number of operations emitted."""
        ops = {b.q: _operations(b, which) for b in self.prog.blocks}
        cost = lambda b: ops[b.q]  # noqa: E731
        blocks = sorted(self.prog.blocks, key=lambda b: (-cost(b), b.q))
        cap = 1.1 * sum(map(cost, blocks)) / n
        bins, load, ents = [[] for _ in range(n)], [0] * n, [set() for _ in range(n)]
        for b in blocks:
            es = set(b.entries)
            fit = [w for w in range(n) if load[w] + cost(b) <= cap] or [min(range(n), key=lambda w: load[w])]
            w = max(fit, key=lambda w: (len(es & ents[w]) - len(es - ents[w]) if ents[w] else -0.5 * len(es), -load[w]))
            bins[w].append(b)
            load[w] += cost(b)
            ents[w] |= es
        return bins

    def powers(self):
        return max(max(js) for js in self.alpha.values())


def _poly(w, name, coefs, var="c0"):
    """name = sum_j coefs[j] var^j (Horner; coefs: expressions)."""
    w(f"double {name} = {coefs[-1]};")
    for c in reversed(coefs[:-1]):
        w(f"{name} = fma({name}, {var}, {c});")


def _xi(lay, core):
    js = lay.alpha[core]
    name = lambda a: f"x{a}" if a in lay.ahead else f"xi[{a}]"  # noqa: E731
    return [name(js[j]) if j in js else "0.0" for j in range(max(js) + 1)]


def _derivative(coefs):
    """Coefficients of the derivative of a polynomial given by expressions."""
    return [c if j == 1 else f"{j}.0 * {c}" for j, c in enumerate(coefs)][1:]


def _sub(w, lines, repl):
    for line in lines:
        for a, b in repl:
            line = line.replace(a, b)
        w(line)


def _blocks(w, lay, part, hot, tangent, body, ahead=lambda blk: None):
    """The blocks of a part, fenced; what is not in LDS (entries, the coefficients of the contraction
    alone, what ahead loads) is loaded one block ahead.  Of the entries only the first AHEAD values: the
    contractions of two moments of high rank read up to 67 from memory, and held ahead of their block they
    spilled the registers of the block before it."""
    first = lambda blk: [e for e in blk.entries if e not in hot][:AHEAD // (1 + tangent)]  # noqa: E731
    for k in range(len(part) + 1):
        if k < len(part):
            for e in first(part[k]):
                g = f"g{k}_"
                w(f"const double {g}{e} = M({e});" + (f" const double {g}d{e} = Md({e});" if tangent else ""))
            if all(b.q != part[k].q for b in part[:k]):
                ahead(part[k])
                for a in lay.alpha[(part[k].q,)].values():
                    w(f"const double x{a} = xi[{a}];")
        if k == 0:
            continue
        blk = part[k - 1]
        w("MTP_TILE_FENCE();")
        w(f"{{  // contraction {blk.q}")
        w.push()
        if lay.e0 in hot:  # again, rather than kept through the blocks
            w(f"const double c0 = M({lay.e0});" + (f" const double c0d = Md({lay.e0});" if tangent else ""))
        loaded = first(blk)
        for e in blk.entries:
            if e not in loaded:
                w(f"double me{e} = M({e});" + (f" double mde{e} = Md({e});" if tangent else ""))
            else:
                w(f"double me{e} = g{k - 1}_{e};" + (f" double mde{e} = g{k - 1}_d{e};" if tangent else ""))
        lay.ahead = set(lay.alpha[(blk.q,)].values())
        body(k - 1, blk)
        lay.ahead = set()
        w.pop()
        w("}")


def _order(lay, part):
    from .emit import _locality_order
    return _locality_order([b for b in part if b.q != lay.q0])


def _basis_out(w, lay, core, b):
    """Stores of the basis values b C_0^j of a core (WB)."""
    js = lay.alpha[core]
    w("if constexpr (WB) {")
    w.push()
    w(f"double p = {b};")
    for j in sorted(js):
        if j > min(js):
            w("p *= c0;")
        w(f"Bo[{js[j]} * ldb] = p;")
    w.pop()
    w("}")


def _core_terms(w, lay, core, b):
    """Energy and C_0-adjoint of a core with value b."""
    coefs = _xi(lay, core)
    _poly(w, "P", coefs)
    w(f"e = fma({b}, P, e);")
    if len(coefs) > 1:
        _poly(w, "dP", _derivative(coefs))
        w(f"c0b = fma({b}, dP, c0b);")


def _forward(w, lay):
    from .emit import _W, _emit_block_forward
    for wi, part in enumerate(lay.parts[0]):
        w("template <bool WB, class MA>")
        w(f"static __device__ __forceinline__ void fwd_wave{wi}(const MA& M, const double* __restrict__ xi, double* __restrict__ crow,")
        w("    double* __restrict__ Bo, long ldb, double& e, double& c0b) {")
        w.push()
        w(f"const double c0 = M({lay.e0});")

        def body(_, blk):
            sub = _W()
            _emit_block_forward(sub, blk)
            w("double cq = 0.0;")
            _sub(w, sub.lines, [(f"C[{blk.q}]", "cq"), ("R ", "double "), ("R(", "double(")])
            core = (blk.q,)
            _basis_out(w, lay, core, "cq")
            _core_terms(w, lay, core, "cq")
            if blk.q in lay.grow:
                w(f"crow[{lay.grow[blk.q]} * 64] = cq;")
            w("MTP_PIN(e); MTP_PIN(c0b);")

        _blocks(w, lay, _order(lay, part), set(lay.hot), False, body)
        if any(b.q == lay.q0 for b in part):
            w("{  // powers of C_0 alone")
            w.push()
            _basis_out(w, lay, (), "c0")
            coefs = _xi(lay, ())
            _poly(w, "P", coefs)
            _poly(w, "dP", _derivative(coefs))
            w("e += P;")
            w("c0b += dP;")
            w.pop()
            w("}")
        w.pop()
        w("}")


def _members(core, q):
    """(multiplicity of q, rest of the core without one q)."""
    rest = list(core)
    rest.remove(q)
    return core.count(q), rest


def _spread(lay, n):
    """Cores and general contractions (other than C_0) for n waves, by their number of terms."""
    tasks = [(2 + len(c), ("core", c)) for c in lay.cores]
    for q in lay.general:
        if q != lay.q0:
            tasks.append((2 + 4 * sum(q in c for c in lay.cores), ("adj", q)))
    bins, load = [[] for _ in range(n)], [0] * n
    for cost, t in sorted(tasks, key=lambda t: (-t[0], t[1])):
        w = load.index(min(load))
        bins[w].append(t)
        load[w] += cost
    return [sorted(b) for b in bins]


def _cores(w, lay):
    for wi, tasks in enumerate(_spread(lay, lay.waves[0])):
        w("template <bool WB, class MA, class CB>")
        w(f"static __device__ __forceinline__ void core_wave{wi}(const MA& M, const double* __restrict__ xi, const double* __restrict__ crow,")
        w("    const CB& cb, double* __restrict__ Bo, long ldb, double& e, double& c0b) {")
        w.push()
        w(f"const double c0 = M({lay.e0});")
        for kind, t in tasks:
            w("{")
            w.push()
            if kind == "core":
                w("const double b = " + " * ".join(f"crow[{lay.grow[q]} * 64]" for q in t) + ";")
                _basis_out(w, lay, t, "b")
                _core_terms(w, lay, t, "b")
            else:
                _poly(w, "s", _xi(lay, (t,)))
                for core in lay.cores:
                    if t in core:
                        k, rest = _members(core, t)
                        w("{")
                        w.push()
                        _poly(w, "P", _xi(lay, core))
                        b = " * ".join(f"crow[{lay.grow[q]} * 64]" for q in rest)
                        w(f"s = fma({'' if k == 1 else f'{k}.0 * '}{b}, P, s);")
                        w.pop()
                        w("}")
                w(f"cb({lay.grow[t]}, s);")
            w.pop()
            w("}")
        w.pop()
        w("}")


def _pieces(blk):
    """A contraction without temporaries in pieces of PIECE entries or a little more (its terms are
    independent, and the reverse of all 28 of two moments of rank 6 held 56 entries at a time)."""
    if blk.n_temp or len(blk.entries) <= 2 * PIECE:
        return [blk]
    out, ops = [], []
    for op in blk.ops:
        ops.append(op)
        ents = sorted({k for o in ops for r in o[1:3] if r is not None for kind, k in [r] if kind == "m"})
        if len(ents) >= PIECE:
            out.append(Block(blk.q, 0, ops, ents))
            ops = []
    if ops:
        out.append(Block(blk.q, 0, ops, sorted({k for o in ops for r in o[1:3] if r is not None for kind, k in [r] if kind == "m"})))
    return out


def _pin(w, blk, tangent, shared):
    """Between the forward and the reverse of a block: the inner sums of the forward come up again in the
    reverse, and the compiler would keep them all (a spill each in the larger blocks) instead of adding
    them again from the entries."""
    from .emit import _group_ops
    if len(_group_ops(blk.ops)) <= PIN_GROUPS or not (tangent or shared > PIN_SHARED):
        return
    for e in blk.entries:
        w(f"MTP_PIN(me{e});" + (f" MTP_PIN(mde{e});" if tangent else ""))


def _touch(lay, parts):
    """Waves that touch each entry (wave order)."""
    touch = defaultdict(list)
    for wi, part in enumerate(parts):
        for e in sorted({e for b in part for e in b.entries}):
            touch[e].append(wi)
    return touch


def _combine(w, name, lay, touch, n, shared):
    rows = {e: k for k, e in enumerate(e for e in sorted(touch) if len(touch[e]) > 1)}
    assert len(rows) <= LDS_ROWS
    for wi in range(n):
        w("template <class OUT>")
        w(f"static __device__ __forceinline__ void {name}{wi}(const double* __restrict__ mbs, double* __restrict__ sh, const OUT& out) {{")
        w.push()
        for k, e in enumerate(shared[wi]):
            ws = touch[e]
            if wi == ws[0]:
                w(f"sh[{rows[e]} * 64] = mbs[{k}];")
            elif wi == ws[-1]:
                w(f"out({e}, sh[{rows[e]} * 64] + mbs[{k}]);")
            else:
                w(f"sh[{rows[e]} * 64] += mbs[{k}];")
        w.pop()
        w("}")
    return rows


def _reverse(w, lay, tangent):
    from .emit import (_W, _emit_block_forward, _emit_block_forward_tangent, _emit_block_reverse,
                       _emit_block_reverse_tangent)
    n = lay.waves[3 if tangent else 1]
    parts = lay.parts[3 if tangent else 1]
    hot = set(lay.thot if tangent else lay.hot)
    touch = _touch(lay, parts)
    shared = [[e for e in sorted(touch) if len(touch[e]) > 1 and wi in touch[e]] for wi in range(n)]
    pre = "t" if tangent else ""
    w(f"static constexpr int {pre.upper()}SHARED[{n}] = {{{', '.join(str(len(s)) for s in shared)}}};")
    for wi, part in enumerate(parts):
        args = "const MA& M, const MA& Md, const CB& cb, const CB& cbd" if tangent else "const MA& M, const CB& cb"
        w("template <class MA, class CB, class OUT>")
        w(f"static __device__ __forceinline__ void {pre}rev_wave{wi}({args}, const double* __restrict__ xi,")
        w("    double* __restrict__ mbs, const OUT& out) {")
        w.push()
        order = [piece for b in _order(lay, part) for piece in _pieces(b)]
        last = {e: k for k, b in enumerate(order) for e in b.entries}
        slot = {e: k for k, e in enumerate(shared[wi])}
        started = set()
        w(f"const double c0 = M({lay.e0});")
        if tangent:
            w(f"const double c0d = Md({lay.e0});")

        def ahead(blk):  # adjoint of a general contraction
            if blk.q in lay.grow:
                g = lay.grow[blk.q]
                w(f"const double cbg{blk.q} = cb({g});" + (f" const double cbdg{blk.q} = cbd({g});" if tangent else ""))

        acc = "bd" if tangent else "b"
        for e in sorted({e for b in order for e in b.entries}):
            w(f"double m{acc}{e};")

        def body(k, blk):
            if blk.q in lay.grow:
                w(f"const double cb = cbg{blk.q};" + (f" const double cbd = cbdg{blk.q};" if tangent else ""))
            else:
                coefs = _xi(lay, (blk.q,))
                _poly(w, "cb", coefs)
                if tangent:
                    if len(coefs) > 1:
                        _poly(w, "dP", _derivative(coefs))
                        w("const double cbd = dP * c0d;")
                    else:
                        w("const double cbd = 0.0;")
            for e in blk.entries:
                if e not in started:
                    started.add(e)
                    w(f"m{acc}{e} = 0.0;")
            sub = _W()
            if tangent:
                _emit_block_forward_tangent(sub, blk, with_output=False)
                _pin(sub, blk, True, max(map(len, shared)))
                for t in range(blk.n_temp):
                    sub(f"R tb{t} = R(0), tbd{t} = R(0);")
                _emit_block_reverse_tangent(sub, blk, {e: e for e in blk.entries})
                repl = [(f"mbd[{e}]", f"mbd{e}") for e in blk.entries]
            else:
                _emit_block_forward(sub, blk, with_output=False)
                _pin(sub, blk, False, max(map(len, shared)))
                for t in range(blk.n_temp):
                    sub(f"R tb{t} = R(0);")
                _emit_block_reverse(sub, blk, lambda r: {"t": f"tb{r[1]}", "m": f"mb{r[1]}", "c": "cb"}[r[0]])
                repl = []
            _sub(w, sub.lines, repl + [("R ", "double "), ("R(", "double(")])
            for e in blk.entries:
                if last[e] == k and e not in slot and e != lay.e0:
                    w(f"out({e}, m{acc}{e});")
                else:  # the block's arithmetic is done here, not where the sum is used at last
                    w(f"MTP_PIN(m{acc}{e});")

        _blocks(w, lay, order, hot, tangent, body, ahead)
        owner = any(b.q == lay.q0 for b in part)
        if owner:  # the adjoint of C_0 itself
            src = "cbd" if tangent else "cb"
            if lay.e0 in started:
                w(f"m{acc}{lay.e0} += {src}({lay.grow[lay.q0]});")
            else:
                w(f"double m{acc}{lay.e0} = {src}({lay.grow[lay.q0]});")
        if lay.e0 not in slot and (owner or lay.e0 in started):
            w(f"out({lay.e0}, m{acc}{lay.e0});")
        for e, k in slot.items():
            w(f"mbs[{k}] = m{acc}{e};")
        if wi == 0:
            for e in range(lay.prog.n_mom):
                if e not in touch:
                    w(f"out({e}, 0.0);")
        w.pop()
        w("}")
    _combine(w, f"{pre}rev_combine", lay, touch, n, shared)


def _forward_tangent(w, lay):
    from .emit import _W, _emit_block_forward_tangent
    n = lay.waves[2]

    def out_terms(core, b, bd):
        """out_alpha = ebar B - dB for the powers of C_0, and the tangent of the C_0-adjoint."""
        js = lay.alpha[core]
        w("{")
        w.push()
        w(f"double p = {b}, pd = {bd};")
        for j in sorted(js):
            if j > min(js):
                w("pd = fma(pd, c0, p * c0d);")
                w("p *= c0;")
            w(f"out[{js[j]} * ld] = fma(ebar, p, -pd);")
        w.pop()
        w("}")
        coefs = _xi(lay, core)
        if len(coefs) > 1:
            d1 = _derivative(coefs)
            w("{")
            w.push()
            _poly(w, "dP", d1)
            if core:
                w(f"c0bd = fma({bd}, dP, c0bd);")
            if len(coefs) > 2:
                d2 = [f"{j * (j - 1)}.0 * {c}" for j, c in enumerate(coefs)][2:]
                _poly(w, "ddP", d2)
                w(f"c0bd = fma({b + ' * ' if core else ''}c0d, ddP, c0bd);")
            w.pop()
            w("}")

    for wi, part in enumerate(lay.parts[2]):
        w("template <class MA, class OUT>")
        w(f"static __device__ __forceinline__ void tfwd_wave{wi}(const MA& M, const MA& Md, const double* __restrict__ xi, double ebar,")
        w("    double* __restrict__ crow, double* __restrict__ cdrow, const OUT& out, long ld, double& c0bd) {")
        w.push()
        w(f"const double c0 = M({lay.e0}), c0d = Md({lay.e0});")

        def body(_, blk):
            sub = _W()
            _emit_block_forward_tangent(sub, blk)
            w("double cq = 0.0, cqd = 0.0;")
            _sub(w, sub.lines, [(f"Cd[{blk.q}]", "cqd"), (f"C[{blk.q}]", "cq"), ("R ", "double "), ("R(", "double(")])
            out_terms((blk.q,), "cq", "cqd")
            if blk.q in lay.grow:
                w(f"crow[{lay.grow[blk.q]} * 64] = cq; cdrow[{lay.grow[blk.q]} * 64] = cqd;")
            w("MTP_PIN(c0bd);")

        _blocks(w, lay, _order(lay, part), set(lay.thot), True, body)
        if any(b.q == lay.q0 for b in part):
            out_terms((), "c0", "c0d")
        w.pop()
        w("}")
    for wi, tasks in enumerate(_spread(lay, n)):
        w("template <class MA, class CB, class OUT>")
        w(f"static __device__ __forceinline__ void tcore_wave{wi}(const MA& M, const MA& Md, const double* __restrict__ xi, double ebar,")
        w("    const double* __restrict__ crow, const double* __restrict__ cdrow, const CB& cbd, const OUT& out, long ld, double& c0bd) {")
        w.push()
        w(f"const double c0 = M({lay.e0}), c0d = Md({lay.e0});")

        def product(qs):
            """b and bd of a product of general contractions."""
            r = [f"crow[{lay.grow[q]} * 64]" for q in qs]
            d = [f"cdrow[{lay.grow[q]} * 64]" for q in qs]
            w(f"double b = {r[0]}, bd = {d[0]};")
            for x, xd in zip(r[1:], d[1:]):
                w(f"bd = fma(bd, {x}, b * {xd});")
                w(f"b *= {x};")

        for kind, t in tasks:
            w("{")
            w.push()
            if kind == "core":
                product(t)
                out_terms(t, "b", "bd")
            else:
                coefs = _xi(lay, (t,))
                w("double s = 0.0;")
                if len(coefs) > 1:
                    _poly(w, "dP", _derivative(coefs))
                    w("s = dP * c0d;")
                for core in lay.cores:
                    if t in core:
                        k, rest = _members(core, t)
                        w("{")
                        w.push()
                        coefs = _xi(lay, core)
                        product(rest)
                        _poly(w, "P", coefs)
                        m = "" if k == 1 else f"{k}.0 * "
                        w(f"s = fma({m}bd, P, s);")
                        if len(coefs) > 1:
                            _poly(w, "dP", _derivative(coefs))
                            w(f"s = fma({m}b * c0d, dP, s);")
                        w.pop()
                        w("}")
                w(f"cbd({lay.grow[t]}, s);")
            w.pop()
            w("}")
        w.pop()
        w("}")


def _dispatch(w, name, n, tparams, params, targs, args):
    w(f"template <int W, {tparams}>")
    w(f"static __device__ __forceinline__ void {name}({params}) {{")
    w.push()
    for k in range(n):
        w(f"{'if' if k == 0 else 'else if'} constexpr (W == {k}) {name}{k}<{targs}>({args});")
    w.pop()
    w("}")


def emit_waves(w, prog: Program):
    waves = WAVES.get(prog.level)
    w(f"static constexpr bool WAVES = {'true' if waves else 'false'};")
    if not waves:
        w("static constexpr int NFWAVE = 1, NRWAVE = 1, NTFWAVE = 1, NTRWAVE = 1;")
        return
    lay = Layout(prog, waves)
    w(f"static constexpr int NFWAVE = {waves[0]}, NRWAVE = {waves[1]}, NTFWAVE = {waves[2]}, NTRWAVE = {waves[3]};")
    w(f"static constexpr int NGEN = {len(lay.general)}, GEN0 = {lay.grow[lay.q0]};")
    for name, rows in (("HOT", lay.hot), ("THOT", lay.thot)):
        at = {e: k for k, e in enumerate(rows)}
        w(f"static constexpr int N{name} = {len(rows)};")
        w(f"static constexpr int {name}_ENTRY[N{name}] = {{{', '.join(map(str, rows))}}};")
        w(f"static constexpr int {name}_ROW[NMOM] = {{{', '.join(str(at.get(e, -1)) for e in range(prog.n_mom))}}};")
    for k in range(2):
        t = _touch(lay, lay.parts[1 + 2 * k])
        w(f"static constexpr int {'T' if k else ''}SHARED_ROWS = {sum(len(v) > 1 for v in t.values())};")
    _forward(w, lay)
    _cores(w, lay)
    _reverse(w, lay, False)
    _forward_tangent(w, lay)
    _reverse(w, lay, True)
    _dispatch(w, "fwd_wave", waves[0], "bool WB, class MA",
              "const MA& M, const double* __restrict__ xi, double* __restrict__ crow, double* __restrict__ Bo, long ldb, double& e, double& c0b",
              "WB, MA", "M, xi, crow, Bo, ldb, e, c0b")
    _dispatch(w, "core_wave", waves[0], "bool WB, class MA, class CB",
              "const MA& M, const double* __restrict__ xi, const double* __restrict__ crow, const CB& cb, double* __restrict__ Bo, long ldb, double& e, double& c0b",
              "WB, MA, CB", "M, xi, crow, cb, Bo, ldb, e, c0b")
    _dispatch(w, "rev_wave", waves[1], "class MA, class CB, class OUT",
              "const MA& M, const CB& cb, const double* __restrict__ xi, double* __restrict__ mbs, const OUT& out",
              "MA, CB, OUT", "M, cb, xi, mbs, out")
    _dispatch(w, "tfwd_wave", waves[2], "class MA, class OUT",
              "const MA& M, const MA& Md, const double* __restrict__ xi, double ebar, double* __restrict__ crow, double* __restrict__ cdrow, const OUT& out, long ld, double& c0bd",
              "MA, OUT", "M, Md, xi, ebar, crow, cdrow, out, ld, c0bd")
    _dispatch(w, "tcore_wave", waves[2], "class MA, class CB, class OUT",
              "const MA& M, const MA& Md, const double* __restrict__ xi, double ebar, const double* __restrict__ crow, const double* __restrict__ cdrow, const CB& cbd, const OUT& out, long ld, double& c0bd",
              "MA, CB, OUT", "M, Md, xi, ebar, crow, cdrow, cbd, out, ld, c0bd")
    _dispatch(w, "trev_wave", waves[3], "class MA, class CB, class OUT",
              "const MA& M, const MA& Md, const CB& cb, const CB& cbd, const double* __restrict__ xi, double* __restrict__ mbs, const OUT& out",
              "MA, CB, OUT", "M, Md, cb, cbd, xi, mbs, out")
    for pre, n in (("", waves[1]), ("t", waves[3])):
        _dispatch(w, f"{pre}rev_combine", n, "class OUT",
                  "const double* __restrict__ mbs, double* __restrict__ sh, const OUT& out", "OUT", "mbs, sh, out")
