"""Pair records of the coefficient gradient: a chunk of atoms bounds them like the other workspace, the
result does not depend on how the pairs are cut, and a captured call with several chunks replays."""
import numpy as np
import pytest
import torch

from helpers import rel_err, small_lattice

pytestmark = pytest.mark.gpu


def _inputs(seed, reps, level, nsp):
    s, p = small_lattice(seed, reps, 3.16, 0.1, level, nsp)
    rng = np.random.default_rng(seed + 1)
    up = lambda x: torch.as_tensor(x, device="cuda")  # noqa: E731
    return s, p, up(s.pos), up(s.species), up(rng.normal(size=(s.n_atoms, 3)))


def test_chunks_bound_the_records():
    from paper_2510_00193_amd import Potential
    s, p, pos, sp, fbar = _inputs(1300, (36, 36, 36), 10, 2)  # 93,312 atoms, 2.5 million pairs of 64 bytes
    pot = Potential.from_params(p, chunk_atoms=4096)
    nl = pot.neighbors(pos, sp, s.cell)
    assert nl.n_pairs > 2.4e6
    print(f"[records] N={s.n_atoms} pairs {nl.n_pairs}", flush=True)
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    a = pot.param_grad(pos, sp, s.cell, 0.3, fbar, nlist=nl)
    torch.cuda.synchronize()
    used = before - torch.cuda.mem_get_info()[0]
    # 4096 atoms: 111,000 records of 64 bytes (7 MB) and 1 KB per atom; every buffer may take whole 2 MB pages
    assert used < 64 << 20, used
    b = Potential.from_params(p).param_grad(pos, sp, s.cell, 0.3, fbar, nlist=nl)
    torch.cuda.synchronize()
    for name, x, y in zip(("d_linear", "d_radial", "d_shift"), a, b):
        # sums of 93,312 atoms in another grouping: sqrt(n) 2^-53 of the sum of magnitudes
        assert rel_err(x.cpu().numpy(), y.cpu().numpy()) < 1e-11, name


@pytest.mark.parametrize("level,nsp,lanes", [(10, 2, 1), (16, 3, 1), (16, 2, 4), (20, 1, 8)])
def test_captured_gradient_in_chunks_replays(level, nsp, lanes):
    """Under capture the offsets of the chunks are not read: every chunk goes through windows of pairs."""
    from paper_2510_00193_amd import Potential
    s, p, pos, sp, fbar = _inputs(1310 + level, (4, 3, 5), level, nsp)
    pot = Potential.from_params(p, chunk_atoms=23, lanes_per_atom=lanes)
    nl = pot.neighbors(pos, sp, s.cell)
    print(f"[records capture L{level}] N={s.n_atoms} lanes {lanes}", flush=True)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        pot.param_grad(pos, sp, s.cell, 0.7, fbar, nlist=nl)  # reserves the workspace
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        got = pot.param_grad(pos, sp, s.cell, 0.7, fbar, nlist=nl)
    other = Potential.from_params(p)
    base = fbar.clone()
    for rep in range(3):
        fbar.copy_(base * (1.0 + 0.25 * rep))
        g.replay()
        ref = other.param_grad(pos, sp, s.cell, 0.7, fbar, nlist=nl)
        torch.cuda.synchronize()
        for name, x, y in zip(("d_linear", "d_radial", "d_shift"), got, ref):
            assert rel_err(x.cpu().numpy(), y.cpu().numpy()) < 1e-11, (rep, name)
