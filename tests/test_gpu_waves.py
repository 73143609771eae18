"""Contraction programs that several waves run per tile of 64 atoms (levels from 12 on): sizes around a
tile's edge, chunks that end inside a tile, every level with another number of waves, energies, forces
and the coefficient gradient against the oracle."""
import numpy as np
import pytest
import torch

import workloads as wl
from helpers import TOL_E, TOL_F, TOL_W, rel_err, small_lattice
from oracle import mtp as om
from oracle import neighbors as onb

pytestmark = pytest.mark.gpu

TOL_GRAD = 1e-9


@pytest.mark.parametrize("level,n,chunk", [
    (12, 65, None), (14, 63, None), (14, 129, 65),
    (16, 2, None), (16, 64, None), (16, 129, 64),
    (20, 1, None), (20, 63, None), (20, 66, 65),
])
def test_tile_edges(level, n, chunk):
    from paper_2510_00193_amd import Potential
    s, p = small_lattice(950 + level, (5, 4, 4), 3.2, 0.08, level, 2)
    s = wl.Structure(np.ascontiguousarray(s.pos[:n]), s.species[:n].copy(), s.cell)
    kw = {"chunk_atoms": chunk} if chunk else {}
    print(f"[waves L{level}] N={n} chunk {chunk}", flush=True)
    model = om.Model.from_params(p)
    nl = onb.neighbor_csr(s.pos, s.cell, p.r_cut)
    ref = om.energy_forces_virial(model, s)
    pot = Potential.from_params(p, **kw)
    pos, sp = torch.as_tensor(s.pos, device="cuda"), torch.as_tensor(s.species, device="cuda")
    out = pot.compute(pos, sp, s.cell, e_atom=True)
    rng = np.random.default_rng(level + n)
    fbar = rng.normal(size=(n, 3))
    got = pot.param_grad(pos, sp, s.cell, 0.7, torch.as_tensor(fbar, device="cuda"))
    torch.cuda.synchronize()
    assert rel_err(out["e_atom"].cpu().numpy(), ref["E_i"].detach().numpy()) < TOL_E
    assert rel_err(out["forces"].cpu().numpy(), ref["F"].detach().numpy()) < TOL_F
    assert rel_err(out["virial"].cpu().numpy(), ref["W"].detach().numpy()) < TOL_W
    want = om.param_vjp(model, s, 0.7, fbar, nl)
    for name, g, r in zip(("d_linear", "d_radial", "d_shift"), got, want):
        assert rel_err(g.cpu().numpy(), r) < TOL_GRAD, name
