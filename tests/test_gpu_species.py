"""Coefficient tables of several species with rows of an even and an odd number of values, up to the
largest table, in one lane per atom and several: evaluations in both precisions and the coefficient
gradient, against the oracle."""
import numpy as np
import pytest
import torch

from helpers import TOL_E, TOL_F, TOL_W, rel_err, small_lattice
from oracle import mtp as om

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("level,nsp,ncheb", [(10, 8, 5), (10, 3, 8), (10, 4, 16), (16, 4, 16), (16, 3, 10), (20, 3, 9),
                                             (2, 8, 16), (10, 1, 2)])
def test_tables_of_several_species(level, nsp, ncheb):
    from paper_2510_00193_amd import Potential
    s, p = small_lattice(1600 + level + nsp, (3, 4, 3), 3.16, 0.1, level, nsp, n_cheb=ncheb)
    model = om.Model.from_params(p)
    ref = om.energy_forces_virial(model, s)
    fbar = np.random.default_rng(1).normal(size=(s.n_atoms, 3))
    grads = om.param_vjp(model, s, 0.4, fbar, ref["nl"])
    pos, sp = torch.as_tensor(s.pos, device="cuda"), torch.as_tensor(s.species, device="cuda")
    for lanes in (1, 4):
        print(f"[species L{level} nsp {nsp} n_cheb {ncheb}] N={s.n_atoms} lanes {lanes}", flush=True)
        pot = Potential.from_params(p, lanes_per_atom=lanes)
        out = pot.compute(pos, sp, s.cell, e_atom=True)
        got = pot.param_grad(pos, sp, s.cell, 0.4, torch.as_tensor(fbar, device="cuda"))
        torch.cuda.synchronize()
        assert rel_err(out["e_atom"].cpu().numpy(), ref["E_i"].detach().numpy()) < TOL_E
        assert rel_err(out["forces"].cpu().numpy(), ref["F"].detach().numpy()) < TOL_F
        assert rel_err(out["virial"].cpu().numpy(), ref["W"].detach().numpy()) < TOL_W
        for name, x, y in zip(("d_linear", "d_radial", "d_shift"), got, grads):
            assert rel_err(x.cpu().numpy(), y) < 1e-9, name
    if level < 20:
        out = Potential.from_params(p, precision="fp32").compute(pos, sp, s.cell)
        torch.cuda.synchronize()
        # the bound of tests/test_gpu_row_stage.py for rows of up to 65 pairs
        assert rel_err(out["forces"].cpu().numpy(), ref["F"].detach().numpy()) < 1e-4
