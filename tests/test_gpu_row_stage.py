"""Rows copied to LDS with 16-byte reads (one lane per atom): every remainder of a read of four and of a
stage of 32 pairs, in waves that end before the last 32 entries of the list and in waves that do not,
in binary64 and binary32, against the oracle.  Binary32: sums of at most 65 terms of 2^-24 each, in
products of at most five moments, with cancellation to a fifth: 65 * 6e-8 * 5 * 5 = 1e-4."""
import numpy as np
import pytest
import torch

from helpers import TOL_E, TOL_F, rel_err
from oracle import mtp as om
from test_gpu_pair_rows import _cluster

pytestmark = pytest.mark.gpu

ROWS = (29, 30, 31, 32, 33, 34, 35, 36, 63, 64, 65)


@pytest.mark.parametrize("precision,tol", [("fp64", None), ("fp32", 1e-4)])
@pytest.mark.parametrize("rows", [ROWS, ROWS[::-1], (2, 3, 4, 5)])
def test_staged_rows(rows, precision, tol):
    from paper_2510_00193_amd import Potential
    s, p = _cluster(rows, np.random.default_rng(900 + len(rows)), 10)
    ref = om.energy_forces_virial(om.Model.from_params(p), s)
    pos, sp = torch.as_tensor(s.pos, device="cuda"), torch.as_tensor(s.species, device="cuda")
    print(f"[row stage {precision}] N={s.n_atoms}", flush=True)
    pot = Potential.from_params(p, precision=precision, lanes_per_atom=1)
    out = pot.compute(pos, sp, s.cell, nlist=pot.neighbors(pos, sp, s.cell), e_atom=True)
    torch.cuda.synchronize()
    assert rel_err(out["e_atom"].cpu().numpy(), ref["E_i"].detach().numpy()) < (tol or TOL_E)
    assert rel_err(out["forces"].cpu().numpy(), ref["F"].detach().numpy()) < (tol or TOL_F)
