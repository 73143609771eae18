"""Row lengths at which the pair kernels change what they do: rows around the 32 pairs a lane stages
at a time, empty rows beside full ones in one wave, lists of fewer than four pairs (the end of the
list is read with 16-byte loads), at a level of one moment part, of two and of four; every
lanes-per-atom setting, against the oracle."""
import numpy as np
import pytest
import torch

import workloads as wl
from helpers import TOL_E, TOL_F, TOL_W, oracle_sizes, rel_err
from oracle import mtp as om

pytestmark = pytest.mark.gpu


def _cluster(rows, rng, level, n_cheb=8):
    """One dense clump per entry of rows (its atoms all see each other) far apart in a large cell, so
    that every atom of clump c has rows[c] neighbours."""
    side = 12.0
    grid = int(np.ceil(len(rows) ** (1.0 / 3.0)))
    cell = np.diag([side * grid] * 3)
    pos = []
    for c, n in enumerate(rows):
        at = side * (np.array([c // (grid * grid), c // grid % grid, c % grid]) + 0.5)
        k = int(np.ceil((n + 1) ** (1.0 / 3.0)))
        site = np.stack(np.meshgrid(*[np.arange(k)] * 3, indexing="ij"), -1).reshape(-1, 3)[:n + 1]
        pos.append(at + 0.75 * (site - (k - 1) / 2.0) + rng.normal(0.0, 0.05, (n + 1, 3)))
    pos = np.ascontiguousarray(np.concatenate(pos))
    n_alpha, n_mu = oracle_sizes(level)
    p = wl.draw_params(rng, level, 2, n_mu, n_cheb, n_alpha, 0.5, 5.0)
    return wl.Structure(pos, rng.integers(0, 2, len(pos)).astype(np.int32), cell), p


@pytest.mark.parametrize("level,rows", [
    (10, (31, 32, 33, 0, 1, 40)),
    (16, (31, 32, 33, 0, 1)),
    (16, (65, 0, 0, 2)),
    (16, (1,)),            # two pairs in all
    (10, (1, 0)),
    (20, (33, 0, 3)),
    (20, (1,)),
])
def test_row_lengths(level, rows):
    from paper_2510_00193_amd import Potential
    s, p = _cluster(rows, np.random.default_rng(800 + level + len(rows)), level, 10 if level == 20 else 8)
    ref = om.energy_forces_virial(om.Model.from_params(p), s)
    assert sorted(set(np.diff(ref["nl"]["off"]))) == sorted(set(rows))
    pos, sp = torch.as_tensor(s.pos, device="cuda"), torch.as_tensor(s.species, device="cuda")
    for k in (1, 2, 4, 8):
        print(f"[rows L{level} {rows}] N={s.n_atoms} lanes {k}", flush=True)
        pot = Potential.from_params(p, lanes_per_atom=k)
        out = pot.compute(pos, sp, s.cell, nlist=pot.neighbors(pos, sp, s.cell), e_atom=True)
        torch.cuda.synchronize()
        assert rel_err(out["e_atom"].cpu().numpy(), ref["E_i"].detach().numpy()) < TOL_E
        assert rel_err(out["forces"].cpu().numpy(), ref["F"].detach().numpy()) < TOL_F
        assert rel_err(out["virial"].cpu().numpy(), ref["W"].detach().numpy()) < TOL_W
