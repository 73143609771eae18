"""A pair at no distance (positions moved after the list was built) has no direction: the energy is
finite, the forces on its atoms are not numbers, and those of atoms away from it are unharmed."""
import numpy as np
import pytest
import torch

from helpers import small_lattice

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("level,lanes", [(10, 1), (10, 4), (14, 1), (16, 1), (16, 8), (20, 1)])
def test_pairs_at_no_distance(level, lanes):
    from paper_2510_00193_amd import Potential
    s, p = small_lattice(1500 + level, (5, 5, 5), 3.16, 0.05, level, 1)
    pos, sp = torch.as_tensor(s.pos, device="cuda"), torch.as_tensor(s.species, device="cuda")
    print(f"[coincident L{level}] N={s.n_atoms} lanes {lanes}", flush=True)
    pot = Potential.from_params(p, lanes_per_atom=lanes)
    nl = pot.neighbors(pos, sp, s.cell)
    # the atom nearest to the cell's centre takes its nearest neighbour's place (no image between them)
    i = int(np.argmin(np.linalg.norm(s.pos - np.diag(s.cell) / 2, axis=1)))
    j = int(np.argsort(np.linalg.norm(s.pos - s.pos[i], axis=1))[1])
    pos[i] = pos[j]
    out = pot.compute(pos, sp, s.cell, nlist=nl, e_atom=True)
    torch.cuda.synchronize()
    f = out["forces"].cpu().numpy()
    assert np.isfinite(out["e_atom"].cpu().numpy()).all()
    assert np.isnan(f[[i, j]]).any(axis=1).all()
    assert np.isfinite(f).all(axis=1).sum() == s.n_atoms - 2
