"""Launches of the one-part pair kernels on both sides of one wave per SIMD (1024 on this GPU): a chunk of
4096 atoms takes the form that has a SIMD to itself, the whole system the other one.  The arithmetic of an
atom is the same in both, so the results are equal bit for bit."""
import numpy as np
import pytest
import torch

from helpers import small_lattice

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("level", [10, 12, 14])
@pytest.mark.parametrize("lanes,reps", [(1, 33), (2, 26), (4, 21), (8, 17)])
def test_forms_for_few_and_many_waves_agree(level, lanes, reps):
    from paper_2510_00193_amd import Potential
    s, p = small_lattice(1100 + level, (reps, reps, reps), 3.16, 0.1, level, 2, n_cheb=7 if level == 12 else 8)
    assert s.n_atoms * lanes > 64 * 1024
    pos, sp = torch.as_tensor(s.pos, device="cuda"), torch.as_tensor(s.species, device="cuda")
    print(f"[alone L{level}] N={s.n_atoms} lanes {lanes}", flush=True)
    few = Potential.from_params(p, lanes_per_atom=lanes, chunk_atoms=4096)
    many = Potential.from_params(p, lanes_per_atom=lanes)
    nl = many.neighbors(pos, sp, s.cell)
    a = few.compute(pos, sp, s.cell, nlist=nl, e_atom=True)
    b = many.compute(pos, sp, s.cell, nlist=nl, e_atom=True)
    torch.cuda.synchronize()
    for k in ("e_atom", "forces", "virial"):
        assert torch.equal(a[k], b[k]), k
    ainv = torch.as_tensor(np.eye(few.n_alpha), device="cuda")
    ga, gb = (q.grade(pos, sp, s.cell, ainv, nlist=nl) for q in (few, many))
    torch.cuda.synchronize()
    assert torch.equal(ga["grade"], gb["grade"])
