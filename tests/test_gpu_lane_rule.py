"""Lanes per atom chosen from the system's size: the default runs, bit for bit, what the setting it stands
for runs, at both ends of each range (256 compute units), and the allocation-free evaluation agrees with
the ordinary one where two lanes are chosen and the chunk has to shrink."""
import pytest
import torch

from helpers import small_lattice

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("level,reps,lanes", [
    (10, (32, 32, 16), 2),   # 32,768 atoms
    (10, (33, 32, 16), 2),   # 33,792: one lane would leave one wave per SIMD
    (12, (32, 32, 32), 2),   # 65,536
    (14, (33, 32, 32), 1),   # 67,584
    (16, (33, 32, 16), 1),   # a level of two parts
])
def test_default_lanes(level, reps, lanes):
    from paper_2510_00193_amd import Potential
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the sizes are those of 256 compute units")
    s, p = small_lattice(1200 + level, reps, 3.16, 0.1, level, 2)
    pos, sp = torch.as_tensor(s.pos, device="cuda"), torch.as_tensor(s.species, device="cuda")
    print(f"[lane rule L{level}] N={s.n_atoms}", flush=True)
    pot = Potential.from_params(p)
    nl = pot.neighbors(pos, sp, s.cell)
    got = pot.compute(pos, sp, s.cell, nlist=nl, e_atom=True)
    same = {}
    for k in (1, 2):
        ref = Potential.from_params(p, lanes_per_atom=k).compute(pos, sp, s.cell, nlist=nl, e_atom=True)
        torch.cuda.synchronize()
        same[k] = all(torch.equal(got[q], ref[q]) for q in ("e_atom", "forces", "virial"))
    assert same == {lanes: True, 3 - lanes: False}


def test_static_evaluation_with_two_lanes_in_small_chunks():
    from paper_2510_00193_amd import Potential
    s, p = small_lattice(1210, (31, 31, 31), 3.16, 0.1, 10, 1)  # 59,582 atoms: 68 MB of 64 unless chunked
    pos, sp = torch.as_tensor(s.pos, device="cuda"), torch.as_tensor(s.species, device="cuda")
    print(f"[lane rule static] N={s.n_atoms}", flush=True)
    pot = Potential.from_params(p)
    nl = pot.neighbors(pos, sp, s.cell)
    a = pot.compute(pos, sp, s.cell, nlist=nl, e_atom=True)
    b = pot.compute_static(pos, sp, s.cell, nl, e_atom=True)
    torch.cuda.synchronize()
    for k in ("energy", "e_atom", "forces", "virial"):
        assert torch.equal(a[k], b[k]), k
