"""Lanes per atom of batches and the persistent pair kernels: with one lane per atom a persistent
schedule, each of whose workgroups takes several tiles, gives what the one-shot launches give bit for
bit and agrees with the oracle; with more lanes the schedule is recorded as the one-shot one it runs."""
import functools

import numpy as np
import pytest
import torch

import workloads as wl
from helpers import rel_err, small_batch
from oracle import mtp as om
from oracle import neighbors as onb

pytestmark = pytest.mark.gpu

COPIES = 560  # of 16 configurations of 8 to 24 atoms: 2,200 tiles of 64 atoms on 2048 workgroups at most


@functools.lru_cache(maxsize=None)
def _inputs(level):
    structs, p = small_batch(1400 + level, 16, level, n_min=8, n_max=24)
    model = om.Model.from_params(p)
    ref = [om.energy_forces_virial(model, s, onb.neighbor_csr(s.pos, s.cell, p.r_cut)) for s in structs]
    return structs, p, ref


def _batch(p, structs, **kw):
    from paper_2510_00193_amd import Batch, Potential
    off, pos, species, cells = wl.batch_arrays(structs)
    return Batch(Potential.from_params(p, **kw), off, torch.as_tensor(pos, device="cuda"),
                 torch.as_tensor(species, device="cuda"), cells)


@pytest.mark.parametrize("level", [10, 16, 20])
def test_persistent_kernels_take_several_tiles(level):
    structs, p, ref = _inputs(level)
    b = _batch(p, structs * COPIES, lanes_per_atom=1)
    n = b.n_atoms
    assert n // 64 > 2048
    print(f"[batch lanes L{level}] {b.n_cfg} configurations, {n} atoms", flush=True)
    rng = np.random.default_rng(level)
    e0 = torch.as_tensor(rng.normal(size=b.n_cfg), device="cuda")
    f0 = torch.as_tensor(rng.normal(size=(n, 3)), device="cuda")
    out = {}
    for pers in (False, True):
        b.schedule(sorted=True, persistent=pers)
        assert b.sizes()["persistent"] == int(pers)
        out[pers] = b.run(b.outputs(), e0, f0)
        torch.cuda.synchronize()
    for k, v in out[False].items():
        assert torch.equal(v, out[True][k]), k
    e = out[True]["energy"].cpu().numpy().reshape(COPIES, -1)
    assert rel_err(e[0], [float(r["E"].detach()) for r in ref]) < 1e-10
    assert rel_err(e[-1], e[0]) < 1e-12
    f = out[True]["forces"].cpu().numpy()[:n // COPIES]
    assert rel_err(f, np.concatenate([r["F"].detach().numpy() for r in ref])) < 1e-10


def test_more_lanes_run_one_shot():
    structs, p, ref = _inputs(10)
    f = np.concatenate([r["F"].detach().numpy() for r in ref])
    for lanes, keeps in ((0, 0), (1, 1), (2, 0), (8, 0)):
        b = _batch(p, structs, lanes_per_atom=lanes)
        b.schedule(persistent=True)
        assert b.sizes()["persistent"] == keeps, lanes
        out = b.run(b.outputs(loss=False))
        torch.cuda.synchronize()
        assert rel_err(out["forces"].cpu().numpy(), f) < 1e-10, lanes
        if not keeps:
            assert b.tune()["persistent"] == 0
