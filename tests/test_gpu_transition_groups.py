"""The transition density's groups of vectors: 2 a thread on grids below 2^17
points (FP64) or 40,000 (FP32), from there on 8 with a remainder in a group of
its own size, and where a packed grid takes 2.75 MB a remainder one vector at a
time.  Every block of 1 to 9 vectors on each side of the limits, through the
apply's Hartree exchange, against the FP64 oracle.

Tolerances as in the other parity tests: FP64 1e-11 of the largest entry,
mixed 2e-6 of the norm.
"""
import dataclasses

import numpy as np
import pytest

import synth
from oracle import basis, model

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2607_20728_amd import bsex  # noqa: E402


# 32,768 and 122,880 points (2 each in FP64, FP32 groups in the second),
# 131,072 (FP64 groups), 184,320 (FP64 one at a time) and 345,600 (FP32 too)
@pytest.mark.parametrize("grid", [(32, 32, 32), (128, 32, 30), (32, 64, 64), (48, 60, 64),
                                  (48, 60, 120)])
def test_groups(grid):
    nv, nb = 3, 9
    cfg = dataclasses.replace(synth.get_config("m0"), name="groups", grid=grid,
                              cell=tuple(0.3 * n for n in grid), ecut=4.0, n_val=nv, n_pdep=5)
    b = basis.Basis(cfg.cell, cfg.grid, cfg.ecut)
    d = synth.make_system(cfg, b.n_pw, n_trial=nb)
    orbs, eps = synth.random_orbitals(b.n_pw, nv, 0, seed=5)
    S = model.System(b, d["site_xyz"], d["site_depth"], d["site_width"], d["pdep"], d["lam"], nv)
    S.set_orbitals(orbs, eps)
    ref = S.apply(d["trial"])
    X = torch.tensor(d["trial"], dtype=torch.float64, device="cuda")
    for prec in (bsex.FP64, bsex.MIXED):
        print(f"[gpu] groups {grid} precision {prec}", flush=True)
        ctx = bsex.init_from_synth(d, orbitals=orbs, eps=eps, precision=prec)
        for k in range(1, nb + 1):
            Y = bsex.apply(ctx, X[:k].contiguous()).cpu().numpy()
            if prec == bsex.FP64:
                assert np.abs(Y - ref[:k]).max() / np.abs(ref[:k]).max() < 1e-11, k
            else:
                assert np.linalg.norm(Y - ref[:k]) / np.linalg.norm(ref[:k]) < 2e-6, k
        ctx.free()
