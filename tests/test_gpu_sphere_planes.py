"""The pruned sphere-plane transforms at the extremes of the rows and columns
they keep: a cell so thin along one in-plane axis that a single row or column
of modes is left, and one where nearly every line holds modes.  Apply against
the FP64 oracle.

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

# cell edges on a (12, n2, n3) grid: |n| <= L sqrt(2 ecut) / 2 pi = 0.45 L
CASES = [((12, 12, 12), (9.0, 1.5, 9.0)),   # n2 = 0 only
         ((12, 12, 12), (9.0, 9.0, 1.5)),   # n3 = 0 only
         ((12, 16, 16), (9.0, 16.5, 16.5)),  # |n| <= 7 of 16
         ((12, 48, 120), (6.0, 50.0, 8.0))]


@pytest.mark.parametrize("grid,cell", CASES)
def test_extents(grid, cell):
    nv = 3
    cfg = dataclasses.replace(synth.get_config("m0"), name="extents", grid=grid, cell=cell,
                              ecut=4.0, n_val=nv, n_pdep=6)
    b = basis.Basis(cfg.cell, cfg.grid, cfg.ecut)
    d = synth.make_system(cfg, b.n_pw, n_trial=2)
    orbs, eps = synth.random_orbitals(b.n_pw, nv, 0, seed=3)
    S = model.System(b, d["site_xyz"], d["site_depth"], d["site_width"], d["pdep"], d["lam"], nv)
    S.set_orbitals(orbs, eps)
    ref = S.apply(d["trial"])
    X = torch.tensor(d["trial"], dtype=torch.float64, device="cuda")
    for prec in (bsex.FP64, bsex.MIXED):
        print(f"[gpu] extents {grid} {cell} precision {prec}", flush=True)
        ctx = bsex.init_from_synth(d, orbitals=orbs, eps=eps, precision=prec)
        Y = bsex.apply(ctx, X).cpu().numpy()
        if prec == bsex.FP64:
            assert np.abs(Y - ref).max() / np.abs(ref).max() < 1e-11
        else:
            assert np.linalg.norm(Y - ref) / np.linalg.norm(ref) < 2e-6
        ctx.free()
