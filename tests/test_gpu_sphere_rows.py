"""The inverse sphere-plane transform at the plane whose padded form leaves one
workgroup on a CU (72 x 72 in FP64), at the row counts where its rule changes:
one row, the most rows of the compact form with 36 lines a batch (35) and with
18 (53), one step beyond each, and every row.  Apply against the FP64 oracle.

Tolerances as in the other parity tests: FP64 1e-11 of the largest entry,
mixed (whose plane is in place) 2e-6 of the norm.
"""
import dataclasses

import numpy as np
import pytest

import synth
from oracle import basis, model

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2607_20728_amd import bsex  # noqa: E402


@pytest.mark.parametrize("m2", [0, 17, 18, 26, 27, 35])
def test_rows(m2):
    # |n2| <= L2 sqrt(2 ecut) / 2 pi = 0.4502 L2
    nv, cell = 3, (6.0, (m2 + 0.3) / 0.4502, 7.0)
    cfg = dataclasses.replace(synth.get_config("m0"), name="rows", grid=(12, 72, 72), cell=cell,
                              ecut=4.0, n_val=nv, n_pdep=6)
    b = basis.Basis(cfg.cell, cfg.grid, cfg.ecut)
    d = synth.make_system(cfg, b.n_pw, n_trial=2)
    orbs, eps = synth.random_orbitals(b.n_pw, nv, 0, seed=m2)
    S = model.System(b, d["site_xyz"], d["site_depth"], d["site_width"], d["pdep"], d["lam"], nv)
    S.set_orbitals(orbs, eps)
    ref = S.apply(d["trial"])
    X = torch.tensor(d["trial"], dtype=torch.float64, device="cuda")
    for prec in (bsex.FP64, bsex.MIXED):
        print(f"[gpu] sphere rows m2 {m2} precision {prec}", flush=True)
        ctx = bsex.init_from_synth(d, orbitals=orbs, eps=eps, precision=prec)
        Y = bsex.apply(ctx, X).cpu().numpy()
        if prec == bsex.FP64:
            assert np.abs(Y - ref).max() / np.abs(ref).max() < 1e-11
        else:
            assert np.linalg.norm(Y - ref) / np.linalg.norm(ref) < 2e-6
        ctx.free()
