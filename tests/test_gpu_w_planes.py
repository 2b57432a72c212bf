"""The W solve with its plane part in one kernel, at every plane size that has
one: the apply (pair potentials and the Poisson solve of K1e) in FP64 and
mixed precision and the coupling apply, against the FP64 oracle.

Tolerances as in the other parity tests: FP64 1e-11 of the largest entry,
mixed 2e-6 of the norm.
"""
import dataclasses

import numpy as np
import pytest

import synth
from oracle import basis, full_bse, model

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2607_20728_amd import bsex  # noqa: E402

PLANES = [(12, 12), (16, 16), (24, 24), (32, 32), (40, 40), (48, 48), (64, 64), (72, 72),
          (48, 120)]


@pytest.mark.parametrize("n2,n3", PLANES)
def test_planes(n2, n3):
    grid = (8, n2, n3)
    cell = tuple(8.0 * n / 12.0 for n in grid)
    nv = 5
    cfg = dataclasses.replace(synth.get_config("m0"), name="planes", grid=grid, cell=cell,
                              ecut=4.0, n_val=nv)
    b = basis.Basis(cfg.cell, cfg.grid, cfg.ecut)
    d = synth.make_system(cfg, b.n_pw, n_trial=2)
    orbs, eps = synth.random_orbitals(b.n_pw, nv, 0, seed=n2 + n3)
    S = model.System(b, d["site_xyz"], d["site_depth"], d["site_width"], d["pdep"], d["lam"], nv)
    S.set_orbitals(orbs, eps)
    ref = S.apply(d["trial"])
    X = torch.tensor(d["trial"], dtype=torch.float64, device="cuda")
    for prec in (bsex.FP64, bsex.MIXED):
        print(f"[gpu] planes {n2} x {n3} precision {prec}", flush=True)
        ctx = bsex.init_from_synth(d, orbitals=orbs, eps=eps, precision=prec)
        Y = bsex.apply(ctx, X).cpu().numpy()
        if prec == bsex.FP64:
            assert np.abs(Y - ref).max() / np.abs(ref).max() < 1e-11
            B = bsex.apply_coupling(ctx, X[:1].contiguous()).cpu().numpy()
            Bref = full_bse.apply_b(S, d["trial"][:1])
            assert np.abs(B - Bref).max() / np.abs(Bref).max() < 1e-11
        else:
            assert np.linalg.norm(Y - ref) / np.linalg.norm(ref) < 2e-6
        ctx.free()
