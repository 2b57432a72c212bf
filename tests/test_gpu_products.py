"""The matrix products at the edges of their tile and split rules: outputs of
up to 16 rows, of one 32 x 32 tile and a remainder, inner lengths from a
single K step to more than 16 splits; and the transition density's groups of
1, 2 and 8 vectors a thread (the last from 2^18 grid points on).  Apply (projector, PDEP products) and
the U vector (its S matrix) against the FP64 oracle.

Tolerances as in the other parity tests: FP64 1e-11 of the largest entry,
mixed 2e-6 of the norm.
"""
import dataclasses

import numpy as np
import pytest

import synth
from oracle import basis, model, solvers

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2607_20728_amd import bsex  # noqa: E402

# grid edge, n_val, n_pdep, trial vectors: n_pw is about 0.11 edge^3
SIZES = [(8, 3, 5, 1), (12, 16, 33, 1), (16, 17, 64, 2), (24, 33, 130, 1), (32, 16, 17, 3),
         (64, 3, 5, 3)]


@pytest.mark.parametrize("n,nv,npd,nb", SIZES)
def test_products(n, nv, npd, nb):
    cell = (8.0 * n / 12.0,) * 3
    cfg = dataclasses.replace(synth.get_config("m0"), name="products", grid=(n,) * 3, cell=cell,
                              ecut=4.0, n_val=nv, n_pdep=npd)
    b = basis.Basis(cfg.cell, cfg.grid, cfg.ecut)
    d = synth.make_system(cfg, b.n_pw, n_trial=nb)
    orbs, eps = synth.random_orbitals(b.n_pw, nv, 0, seed=n)
    S = model.System(b, d["site_xyz"], d["site_depth"], d["site_width"], d["pdep"], d["lam"], nv)
    S.set_orbitals(orbs, eps)
    ref = S.apply(d["trial"])
    uref = solvers.u_vector(S, d["trial"][0])
    X = torch.tensor(d["trial"], dtype=torch.float64, device="cuda")
    for prec in (bsex.FP64, bsex.MIXED):
        print(f"[gpu] products {n} {nv} {npd} {nb} precision {prec}", flush=True)
        ctx = bsex.init_from_synth(d, orbitals=orbs, eps=eps, precision=prec)
        Y = bsex.apply(ctx, X).cpu().numpy()
        U = bsex.u_vector(ctx, X[0]).cpu().numpy()
        for got, want in ((Y, ref), (U, uref)):
            if prec == bsex.FP64:
                assert np.abs(got - want).max() / np.abs(want).max() < 1e-11
            else:
                assert np.linalg.norm(got - want) / np.linalg.norm(want) < 2e-6
        ctx.free()
