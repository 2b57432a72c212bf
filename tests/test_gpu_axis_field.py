"""The potential's part of H x inside one axis-1 pass, at axis lengths of one
(the separate passes), two, three and four butterfly passes: ground-state
eigenvalues against the dense eigenproblem, and the Z-vector of the mixed mode
(its FP32 operator) against the FP64 one.

Tolerances: eigenvalues 1e-9 from residuals of 1e-8 (quadratic, and the
residual bound itself is 1e-8); Z to 1e-5 of its norm from relative residuals
of 1e-8 each, at a condition number below 500 (spectrum up to 6, gaps from
0.016 up).
"""
import dataclasses

import numpy as np
import pytest

import synth
from oracle import basis, model

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2607_20728_amd import bsex  # noqa: E402


@pytest.mark.parametrize("n1", [8, 12, 20, 24, 30, 36, 48, 60, 72, 96, 120, 128])
def test_axis_lengths(n1):
    print(f"[gpu] field pass {n1}", flush=True)
    grid, cell = (n1, 12, 12), (0.6 * n1, 5.0, 5.0)
    cfg = dataclasses.replace(synth.get_config("m0"), name="field", grid=grid, cell=cell,
                              ecut=4.0, n_val=3, n_pdep=6)
    b = basis.Basis(cfg.cell, cfg.grid, cfg.ecut)
    d = synth.make_system(cfg, b.n_pw, n_trial=1)
    S = model.System(b, d["site_xyz"], d["site_depth"], d["site_width"], d["pdep"], d["lam"], 3)
    S.ground_state(n_extra=2)
    ctx = bsex.init_from_synth(d, gs_tol=1e-8, n_extra=2, precision=bsex.MIXED)
    _, eps = bsex.get_orbitals(ctx, 3)
    assert np.abs(eps - S.eps_all[:3]).max() < 1e-9
    X = torch.tensor(d["trial"][0], dtype=torch.float64, device="cuda")
    Zm, _ = bsex.zvector_solve(ctx, X, tol=1e-8)
    bsex.set_precision(ctx, bsex.FP64)
    Z, _ = bsex.zvector_solve(ctx, X, tol=1e-8)
    assert float(torch.linalg.norm(Zm - Z) / torch.linalg.norm(Z)) < 1e-5
    ctx.free()
