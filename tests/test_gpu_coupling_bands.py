"""The coupling apply with several bands' pair grids per pass, against the FP64
oracle: an even number of bands in passes of an odd 7 (fields 7, 14 begin in
the second half of a packed grid) with a remainder of 6, an odd number (whose
last grid is half empty) in passes of 6 with a remainder of 3.

Tolerance as in the other parity tests: 1e-11 of the largest entry.
"""
import dataclasses

import numpy as np
import pytest

import synth
from oracle import basis, full_bse, model

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2607_20728_amd import bsex  # noqa: E402


@pytest.mark.parametrize("n1,nv", [(120, 20), (128, 21)])
def test_band_passes(n1, nv):
    print(f"[gpu] coupling bands {n1} {nv}", flush=True)
    cfg = dataclasses.replace(synth.get_config("m0"), name="bands", grid=(n1, 12, 12),
                              cell=(0.6 * n1, 5.0, 5.0), ecut=4.0, n_val=nv, n_pdep=9)
    b = basis.Basis(cfg.cell, cfg.grid, cfg.ecut)
    d = synth.make_system(cfg, b.n_pw, n_trial=2)
    orbs, eps = synth.random_orbitals(b.n_pw, nv, 0, seed=n1)
    S = model.System(b, d["site_xyz"], d["site_depth"], d["site_width"], d["pdep"], d["lam"], nv)
    S.set_orbitals(orbs, eps)
    X = torch.tensor(d["trial"], dtype=torch.float64, device="cuda")
    ctx = bsex.init_from_synth(d, orbitals=orbs, eps=eps)
    B = bsex.apply_coupling(ctx, X).cpu().numpy()
    ref = full_bse.apply_b(S, d["trial"])
    assert np.abs(B - ref).max() / np.abs(ref).max() < 1e-11
    ctx.free()
