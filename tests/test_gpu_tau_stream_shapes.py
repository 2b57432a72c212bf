"""The compiled launch shapes of the tau stream that larger band counts choose:
with 8 trial vectors (two a lane) and 4 (one a lane), 512 and 1024 threads at 2
and 4 grid points per workgroup in FP64 and at 2 in FP32, and 1 point in FP32.
Together with test_gpu_tau_stream.py every pair of points and threads that the
rules can choose runs in both forms.

Tolerances as there: FP64 1e-11 of the largest entry, mixed 2e-6 of the norm.
"""
import dataclasses

import numpy as np
import pytest

import synth
from oracle import basis, model

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2607_20728_amd import bsex  # noqa: E402

ODD = ((18, 15, 9), (9.0, 8.0, 5.0), 11.0)  # 2,430 points, no multiple of 4
EVEN = ((16, 16, 16), (8.0, 8.0, 8.0), 12.0)
# points x threads, FP64 with 8 / 4 vectors, FP32 with 8 / 4
CASES = [(ODD, 200),   # 2 x 512 / 256, 2 x 256 / 256
         (ODD, 300),   # 2 x 1024 / 256, 2 x 512 / 256
         (EVEN, 190),  # 4 x 1024 / 512, 4 x 512 / 256
         (EVEN, 290),  # 4 x 1024 / 1024, 2 x 512 / 256
         (EVEN, 350),  # 2 x 1024 / 512, 2 x 512 / 256
         (EVEN, 520),  # 2 x 1024 / 1024, 2 x 1024 / 512
         (EVEN, 700),  # 1 x 512, 2 x 1024 / 1024
         (EVEN, 810)]  # 1 x 512, 1 x 512


@pytest.mark.parametrize("system,nv", CASES)
def test_shapes(system, nv):
    grid, cell, ecut = system
    cfg = dataclasses.replace(synth.get_config("m0"), name="shapes", grid=grid, cell=cell,
                              ecut=ecut, n_val=nv)
    b = basis.Basis(cfg.cell, cfg.grid, cfg.ecut)
    d = synth.make_system(cfg, b.n_pw, n_trial=8)
    orbs, eps = synth.random_orbitals(b.n_pw, nv, 0, seed=nv)
    S = model.System(b, d["site_xyz"], d["site_depth"], d["site_width"], d["pdep"], d["lam"], nv)
    S.set_orbitals(orbs, eps)
    bands = sorted({0, nv // 2, nv - 1})
    ref = S.apply_bands(d["trial"], bands)
    X = torch.tensor(d["trial"], dtype=torch.float64, device="cuda")
    for prec in (bsex.FP64, bsex.MIXED):
        print(f"[gpu] stream shapes {grid} N_v {nv} precision {prec}", flush=True)
        ctx = bsex.init_from_synth(d, orbitals=orbs, eps=eps, precision=prec)
        for nb in (4, 8):
            Y = bsex.apply(ctx, X[:nb].contiguous())[:, bands].cpu().numpy()
            if prec == bsex.FP64:
                assert np.abs(Y - ref[:nb]).max() / np.abs(ref[:nb]).max() < 1e-11, nb
            else:
                assert np.linalg.norm(Y - ref[:nb]) / np.linalg.norm(ref[:nb]) < 2e-6, nb
        ctx.free()
