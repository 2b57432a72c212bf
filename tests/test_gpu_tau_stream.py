"""Every launch shape of the tau stream against the FP64 oracle: 8, 4, 2 and 1
grid points per workgroup, 256 to 1024 threads, one or two trial vectors per
lane, odd band counts, and the partial launches that accumulate over tiles
rebuilt inside the apply.

Tolerances: the FP64 apply is linear with O(log N_r) rounding per transform and
O(N_v) in the tau sums, 1e-11 of the largest entry; the mixed form has FP32
grids and tau under the FP64 diagonal, 2e-6 of the norm.
"""
import dataclasses

import numpy as np
import pytest

import synth
from oracle import basis, model

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2607_20728_amd import bsex  # noqa: E402

# (grid, ecut, n_val): points per workgroup and threads (FP64, 8 vectors)
SHAPES = [((12, 12, 12), 6.0, 3),     # 8 points, one block
          ((12, 12, 12), 6.0, 24),    # 8 points, the largest band count
          ((12, 12, 12), 6.0, 25),    # 4 points, 256 threads, odd
          ((12, 12, 12), 6.0, 105),   # 4 points, 512 threads
          ((12, 12, 12), 6.0, 160),   # 4 points, 1024 threads
          ((9, 10, 15), 4.0, 31),     # 2 points: the grid is no multiple of 4
          ((16, 16, 16), 12.0, 610),  # 1 point: two do not fit the LDS
          # lengths of the storing axis-1 transform: three passes (two of its
          # buffers), its shortest tiles, and a last tile that is not full
          ((30, 12, 12), 6.0, 9), ((80, 9, 10), 4.0, 17), ((128, 12, 12), 6.0, 9)]


def _system(grid, ecut, nv):
    cfg = dataclasses.replace(synth.get_config("m0"), name="stream", grid=grid, ecut=ecut,
                              n_val=nv)
    b = basis.Basis(cfg.cell, cfg.grid, cfg.ecut)
    d = synth.make_system(cfg, b.n_pw, n_trial=9)
    orbs, eps = synth.random_orbitals(b.n_pw, nv, 0, seed=nv)
    S = model.System(b, d["site_xyz"], d["site_depth"], d["site_width"], d["pdep"], d["lam"], nv)
    S.set_orbitals(orbs, eps)
    return S, d, orbs, eps


@pytest.mark.parametrize("grid,ecut,nv", SHAPES)
def test_stream_shapes(grid, ecut, nv):
    S, d, orbs, eps = _system(grid, ecut, nv)
    bands = sorted({0, nv // 2, nv - 1})
    ref = S.apply_bands(d["trial"], bands)
    X = torch.tensor(d["trial"], dtype=torch.float64, device="cuda")
    block = 64 * int(np.prod(grid)) * 8
    forms = [("whole", {}), ("partial", dict(tau_budget_bytes=block)),
             ("mixed", dict(precision=bsex.MIXED))]
    for label, kw in forms:
        print(f"[gpu] stream {grid} N_v {nv} {label}", flush=True)
        ctx = bsex.init_from_synth(d, orbitals=orbs, eps=eps, **kw)
        for nb in (1, 4, 5, 8, 9):
            Y = bsex.apply(ctx, X[:nb].contiguous())[:, bands].cpu().numpy()
            if label == "mixed":
                err = np.linalg.norm(Y - ref[:nb]) / np.linalg.norm(ref[:nb])
                assert err < 2e-6, (label, nb, err)
            else:
                err = np.abs(Y - ref[:nb]).max() / np.abs(ref[:nb]).max()
                assert err < 1e-11, (label, nb, err)
        ctx.free()
