"""Every kernel that makes a sphere-plane pass has its row in the stage table of
profsummary: the names are read from the sources, so one that is renamed or
added without the table following fails here.
"""
import glob
import os
import re
import sqlite3
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
INV, FWD = "inverse plane pass, sphere -> planes", "forward plane pass, planes -> sphere"


def _kernels():
    names = set()
    for f in glob.glob(os.path.join(ROOT, "paper_2607_20728_amd", "csrc", "*")):
        if f.endswith((".h", ".hip")):
            with open(f) as fh:
                names |= set(re.findall(r"void\s+(k_sphere_(?:inv|fwd)_\w+)\(", fh.read()))
    return sorted(names)


def test_sources_have_both_directions():
    assert {n[9:12] for n in _kernels()} == {"inv", "fwd"}


@pytest.mark.parametrize("name,label", [(n + "<72, 72>", INV if "_inv_" in n else FWD)
                                        for n in _kernels()]
                         + [("k_fft_plane<1, 1, 0>", INV), ("k_fft_plane<-1, 0, 1>", FWD),
                            ("k_fft_plane_ct<72, 72, 1, 1, 0>", INV),
                            ("k_fft_plane_ct<72, 72, -1, 0, 1>", FWD)])
def test_stage_row(tmp_path, name, label):
    db = str(tmp_path / "s_results.db")
    con = sqlite3.connect(db)
    con.execute("create table kernels (name text, grid_x int, workgroup_x int, lds_size int, "
                "vgpr_count int, accum_vgpr_count int, duration int, start int)")
    seq = [(f"void bsex::f64::{name}(x)", 3000, 2_000_000),
           ("void bsex::k_tau_stream_qs<2, 1024, 2, true, double>(x)", 5000, 50_000_000)] * 3
    con.executemany("insert into kernels values (?, ?, 256, 0, 0, 0, ?, ?)",
                    [(n, g, d, i) for i, (n, g, d) in enumerate(seq)])
    con.commit()
    con.close()
    out = subprocess.run([sys.executable, "-m", "paper_2607_20728_amd.profsummary", "stages", db,
                          "--grid", "72", "72", "72", "--planes", "35", "--npw", "21079", "--nv",
                          "432", "--nb", "8", "--prec", "f64", "--stream-bytes", "300e9"],
                         capture_output=True, text=True, check=True, cwd=ROOT).stdout
    rows = [ln.split("|") for ln in out.splitlines() if ln.startswith(f"| {label} (`{name}`)")]
    assert len(rows) == 1 and rows[0][3].strip() == "2.00"
