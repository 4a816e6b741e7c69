"""Tiles painted by several workgroups: the parts' sums are integers, so the mesh has the bits of the
one painted a workgroup to a tile.  The split needs room for the parts in the spectrum buffer: an
estimate of the monopole alone (one field) has none and paints whole tiles."""
import numpy as np
import pytest

from gpu_common import say

pytestmark = pytest.mark.gpu

pw = pytest.importorskip("paper_2102_08384_amd.pw")


@pytest.mark.parametrize("n_mesh,prec,assign", [(16, pw.PW_FP64, pw.PW_TSC), (32, pw.PW_FP32, pw.PW_CIC),
                                                (64, pw.PW_FP64, pw.PW_CIC), (128, pw.PW_FP32, pw.PW_TSC)])
def test_parts_sum_to_the_mesh(n_mesh, prec, assign):
    say(f"paint in parts {n_mesh}^3 prec {prec} assign {assign}")
    dt = np.float64 if prec == pw.PW_FP64 else np.float32
    rng = np.random.default_rng(900 + n_mesh)
    # a dense clump inside one tile, a smooth sheet, a few particles elsewhere and empty tiles
    pos = np.concatenate([rng.normal(0, 4, (150_001, 3)) + (40, 40, 1040),
                          rng.uniform(-400, 400, (120_000, 3)) * (1, 1, 0.05) + (0, 0, 1000),
                          rng.uniform(-450, 450, (50, 3)) + (0, 0, 1000)])
    rng.shuffle(pos)
    xyzw = np.concatenate([pos, rng.uniform(0.5, 1.5, (len(pos), 1))], axis=1).astype(dt)
    base = dict(stat=pw.PW_PK, los=pw.PW_BISECTOR, assign=assign, prec=prec, n_mesh=n_mesh, box_len=1000.0,
                box_origin=(-500.0, -500.0, 500.0), bin_lo=0.005, bin_width=0.01, n_bins=4)
    meshes = []
    with pw.Context(0) as ctx:
        for ell_max, order in ((0, 0), (4, 4)):
            ctx.estimate(pw.Config(ell_max=ell_max, order=order, **base), xyzw[:50_000], xyzw[50_000:],
                         ran_nbar=np.full(len(pos) - 50_000, 1e-4, dtype=dt))
            meshes.append(ctx.inspect(0, dt))
    assert np.any(meshes[0] != 0)
    assert np.array_equal(meshes[0], meshes[1])
