"""The lists of occupied rows and planes: a thin catalog moved by whole cells has the same monopole
power, wherever its planes fall among the wavefronts that compact the list."""
import numpy as np
import pytest

from gpu_common import say

pytestmark = pytest.mark.gpu

pw = pytest.importorskip("paper_2102_08384_amd.pw")


@pytest.mark.parametrize("n_mesh", [16, 64, 128, 512])
def test_planes_found_anywhere(n_mesh):
    rng = np.random.default_rng(70 + n_mesh)
    # eighths of a cell: every shift is exact, so the deposits are the same numbers in other cells
    pos = rng.integers(0, 8 * n_mesh, (1500, 3)).astype(np.float64) / 8
    pos[:, 2] = rng.integers(0, 8 * 4, 1500) / 8
    origin = 1024.0
    cfg = pw.Config(stat=pw.PW_PK, los=pw.PW_BISECTOR, assign=pw.PW_CIC, prec=pw.PW_FP64, n_mesh=n_mesh,
                    box_len=float(n_mesh), box_origin=(origin,) * 3, ell_max=0, order=0, bin_lo=0.1, bin_width=0.5,
                    n_bins=4)
    out = []
    with pw.Context(0) as ctx:
        for z0 in (2, 7, n_mesh // 2 - 2, n_mesh - 6):
            say("occupied planes", n_mesh, z0)
            p = pos + (0, 0, z0) + origin
            xyzw = np.concatenate([p, np.ones((len(p), 1))], axis=1)
            r = ctx.estimate(cfg, xyzw[:500], xyzw[500:], ran_nbar=np.full(1000, 1e-3))
            out.append((r["values"][0], r["norm"]))
    (v, (_, I, S)) = out[0]
    assert np.all(np.isfinite(v)) and np.any(v != 0)
    # FP64 transform: about log2(512^3) = 27 roundings of 1e-16 on each side of P, and P before the
    # shot noise S / I is taken off is at least of its size
    bound = 1e-12 * (np.abs(v) + abs(S / I))
    for w, norm in out[1:]:
        assert np.all(np.abs(w - v) <= bound)
        assert norm == out[0][1]
