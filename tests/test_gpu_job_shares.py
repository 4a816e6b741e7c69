"""Row passes whose jobs are shared out over workgroups (small meshes): per-order and whole estimates
with one job, with fewer jobs than shares, and with a last share longer than the others."""
import numpy as np
import pytest

from oracle.estimators import pk_bisector, xi_bisector

from gpu_common import say, rounded, oracle_cfg, max_err_per_ell, uniform_catalog

pytestmark = pytest.mark.gpu

pw = pytest.importorskip("paper_2102_08384_amd.pw")


@pytest.mark.parametrize("stat", [pw.PW_PK, pw.PW_XI])
@pytest.mark.parametrize("n_mesh,ell_max,order", [(16, 0, 0), (16, 2, 2), (32, 4, 4), (64, 2, 4)])
def test_job_shares(stat, n_mesh, ell_max, order):
    say("job shares", "pk" if stat == pw.PW_PK else "xi", n_mesh, ell_max, order)
    gal, ran = uniform_catalog(500 + n_mesh + ell_max, 2001, 6001, (0, 0, 1100), 600)
    bins = dict(bin_lo=0.004, bin_width=0.012, n_bins=6) if stat == pw.PW_PK else dict(bin_lo=0.0, bin_width=60.0,
                                                                                       n_bins=6)
    cfg = pw.Config(stat=stat, los=pw.PW_BISECTOR, assign=pw.PW_CIC, prec=pw.PW_FP64, n_mesh=n_mesh, box_len=800.0,
                    box_origin=(-400.0, -400.0, 700.0), ell_max=ell_max, order=order, **bins)
    gx, g64 = rounded(gal, np.float64)
    rx, r64 = rounded(ran, np.float64)
    with pw.Context(0) as ctx:
        res = ctx.estimate(cfg, gx, rx, ran_nbar=ran["nbar"])
    ref = (pk_bisector if stat == pw.PW_PK else xi_bisector)(g64, r64, oracle_cfg(cfg))
    err = max_err_per_ell(res["values"], ref.values)
    say("per-ell err", err)
    assert np.array_equal(res["counts"], ref.counts)
    assert np.all(err < 1e-10)  # FP64 transforms and sums: a few hundred roundings of 1e-16
