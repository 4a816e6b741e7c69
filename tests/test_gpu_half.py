"""xi_l from half of the separations (real spectra, two fields to an inverse transform): the smallest
and largest sets of planes, odd field counts, odd-parity fields, and a last bin that touches L/2."""
import dataclasses

import numpy as np
import pytest

from oracle.estimators import xi_bisector, xi_midpoint

from gpu_common import say, rounded, oracle_cfg, max_err_per_ell, uniform_catalog

pytestmark = pytest.mark.gpu

pw = pytest.importorskip("paper_2102_08384_amd.pw")


@pytest.fixture(scope="module")
def ctx():
    c = pw.Context(0)
    yield c
    c.close()


# box 800: H = 50 at 16^3, 25 at 32^3, 12.5 at 64^3; bins (lo, width, n)
@pytest.mark.parametrize("los,parity,n_mesh,prec,ell_max,order,bins", [
    ("midpoint", "even", 16, pw.PW_FP64, 4, 4, (10.0, 50.0, 1)),     # the planes z = 0, 1 alone
    ("midpoint", "even", 16, pw.PW_FP64, 2, 2, (0.0, 100.0, 4)),     # every separation below L/2
    ("midpoint", "all", 16, pw.PW_FP64, 4, 3, (0.0, 100.0, 4)),      # fields odd in D
    ("midpoint", "all", 32, pw.PW_FP32, 2, 1, (0.0, 60.0, 6)),       # 6 + 10 fields, pairs across parities
    ("midpoint", "even", 64, pw.PW_FP32, 0, 0, (0.0, 30.0, 5)),      # one field
    ("bisector", "even", 16, pw.PW_FP64, 4, 4, (0.0, 100.0, 4)),     # 15 targets
    ("bisector", "even", 64, pw.PW_FP32, 2, 2, (0.0, 25.0, 4)),
    # bins that end at L/2, whose last one takes in the axis cells at N/2 by rounding
    ("midpoint", "even", 16, pw.PW_FP64, 2, 2, (120.56978104822326, 39.91860270739668, 7)),
    ("midpoint", "all", 16, pw.PW_FP64, 2, 1, (120.56978104822326, 39.91860270739668, 7)),
    ("bisector", "even", 16, pw.PW_FP64, 2, 2, (66.36278373170074, 47.6624594668999, 7)),
])
def test_half_sets(ctx, los, parity, n_mesh, prec, ell_max, order, bins):
    say("xi from half sets", los, parity, n_mesh, prec, ell_max, order, bins)
    dt = np.float64 if prec == pw.PW_FP64 else np.float32
    gal, ran = uniform_catalog(70 + n_mesh + order, 3001, 9001, (0, 0, 1100), 400)
    cfg = pw.Config(stat=pw.PW_XI, los=pw.PW_MIDPOINT if los == "midpoint" else pw.PW_BISECTOR, assign=pw.PW_TSC,
                    prec=prec, n_mesh=n_mesh, box_len=800.0, box_origin=(-400.0, -400.0, 700.0), ell_max=ell_max,
                    order=order, bin_lo=bins[0], bin_width=bins[1], n_bins=bins[2],
                    midpoint_parity=pw.PW_PARITY_ALL if parity == "all" else pw.PW_PARITY_EVEN)
    gx, g64 = rounded(gal, dt)
    rx, r64 = rounded(ran, dt)
    res = ctx.estimate(cfg, gx, rx, ran_nbar=ran["nbar"].astype(dt))
    est = xi_midpoint if los == "midpoint" else xi_bisector
    ref = est(g64, r64, dataclasses.replace(oracle_cfg(cfg), parity=parity))
    err = max_err_per_ell(res["values"], ref.values)
    say("per-ell err", err)
    assert np.array_equal(res["counts"], ref.counts)
    # FP64 transforms and sums: a few hundred roundings of 1e-16; FP32: the estimator's 1e-4 bound
    assert np.all(err < (1e-10 if prec == pw.PW_FP64 else 1e-4))
