"""Midpoint P_l from half of the separations (meshes from 64^3 on) in double precision, with k-bins that
take in the Nyquist frequency: several steps of g fields, alpha = 2 and 4, odd and even alpha side by
side, more A fields than one step of rows, and (128^3) columns shared by two wavefronts, against the
oracle's stored values.  The planes at N/2, where the mirror of an index is not the opposite separation,
are worth 1e-4 of P_l, so only a tight bound holds them."""
import json
import os

import numpy as np
import pytest

from gpu_common import say, rounded, max_err_per_ell, uniform_catalog

pytestmark = pytest.mark.gpu

pw = pytest.importorskip("paper_2102_08384_amd.pw")

with open(os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden", "mid_pk_planes.json")) as fh:
    GOLD = json.load(fh)


def _run(ctx, c, prec, cat):
    dt = np.float64 if prec == pw.PW_FP64 else np.float32
    cfg = pw.Config(stat=pw.PW_PK, los=pw.PW_MIDPOINT, assign=c["assign"], prec=prec, n_mesh=c["n_mesh"],
                    box_len=c["box_len"], box_origin=tuple(c["box_origin"]), ell_max=c["ell_max"], order=c["order"],
                    bin_lo=c["bin_lo"], bin_width=c["bin_width"], n_bins=c["n_bins"],
                    midpoint_parity=pw.PW_PARITY_ALL if c["parity"] == "all" else pw.PW_PARITY_EVEN)
    (gx, _), (rx, _) = (rounded(k, dt) for k in cat)
    return ctx.estimate(cfg, gx, rx, ran_nbar=cat[1]["nbar"].astype(dt))


@pytest.fixture(scope="module")
def catalog():
    return uniform_catalog(**GOLD["catalog"])


@pytest.mark.parametrize("c", GOLD["cases"], ids=lambda c: f"{c['n_mesh']}-l{c['ell_max']}-o{c['order']}-{c['parity']}")
def test_half_planes(catalog, c):
    say("midpoint half planes", {k: v for k, v in c.items() if k not in ("values", "counts")})
    with pw.Context(0) as ctx:
        res = _run(ctx, c, pw.PW_FP64, catalog)
    assert np.array_equal(res["counts"], c["counts"])
    err = max_err_per_ell(res["values"], np.array(c["values"]))
    say("per-ell err", err)
    assert np.all(err < 1e-10)  # FP64 transforms and sums: a few hundred roundings of 1e-16


@pytest.mark.parametrize("prec", [pw.PW_FP64, pw.PW_FP32])
def test_every_field_grouping(catalog, prec):
    """The inverse y pass with one, two, four and seven fields to a workgroup (a partial last group
    among them), and the autotuner's choice, give the default's multipoles."""
    c = next(c for c in GOLD["cases"] if (c["n_mesh"], c["ell_max"], c["parity"]) == (64, 4, "all"))
    say("midpoint half planes, every field grouping, prec", prec)
    with pw.Context(0) as ctx:
        ctx.set_tuning(0)
        base = _run(ctx, c, prec, catalog)["values"]
        for mode in (2, 3, 4, 5, 6, 7, 1):
            ctx.set_tuning(mode)
            got = _run(ctx, c, prec, catalog)["values"]
            # the same transforms of every field; FP64 shell sums in another order
            assert np.max(np.abs(got - base)) <= 1e-12 * np.max(np.abs(base)), mode
    assert np.all(max_err_per_ell(base, np.array(c["values"])) < (1e-10 if prec == pw.PW_FP64 else 1e-4))
    assert any(e["key"].startswith("iy:") for e in pw.tune_entries())
