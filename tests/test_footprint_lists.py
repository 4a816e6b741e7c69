"""Device footprint of estimates with many fields on a small mesh: the field lists are part of the fixed
allowance for small tables, so a budget that once held such an estimate still does."""
import pytest

pw = pytest.importorskip("paper_2102_08384_amd.pw")


@pytest.mark.parametrize("prec,ell_max,order,held", [(pw.PW_FP32, 8, 8, 77_979_432), (pw.PW_FP32, 6, 8, 63_226_816),
                                                     (pw.PW_FP64, 8, 8, 154_853_012), (pw.PW_FP64, 8, 6, 116_961_684)])
def test_field_lists_need_no_more_budget(prec, ell_max, order, held):
    cfg = pw.Config(stat=pw.PW_XI, los=pw.PW_MIDPOINT, prec=prec, n_mesh=16, ell_max=ell_max, order=order, bin_lo=0.0,
                    bin_width=30.0, n_bins=4, midpoint_parity=pw.PW_PARITY_ALL)
    assert pw.footprint(cfg, 100_003, 500_001) <= held
