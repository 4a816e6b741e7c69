"""Write the expected values of tests/test_gpu_mid_planes.py with the FP64 oracle.

    python tests/golden/make_mid_pk_planes.py

Midpoint P_l (Sections 3.2 and 3.3) of a uniform catalog at 64^3 and 128^3, with k-bins that
take in the Nyquist frequency: the meshes on which the library keeps only half of the
separations.  Nothing here calls the library.
"""
import json
import os
import sys
import time

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(os.path.dirname(HERE))
sys.path.insert(0, ROOT)
sys.path.insert(0, os.path.join(ROOT, "tests"))

import numpy as np  # noqa: E402

from gpu_common import rounded, uniform_catalog  # noqa: E402
from oracle.estimators import Config, pk_midpoint  # noqa: E402

CATALOG = dict(seed=620, n_gal=3001, n_ran=9001, center=(0, 0, 1000), side=440)
CASES = [(64, 4, 4, "even"), (64, 4, 4, "all"), (64, 6, 4, "even"), (128, 4, 4, "even"), (128, 4, 4, "all")]


def main():
    gal, ran = (rounded(c, np.float64)[1] for c in uniform_catalog(**CATALOG))
    rows = []
    for n_mesh, ell_max, order, parity in CASES:
        c = dict(n_mesh=n_mesh, box_len=1000.0, box_origin=[-500.0, -500.0, 500.0], assign=3, ell_max=ell_max,
                 order=order, parity=parity, bin_lo=0.004, bin_width=0.0125, n_bins=n_mesh // 4)
        t = time.time()
        res = pk_midpoint(gal, ran, Config(N=n_mesh, L=c["box_len"], b0=tuple(c["box_origin"]), assign=3,
                                           ells=tuple(range(0, ell_max + 1, 2)), order=order, compensate=True,
                                           bin_lo=c["bin_lo"], bin_width=c["bin_width"], n_bins=c["n_bins"],
                                           parity=parity))
        rows.append(dict(c, values=res.values.tolist(), counts=res.counts.tolist()))
        print(f"[golden] {n_mesh}^3 l<={ell_max} order {order} {parity}: {time.time() - t:.0f} s", flush=True)
    with open(os.path.join(HERE, "mid_pk_planes.json"), "w") as fh:
        json.dump({"catalog": CATALOG, "cases": rows}, fh, indent=1)


if __name__ == "__main__":
    main()
