"""Paint of crowded tiles in parts (paint_cut): the list and the parts' blocks fit their scratch memory
whatever the tile counts, and a mesh painted in parts has the bits of the one painted whole (a
memory-lean plan of a small k-sphere leaves no scratch for parts), on 64, 512 and 4096 tiles, with room
for every part and with the little of a single field: one tile with most of the catalog, many just above
and below a part's size."""
import ctypes

import numpy as np
import pytest

from gpu_common import say

pw = pytest.importorskip("paper_2102_08384_amd.pw")

MOST_OF_TILE = 16


class _Cut(ctypes.Structure):
    _fields_ = [("per", ctypes.c_int), ("most", ctypes.c_int), ("room", ctypes.c_int), ("list_bytes", ctypes.c_int), ("mem", ctypes.c_void_p)]


def paint_cut(n_mesh, n_part, scratch_bytes):
    fn = pw._lib["_ZN2pw9paint_cutEilPvm"]
    fn.restype, fn.argtypes = _Cut, [ctypes.c_int, ctypes.c_long, ctypes.c_void_p, ctypes.c_ulong]
    return fn(n_mesh, n_part, ctypes.c_void_p(4096), scratch_bytes)


def listed(counts, cut):
    per = cut.per
    if cut.room:  # the scan's rule where room is short
        free = cut.room - np.count_nonzero(counts)
        per = max(per, -(-int(counts.sum()) // free)) if free > 0 else int(counts.sum())
    parts = np.minimum(-(-counts // per), MOST_OF_TILE)
    return int(parts[parts > 1].sum())


@pytest.mark.parametrize("n_mesh", [16, 32, 64, 128, 256, 512])
def test_parts_fit(n_mesh):
    rng = np.random.default_rng(n_mesh)
    ntiles, seen, tight = max(1, n_mesh // 16) ** 3, 0, 0
    for _ in range(400):
        n = int(10 ** rng.uniform(0, 9.3))
        scratch = int(10 ** rng.uniform(2, 10.5))
        cut = paint_cut(n_mesh, n, scratch)
        if cut.per == 0:
            assert cut.most == 0
            continue
        seen += 1
        tight += cut.room > 0
        assert n_mesh < 512 and 2 <= cut.most <= 1024
        assert cut.list_bytes >= 8 + 16 * (ntiles + cut.most) and cut.list_bytes % 256 == 0
        assert cut.list_bytes + cut.most * 18 ** 3 * 8 <= scratch
        over = n // (cut.per + 1)  # as many tiles as can hold one record more than a part
        for counts in ([n], [cut.per + 1] * over + [n - over * (cut.per + 1)], [cut.per] * (n // cut.per),
                       rng.multinomial(n, rng.dirichlet(np.full(ntiles, 0.05)))):
            assert listed(np.asarray(counts), cut) <= cut.most
    assert (seen > 20 and tight > 5) == (n_mesh < 512)


@pytest.mark.gpu
@pytest.mark.parametrize("n_mesh,prec,assign", [(64, pw.PW_FP32, pw.PW_TSC), (64, pw.PW_FP64, pw.PW_CIC), (128, pw.PW_FP32, pw.PW_TSC), (128, pw.PW_FP64, pw.PW_CIC),
                                                (256, pw.PW_FP64, pw.PW_TSC), (256, pw.PW_FP32, pw.PW_CIC)])
def test_parts_sum_to_the_mesh_of_many_tiles(n_mesh, prec, assign):
    say(f"paint in parts, many tiles: {n_mesh}^3 prec {prec} assign {assign}")
    dt = np.float64 if prec == pw.PW_FP64 else np.float32
    n = 1_300_001 if n_mesh == 256 else 700_001
    side = 16000.0 / n_mesh  # of a tile, box 1000
    rng = np.random.default_rng(40 + n_mesh)
    # half of the catalog in one tile, a fifth in two more, the rest in a slab of crowded and thin tiles
    at = ((3, 2, 1), (0, 1, 3), (1, 1, 3)) if n_mesh == 64 else ((3, 2, 4), (5, 5, 5), (6, 5, 5))
    u = [rng.uniform(0.05, 0.95, (n // k, 3)) * side + np.array(a) * side for k, a in zip((2, 10, 10), at)]
    u.append(rng.uniform(0, 1, (n - sum(map(len, u)), 3)) * (990, 990, 60))
    pos = np.concatenate(u) + (-500, -500, 500)
    rng.shuffle(pos)
    xyzw = np.concatenate([pos, rng.uniform(0.5, 1.5, (n, 1))], axis=1).astype(dt)
    split = n // 4
    base = dict(stat=pw.PW_PK, los=pw.PW_BISECTOR, assign=assign, prec=prec, n_mesh=n_mesh, box_len=1000.0,
                box_origin=(-500.0, -500.0, 500.0), ell_max=4, order=4, bin_lo=0.005, bin_width=0.01, n_bins=2)
    meshes = []
    with pw.Context(0) as ctx:
        # no room, room for every part, room of one field
        for kind in (dict(memory_lean=1), dict(), dict(los=pw.PW_MIDPOINT, ell_max=0, order=0)):
            ctx.estimate(pw.Config(**{**base, **kind}), xyzw[:split], xyzw[split:],
                         ran_nbar=np.full(n - split, 1e-4, dtype=dt))
            meshes.append(ctx.inspect(0, dt))
            if "memory_lean" in kind:  # its scratch is the k-sphere: 49 fields of slots padded to 128 bytes
                cut = paint_cut(n_mesh, n, ctx.inspect(1, np.uint8).nbytes + 49 * 128)
                assert cut.per == 0 or 0 < cut.room < 16  # no more room than occupied tiles (the slab's 16): none is cut
            elif not kind:  # at least the x pass's output: 49 fields of n_mesh^2 rows of 128 bytes
                cut = paint_cut(n_mesh, n, 49 * n_mesh ** 2 * 128)
                assert 0 < cut.per < n // 10
            else:  # one field of n_mesh^2 rows of n_mesh / 2 + 1 values, padded to 128 bytes
                row = -(-(n_mesh // 2 + 1) * 2 * np.dtype(dt).itemsize // 128) * 128
                cut = paint_cut(n_mesh, n, n_mesh ** 2 * row)
                assert cut.per > 0 and (cut.room > 0) == (n_mesh < 256)
    assert np.any(meshes[0] != 0)
    assert np.array_equal(meshes[0], meshes[1]) and np.array_equal(meshes[0], meshes[2])
