"""The automatic launch shape's rule for 8-wavefront workgroups (host only):
one workgroup per compute unit where a slice then has at most one column per
lane, two per unit where it would have more or where nothing is pruned, and
fewer than one where a workgroup holds little for its merge."""
import ctypes

import numpy as np
import pytest

import paper_2608_01536_amd as celty

FAKE = 0x10000


@pytest.mark.parametrize("M,K,density,cols,blocks", [
    (4096, 11008, 0.5, 344, 256),     # one per unit
    (5120, 12800, 0.5, 512, 250),     # exactly one column per lane
    (5120, 12801, 0.5, 256, 510),     # more: two per unit
    (5120, 13824, 0.5, 272, 510),
    (7168, 7168, 0.5, 399, 252),
    (7168, 7168, 1.0, 200, 504),      # nothing pruned
    (7168, 7168, 0.93, 399, 252),     # just under 15/16
    (4096, 4096, 0.5, 128, 256),      # heavy enough for its merge
    (4096, 4096, 0.3, 152, 216),      # light: 112 bytes per ticket
    (4096, 4096, 0.1, 256, 128),      # never below 128
    (512, 2048, 0.1, 64, 64),         # already below
    (8192, 8192, 0.5, 256, 256),      # 16 wavefronts: as before
])
def test_automatic_slices(M, K, density, cols, blocks):
    R = celty.default_tile_rows(M, K)
    d = celty.celty_rlc_csc(2, M, K, R, -(-M // R), 4, int(M * K * density) // 8, 0, 0, 0, 1.0, 0, FAKE, FAKE, FAKE, FAKE)
    out, n = celty.celty_launch(), ctypes.c_int64()
    assert celty._plan(ctypes.byref(d), None, ctypes.byref(out), ctypes.byref(n), None) == celty.CELTY_OK
    assert (out.cols_per_block, n.value) == (cols, blocks)


def test_tall_tiles_keep_their_slices():
    # 8 wavefronts asked for on a tall tile: wider slices would not leave the
    # tile room in LDS
    M, K, R = 200000, 15000, 39000
    d = celty.celty_rlc_csc(2, M, K, R, -(-M // R), 4, 3 * 10 ** 6, 0, 0, 0, 1.0, 0, FAKE, FAKE, FAKE, FAKE)
    out, n = celty.celty_launch(), ctypes.c_int64()
    L = celty.celty_launch(0, 8, 0, 0)
    assert celty._plan(ctypes.byref(d), ctypes.byref(L), ctypes.byref(out), ctypes.byref(n), None) == celty.CELTY_OK
    assert (out.cols_per_block, n.value) == (239, 378)


def _cut(M, K, groups, R=None, launch=None, layout=celty.LAYOUT_RLC, nnz=0):
    """(columns, wavefronts, workgroups) of the plan."""
    R = R or celty.default_tile_rows(M, K)
    d = celty.celty_rlc_csc(2, M, K, R, -(-M // R), 4, groups, nnz, nnz, 0, 1.0, layout, FAKE, FAKE, FAKE, FAKE)
    out, n = celty.celty_launch(), ctypes.c_int64()
    L = None if launch is None else ctypes.byref(celty.celty_launch(*launch))
    assert celty._plan(ctypes.byref(d), L, ctypes.byref(out), ctypes.byref(n), None) == celty.CELTY_OK
    return out.cols_per_block, out.waves_per_block, n.value


# the stored groups of uniform masks at weight sparsities of 90 and 95 %, and of 97.5 % in the fourth
@pytest.mark.parametrize("M,K,groups,cols,blocks", [
    (6732, 10452, 1136000, 320, 462),   # ws 90: near two per unit, not cut to something uneven between
    (5838, 15932, 1096000, 384, 504),   # ws 95: nor to more than one column per lane
    (4636, 15004, 826000, 320, 470),
    (1000, 40000, 250000, 640, 252),    # slices of several columns per lane already: kept
    (624, 23864, 184000, 508, 141),     # the fewest slices with one column per lane
    (953, 11184, 129000, 350, 128),
])
def test_light_slices_stay_within_one_per_unit_and_one_column_per_lane(M, K, groups, cols, blocks):
    assert _cut(M, K, groups) == (cols, 8, blocks)


@pytest.mark.parametrize("M,K,density,layout,launch,want", [
    # several groups per lane: neither rule
    (7168, 7168, 0.5, celty.LAYOUT_RLC, (0, 0, 2, 0), (200, 8, 504)),
    (4096, 4096, 0.2, celty.LAYOUT_RLC, (0, 0, 2, 0), (128, 8, 256)),
    (7168, 7168, 0.5, celty.LAYOUT_RLC, (0, 0, 4, 0), (200, 8, 504)),
    (4096, 4096, 0.2, celty.LAYOUT_RLC, (0, 0, 4, 0), (128, 8, 256)),
    # the swizzled tile and the 16-bit rows: as the plain kernel
    (7168, 7168, 0.5, celty.LAYOUT_RLC, (0, 0, 0, 1), (399, 8, 252)),
    (7168, 7168, 0.5, celty.LAYOUT_ROWS16, (0, 0, 0, 0), (399, 8, 252)),
    # interleaved: the plain kernel's slices (so the same y), with 16 wavefronts
    # where the plain kernel gives up the second workgroup
    (7168, 7168, 0.5, celty.LAYOUT_INTERLEAVED, (0, 0, 0, 0), (399, 16, 252)),
    (7168, 7168, 0.5, celty.LAYOUT_INTERLEAVED, (0, 8, 0, 0), (200, 8, 504)),
    (4096, 11008, 0.5, celty.LAYOUT_INTERLEAVED, (0, 0, 0, 0), (344, 16, 256)),
    (5120, 5120, 0.4, celty.LAYOUT_INTERLEAVED, (0, 0, 0, 0), (205, 8, 250)),
    (4096, 4096, 0.5, celty.LAYOUT_INTERLEAVED, (0, 0, 0, 0), (128, 8, 256)),
    (8192, 8192, 0.5, celty.LAYOUT_INTERLEAVED, (0, 0, 0, 0), (256, 16, 256)),
])
def test_slices_of_the_other_walks(M, K, density, layout, launch, want):
    assert _cut(M, K, int(M * K * density) // 8, layout=layout, launch=launch) == want


@pytest.mark.parametrize("M,K,ws", [(4096, 4096, 80), (4096, 4096, 70), (3001, 1003, 75), (2048, 2048, 60)])
def test_light_slices_are_the_same_in_every_layout(M, K, ws):
    # a layout's stored groups depend on its padding and alignment; the slices
    # set the grids, and with them y's last bits, so they may not
    rng = np.random.default_rng(M + K + ws)
    W = (rng.standard_normal((M, K), dtype=np.float32) * 0.02).astype(np.float16)
    mask = (rng.random((M, K), dtype=np.float32) >= ws / 100).astype(np.uint8)
    cuts = set()
    for layout in (celty.LAYOUT_RLC, celty.LAYOUT_ROWS16, celty.LAYOUT_INTERLEAVED):
        groups, nnz, _ = celty.celty_encode_plan(W, mask, celty.default_tile_rows(M, K), layout)
        cuts.add(_cut(M, K, groups, layout=layout, nnz=nnz))
    assert len(cuts) == 1, cuts
