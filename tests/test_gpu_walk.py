"""GPU parity of the one-group-per-lane walk at the sizes where its bookkeeping
can go wrong: segments found from head bits (64 heads in a pass, heads on a
pass's first and last position, more than 64 segments in one build of the
bits, walks longer than one build, more than 64 heads left for the next
build), ranges that start inside a segment, and walks of one pass, of the
ring's depth and of one more, in the ring of three passes and in that of two.
Which ring a case takes and what it leaves for a second build are computed
from the encoded matrix and asserted.

The kernels with several groups per lane find their segments another way and
sum the same products on the same grids, so y must agree bit for bit; it is
also checked against the fp64 definition (the oracle) within 2e-3, the
library's parity bar."""
import numpy as np
import pytest

import workloads
from oracle import spmspv as ref

pytestmark = pytest.mark.gpu

TOL = 2e-3

BUILD = 30   # passes whose heads are marked in one build

# label, M, K, ws, as, R, cols, waves
CASES = [
    ("one_group", 8, 1, 0, 0, 8, 1, 2),
    ("one_group_segments", 40, 2000, 0, 0, 8, 1000, 2),         # 64 heads in every pass, 500 groups a wavefront
    ("one_group_segments_ragged", 50, 3000, 30, 20, 7, 999, 2),
    ("heads_on_pass_edges", 512, 129, 0, 0, 512, 129, 2),       # 64 groups per segment
    ("heads_off_pass_edges", 520, 130, 0, 0, 520, 130, 4),      # 65 groups per segment
    ("segments_64", 300, 64, 50, 0, 256, 64, 4),
    ("segments_65", 300, 65, 50, 0, 256, 65, 4),
    ("more_than_one_build", 2048, 300, 0, 0, 2048, 300, 2),     # 600 passes a wavefront
    ("builds_of_short_segments", 96, 4096, 0, 0, 16, 1024, 2),  # 2 groups per segment, 16 passes
    ("builds_of_short_segments_long", 32, 4096, 0, 0, 32, 1024, 2),
    ("depth_and_one_more", 2048, 64, 0, 50, 1024, 64, 16),
    ("many_workgroups", 5120, 2000, 50, 30, 512, 40, 8),        # over 256 of 8 wavefronts, 2 passes each
    ("second_build_of_many_heads", 96, 2048, 0, 0, 48, 1024, 2),
    ("two_pass_ring", 4090, 2203, 0, 0, 512, 67, 8),
    ("two_pass_ring_ragged", 4333, 4100, 40, 30, 509, 141, 8),
    ("two_pass_ring_second_build", 12336, 2700, 0, 0, 48, 2700, 8),
    ("wide_slices", 1024, 6000, 60, 40, 256, 4096, 8),          # 8 columns per lane in the selection
]


def ring_depth(celty, enc, launch):
    """Passes in flight of a launch with one group per lane: two where over 256
    workgroups of 8 wavefronts walk an estimated 4 to 16 passes each (half of
    the stored groups taken as active), else three."""
    plan = celty.celty_spmspv_plan(enc, launch)
    passes = 0.5 * enc.n_groups / (plan["blocks"] * plan["waves_per_block"] * 64)
    return 2 if plan["waves_per_block"] == 8 and plan["blocks"] > 256 and 4 <= passes <= 16 else 3


def heads_of_later_builds(enc, x, tau, cols, waves):
    """The most segments that start in a wavefront's range past its first
    build (equal ranges: fewer than 16 wavefronts)."""
    assert waves < 16
    xf = np.abs(np.asarray(x, dtype=np.float32))
    counts = np.diff(enc.gptr.astype(np.int64)).reshape(enc.T, enc.K) * (xf > np.float32(tau))
    most = 0
    for t in range(enc.T):
        for k0 in range(0, enc.K, cols):
            c = counts[t, k0:k0 + cols]
            ends = np.cumsum(c[c > 0])
            starts = ends - c[c > 0]
            n = int(ends[-1]) if len(ends) else 0
            for w in range(waves):
                lo, hi = w * n // waves + 64 * BUILD, (w + 1) * n // waves
                most = max(most, int(np.count_nonzero((starts > lo) & (starts < hi))))
    return most


@pytest.mark.parametrize("label,M,K,ws,as_,R,cols,waves", CASES, ids=[c[0] for c in CASES])
def test_walk(label, M, K, ws, as_, R, cols, waves):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2608_01536_amd as celty
    print(f"walk {label}", flush=True)
    dev = torch.device("cuda:0")
    p = workloads.random_small(9000 + len(label), M, K, ws=ws, as_=as_)
    enc = celty.celty_encode(p.W, p.mask, R)
    assert ring_depth(celty, enc, (cols, waves, 1)) == (2 if label.startswith("two_pass_ring") else 3)
    if "second_build" in label:
        assert heads_of_later_builds(enc, p.x, p.tau, cols, waves) > (64 if "many_heads" in label else 0)
    W = enc.to_device(dev)
    x = torch.from_numpy(np.ascontiguousarray(p.x).view(np.int16)).to(dev)
    wsp = celty.new_workspace(W, dev)
    out = {}
    for groups in (1, 2, 4):
        y = torch.full((M,), 0x7C01, dtype=torch.int16, device=dev)   # NaN bits
        celty.celty_spmspv_ex(W, x, p.tau, y, wsp, (cols, waves, groups))
        torch.cuda.synchronize()
        assert int(wsp.count_nonzero()) == 0
        out[groups] = y.cpu().numpy().view(np.uint16)
    err = ref.rel_error(out[1].view(np.float16).astype(np.float64), ref.spmspv_dense_fp64(p.W, p.mask, p.x, p.tau))
    assert err <= TOL, err
    assert np.array_equal(out[1], out[2]) and np.array_equal(out[1], out[4])
