"""GPU parity of the one-group-per-lane walk at the sizes where its bookkeeping
can go wrong: segments found from head bits (64 heads in a pass, heads on a
pass's first and last position, more than 64 segments in one build of the
bits, walks longer than one build), ranges that start inside a segment, and
walks of one pass, of the ring's depth and of one more.

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
    ("two_pass_ring", 5120, 2000, 50, 30, 512, 40, 8),          # over 256 workgroups of 8 wavefronts
    ("wide_slices", 1024, 6000, 60, 40, 256, 4096, 8),          # 8 columns per lane in the selection
]


@pytest.mark.parametrize("label,M,K,ws,as_,R,cols,waves", CASES, ids=[c[0] for c in CASES])
def test_walk(label, M, K, ws, as_, R, cols, waves):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2608_01536_amd as celty
    print(f"walk {label}", flush=True)
    dev = torch.device("cuda:0")
    p = workloads.random_small(9000 + len(label), M, K, ws=ws, as_=as_)
    W = celty.celty_encode(p.W, p.mask, R).to_device(dev)
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
