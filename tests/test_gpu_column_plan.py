"""dK/dV work plan: key blocks cut into parts, and the per-KV-head or shared
work queues, against the fp64 oracle.

The shapes sit on the plan's lines: the longest block with no parts and one
row-step more, groups whose steps do not divide into equal parts, KV heads
that divide the CUs (a queue each) and that do not (one queue), more items
than workgroups, several traces of which only some are cut.
"""
import pytest
import torch

from paper_2609_35750_amd import inputs
from tests.gpu_helpers import gpu_fwd_bwd
from tests.test_gpu_parity import _parity

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def kvs():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_35750_amd import kvs as k

    return k


CASES = [
    # lengths, Hq, Hkv, D, p, w, s, strategy
    ([1024], 2, 2, 128, 64, 300, 20, "keep_all"),       # 16 steps: never cut
    ([1025], 2, 2, 128, 64, 300, 20, "keep_all"),       # 17 steps
    ([1500], 9, 3, 64, 100, 200, 30, "latest_only"),    # one queue, odd group
    ([1300], 12, 12, 128, 33, 97, 13, "last2"),         # one queue, many KV heads
    ([1601], 10, 2, 128, 130, 350, 40, "keep_all"),     # 130 steps in parts of unequal length
    ([900, 900, 900], 8, 1, 64, 64, 128, 32, "keep_all"),
    ([2100], 16, 8, 64, 256, 400, 64, "keep_all"),
    ([17, 1300, 0, 640, 1, 1299, 128, 64] * 3, 16, 2, 128, 40, 120, 16, "last2"),
    ([200] * 40, 8, 8, 64, 16, 60, 8, "keep_all"),      # 640 whole items on 256 workgroups
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: f"B{len(c[0])}_L{max(c[0])}_H{c[1]}x{c[2]}_D{c[3]}")
def test_column_plan(kvs, case):
    lengths, Hq, Hkv, D, p, w, s, strategy = case
    wl = inputs.custom_workload(f"plan_L{max(lengths)}", Hq, Hkv, D, lengths, p, w, s, strategy, seed=sum(lengths))
    cu = wl.cu_seqlens() if wl.varlen else None
    e = wl.evict_at()
    B = wl.B if wl.B > 1 and not wl.varlen else None
    _parity(kvs, wl, e, cu=cu, B=B)
    t = inputs.make_tensors(wl)
    a, b = (gpu_fwd_bwd(kvs, t["q"], t["k"], t["v"], t["do"], e, wl.softmax_scale, cu_seqlens=cu,
                        max_seqlen=wl.T if wl.varlen else None, B=B) for _ in range(2))
    for key in ("dq", "dk", "dv"):
        assert torch.equal(a[key], b[key]), key
