"""dK/dV column kernel, where its two row halves and its ring of three tiles
begin: one to five steps of 64 rows, the last of them with rows in one half
only or a single row, blocks whose second half of keys or rows is absent, and
groups that put one to three q-heads between two steps of rows.  Against the
fp64 oracle; dK and dV are also the same in two runs.
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


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("G", [1, 2, 3])
@pytest.mark.parametrize("lengths", [[1], [32], [33, 64, 65, 96], [97, 128, 129], [160, 161, 192, 193], [257, 31, 0, 289]],
                         ids=lambda x: "_".join(map(str, x)))
def test_column_rows(kvs, lengths, G, D):
    wl = inputs.custom_workload(f"rows_{lengths[0]}", 2 * G, 2, D, lengths, 8, 24, 5, "keep_all", seed=sum(lengths) + G)
    cu = wl.cu_seqlens() if wl.varlen else None
    e = wl.evict_at()
    _parity(kvs, wl, e, cu=cu, B=None)
    t = inputs.make_tensors(wl)
    a, b = (gpu_fwd_bwd(kvs, t["q"], t["k"], t["v"], t["do"], e, wl.softmax_scale, cu_seqlens=cu,
                        max_seqlen=wl.T if wl.varlen else None) for _ in range(2))
    for key in ("dk", "dv"):
        assert torch.equal(a[key], b[key]), key
