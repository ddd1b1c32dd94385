"""Rounding of the paged decode: the bf16 probabilities of a tile of 32 slots are
taken against the tile's own maximum, so that a result does not lose precision
with the length of the run of tiles one wave walks.

A model with exactly these roundings (everything else in 64 bits) gives the
same bf16 outputs but for values that a 32-bit sum puts on the other side of a
rounding boundary: the sums' error is a few 2^-24 of the largest term against
a bf16 spacing of 2^-8, so fewer than 2 values in 100 may differ (probabilities
against a running maximum change about half of the values).
"""
import math

import pytest
import torch

from paper_2609_35750_amd import inputs
from tests.gpu_helpers import announce

pytestmark = pytest.mark.gpu


def _model(q, k, v, scale):
    """O [G, D] (bf16 values) of one KV head: q [G, D], k and v [n, D], all fp64 holding bf16 values."""
    s2 = torch.tensor(scale * 1.4426950408889634, dtype=torch.float32).double()
    x = (k @ q.t().contiguous()).float().double() * s2          # [n, G], log2 units
    m = x.max(0).values
    num, den = torch.zeros(q.shape[0], v.shape[1], dtype=torch.float64, device=q.device), 0.0
    for t in range(0, k.shape[0], 32):
        xt = x[t:t + 32]
        mt = xt.max(0).values
        p = torch.exp2(xt - mt)
        w = torch.exp2(mt - m)
        num += w[:, None] * (p.to(torch.bfloat16).double().t().contiguous() @ v[t:t + 32])
        den = den + w * p.sum(0)
    return (num / den[:, None]).to(torch.bfloat16).double()


@pytest.mark.parametrize("lens,Hkv,G,D,width", [
    ([5000], 2, 4, 64, 400),                           # short units: two tiles
    ([33, 448, 1000, 32, 2000, 777] * 4, 8, 3, 64, 300),
    ([200 + 40 * i for i in range(48)], 4, 8, 128, 160),
    ([300] * 300, 4, 2, 128, 19),                      # one unit a sequence
], ids=["one", "ragged_d64", "ragged_d128", "many"])
def test_decode_rounds_by_tile(lens, Hkv, G, D, width):
    from paper_2609_35750_amd import paged

    dev = torch.device("cuda:0")
    announce(f"decode rounding S={len(lens)} max={max(lens)} Hkv={Hkv} G={G} D={D}")
    S, bs, scale = len(lens), 16, 1.0 / math.sqrt(D)
    cache = paged.PagedKVCache(sum(-(-n // bs) for n in lens), bs, S, width, Hkv, D, device=dev)
    kv = []
    for s, n in enumerate(lens):
        k, v = (inputs.randn_bf16((n, Hkv, D), 300 + 2 * s + i).to(dev) for i in range(2))
        kv.append((k, v))
        cache.append(s, range(n), k, v)
    q = inputs.randn_bf16((S, Hkv * G, D), 299).to(dev)
    o = cache.decode(q, scale)[0].double()
    ref = torch.stack([torch.cat([_model(q[s, g * G:(g + 1) * G].double(), kv[s][0][:, g].double(),
                                         kv[s][1][:, g].double(), scale) for g in range(Hkv)]) for s in range(S)])
    differ = float((o != ref).double().mean())
    print(f"[rounding] {differ:.2%} of {o.numel()} values differ", flush=True)
    assert differ < 0.02
