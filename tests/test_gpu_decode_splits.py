"""Paged decode across key-split counts, against the fp64 oracle.

The decode cuts a sequence's slots into splits of whole 32-slot tiles and a
merge kernel combines them; both change shape with the number of sequences,
KV heads and live tiles.  The cases sit where that can go wrong: one split,
split counts around the merge's wave and pass sizes, sequences of a tile more
or less than a split, empty and one-slot sequences beside a long one, tables
much wider than what is live.
"""
import math

import pytest
import torch

from oracle import paged as opg
from paper_2609_35750_amd import inputs
from tests.gpu_helpers import announce, assert_close, assert_lse, to_f64

pytestmark = pytest.mark.gpu

CASES = [
    # live entries per sequence, Hkv, G, D, block size, table width in blocks
    ([1], 1, 1, 128, 1, 1),
    ([31, 32, 33, 0, 1], 2, 4, 128, 16, 3),
    ([1024], 8, 4, 128, 16, 64),             # 32 tiles: the widest split of a short sequence
    ([1153, 0, 96], 8, 2, 64, 16, 400),      # table far wider than what is live
    ([4100, 129, 1, 0, 640, 127], 4, 5, 128, 5, 900),
    ([9001], 1, 8, 64, 1, 9100),             # one KV head: the most splits of a sequence
    ([300] * 70 + [2000, 0, 17], 8, 1, 128, 16, 130),   # more than 64 sequences
    ([60 + 7 * i for i in range(140)], 8, 2, 64, 16, 70),   # more than 128 sequences: three registers a lane
]

# The same for batches whose units are listed by a plan kernel (more than 256
# sequences, or more than three rounds of waves), and for those under a narrow
# table, where every sequence is one unit.
LISTED = [
    ([40 + 9 * (i % 31) for i in range(257)], 2, 2, 64, 16, 70),
    ([0, 3000] + [0, 17, 65, 33] * 63 + [1, 2500, 0], 8, 4, 128, 16, 190),
    ([64 * (i % 3) for i in range(599)] + [5000], 8, 1, 64, 16, 320),
    ([100] * 300 + [0] * 300, 4, 2, 128, 16, 300),     # equal ones and empty ones under a wide table
    ([(7 * i) % 41 for i in range(5003)] + [2000], 1, 2, 64, 16, 126),   # more than the plan's threads hold
    ([300, 0, 700] * 80, 16, 1, 128, 16, 200),         # 3,840 waves at 1,024 a round, fewer than 256 sequences
    ([128, 0, 31] * 5, 3, 2, 64, 16, 8),               # one unit each: four tiles wide
    ([(11 * i) % 513 for i in range(256)], 8, 2, 128, 16, 32),   # one unit each: 16 tiles, two rounds
]


@pytest.mark.parametrize("case", CASES + LISTED, ids=lambda c: f"S{len(c[0])}_max{max(c[0])}_Hkv{c[1]}_G{c[2]}_D{c[3]}_bs{c[4]}")
def test_decode_split_shapes(case):
    from paper_2609_35750_amd import paged

    lens, Hkv, G, D, bs, width = case
    dev = torch.device("cuda:0")
    announce(f"decode splits lens={lens[:6]} S={len(lens)} Hkv={Hkv} G={G} D={D} bs={bs} width={width}")
    S, Hq, scale = len(lens), Hkv * G, 1.0 / math.sqrt(D)
    cache = paged.PagedKVCache(sum(-(-n // bs) for n in lens) + 1, bs, S, width, Hkv, D, device=dev)
    kv = []
    for s, n in enumerate(lens):
        k, v = inputs.randn_bf16((n, Hkv, D), 1000 + 2 * s), inputs.randn_bf16((n, Hkv, D), 1001 + 2 * s)
        kv.append((k, v))
        if n:
            cache.append(s, range(n), k.to(dev), v.to(dev))
    q = inputs.randn_bf16((S, Hq, D), 999)
    o, lse = cache.decode(q.to(dev), scale)
    o2, lse2 = cache.decode(q.to(dev), scale)
    assert torch.equal(o.view(torch.int16), o2.view(torch.int16)) and torch.equal(lse, lse2)
    o, lse = to_f64(o), to_f64(lse)
    for s, n in enumerate(lens):
        if n == 0:
            assert (o[s] == 0).all() and (lse[s] == float("-inf")).all()
            continue
        ro, rl = opg.decode(q[s], kv[s][0], kv[s][1], range(n), scale)
        assert_close(f"seq {s} ({n} live) O", o[s], ro)
        assert_lse(f"seq {s} ({n} live)", lse[s], rl)
