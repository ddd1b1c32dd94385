"""Workspaces between what a call takes and what the query gives.

The backward cuts as many key blocks as its workspace holds partial sums for.
dQ does not depend on that; dK and dV are the same sums in another order (32-bit
sums, rounded once: at most one bf16 spacing apart, and different in few
values).  A byte less than the least is refused; the bytes around the workspace
stay as they are.  The paged decode takes the query's size, and with a wide table
that of equal splits, which may hold a few units less; partial results in either
layout of their rows.
"""
import ctypes
import math

import numpy as np
import pytest
import torch

from oracle import paged as opg
from paper_2609_35750_amd import inputs
from tests.gpu_helpers import announce, assert_close, assert_lse, to_f64, ulp_bf16

pytestmark = pytest.mark.gpu

GUARD = 4096


def _up(n):
    return (n + 255) // 256 * 256


def _call(fn, sizes, device):
    """fn(workspace pointer, bytes) -> status for every size; the guard bytes must survive."""
    for n in sizes:
        buf = torch.full((GUARD + n + GUARD,), 0x5B, dtype=torch.uint8, device=device)
        yield n, fn(buf.data_ptr() + GUARD, n)
        torch.cuda.synchronize()
        b = buf.cpu().numpy()
        assert (b[:GUARD] == 0x5B).all() and (b[GUARD + n:] == 0x5B).all(), n


@pytest.mark.parametrize("lens,Hq,Hkv,D", [
    ([2100], 16, 8, 128),
    ([1500, 33, 900, 0, 1], 9, 3, 64),      # one queue for all heads
    ([640], 64, 64, 64),                    # never cut: more blocks than workgroups
    ([8300], 2, 1, 64),                     # above 8,192 tokens some partial sums are always needed
], ids=lambda x: str(x))
def test_backward_workspace_sizes(lens, Hq, Hkv, D):
    from paper_2609_35750_amd import kvs

    lib, dev = kvs.lib, torch.device("cuda:0")
    announce(f"workspace lens={lens} Hq={Hq} Hkv={Hkv} D={D}")
    wl = inputs.custom_workload("workspace", Hq, Hkv, D, lens, 64, 200, 20, "keep_all", seed=len(lens))
    B, N, T = len(lens), sum(lens), max(lens)
    t = inputs.make_tensors(wl)
    q, k, v, do = (t[n].to(dev).contiguous() for n in ("q", "k", "v", "do"))
    e = torch.from_numpy(np.asarray(wl.evict_at(), dtype=np.int32)).to(dev)
    cu = torch.from_numpy(np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)).to(dev)
    scale = wl.softmax_scale
    o, lse = kvs.kvs_evict_attn_fwd(q, k, v, e, scale, cu, T)
    full = kvs.kvs_evict_attn_bwd(do, q, k, v, o, lse, e, scale, cu, T)

    query = lib.kvs_evict_attn_varlen_bwd_workspace(B, N, T, Hq, Hkv, D)
    blocks = B * -(-T // 128)
    least = _up(8 * (B + N // 64 + 2)) + 2 * _up(4 * Hq * N) + 2 * _up(8 * blocks)
    if T > 8192:
        cap = min(2048 // Hkv, blocks * -(-(-(-T // 64)) // 64))
        least += _up(8 * (blocks + cap)) - _up(8 * blocks) + _up(cap * Hkv * 1024 * D)
    dq, dk, dv = torch.empty_like(q), torch.empty_like(k), torch.empty_like(v)
    stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)

    def call(ws, n):
        for x in (dq, dk, dv):
            x.fill_(math.nan)
        return lib.kvs_evict_attn_varlen_bwd(
            do.data_ptr(), q.data_ptr(), k.data_ptr(), v.data_ptr(), o.data_ptr(), lse.data_ptr(), e.data_ptr(),
            cu.data_ptr(), dq.data_ptr(), dk.data_ptr(), dv.data_ptr(), B, N, T, Hq, Hkv, D, scale, ws, n, stream)

    assert query >= least
    for n, st in _call(call, sorted({least, least + 1024 * D * Hkv * 3 + 5000, (least + query) // 2, query}), dev):
        assert st == kvs.KVS_OK, (n, lib.kvs_last_error())
        assert torch.equal(dq.view(torch.int16), full[0].view(torch.int16))
        for a, b in ((dk, full[1]), (dv, full[2])):
            x, y = (z.double().cpu().numpy() for z in (a, b))
            assert (np.abs(x - y) <= ulp_bf16(np.maximum(np.abs(x), np.abs(y))) + 1e-5).all()
            assert (x != y).mean() < 0.02
    for n, st in _call(call, [least - 1], dev):
        assert st == kvs.KVS_ERR_WORKSPACE


@pytest.mark.parametrize("lens,Hkv,G,D,width", [
    ([3000], 4, 2, 128, 200),                       # a row for every unit
    ([900, 33, 0, 1500] * 40, 8, 2, 64, 100),       # rows for the cut sequences only
    ([200, 1700] * 100, 8, 1, 128, 110),
    ([70] * 290 + [2000], 8, 4, 128, 130),          # the same, units listed
    ([2000] + [0, 70] * 160, 1, 2, 64, 130),
    ([600] * 64, 8, 2, 128, 300),                   # equal splits: two a sequence, and no room for the lookup
], ids=lambda x: f"S{len(x)}" if isinstance(x, list) else str(x))
def test_decode_workspace_sizes(lens, Hkv, G, D, width):
    from paper_2609_35750_amd import kvs, paged

    lib, dev, bs = kvs.lib, torch.device("cuda:0"), 16
    announce(f"decode workspace S={len(lens)} Hkv={Hkv} G={G} D={D} width={width}")
    S, Hq, scale = len(lens), Hkv * G, 1.0 / math.sqrt(D)
    cache = paged.PagedKVCache(sum(-(-n // bs) for n in lens), bs, S, width, Hkv, D, device=dev)
    kv = [[inputs.randn_bf16((n, Hkv, D), 700 + 2 * s + i) for i in range(2)] for s, n in enumerate(lens)]
    for s, n in enumerate(lens):
        if n:
            cache.append(s, range(n), kv[s][0].to(dev), kv[s][1].to(dev))
    q = inputs.randn_bf16((S, Hq, D), 699)
    qd = q.to(dev)
    table, nblk = cache.device_tables()
    ref = [opg.decode(q[s], kv[s][0], kv[s][1], range(n), scale) for s, n in enumerate(lens)]

    query = lib.kvs_paged_decode_workspace(S, Hq, Hkv, D, width, bs)
    rows = S * Hq * min(-(-(1024 if D == 128 else 2048) // (S * Hkv)), max(1, width * bs // 128))
    least = _up(rows * D * 4) + _up(rows * 8)
    if S == 1:   # a table of 25 splits of four tiles, but 50 units of two
        least = query
    o, lse = torch.empty_like(qd), torch.empty((S, Hq), dtype=torch.float32, device=dev)
    stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)

    def call(ws, n):
        o.fill_(math.nan), lse.fill_(math.nan)
        return lib.kvs_paged_decode(qd.data_ptr(), cache.k.data_ptr(), cache.v.data_ptr(), cache.slot_pos.data_ptr(),
                                    table.data_ptr(), nblk.data_ptr(), o.data_ptr(), lse.data_ptr(), S, Hq, Hkv, D,
                                    cache.num_blocks, bs, width, scale, ws, n, stream)

    for n, st in _call(call, sorted({least, query}), dev):
        assert st == kvs.KVS_OK, (n, lib.kvs_last_error())
        x, y = to_f64(o), to_f64(lse)
        live = [s for s in range(S) if lens[s]]
        assert_close(f"{n} bytes: O", x[live], np.stack([ref[s][0] for s in live]))
        assert_lse(f"{n} bytes", y[live], np.stack([ref[s][1] for s in live]))
        for s in range(S):
            assert lens[s] or ((x[s] == 0).all() and (y[s] == -math.inf).all())
    for n, st in _call(call, [least - 1], dev):
        assert st == kvs.KVS_ERR_WORKSPACE
