"""Host side of the streamed paged cache: the block manager against a plain
model over random calls (CPU), and the updates that take the slots from host
lists as runs against the ones that read device lists (GPU)."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2609_35750_amd import inputs


class Model:
    """Blocks, free list and positions as plain Python containers."""

    def __init__(self, nb, bs, ns, mb):
        self.bs, self.mb = bs, mb
        self.free = list(range(nb - 1, -1, -1))
        self.blocks = [[] for _ in range(ns)]
        self.fill = [bs] * ns
        self.live = {}
        self.slot = [{} for _ in range(ns)]

    def append(self, s, pos):
        if any(p < 0 for p in pos) or len(set(pos)) != len(pos) or any(p in self.slot[s] for p in pos):
            return None
        need = max(0, -(-(len(pos) - (self.bs - self.fill[s])) // self.bs))
        if need > len(self.free) or len(self.blocks[s]) + need > self.mb:
            return None
        out = []
        for p in pos:
            if self.fill[s] == self.bs:
                self.blocks[s].append(self.free.pop())
                self.fill[s] = 0
            b = self.blocks[s][-1]
            out.append(b * self.bs + self.fill[s])
            self.fill[s] += 1
            self.live[b] = self.live.get(b, 0) + 1
            self.slot[s][p] = out[-1]
        return out

    def evict(self, s, pos):
        if len(set(pos)) != len(pos) or any(p not in self.slot[s] for p in pos):
            return None
        out = []
        for p in pos:
            out.append(self.slot[s].pop(p))
            b = out[-1] // self.bs
            self.live[b] -= 1
            if self.live[b] == 0:
                if self.blocks[s][-1] == b:
                    self.fill[s] = self.bs
                self.blocks[s].remove(b)
                self.free.append(b)
        return out


@pytest.mark.parametrize("bs", [1, 5, 16])
def test_block_manager_matches_model(bs):
    from paper_2609_35750_amd.kvs import KvsError
    from paper_2609_35750_amd.paged import BlockManager

    rng = np.random.default_rng(bs)
    nb, ns, mb = 60, 3, 40
    bm, m = BlockManager(nb, bs, ns, mb), Model(nb, bs, ns, mb)
    far = [0, 255, 256, 257, 1 << 20, (1 << 31) - 400]   # pages of their own, and their edges

    def call(f, *a):
        try:
            return f(*a).tolist()
        except KvsError:
            return None

    for it in range(1500):
        s = int(rng.integers(ns))
        have = list(m.slot[s])
        if rng.random() < 0.55 or not have:
            start = int(rng.choice(far)) + int(rng.integers(0, 280))
            pos = list(range(start, start + int(rng.integers(1, 40))))
            if rng.random() < 0.1:
                pos.append(pos[0] if rng.random() < 0.5 else -1)
            assert call(bm.append, s, pos) == m.append(s, pos), it
        else:
            pos = [int(x) for x in rng.permutation(have)[: int(rng.integers(1, len(have) + 1))]]
            if rng.random() < 0.1:
                pos.append(pos[0] if rng.random() < 0.5 else 77_777_777)
            assert call(bm.evict, s, pos) == m.evict(s, pos), it
        assert bm.free_blocks() == len(m.free) and bm.live(s) == len(m.slot[s])
        if it % 50 == 0:
            table, n = bm.tables()
            assert [table[i, : n[i]].tolist() for i in range(ns)] == m.blocks
    for s in range(ns):
        assert bm.release(s).tolist() == sorted(m.slot[s].values())
    assert bm.free_blocks() == nb


LISTS = {
    "one": [7],
    "up": list(range(3, 40)),
    "down": list(range(50, 9, -1)),
    "blocks": [16 * b + r for b in (5, 2, 9, 8) for r in range(16)],
    "zigzag": [10, 11, 10 + 5, 14, 13, 20, 22, 21, 23],
    "limit": [2 * i for i in range(512)],          # as many runs as the host call takes
    "long and short": [1900 - 2 * i for i in range(90)] + list(range(1400)) + [1720, 1719, 1710] + list(range(1999, 1949, -1)),
    "out of range": [-1, 0, 1, 2045, 2046, 2047, 2048, 2049, (1 << 31) - 1],
}


@pytest.mark.gpu
@pytest.mark.parametrize("name", LISTS)
@pytest.mark.parametrize("D,bs", [(64, 16), (128, 1)])
def test_host_lists_match_device_lists(name, D, bs):
    from paper_2609_35750_amd import kvs, paged

    dev, lib = torch.device("cuda:0"), kvs.lib
    Hkv, nb = 3, 2048 // bs
    slots = np.asarray(LISTS[name], dtype=np.int32)
    n = slots.size
    pos = np.arange(100, 100 + n, dtype=np.int32)
    pos[n // 2:] += 9   # a gap in the positions ends a run
    kn, vn = (inputs.randn_bf16((n, Hkv, D), 5 + i).to(dev) for i in range(2))
    caches = []
    for host in (True, False):
        k, v = (torch.zeros((nb, Hkv, bs, D), dtype=torch.bfloat16, device=dev) for _ in range(2))
        sp = torch.full((2048,), -1, dtype=torch.int32, device=dev)
        if host:
            p = lambda a: a.ctypes.data_as(ctypes.c_void_p)   # noqa: E731
            stream = torch.cuda.current_stream().cuda_stream
            assert lib.kvs_paged_append_host(kn.data_ptr(), vn.data_ptr(), p(pos), p(slots), n, k.data_ptr(),
                                             v.data_ptr(), sp.data_ptr(), nb, bs, Hkv, D, stream) == kvs.KVS_OK
        else:
            paged.kvs_paged_append(kn, vn, torch.from_numpy(pos).to(dev), torch.from_numpy(slots).to(dev), k, v, sp,
                                   bs)
        full = sp.clone()
        gone = np.ascontiguousarray(slots[n // 3:])
        if host:
            assert lib.kvs_paged_evict_host(p(gone), gone.size, sp.data_ptr(), nb, bs, stream) == kvs.KVS_OK
        else:
            paged.kvs_paged_evict(torch.from_numpy(gone).to(dev), sp, nb, bs)
        caches.append((k.view(torch.int16), v.view(torch.int16), full, sp))
    for a, b in zip(*caches):
        assert torch.equal(a, b)


@pytest.mark.gpu
def test_too_many_runs_fall_back():
    from paper_2609_35750_amd import kvs, paged

    dev = torch.device("cuda:0")
    n, Hkv, D = 1300, 1, 64
    cache = paged.PagedKVCache(4096, 1, 2, 4096, Hkv, D, device=dev)
    for i in range(n):   # blocks of two sequences alternate: evicted and handed out again out of order
        cache.bm.append(i % 2, [i])
    order = np.random.default_rng(3).permutation(np.arange(0, n, 2))
    cache.bm.evict(0, order)
    kn, vn = (inputs.randn_bf16((order.size, Hkv, D), 8 + i).to(dev) for i in range(2))
    slots = cache.append(0, np.arange(5000, 5000 + order.size), kn, vn)
    assert np.count_nonzero(np.abs(np.diff(slots)) != 1) > 512
    sp = cache.slot_pos.cpu().numpy()
    np.testing.assert_array_equal(sp[slots], np.arange(5000, 5000 + order.size))
    got = cache.k.view(torch.int16).cpu().numpy().reshape(-1, Hkv, D)[slots]
    np.testing.assert_array_equal(got, kn.view(torch.int16).cpu().numpy())
    cache.evict(0, np.random.default_rng(4).permutation(np.arange(5000, 5000 + order.size)))
    assert (cache.slot_pos.cpu().numpy()[slots] == -1).all()


@pytest.mark.gpu
def test_host_lists_are_not_captured():
    """A list the host holds is refused by a capturing stream, and a replay changes nothing."""
    from paper_2609_35750_amd import kvs

    dev, lib = torch.device("cuda:0"), kvs.lib
    Hkv, D, bs, nb, n = 2, 64, 16, 8, 20
    slots, pos = np.arange(n, dtype=np.int32), np.arange(n, dtype=np.int32)
    kn = torch.ones((n, Hkv, D), dtype=torch.bfloat16, device=dev)
    k, v = (torch.zeros((nb, Hkv, bs, D), dtype=torch.bfloat16, device=dev) for _ in range(2))
    sp = torch.full((nb * bs,), -1, dtype=torch.int32, device=dev)
    count = torch.zeros(1, device=dev)
    p = lambda a: a.ctypes.data_as(ctypes.c_void_p)   # noqa: E731

    def both():
        stream = torch.cuda.current_stream().cuda_stream
        return (lib.kvs_paged_append_host(kn.data_ptr(), kn.data_ptr(), p(pos), p(slots), n, k.data_ptr(),
                                          v.data_ptr(), sp.data_ptr(), nb, bs, Hkv, D, stream),
                lib.kvs_paged_evict_host(p(slots), n, sp.data_ptr(), nb, bs, stream))

    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        count += 1
        st = both()
    assert st == (kvs.KVS_ERR_UNSUPPORTED, kvs.KVS_ERR_UNSUPPORTED)
    for _ in range(3):
        g.replay()
        torch.cuda.synchronize()
    assert count.item() == 3 and (k == 0).all() and (sp == -1).all()
    assert both() == (kvs.KVS_OK, kvs.KVS_OK)


@pytest.mark.gpu
@pytest.mark.parametrize("down", [False, True])
def test_one_long_run_beside_short_ones(down):
    """So unequal that appends and evictions both share the runs' work by a list of first workgroups."""
    from paper_2609_35750_amd import kvs, paged

    dev, lib = torch.device("cuda:0"), kvs.lib
    Hkv, D, bs, nb = 1, 64, 16, 1024
    slots = np.asarray([13000 + 2 * i for i in range(60)] + list(range(12000)) + [13400 - 2 * i for i in range(60)],
                       dtype=np.int32)
    if down:
        slots = np.ascontiguousarray(slots[::-1])
    n = slots.size
    pos = np.arange(7, 7 + n, dtype=np.int32)
    kn, vn = (inputs.randn_bf16((n, Hkv, D), 50 + i).to(dev) for i in range(2))
    p = lambda a: a.ctypes.data_as(ctypes.c_void_p)   # noqa: E731
    stream = torch.cuda.current_stream().cuda_stream
    caches = []
    for host in (True, False):
        k, v = (torch.zeros((nb, Hkv, bs, D), dtype=torch.bfloat16, device=dev) for _ in range(2))
        sp = torch.full((nb * bs,), -1, dtype=torch.int32, device=dev)
        if host:
            assert lib.kvs_paged_append_host(kn.data_ptr(), vn.data_ptr(), p(pos), p(slots), n, k.data_ptr(),
                                             v.data_ptr(), sp.data_ptr(), nb, bs, Hkv, D, stream) == kvs.KVS_OK
        else:
            paged.kvs_paged_append(kn, vn, torch.from_numpy(pos).to(dev), torch.from_numpy(slots).to(dev), k, v, sp, bs)
        full = sp.clone()
        gone = np.ascontiguousarray(slots[30:])
        if host:
            assert lib.kvs_paged_evict_host(p(gone), gone.size, sp.data_ptr(), nb, bs, stream) == kvs.KVS_OK
        else:
            paged.kvs_paged_evict(torch.from_numpy(gone).to(dev), sp, nb, bs)
        caches.append((k.view(torch.int16), v.view(torch.int16), full, sp))
    for a, b in zip(*caches):
        assert torch.equal(a, b)
