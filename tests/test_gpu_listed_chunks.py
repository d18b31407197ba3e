"""Transfers without staging whose chunks lie in pool slots of any order: one launch takes a
list of up to 256 chunks.  Byte for byte against the CPU oracle at the lengths around that
limit, with chunks that the store skips, with runs long enough to go unlisted, with rows of
every kind, layer by layer, and with "link_groups" 0, where launches take no list."""
import zlib

import numpy as np
import pytest

import oracle
from paper_2510_09665_amd import workloads as W

pytestmark = pytest.mark.gpu

ROWS = {
    "rows_of_16": dict(L=3, P=2, H=2, D=32, e=2, BS=4, NB=700, CT=4),
    "wide_hnd": dict(L=2, P=2, H=3, D=33, e=1, BS=4, NB=700, CT=4, layout="HND"),
    "narrow": dict(L=2, P=1, H=2, D=3, e=1, BS=4, NB=1300, CT=8),
}


def _fragment(c, g, n, rng, run):
    """Fills the pool and frees runs of up to `run` slots until n are free."""
    total = c.pool_slots()
    other = (1 << 32) + np.arange(total, dtype=np.uint64)
    c.put_host(other, np.zeros(total * g.chunk_bytes, dtype=np.uint8))
    free, at = [], 0
    while len(free) < n:
        k = int(min(rng.integers(1, run + 1), n - len(free)))
        free += list(range(at, at + k))
        at += k + 1
    c.clear(other[free])


@pytest.mark.parametrize("rows", list(ROWS))
@pytest.mark.parametrize("n,run", [(2, 1), (256, 1), (257, 1), (290, 3), (600, 270)])
@pytest.mark.parametrize("how", ["by_size", "layers", "no_list"])
def test_scattered_slots_match_oracle(rows, n, run, how):
    from gpu_util import PagedKV, assert_layers_equal, slots_to_device
    from paper_2510_09665_amd import lmc
    g = W.KVGeometry(**ROWS[rows])
    rng = np.random.default_rng(zlib.crc32(("%s %d" % (rows, n)).encode()))
    n_tok = n * g.CT
    assert n_tok <= g.n_slots
    slots, tau = (rng.permutation(g.n_slots)[:n_tok].astype(np.int64) for _ in range(2))
    slots[rng.integers(0, n_tok, 2)] = -1
    src, dst = PagedKV(g, np.arange(g.NB), rng), PagedKV(g, np.arange(g.NB), fill="sentinel")
    want = oracle.gather(g, src.host, slots)
    ids = rng.permutation(1 << 20)[:n].astype(np.uint64)
    old = np.arange(n // 2, n // 2 + n // 5)               # stored before: the store skips them
    with lmc.Context(g, (2 * n + 2) * g.chunk_bytes, staging_chunks=2,
                     flags=lmc.LMC_FLAG_DIRECT if how == "layers" else 0) as c:
        if how == "no_list":
            c.tune("link_groups", 0)
        _fragment(c, g, n, rng, run)
        if old.size:
            c.put_host(ids[old], want[old])
        c.reset_stats()
        d_slots, d_tau = slots_to_device(slots), slots_to_device(tau)
        if how == "layers":
            t = c.store_begin(d_slots, ids)
            for l in range(g.L):
                c.store_layers(t, l, 1, src.dev)
        else:
            c.store(src.dev, d_slots, ids)
        c.wait()
        st = c.get_stats()
        assert st["chunks_stored"] == n - old.size and st["bytes_d2h"] == (n - old.size) * g.chunk_bytes
        if how == "by_size" and run == 1:
            assert st["gather_launches"] <= 2 + n // 256      # and not one for each run of slots
        for i in range(n):
            assert np.array_equal(c.get_host(ids[i]), want[i]), i
        if how == "layers":
            c.retrieve_layerwise(ids, d_tau, dst.dev, 1)
        else:
            c.retrieve(ids, d_tau, dst.dev)
        c.wait()
        assert c.get_stats()["bytes_h2d"] == n * g.chunk_bytes
    oracle.scatter(g, want, tau, dst.host)
    assert_layers_equal([d.cpu().numpy() for d in dst.dev], dst.host, rows)


def test_cost_of_a_call_grows_with_its_chunks_and_no_faster():
    """"link_groups" 0 and every other pool slot taken: a launch for each chunk.  Four times the
    chunks take about four times as long to enqueue; a search that begins anew for each launch took
    ten times."""
    import time
    import torch
    from gpu_util import slots_to_device
    from paper_2510_09665_amd import lmc
    g = W.KVGeometry(L=1, P=1, H=1, D=16, e=1, BS=4, NB=4, CT=4)
    most = 131072
    layers = [torch.zeros(g.layer_bytes, dtype=torch.uint8, device="cuda")]
    slots = slots_to_device(np.tile(np.arange(g.CT, dtype=np.int64), most))
    with lmc.Context(g, 2 * most * g.chunk_bytes, staging_chunks=2) as c:
        c.tune("link_groups", 0)
        other = (1 << 32) + np.arange(2 * most, dtype=np.uint64)
        c.put_host(other, np.zeros(2 * most * g.chunk_bytes, dtype=np.uint8))
        c.clear(other[::2])
        took = {}
        for n in (most // 4, most) * 3:
            ids = np.arange(1, n + 1, dtype=np.uint64)
            torch.cuda.synchronize()
            t = time.perf_counter()
            ticket = c.store(layers, slots, ids)
            took[n] = min(took.get(n, 1e9), time.perf_counter() - t)
            c.wait(ticket)
            c.clear(ids)
        assert c.get_stats()["gather_launches"] == 3 * (most + most // 4)
        assert took[most] < 6.5 * took[most // 4], took
