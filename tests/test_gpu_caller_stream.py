"""Bulk retrieves without staging run on the caller's own stream: behind what is on it, before
what follows, with the ticket independent of that stream's life.  Bytes against the CPU oracle."""
import ctypes
import threading

import numpy as np
import pytest

import oracle
from paper_2510_09665_amd import workloads as W

pytestmark = pytest.mark.gpu


def _hip():
    with open("/proc/self/maps") as maps:
        path = next(line.split()[-1] for line in maps if "libamdhip64" in line)
    return ctypes.CDLL(path)


def _case(n, seed):
    from gpu_util import PagedKV, slots_to_device
    g = W.geometry("tiny", NB=256)
    rng = np.random.default_rng(seed)
    slots, tau = (rng.permutation(g.n_slots)[:n * g.CT].astype(np.int64) for _ in range(2))
    src, dst = PagedKV(g, np.arange(g.NB), rng), PagedKV(g, np.arange(g.NB), fill="sentinel")
    want = oracle.gather(g, src.host, slots)
    oracle.scatter(g, want, tau, dst.host)
    return g, src, dst, slots_to_device(slots), slots_to_device(tau), np.arange(1, 1 + n, dtype=np.uint64)


@pytest.mark.parametrize("n", [1, 5])
@pytest.mark.parametrize("kind", ["null", "own", "destroyed", "caller_does_not_wait"])
def test_behind_a_store_and_before_a_consumer(n, kind):
    """Store, retrieve and a consumer of the pages with no host wait between; the retrieve's
    stream has work in front of it (the slot mapping arrives there), and in one case it is
    destroyed before the ticket is asked for."""
    import torch
    from gpu_util import assert_layers_equal
    from paper_2510_09665_amd import lmc
    g, src, dst, d_slots, d_tau, ids = _case(n, 3 + n)
    hip = _hip()
    raw = ctypes.c_void_p()
    if kind == "destroyed":
        assert hip.hipStreamCreateWithFlags(ctypes.byref(raw), 1) == 0
    own = torch.cuda.Stream()
    handle = {"null": None, "destroyed": raw.value}.get(kind, own.cuda_stream)
    outside = torch.cuda.default_stream() if kind == "null" else torch.cuda.ExternalStream(handle)
    with lmc.Context(g, (n + 1) * g.chunk_bytes, staging_chunks=2) as c:
        if kind == "caller_does_not_wait":
            c.tune("caller_waits", 0)
        late = torch.full_like(d_tau, -1)
        busy = torch.zeros(64 << 20, dtype=torch.uint8, device="cuda")
        torch.cuda.synchronize()
        t0 = c.store(src.dev, d_slots, ids)
        with torch.cuda.stream(outside):
            for _ in range(4):
                busy.add_(1)
            late.copy_(d_tau)
        t1 = c.retrieve(ids, late, dst.dev, handle)
        seen = None
        if kind == "caller_does_not_wait":
            c.wait(t1)
        with torch.cuda.stream(outside):
            seen = [d.clone() for d in dst.dev]
        if kind == "destroyed":
            outside.synchronize()
            assert hip.hipStreamDestroy(raw) == 0
        c.wait(t1)
        assert c.test(t0) and c.test(t1)
        torch.cuda.synchronize()
        assert_layers_equal([d.cpu().numpy() for d in dst.dev], dst.host, "pages")
        assert_layers_equal([d.cpu().numpy() for d in seen], dst.host, "consumer on the caller's stream")
        assert c.get_stats()["chunks_retrieved"] == n
        c.clear(ids)                                     # no count stays on the chunks


def test_threads_with_streams_of_their_own():
    """Four threads load from one context, each on its own stream, again and again."""
    import torch
    from gpu_util import PagedKV, assert_layers_equal, slots_to_device
    from paper_2510_09665_amd import lmc
    g = W.geometry("tiny", NB=256)
    rng = np.random.default_rng(17)
    src = PagedKV(g, np.arange(g.NB), rng)
    slots = rng.permutation(g.n_slots)[:4 * g.CT].astype(np.int64)
    want = oracle.gather(g, src.host, slots)
    ids = np.arange(1, 5, dtype=np.uint64)
    with lmc.Context(g, 4 * g.chunk_bytes, staging_chunks=2) as c:
        c.store(src.dev, slots_to_device(slots), ids)
        c.wait()
        work = []
        for i in range(4):
            dst = PagedKV(g, np.arange(g.NB), fill="sentinel")
            tau = rng.permutation(g.n_slots)[:4 * g.CT].astype(np.int64)
            oracle.scatter(g, want, tau, dst.host)
            work.append((dst, slots_to_device(tau), torch.cuda.Stream()))
        torch.cuda.synchronize()
        errors = []

        def load(dst, d_tau, stream):
            try:
                for k in range(25):
                    t = c.retrieve(ids, d_tau, dst.dev, stream)
                    if k % 5 == 4:
                        c.wait(t)
            except Exception as e:
                errors.append(e)

        threads = [threading.Thread(target=load, args=w) for w in work]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
        c.wait()
        assert not errors
        for dst, _, _ in work:
            assert_layers_equal([d.cpu().numpy() for d in dst.dev], dst.host, "thread")
        c.clear(ids)
