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


def _products(stream, n=40):
    """Some milliseconds of work on a stream."""
    import torch
    with torch.cuda.stream(stream):
        a = torch.ones(4096, 4096, device="cuda", dtype=torch.bfloat16)
        for _ in range(n):
            a = (a @ a).clamp_(-1, 1)
    return a


@pytest.mark.parametrize("first,second", [("bulk", "other"), ("layers", "other"), ("layers", "same"), ("bulk", "null")])
def test_retrieves_into_the_same_pages_take_effect_in_the_order_of_the_calls(first, second):
    """The first retrieve has to wait for what is on its stream; the second, from a stream that is
    idle, fills the same pages with another chunk, and the pages end up with that one."""
    import torch
    from gpu_util import PagedKV, assert_layers_equal, slots_to_device
    from paper_2510_09665_amd import lmc
    g = W.geometry("tiny", NB=256)
    rng = np.random.default_rng(31)
    src, dst = PagedKV(g, np.arange(g.NB), rng), PagedKV(g, np.arange(g.NB), fill="sentinel")
    slots = rng.permutation(g.n_slots)[:2 * g.CT].astype(np.int64)
    tau = rng.permutation(g.n_slots)[:g.CT].astype(np.int64)
    oracle.scatter(g, oracle.gather(g, src.host, slots)[1:], tau, dst.host)
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    with lmc.Context(g, 2 * g.chunk_bytes, staging_chunks=2) as c:
        c.wait(c.store(src.dev, slots_to_device(slots), [1, 2]))
        d_tau = slots_to_device(tau)
        torch.cuda.synchronize()
        keep = _products(a)
        assert not a.query()
        if first == "bulk":
            c.retrieve([1], d_tau, dst.dev, a)
        else:
            c.retrieve_layerwise([1], d_tau, dst.dev, 1, a)
        c.retrieve([2], d_tau, dst.dev, {"other": b, "same": a, "null": None}[second])
        c.wait()
        torch.cuda.synchronize()
        del keep
        assert_layers_equal([d.cpu().numpy() for d in dst.dev], dst.host, "pages")


def test_beside_a_store_from_a_stream_in_its_hardware_queue():
    """A small retrieve from a stream that shares a hardware queue with a stream of a large store
    comes back long before the store does."""
    import time
    import torch
    from gpu_util import slots_to_device
    from paper_2510_09665_amd import lmc
    g = W.geometry("llama3_8b", L=8, NB=4096)
    n, rng = 128, np.random.default_rng(37)
    blocks = rng.permutation(g.NB)
    d_ss = slots_to_device(W.slots_from_blocks(g, blocks[:n * 16], n * g.CT))
    d_ts = slots_to_device(W.slots_from_blocks(g, blocks[n * 16:(n + 1) * 16], g.CT))
    layers = [torch.zeros(g.layer_bytes, dtype=torch.uint8, device="cuda") for _ in range(g.L)]
    ids = np.arange(1, n + 1, dtype=np.uint64)
    producer, streams = torch.cuda.Stream(), [torch.cuda.Stream() for _ in range(12)]
    for s in streams + [producer]:
        with torch.cuda.stream(s):
            torch.zeros(1, device="cuda").add_(1)          # a stream gets its queue when it is first used
    torch.cuda.synchronize()
    with lmc.Context(g, (n + 1) * g.chunk_bytes, staging_chunks=8) as c:
        c.put_host([9999], np.zeros(g.chunk_bytes, dtype=np.uint8))
        masks = [c.probe_stream(s) for s in streams]
        # bits 2 to 4: the streams of a store; bit 5: the scatter stream
        sharing = [s for s, m in zip(streams, masks) if m & 0b011100 and not m & 0b100000][:4]
        if not sharing:
            pytest.skip("no stream shares a queue with the store's: %s" % masks)
        for s in sharing:
            c.wait(c.store(layers, d_ss, ids, producer))   # what a first pass costs is behind it
            c.clear(ids)
            t0 = time.perf_counter()
            stored = c.store(layers, d_ss, ids, producer)
            time.sleep(0.002)
            t1 = time.perf_counter()
            loaded = c.retrieve([9999], d_ts, layers, s)
            while not c.test(loaded):
                pass
            t2 = time.perf_counter()
            c.wait(stored)
            t3 = time.perf_counter()
            c.clear(ids)
            torch.cuda.synchronize()
            assert t2 - t1 < (t3 - t0) / 3, ("retrieve %.1f of %.1f ms" % ((t2 - t1) * 1e3, (t3 - t0) * 1e3), masks)


def test_the_per_thread_stream_is_another_one_in_each_thread():
    """Two threads name hipStreamPerThread: one name, two streams.  The first thread's is busy, the
    second's is not; the pages they both fill end up as the second call left them."""
    import torch
    from gpu_util import PagedKV, assert_layers_equal, slots_to_device
    from paper_2510_09665_amd import lmc
    per_thread = 2                                          # hipStreamPerThread
    g = W.geometry("tiny", NB=256)
    rng = np.random.default_rng(43)
    src, dst = PagedKV(g, np.arange(g.NB), rng), PagedKV(g, np.arange(g.NB), fill="sentinel")
    slots = rng.permutation(g.n_slots)[:2 * g.CT].astype(np.int64)
    tau = rng.permutation(g.n_slots)[:g.CT].astype(np.int64)
    oracle.scatter(g, oracle.gather(g, src.host, slots)[1:], tau, dst.host)
    with lmc.Context(g, 2 * g.chunk_bytes, staging_chunks=2) as c:
        c.wait(c.store(src.dev, slots_to_device(slots), [1, 2]))
        d_tau = slots_to_device(tau)
        torch.cuda.synchronize()
        errors, keep = [], []

        def load(chunk, products):
            try:
                if products:
                    keep.append(_products(torch.cuda.ExternalStream(per_thread), products))
                c.retrieve([chunk], d_tau, dst.dev, per_thread)
            except Exception as e:
                errors.append(e)

        for args in ((1, 40), (2, 0)):
            t = threading.Thread(target=load, args=args)
            t.start()
            t.join()
        assert not errors, errors
        c.wait()
        torch.cuda.synchronize()
        assert_layers_equal([d.cpu().numpy() for d in dst.dev], dst.host, "pages")


def test_a_retrieve_that_fails_on_the_callers_stream_can_be_repeated():
    """Every checked HIP call of a retrieve on the caller's stream fails once (on the host): no count
    stays on the chunks, and the call made again fills the pages."""
    import torch
    from gpu_util import assert_layers_equal
    from paper_2510_09665_amd import lmc
    g, src, dst, d_slots, d_tau, ids = _case(5, 61)
    stream = torch.cuda.Stream()
    with lmc.Context(g, 5 * g.chunk_bytes, staging_chunks=2) as c:
        c.wait(c.store(src.dev, d_slots, ids))
        torch.cuda.synchronize()
        failures = 0
        for nth in range(1, 50):
            c.tune("fail_hip_after", nth)
            try:
                t = c.retrieve(ids, d_tau, dst.dev, stream)
            except lmc.LMCError as e:
                assert e.status == lmc.LMC_ERR_HIP, e
                failures += 1
                assert c.lookup(ids) == ids.size
                continue
            c.tune("fail_hip_after", 0)
            c.wait(t)
            break
        else:
            raise AssertionError("the retrieve never got through")
        assert failures >= 4, failures        # launch, event and wait behind it, the ticket's event
        c.clear(ids)                          # BUSY if a count had stayed
        assert_layers_equal([d.cpu().numpy() for d in dst.dev], dst.host, "pages")
