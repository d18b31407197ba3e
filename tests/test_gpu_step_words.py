"""Layer-wise retrieves without staging run as one launch whose steps count themselves off at words
in device memory; consumers wait for the words' values.  Byte for byte against the CPU oracle,
every layer read as soon as its wait returns, by a stream whose caches hold the pages as they were
before: rows of every kind, steps that do not divide the layers, steps with fewer tiles than
workgroups, chunks back to back and in scattered slots, tokens without a page."""
import zlib

import numpy as np
import pytest

import oracle
from paper_2510_09665_amd import workloads as W

pytestmark = pytest.mark.gpu

SHAPES = {
    "rows_of_256": dict(L=7, P=2, H=1, D=128, e=2, BS=16, NB=96, CT=64),
    "rows_of_2048": dict(L=5, P=2, H=8, D=128, e=2, BS=16, NB=96, CT=128),
    "mla": dict(L=6, P=1, H=1, D=576, e=1, BS=64, NB=40, CT=256),
    "hnd": dict(L=4, P=2, H=4, D=64, e=2, BS=16, NB=64, CT=64, layout="HND"),
    "wide_row216": dict(L=5, P=2, H=3, D=72, e=1, BS=16, NB=56, CT=64),
    "wide_hnd_run33": dict(L=3, P=2, H=3, D=33, e=1, BS=4, NB=90, CT=32, layout="HND"),
    "narrow_8": dict(L=3, P=1, H=1, D=4, e=2, BS=4, NB=90, CT=32),
    "narrow_4": dict(L=3, P=2, H=1, D=6, e=2, BS=4, NB=90, CT=32),
    "narrow_2": dict(L=3, P=2, H=1, D=5, e=2, BS=4, NB=90, CT=32),
    "narrow_1": dict(L=3, P=1, H=1, D=5, e=1, BS=4, NB=90, CT=32),
}


def _request(g, n, rng):
    tau = rng.permutation(g.n_slots)[:n * g.CT].astype(np.int64)
    tau[rng.integers(0, n * g.CT, 2)] = -1
    return tau


def _pool(c, g, n, scattered, rng):
    """n chunks of random bytes in the pool, at every other slot in random order if scattered."""
    want = rng.integers(0, 256, (n, g.chunk_bytes), dtype=np.uint8)
    ids = np.arange(1, n + 1, dtype=np.uint64)
    if scattered:
        other = (1 << 40) + np.arange(2 * n, dtype=np.uint64)
        c.put_host(other, np.zeros((2 * n, g.chunk_bytes), dtype=np.uint8))
        c.clear(other[::2])
    for i in rng.permutation(n) if scattered else range(n):
        c.put_host(ids[i:i + 1], want[i])
    return want, ids


@pytest.mark.parametrize("shape", list(SHAPES))
@pytest.mark.parametrize("n,step,scattered,groups", [(1, 1, False, 64), (1, 2, False, 1), (2, 3, False, 64), (3, 1, True, 5),
                                                     (2, 99, True, 64)])
def test_each_layer_is_there_when_its_wait_returns(shape, n, step, scattered, groups):
    import torch
    from gpu_util import assert_layers_equal, slots_to_device
    from paper_2510_09665_amd import lmc
    g = W.KVGeometry(**SHAPES[shape])
    rng = np.random.default_rng(zlib.crc32(("%s %d %d" % (shape, n, step)).encode()))
    consumer = torch.cuda.Stream()
    with lmc.Context(g, 2 * n * g.chunk_bytes, staging_chunks=2) as c:
        want, ids = _pool(c, g, n, scattered, rng)
        c.tune("link_groups", groups)         # two to a workgroup: an odd number leaves a half without work
        c.reset_stats()
        for again in range(3):
            tau = _request(g, n, rng)
            host = [W.sentinel_layer(g, l) for l in range(g.L)]
            dev = [torch.from_numpy(h).cuda() for h in host]
            d_tau = slots_to_device(tau)
            oracle.scatter(g, want, tau, host)
            torch.cuda.synchronize()
            with torch.cuda.stream(consumer):
                before = [d.clone() for d in dev]         # the pages as they are now, in the caches
            t = c.retrieve_layerwise(ids, d_tau, dev, step, consumer)
            seen = []
            for l in range(g.L):
                c.wait_layer(t, l, consumer)
                with torch.cuda.stream(consumer):
                    seen.append(dev[l].clone())
            consumer.synchronize()
            assert_layers_equal([d.cpu().numpy() for d in seen], host, "as each wait returned, pass %d" % again)
            c.wait(t)
            c.wait_layer(t, 0, consumer)                    # finished: nothing to wait for
            del before
        assert c.get_stats()["scatter_launches"] == 3 * -(-g.L // min(step, g.L))
        assert c.get_stats()["bytes_h2d"] == 3 * n * g.chunk_bytes


def test_slot_outside_the_pages_is_reported_and_the_rest_is_carried_out():
    import torch
    from gpu_util import assert_layers_equal, slots_to_device
    from paper_2510_09665_amd import lmc
    g = W.KVGeometry(**SHAPES["rows_of_256"])
    rng = np.random.default_rng(3)
    with lmc.Context(g, 4 * g.chunk_bytes, staging_chunks=2) as c:
        want, ids = _pool(c, g, 2, False, rng)
        tau = _request(g, 2, rng)
        host = [W.sentinel_layer(g, l) for l in range(g.L)]
        dev = [torch.from_numpy(h).cuda() for h in host]
        bad = tau.copy()
        bad[5] = g.n_slots
        tau[5] = -1
        oracle.scatter(g, want, tau, host)
        d_bad = slots_to_device(bad)
        t = c.retrieve_layerwise(ids, d_bad, dev, 2, torch.cuda.current_stream())
        with pytest.raises(lmc.LMCError) as e:
            c.wait(t)
        assert e.value.status == lmc.LMC_ERR_BADSLOT
        assert_layers_equal([d.cpu().numpy() for d in dev], host)


@pytest.mark.parametrize("kind", ["null", "per_thread", "blocking", "copy_engine"])
def test_every_kind_of_consumer(kind):
    """The null stream, a blocking stream, one name for many streams, and copies to the host behind the
    waits; two retrieves into the same pages under way at once, the later one's bytes stay."""
    import torch
    from gpu_util import assert_layers_equal, slots_to_device
    from paper_2510_09665_amd import lmc
    g = W.KVGeometry(**SHAPES["rows_of_2048"])
    rng = np.random.default_rng(17)
    stream = torch.cuda.Stream() if kind == "copy_engine" else None
    handle = {"null": None, "per_thread": 2, "blocking": torch.cuda.ExternalStream(0), "copy_engine": stream}[kind]
    with lmc.Context(g, 5 * g.chunk_bytes, staging_chunks=2) as c:
        want, ids = _pool(c, g, 4, False, rng)
        tau = _request(g, 2, rng)
        host = [W.sentinel_layer(g, l) for l in range(g.L)]
        dev = [torch.from_numpy(h).cuda() for h in host]
        d_tau = slots_to_device(tau)
        oracle.scatter(g, want[2:], tau, host)
        out = [torch.empty(g.layer_bytes, dtype=torch.uint8, pin_memory=True) for _ in range(g.L)]
        torch.cuda.synchronize()
        c.retrieve_layerwise(ids[:2], d_tau, dev, 1, handle)
        t = c.retrieve_layerwise(ids[2:], d_tau, dev, 2, handle)
        for l in range(g.L):
            c.wait_layer(t, l, handle)
            if kind == "copy_engine":
                with torch.cuda.stream(stream):
                    out[l].copy_(dev[l], non_blocking=True)
        if kind == "copy_engine":
            stream.synchronize()
            assert_layers_equal([o.numpy() for o in out], host)
        c.wait(t)
        torch.cuda.synchronize()
        assert_layers_equal([d.cpu().numpy() for d in dev], host)


@pytest.mark.parametrize("shape", ["rows_of_256", "wide_row216", "narrow_4"])
@pytest.mark.parametrize("library_stream", [False, True])
def test_bulk_retrieves_hand_over_by_word(shape, library_stream):
    """Small retrieves one behind another into the same pages, from two streams in turn or from one (on
    whose own stream the kernels then run); a reader on the stream of each, whose caches hold the pages
    as they were, sees that retrieve's bytes, and the last one's stay."""
    import torch
    from gpu_util import assert_layers_equal, slots_to_device
    from paper_2510_09665_amd import lmc
    g = W.KVGeometry(**SHAPES[shape])
    rng = np.random.default_rng(zlib.crc32(shape.encode()) + 5)
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    with lmc.Context(g, 8 * g.chunk_bytes, staging_chunks=2) as c:
        want, ids = _pool(c, g, 4, True, rng)
        tau = _request(g, 2, rng)
        d_tau = slots_to_device(tau)
        dev = [torch.from_numpy(W.sentinel_layer(g, l)).cuda() for l in range(g.L)]
        hosts = []
        for first in (0, 2):
            hosts.append([W.sentinel_layer(g, l) for l in range(g.L)])
            oracle.scatter(g, want[first:first + 2], tau, hosts[-1])
        torch.cuda.synchronize()
        seen = []
        for k in range(12):
            s = b if library_stream and k % 3 == 1 else a
            with torch.cuda.stream(s):
                c.retrieve(ids[2 * (k % 2):2 * (k % 2) + 2], d_tau, dev, s)
                seen.append([d.clone() for d in dev])
            (a if s is b else b).wait_stream(s)            # the next retrieve finds the pages read
        t = c.retrieve(ids[:2], d_tau, dev, a)
        c.wait(t)
        assert c.test(t)
        torch.cuda.synchronize()
        for k, one in enumerate(seen):
            assert_layers_equal([d.cpu().numpy() for d in one], hosts[k % 2], "retrieve %d" % k)
        assert_layers_equal([d.cpu().numpy() for d in dev], hosts[0])


def test_while_another_stream_is_captured():
    """The call and its waits go on, and nothing of them gets into the graph."""
    import torch
    from gpu_util import assert_layers_equal, slots_to_device
    from paper_2510_09665_amd import lmc
    g = W.KVGeometry(**SHAPES["rows_of_256"])
    rng = np.random.default_rng(29)
    consumer, captured = torch.cuda.Stream(), torch.cuda.Stream()
    with lmc.Context(g, 4 * g.chunk_bytes, staging_chunks=2) as c:
        want, ids = _pool(c, g, 2, False, rng)
        tau = _request(g, 2, rng)
        host = [W.sentinel_layer(g, l) for l in range(g.L)]
        dev = [torch.from_numpy(h).cuda() for h in host]
        d_tau = slots_to_device(tau)
        x = torch.zeros(64, device="cuda")
        oracle.scatter(g, want, tau, host)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=captured, capture_error_mode="relaxed"):
            t = c.retrieve_layerwise(ids, d_tau, dev, 1, consumer)
            for l in range(g.L):
                c.wait_layer(t, l, consumer)
            x.add_(1)
        c.wait(t)
        consumer.synchronize()
        for _ in range(3):
            graph.replay()
        torch.cuda.synchronize()
        assert_layers_equal([d.cpu().numpy() for d in dev], host)
        assert x.cpu().tolist() == [3.0] * 64


@pytest.mark.parametrize("how", ["in_turn", "last_first", "destroyed"])
def test_layers_of_one_step_are_waited_for_once_by_each_stream(how):
    """Two streams that wait for the same layers in turn, a stream that waits for the last layer before the
    first, and a stream that is destroyed behind its wait, after which another may have its handle."""
    import ctypes
    import torch
    from gpu_util import assert_layers_equal, slots_to_device
    from paper_2510_09665_amd import lmc
    g = W.KVGeometry(L=6, P=2, H=8, D=128, e=2, BS=16, NB=256, CT=256)
    rng = np.random.default_rng(51)
    with open("/proc/self/maps") as maps:
        hip = ctypes.CDLL(next(line.split()[-1] for line in maps if "libamdhip64" in line))
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    with lmc.Context(g, 5 * g.chunk_bytes, staging_chunks=2) as c:
        want, ids = _pool(c, g, 4, False, rng)
        tau = _request(g, 4, rng)
        host = [W.sentinel_layer(g, l) for l in range(g.L)]
        dev = [torch.from_numpy(h).cuda() for h in host]
        d_tau = slots_to_device(tau)
        oracle.scatter(g, want, tau, host)
        for again in range(3):
            for l, d in enumerate(dev):
                d.copy_(torch.from_numpy(W.sentinel_layer(g, l)))
            before = []
            for s in (a, b):
                with torch.cuda.stream(s):
                    before.append([d.clone() for d in dev])     # the pages as they are now, in the caches
            torch.cuda.synchronize()
            t = c.retrieve_layerwise(ids, d_tau, dev, 3)        # two steps
            seen = {}
            if how == "destroyed":
                raw = ctypes.c_void_p()
                assert hip.hipStreamCreateWithFlags(ctypes.byref(raw), 1) == 0
                c.wait_layer(t, 0, raw.value)
                assert hip.hipStreamDestroy(raw) == 0
                made = []
                for _ in range(4):
                    assert hip.hipStreamCreateWithFlags(ctypes.byref(raw), 1) == 0
                    made.append(raw.value)
                for k, h in enumerate(made):
                    c.wait_layer(t, 1, h)
                    with torch.cuda.stream(torch.cuda.ExternalStream(h)):
                        seen[1, k] = dev[1].clone()
                torch.cuda.synchronize()
                for h in made:
                    assert hip.hipStreamDestroy(ctypes.c_void_p(h)) == 0
            else:
                for l in (range(g.L) if how == "in_turn" else reversed(range(g.L))):
                    for s in (a, b) if how == "in_turn" else (a,):
                        c.wait_layer(t, l, s)
                        with torch.cuda.stream(s):
                            seen[l, s] = dev[l].clone()
            torch.cuda.synchronize()
            for (l, _), d in seen.items():
                assert np.array_equal(d.cpu().numpy(), host[l]), (again, l)
            c.wait(t)
            assert_layers_equal([d.cpu().numpy() for d in dev], host)
            del before


def test_events_recorded_on_streams_that_are_gone_go_on_in_use():
    """A busy stream that stores, a stream that waits for layers and is destroyed, and one that is probed: the events
    recorded on them come back as those of other calls, and go with the context."""
    import ctypes
    import torch
    from conftest import _hip_runtime
    from gpu_util import assert_layers_equal, slots_to_device
    from paper_2510_09665_amd import lmc
    g = W.KVGeometry(L=6, P=2, H=8, D=128, e=2, BS=16, NB=256, CT=256)
    rng = np.random.default_rng(67)
    hip = _hip_runtime()
    for _ in range(2):
        with lmc.Context(g, 9 * g.chunk_bytes, staging_chunks=2) as c:
            want, ids = _pool(c, g, 4, False, rng)
            new = np.arange(100, 104, dtype=np.uint64)
            tau = _request(g, 4, rng)
            host = [W.sentinel_layer(g, l) for l in range(g.L)]
            dev = [torch.from_numpy(h).cuda() for h in host]
            d_tau = slots_to_device(tau)
            oracle.scatter(g, want, tau, host)
            kept = oracle.gather(g, host, tau)
            for k in range(12):
                for l, d in enumerate(dev):
                    d.copy_(torch.from_numpy(W.sentinel_layer(g, l)))
                torch.cuda.synchronize()
                c.tune("direct_retrieve_below", 0 if k % 3 == 2 else 64 << 20)
                c.tune("direct_store_below", 0 if k % 3 == 1 else 64 << 20)
                made = []
                for _ in range(3):
                    raw = ctypes.c_void_p()
                    assert hip.hipStreamCreateWithFlags(ctypes.byref(raw), 1) == 0
                    made.append(raw)
                t = c.retrieve_layerwise(ids, d_tau, dev, 1 + k % 4)
                for raw in made:
                    for l in range(g.L):
                        c.wait_layer(t, l, raw.value)
                if k == 5:
                    c.probe_stream(made[0].value)
                with torch.cuda.stream(torch.cuda.ExternalStream(made[1].value)):
                    torch.cuda._sleep(1 << 18)
                u = c.store(dev, d_tau, new, made[1].value)
                for raw in made:
                    assert hip.hipStreamDestroy(raw) == 0
                c.wait(u)
                assert c.test(t)
                for i, w in zip(new, kept):
                    assert np.array_equal(c.get_host(i), w), k
                c.clear(new)
                torch.cuda.synchronize()
                assert_layers_equal([d.cpu().numpy() for d in dev], host, "pass %d" % k)
