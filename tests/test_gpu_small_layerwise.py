"""Layer-wise calls that skip staging by their size.  Bytes
against the CPU oracle; every layer is read as soon as its wait returns."""
import numpy as np
import pytest

import oracle
from paper_2510_09665_amd import workloads as W

pytestmark = pytest.mark.gpu


def _setup(n, seed, name="llama3_8b", **kw):
    import torch
    from gpu_util import PagedKV, slots_to_device
    g = W.geometry(name, **dict(dict(L=8, NB=128), **kw))
    rng = np.random.default_rng(seed)
    blocks = rng.permutation(g.NB)
    per = n * g.CT // g.BS
    slots = W.slots_from_blocks(g, blocks[:per], n * g.CT)
    tau = W.slots_from_blocks(g, blocks[per:2 * per], n * g.CT)
    src = PagedKV(g, np.arange(g.NB), rng)
    dst = PagedKV(g, np.arange(g.NB), fill="sentinel")
    want = oracle.gather(g, src.host, slots)
    oracle.scatter(g, want, tau, dst.host)
    torch.cuda.synchronize()
    return g, src, dst, want, slots_to_device(slots), slots_to_device(tau), np.arange(1, 1 + n, dtype=np.uint64)


@pytest.mark.parametrize("steps,staged", [((1,) * 8, ()), ((1,) * 8, (0, 2, 4, 6)), ((1,) * 8, (1, 3, 5, 7)), ((1, 2, 1, 3, 1), (1, 3)),
                                          ((3, 1, 4), (0, 2)), ((2, 2, 2, 1, 1), (0, 1, 2)), ((2, 2, 2, 1, 1), (2,)),
                                          ((8,), ()), ((4, 4), ()), ((3, 3, 2), ()), ((7, 1), (0,)), ((1, 1, 1, 1, 3, 1), (4,)), ((1, 7), (1,)), ((8,), (0,))])
@pytest.mark.parametrize("how", ["behind_a_producer", "idle", "timed"])
def test_store_steps_of_any_size(steps, staged, how):
    """Steps of one store with staging (`staged`: which) and without, behind each other in every order, in turn on
    two streams where the caller's is idle: a store whose last step goes without staging has ended when the
    copies of the others have, and only one that has none of them says so by the word."""
    import torch
    from paper_2510_09665_amd import lmc
    g, src, dst, want, d_slots, d_tau, ids = _setup(2, sum(i * s for i, s in enumerate(steps)))
    stream = torch.cuda.Stream()
    with lmc.Context(g, 3 * g.chunk_bytes, staging_chunks=2, flags=lmc.LMC_FLAG_TIMING if how == "timed" else 0) as c:
        for again in range(4):
            live = [torch.zeros_like(d) if how == "behind_a_producer" else d for d in src.dev]
            torch.cuda.synchronize()
            t = c.store_begin(d_slots, ids, stream)
            l = 0
            for i, k in enumerate(steps):
                if how == "behind_a_producer":               # filled layer by layer on the caller's stream
                    with torch.cuda.stream(stream):
                        for x in range(l, l + k):
                            live[x].copy_(src.dev[x])
                c.tune("direct_store_below", 0 if i in staged else 64 << 20)
                c.store_layers(t, l, k, live, stream)
                l += k
            assert l == g.L
            c.wait_layer(t, 0, stream)
            c.wait(t)
            for i, w in zip(ids, want):
                assert np.array_equal(c.get_host(i), w)
            assert c.get_stats()["bytes_d2h"] == (again + 1) * 2 * g.chunk_bytes
            c.tune("expect_groups_staged", (again + 1) * len(staged))
            c.tune("expect_stores_told", again + 1 if not staged and how != "timed" else 0)
            c.clear(ids)
            c.put_host(ids, want ^ 255)                       # the slots hold other bytes before the next pass
            c.clear(ids)


@pytest.mark.parametrize("n,k,staged", [(1, 1, False), (2, 3, False), (2, 8, False), (2, 1, True)])
def test_retrieve_behind_the_store_and_each_layer_at_once(n, k, staged):
    """Layer-wise store, layer-wise retrieve and a reader of every layer, no host wait between."""
    import torch
    from gpu_util import assert_layers_equal
    from paper_2510_09665_amd import lmc
    g, src, dst, want, d_slots, d_tau, ids = _setup(n, 11 * n + k)
    consumer = torch.cuda.Stream()
    with lmc.Context(g, 3 * g.chunk_bytes, staging_chunks=2) as c:
        if staged:
            c.tune("direct_store_below", 0)
            c.tune("direct_retrieve_below", 0)
        t0 = c.store_begin(d_slots, ids)
        for l in range(g.L):
            c.store_layers(t0, l, 1, src.dev)
        t1 = c.retrieve_layerwise(ids, d_tau, dst.dev, k)
        seen = []
        for l in range(g.L):
            c.wait_layer(t1, l, consumer)
            with torch.cuda.stream(consumer):
                seen.append(dst.dev[l].clone())
        consumer.synchronize()
        assert_layers_equal([d.cpu().numpy() for d in seen], dst.host, "as each wait returned")
        c.wait(t1)
        assert c.get_stats()["scatter_launches"] == -(-g.L // k)
        c.clear(ids)


def test_wait_covers_a_layerwise_store_that_ends_behind_a_newer_ticket():
    """A layer-wise store is begun, a small store follows and is done, then the layers are
    submitted: waiting for the newer ticket waits for the older one too."""
    from paper_2510_09665_amd import lmc
    g, src, dst, want, d_slots, d_tau, ids = _setup(2, 5, L=32, NB=64)
    with lmc.Context(g, 3 * g.chunk_bytes, staging_chunks=2) as c:
        c.tune("direct_store_below", 3 * g.chunk_bytes)
        t0 = c.store_begin(d_slots, ids)
        t1 = c.store(src.dev, d_slots, [77])
        for l in range(g.L):
            c.store_layers(t0, l, 1, src.dev)
        c.wait(t1)
        assert c.test(t0)
        for i, w in zip(ids, want):
            assert np.array_equal(c.get_host(i), w)


def test_a_staged_layerwise_store_that_fails_is_taken_back_as_a_whole():
    from paper_2510_09665_amd import lmc
    g, src, dst, want, d_slots, d_tau, ids = _setup(3, 23, name="tiny", L=4, NB=128)
    with lmc.Context(g, 3 * g.chunk_bytes, staging_chunks=2) as c:
        c.tune("direct_store_below", 0)
        failures = 0
        for nth in range(1, 200):
            t = c.store_begin(d_slots, ids)
            try:
                for l in range(g.L):
                    if l == 2:
                        c.tune("fail_hip_after", nth)
                    c.store_layers(t, l, 1, src.dev)
            except lmc.LMCError as e:
                assert e.status == lmc.LMC_ERR_HIP, e
                failures += 1
                assert c.lookup(ids) == 0 and c.get_stats()["pool_slots_used"] == 0
                c.wait()
                continue
            c.tune("fail_hip_after", 0)
            c.wait(t)
            break
        else:
            raise AssertionError("the store never got through")
        assert failures >= 3
        for i, w in zip(ids, want):
            assert np.array_equal(c.get_host(i), w)


@pytest.mark.parametrize("flag", [False, True])
@pytest.mark.parametrize("what", ["retrieve", "store"])
def test_captured_into_a_graph(what, flag):
    """Layer-wise calls from a stream that is being captured, with a wait for every layer: the
    graph holds the launches and moves the bytes of the moment each time it is replayed."""
    import torch
    from gpu_util import assert_layers_equal
    from paper_2510_09665_amd import lmc
    g, src, dst, want, d_slots, d_tau, ids = _setup(2, 41, name="tiny", L=4, NB=128)
    untouched = [d.clone() for d in dst.dev]
    stream = torch.cuda.Stream()
    with lmc.Context(g, 3 * g.chunk_bytes, staging_chunks=2, flags=lmc.LMC_FLAG_DIRECT if flag else 0) as c:
        if what == "retrieve":
            c.wait(c.store(src.dev, d_slots, ids))
        graph = torch.cuda.CUDAGraph()
        torch.cuda.synchronize()
        with torch.cuda.graph(graph, stream=stream, capture_error_mode="relaxed"):
            if what == "retrieve":
                t = c.retrieve_layerwise(ids, d_tau, dst.dev, 1, stream)
            else:
                t = c.store_begin(d_slots, ids, stream)
                for l in range(g.L):
                    c.store_layers(t, l, 1, src.dev, stream)
            for l in range(g.L):
                c.wait_layer(t, l, stream)
        for replay in range(3):
            if what == "retrieve":
                for d, u in zip(dst.dev, untouched):
                    d.copy_(u)
            else:
                for d in src.dev:
                    d.bitwise_xor_(255)               # other bytes each time
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            if what == "retrieve":
                assert_layers_equal([d.cpu().numpy() for d in dst.dev], dst.host, "replay %d" % replay)
            else:
                for i, w in zip(ids, want):
                    assert np.array_equal(c.get_host(i), w ^ (255 if replay % 2 == 0 else 0)), replay
        del graph


@pytest.mark.parametrize("name,n,kw", [("llama3_8b", 1, dict(L=8, NB=64)),                     # steps of 1 MiB
                                       ("llama3_8b", 2, dict(L=5, NB=96, layout="HND")),
                                       ("llama3_8b", 3, dict(L=3, H=5, D=108, NB=96)),         # 1080-byte rows, in pieces
                                       ("llama3_8b", 40, dict(L=4, H=1, D=33, e=1, CT=208, NB=1100))])   # rows that do not tell
@pytest.mark.parametrize("how", ["idle", "busy_between", "another_between", "mixed", "odd_groups", "one_stream", "captured_between",
                                 "late_mapping"])
def test_store_steps_on_two_streams_in_turn(name, n, kw, how):
    """Steps of 0.5 MiB and more from a stream that is idle: every byte is in the pool when the wait returns, and
    a retrieve issued right behind sees all of them.  The slot mapping comes late on another stream, the
    stream becomes busy, another operation comes, a staged step follows, or another stream is captured
    between two steps."""
    import torch
    from gpu_util import assert_layers_equal
    from paper_2510_09665_amd import lmc
    g, src, dst, want, d_slots, d_tau, ids = _setup(n, 61 + n, name=name, **kw)
    stream, other = torch.cuda.Stream(), torch.cuda.Stream()
    x = torch.zeros(1 << 22, device="cuda")
    with lmc.Context(g, (2 * n + 2) * g.chunk_bytes, staging_chunks=n) as c:
        if how == "odd_groups":
            c.tune("link_groups", 7)
        if how == "one_stream":
            c.tune("store_step_streams", 1)
        for again in range(6):
            for d in src.dev:
                d.bitwise_xor_(255)
            torch.cuda.synchronize()
            if how == "late_mapping":
                late = torch.full_like(d_slots, -1)
                with torch.cuda.stream(other):
                    for _ in range(100):
                        x.add_(1)
                    late.copy_(d_slots)
                t = c.store_begin(late, ids, other)
            else:
                t = c.store_begin(d_slots, ids, stream)
            graph = None
            for l in range(g.L):
                if l == 1 and how == "busy_between":
                    with torch.cuda.stream(stream):
                        for _ in range(20):
                            x.add_(1)
                if l == 2 and how == "another_between":
                    c.store(src.dev, d_slots[:g.CT], np.array([1 << 40], dtype=np.uint64), other)
                if how == "mixed" and l == 2:
                    c.tune("direct_store_below", 0)
                if how == "captured_between" and l == 1:
                    graph = torch.cuda.CUDAGraph()
                    with torch.cuda.graph(graph, stream=other, capture_error_mode="relaxed"):
                        c.store_layers(t, l, 1, src.dev, stream)
                        x.add_(1)
                else:
                    c.store_layers(t, l, 1, src.dev, stream)
            if again % 2:
                u = c.retrieve(ids, d_tau, dst.dev, other)
                c.wait(u)
                torch.cuda.synchronize()
                assert_layers_equal([d.cpu().numpy() for d in dst.dev], dst.host, "pass %d" % again)
            c.wait(t)
            flip = 255 if again % 2 == 0 else 0
            for i, w in zip(ids, want):
                assert np.array_equal(c.get_host(i), w ^ flip), (again, i)
            c.wait()
            c.tune("direct_store_below", 64 << 20)
            c.clear(ids)
            c.clear(np.array([1 << 40], dtype=np.uint64))
            del graph
        if how in ("idle", "odd_groups", "one_stream") and "e" not in kw:
            c.tune("expect_stores_told", 6)


@pytest.mark.parametrize("kw", [dict(L=8, NB=64), dict(L=6, H=1, NB=64), dict(L=5, H=1, D=33, e=1, CT=208, NB=64)],
                         ids=["steps_of_1_mib", "small_steps", "rows_that_do_not_count"])
@pytest.mark.parametrize("how", ["words", "no_value_waits_any_more", "timed", "after_all"])
def test_pages_may_be_written_again_behind_the_wait_for_a_stored_layer(kw, how):
    """A stream that waits for a layer of a store writes the layer's pages: the pool has what was in them before."""
    import torch
    from paper_2510_09665_amd import lmc
    g, src, dst, want, d_slots, d_tau, ids = _setup(1, 83, **kw)
    stream, writer = torch.cuda.Stream(), torch.cuda.Stream()
    with lmc.Context(g, 3 * g.chunk_bytes, staging_chunks=1, flags=lmc.LMC_FLAG_TIMING if how == "timed" else 0) as c:
        for again in range(4):
            live = [d.clone() for d in src.dev]
            torch.cuda.synchronize()
            t = c.store_begin(d_slots, ids, stream)
            for l in range(g.L):
                c.store_layers(t, l, 1, live, stream)
                if how == "no_value_waits_any_more":
                    c.tune("value_waits", 0)
                if how != "after_all":
                    c.wait_layer(t, l, writer)
                    with torch.cuda.stream(writer):
                        live[l].fill_(0xEE)
                c.tune("value_waits", 1)
            if how == "after_all":
                for l in reversed(range(g.L)):
                    c.wait_layer(t, l, writer)
                    with torch.cuda.stream(writer):
                        live[l].fill_(0xEE)
            c.wait(t)
            for i, w in zip(ids, want):
                assert np.array_equal(c.get_host(i), w), again
            torch.cuda.synchronize()
            c.clear(ids)


@pytest.mark.parametrize("step", [1, 4])
def test_waits_for_a_stored_layer_are_skipped_where_they_are_over(step):
    """A stream that already waits for a step, and a store that has ended: nothing is enqueued, and the next call on
    the stream finds it idle.  Waits in every order, by two streams in turn, while layers are still handed in."""
    import time
    import torch
    from paper_2510_09665_amd import lmc
    g, src, dst, want, d_slots, d_tau, ids = _setup(1, 97 + step, L=16, NB=64)
    stream, writer, third = (torch.cuda.Stream() for _ in range(3))
    with lmc.Context(g, 3 * g.chunk_bytes, staging_chunks=1) as c:
        for again in range(4):
            live = [d.clone() for d in src.dev]
            torch.cuda.synchronize()
            t = c.store_begin(d_slots, ids, stream)
            for l in range(0, g.L, step):
                c.store_layers(t, l, step, live, stream)
                if again % 2:
                    for k in range(l + step - 1, -1, -1):      # the newest first, by two streams in turn
                        for s in (writer, third):
                            c.wait_layer(t, k, s)
                    with torch.cuda.stream(writer if l // step % 2 else third):
                        for k in range(l, l + step):
                            live[k].fill_(0xEE)
            if again == 2:
                time.sleep(0.01)                              # in the pool long ago, and nobody has looked
                assert writer.query()
                for l in range(g.L):
                    c.wait_layer(t, l, writer)
                assert writer.query()                          # nothing stands on the stream
            for l in range(g.L):
                c.wait_layer(t, l, writer)
                with torch.cuda.stream(writer):
                    live[l].fill_(0xEE)
            c.wait(t)
            for i, w in zip(ids, want):
                assert np.array_equal(c.get_host(i), w), again
            torch.cuda.synchronize()
            c.clear(ids)


def test_a_step_without_a_partner_has_all_groups():
    """With so few groups that they, and not the link, set the pace, a store in one or two calls takes as long where
    steps go on two streams in turn as where they go on one."""
    import time
    import torch
    from paper_2510_09665_amd import lmc
    g, src, dst, want, d_slots, d_tau, ids = _setup(1, 3, L=16, NB=64)
    stream = torch.cuda.Stream()
    with lmc.Context(g, 2 * g.chunk_bytes, staging_chunks=1) as c:
        c.tune("link_groups", 8)
        for calls in (1, 2):
            took = {}
            for streams in (1, 2, 1, 2):
                c.tune("store_step_streams", streams)
                for _ in range(4):
                    c.clear(ids)
                    torch.cuda.synchronize()
                    begin = time.perf_counter()
                    t = c.store_begin(d_slots, ids, stream)
                    for i in range(calls):
                        c.store_layers(t, i * g.L // calls, g.L // calls, src.dev, stream)
                    c.wait(t)
                    took.setdefault(streams, []).append(time.perf_counter() - begin)
            assert np.array_equal(c.get_host(ids[0]), want[0])
            # half of the groups took 1.9 times as long
            assert min(took[2]) < 1.3 * min(took[1]), (calls, took)
