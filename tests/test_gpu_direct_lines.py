"""Which calls skip staging by their size.  Retrieves: up to 256 MiB, up to 512 MiB layer by layer in
steps of at most 8 MiB, up to 64 MiB beside a store that is under way.  Layer-wise stores: up to 64 MiB,
up to 256 MiB steps of at most 2 MiB, which one store may mix with staged ones, and of any size from a
stream that is idle.  Where a line is set, up to that.  Once a stream has been found that a direction does not
hold up: retrieves up to 64 MiB, up to 512 layer by layer in steps of at most 3 MiB; no steps of stores of more
than 2 MiB that have a producer at work.  At each line, the last size on this side and the first on the other: the trace says
whether copies between staging and the pool were made, and the bytes are the same either way."""
import numpy as np
import pytest

from paper_2510_09665_amd import workloads as W

pytestmark = pytest.mark.gpu

MIB = 1 << 20
CHUNKS = 65
# chunks of 8 MiB, 128 KiB a layer
G = W.KVGeometry(L=64, P=2, H=1, D=32, e=2, BS=32, NB=2 * CHUNKS * 32, CT=1024)


@pytest.fixture(scope="module")
def kv():
    import torch
    gen = torch.Generator(device="cuda").manual_seed(7)
    pages = torch.empty((G.L, G.layer_bytes // 8), dtype=torch.int64, device="cuda").random_(generator=gen)
    blocks = np.split(np.random.default_rng(7).permutation(G.NB), 2)
    t = np.arange(CHUNKS * G.CT)
    slots = [torch.from_numpy(b[t // G.BS].astype(np.int64) * G.BS + t % G.BS).cuda() for b in blocks]
    return pages, [torch.from_numpy(b).cuda() for b in blocks], slots


@pytest.mark.parametrize("chunks,step,store,line,direct", [
    (32, 0, False, None, True), (33, 0, False, None, False),
    (32, 64, False, None, True), (33, 64, False, None, False),              # one step: as bulk
    (64, 1, False, None, True), (65, 1, False, None, False),                # 512 MiB, steps of 8 MiB
    (33, 1, False, None, True), (33, 2, False, None, False),                # steps of 8.25 MiB
    (8, 0, True, None, True), (9, 0, True, None, False),
    (8, 1, True, None, True), (9, 1, True, None, False),
    (2, 0, False, 16, True), (3, 0, False, 16, False), (3, 1, False, 16, False), (1, 1, False, 0, False),
    (33, 0, False, 264, True), (9, 0, True, 264, True),
])
def test_lines(kv, chunks, step, store, line, direct):
    import torch
    from paper_2510_09665_amd import lmc
    pages, blocks, slots = kv
    per, n = G.CT // G.BS, chunks * G.CT
    layers = [p.view(torch.uint8) for p in pages.unbind(0)]
    for l in layers:
        W.page_view(G, l)[:, blocks[1]] = 0x5A
    torch.cuda.synchronize()
    with lmc.Context(G, (chunks + 1) * G.chunk_bytes, staging_chunks=8) as c:
        ids = np.arange(1, chunks + 1, dtype=np.uint64)
        c.store(layers, slots[0][:n], ids)
        c.wait()
        if line is not None:
            c.tune("direct_retrieve_below", line * MIB)
        c.tune("trace", 1)
        if store:      # under way until its last layers are handed in
            other = c.store_begin(slots[0][:G.CT], np.array([1 << 40], dtype=np.uint64))
        if step:
            t = c.retrieve_layerwise(ids, slots[1][:n], layers, step)
        else:
            t = c.retrieve(ids, slots[1][:n], layers)
        while not c.test(t):
            pass
        if store:
            c.store_layers(other, 0, G.L, layers)
        c.wait()
        copies = [r for r in c.trace_read()[0] if r["stage"] == lmc.LMC_STAGE_H2D]
        assert (not copies) == direct
    for l in layers:
        v = W.page_view(G, l)
        assert torch.equal(v[:, blocks[1][:chunks * per]], v[:, blocks[0][:chunks * per]])
        assert (v[:, blocks[1][chunks * per:]] == 0x5A).all()


@pytest.mark.parametrize("chunks,steps,busy,line,staged", [
    (8, (64,), True, None, 0), (9, (64,), True, None, 1),                  # 64 MiB
    (9, (1,) * 64, True, None, 0), (16, (1,) * 64, True, None, 0), (17, (1,) * 64, True, None, 64),   # steps of 2 MiB
    (9, (1, 2, 1, 60), True, None, 2), (16, (2, 1, 61), True, None, 2),    # mixed
    (9, (64,), False, None, 0), (17, (1, 31, 32), False, None, 0), (32, (8,) * 8, False, None, 0),
    (33, (1,) * 64, True, None, 64), (33, (32, 32), False, None, 2),       # 256 MiB
    (2, (64,), False, 16, 0), (3, (1,) * 64, False, 16, 64), (1, (32, 32), False, 0, 2),
])
def test_lines_of_layerwise_stores(kv, chunks, steps, busy, line, staged):
    import torch
    from paper_2510_09665_amd import lmc
    pages, blocks, slots = kv
    n, per = chunks * G.CT, G.CT // G.BS
    layers = [p.view(torch.uint8) for p in pages.unbind(0)]
    stream = torch.cuda.Stream()
    work = torch.ones(4096, 4096, device="cuda", dtype=torch.bfloat16)
    torch.cuda.synchronize()
    with lmc.Context(G, chunks * G.chunk_bytes, staging_chunks=chunks) as c:
        ids = np.arange(1, chunks + 1, dtype=np.uint64)
        if line is not None:
            c.tune("direct_store_below", line * MIB)
        c.tune("trace", 1)
        if busy:
            with torch.cuda.stream(stream):
                for _ in range(400):
                    work = (work @ work).clamp_(-1, 1)
        t, l = c.store_begin(slots[0][:n], ids, stream), 0
        for k in steps:
            c.store_layers(t, l, k, layers, stream)
            l += k
        assert not busy or not stream.query()
        assert l == G.L
        c.wait(t)
        assert sum(r["stage"] == lmc.LMC_STAGE_D2H for r in c.trace_read()[0]) == staged
        rows = torch.stack([W.page_view(G, x)[:, blocks[0][:chunks * per]] for x in layers])     # [L][P][block][bytes]
        want = rows.view(G.L, G.P, chunks, -1).permute(2, 0, 1, 3).reshape(chunks, -1).cpu().numpy()
        for i in ids:
            assert np.array_equal(c.chunk_acquire(i), want[int(i) - 1]), i
            c.chunk_release(i)


def _place(c, streams, bits):
    """Probes until a stream overlaps with the direction; True if one does (it takes three hardware queues)."""
    return any((c.probe_stream(s) & bits) == 0 for s in streams)


@pytest.mark.parametrize("chunks,step,line,again,direct", [
    (8, 0, None, False, True), (9, 0, None, False, False), (8, 64, None, False, True), (9, 64, None, False, False),
    (24, 1, None, False, True), (25, 1, None, False, False), (9, 2, None, False, True), (13, 2, None, False, False),
    (9, 0, 264, False, True), (33, 0, 264, False, True), (2, 1, 8, False, False),
    (32, 0, None, True, True), (64, 1, None, True, True),       # the library's streams placed anew
])
def test_lines_where_a_stream_overlaps_with_retrieves(kv, chunks, step, line, again, direct):
    import torch
    from paper_2510_09665_amd import lmc
    pages, blocks, slots = kv
    per, n = G.CT // G.BS, chunks * G.CT
    layers = [p.view(torch.uint8) for p in pages.unbind(0)]
    for l in layers:
        W.page_view(G, l)[:, blocks[1]] = 0x5A
    torch.cuda.synchronize()
    with lmc.Context(G, max(4, chunks) * G.chunk_bytes, staging_chunks=8) as c:
        if not _place(c, [torch.cuda.Stream() for _ in range(16)], 0x23):
            pytest.skip("every stream shares a hardware queue with the retrieves")
        ids = np.arange(1, chunks + 1, dtype=np.uint64)
        c.wait(c.store(layers, slots[0][:n], ids))
        assert c.test(1)
        if again:
            c.tune("arrange_streams", 1)
        if line is not None:
            c.tune("direct_retrieve_below", line * MIB)
        c.tune("trace", 1)
        if step:
            t = c.retrieve_layerwise(ids, slots[1][:n], layers, step)
        else:
            t = c.retrieve(ids, slots[1][:n], layers)
        c.wait(t)
        copies = [r for r in c.trace_read()[0] if r["stage"] == lmc.LMC_STAGE_H2D]
        assert (not copies) == direct
    for l in layers:
        v = W.page_view(G, l)
        assert torch.equal(v[:, blocks[1][:chunks * per]], v[:, blocks[0][:chunks * per]])
        assert (v[:, blocks[1][chunks * per:]] == 0x5A).all()


@pytest.mark.parametrize("chunks,steps,busy,line,staged", [
    (8, (64,), True, None, 1), (8, (2,) * 32, True, None, 0), (8, (3,) + (2,) * 29 + (3,), True, None, 2),
    (8, (3,) + (2,) * 29 + (3,), False, None, 0), (16, (1,) * 64, True, None, 0), (1, (32, 32), True, None, 2),
    (1, (16,) * 4, True, None, 0), (8, (64,), True, 64, 0),
])
def test_lines_of_layerwise_stores_where_a_stream_overlaps_with_stores(kv, chunks, steps, busy, line, staged):
    import torch
    from paper_2510_09665_amd import lmc
    pages, blocks, slots = kv
    n, per = chunks * G.CT, G.CT // G.BS
    layers = [p.view(torch.uint8) for p in pages.unbind(0)]
    stream = torch.cuda.Stream()
    with lmc.Context(G, chunks * G.chunk_bytes, staging_chunks=chunks) as c:
        if not _place(c, [torch.cuda.Stream() for _ in range(16)], 0x1c):
            pytest.skip("every stream shares a hardware queue with the stores")
        ids = np.arange(1, chunks + 1, dtype=np.uint64)
        if line is not None:
            c.tune("direct_store_below", line * MIB)
        c.tune("trace", 1)
        if busy:
            with torch.cuda.stream(stream):
                torch.cuda._sleep(1 << 26)
        t, l = c.store_begin(slots[0][:n], ids, stream), 0
        for k in steps:
            c.store_layers(t, l, k, layers, stream)
            l += k
        assert not busy or not stream.query()
        c.wait(t)
        assert sum(r["stage"] == lmc.LMC_STAGE_D2H for r in c.trace_read()[0]) == staged
        rows = torch.stack([W.page_view(G, x)[:, blocks[0][:chunks * per]] for x in layers])     # [L][P][block][bytes]
        want = rows.view(G.L, G.P, chunks, -1).permute(2, 0, 1, 3).reshape(chunks, -1).cpu().numpy()
        for i in ids:
            assert np.array_equal(c.chunk_acquire(i), want[int(i) - 1]), i
            c.chunk_release(i)
