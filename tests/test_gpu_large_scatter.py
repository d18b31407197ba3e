"""Scatters inside HBM of 192 MiB and more whose pages hold 8 KiB, or rows of 1 KiB and whole lines, in one
piece write at system scope and in the plain order of the tiles: the sizes around that line, rows that qualify and rows that do
not, on two streams at once, against the pages built by indexing."""
import numpy as np
import pytest

from paper_2510_09665_amd import workloads as W

pytestmark = pytest.mark.gpu

# rows of 1 KiB; of 576 bytes back to back; of 576 bytes in one-token pages; by head
SHAPES = [dict(L=2, P=1, H=4, D=128, e=2, BS=16), dict(L=2, P=1, H=1, D=576, e=1, BS=16),
          dict(L=2, P=1, H=1, D=576, e=1, BS=1), dict(L=2, P=1, H=4, D=128, e=2, BS=16, layout="HND")]


@pytest.mark.parametrize("shape", range(len(SHAPES)))
@pytest.mark.parametrize("beside", [-1, 0, 1])
def test_around_the_line(shape, beside):
    import torch
    from gpu_util import slots_to_device
    from paper_2510_09665_amd import lmc
    kw = dict(SHAPES[shape], CT=64)
    row = kw["H"] * kw["D"] * kw["e"]
    tiles_per_chunk = 2 * -(-64 * row // 4096)
    n = 49152 // tiles_per_chunk + beside
    blocks = -(-n * 64 // kw["BS"])
    g = W.KVGeometry(NB=blocks + 7, **kw)
    gen = torch.Generator(device="cuda").manual_seed(shape)
    r = np.random.default_rng(shape)
    order = r.permutation(g.NB)
    t = np.arange(n * 64)
    slots = order[t // g.BS].astype(np.int64) * g.BS + t % g.BS
    slots[r.integers(0, slots.size, 5)] = -1
    d_slots = slots_to_device(slots)
    bufs = [torch.randint(0, 256, (n * g.chunk_bytes,), dtype=torch.uint8, device="cuda", generator=gen) for _ in range(2)]
    outs = [[torch.full((g.layer_bytes,), 0x5A, dtype=torch.uint8, device="cuda") for _ in range(g.L)] for _ in range(2)]
    streams = [torch.cuda.Stream() for _ in range(2)]
    torch.cuda.synchronize()
    with lmc.Context(g, g.chunk_bytes) as c:
        for _ in range(2):
            for s, b, o in zip(streams, bufs, outs):
                c.scatter(b, d_slots, n, o, s)
        torch.cuda.synchronize()
    keep = torch.from_numpy(slots >= 0).cuda()
    for b, o in zip(bufs, outs):
        chunks = b.view(n, g.L, 64, g.H, g.D * g.e)
        for l in range(g.L):
            rows = chunks[:, l].reshape(n * 64, g.H, -1)[keep]
            want = torch.full((g.layer_bytes,), 0x5A, dtype=torch.uint8, device="cuda")
            sl = d_slots[keep]
            if g.layout == "HND":
                v = want.view(g.NB, g.H, g.BS, -1)
                v.transpose(1, 2)[sl // g.BS, sl % g.BS] = rows
            else:
                want.view(g.NB * g.BS, g.H, -1)[sl] = rows
            assert torch.equal(o[l], want), l


@pytest.mark.parametrize("beside", [-1, 0, 1])
@pytest.mark.parametrize("kw", [dict(H=1, D=576, e=1, BS=16, CT=16), dict(H=1, D=128, e=2, BS=16, CT=16),
                                dict(H=1, D=512, e=2, BS=1, CT=3)], ids=str)
def test_planes_shorter_than_their_tiles(kw, beside):
    """The line is in bytes, whatever the number of tiles that they take."""
    import torch
    from gpu_util import slots_to_device
    from paper_2510_09665_amd import lmc
    g = W.KVGeometry(L=3, P=2, NB=2500, **kw)
    n = -(-(192 << 20) // g.chunk_bytes) + beside
    r = np.random.default_rng(n)
    # more tokens than the pages hold: a slot is taken once, the other tokens have none
    slots = np.full(n * g.CT, -1, dtype=np.int64)
    taken = r.permutation(n * g.CT)[:min(n * g.CT, g.n_slots - 5)]
    slots[taken] = r.permutation(g.n_slots)[:taken.size]
    d_slots = slots_to_device(slots)
    buf = torch.randint(0, 256, (n * g.chunk_bytes,), dtype=torch.uint8, device="cuda")
    out = [torch.full((g.layer_bytes,), 0x5A, dtype=torch.uint8, device="cuda") for _ in range(g.L)]
    torch.cuda.synchronize()
    with lmc.Context(g, g.chunk_bytes) as c:
        c.scatter(buf, d_slots, n, out, torch.cuda.current_stream())
        torch.cuda.synchronize()
    keep = d_slots >= 0
    chunks = buf.view(n, g.L, g.P, g.CT, -1)
    for l in range(g.L):
        want = torch.full((g.layer_bytes,), 0x5A, dtype=torch.uint8, device="cuda")
        for p in range(g.P):
            want.view(g.P, g.n_slots, -1)[p, d_slots[keep]] = chunks[:, l, p].reshape(n * g.CT, -1)[keep]
        assert torch.equal(out[l], want), l
