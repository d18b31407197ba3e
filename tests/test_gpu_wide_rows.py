"""Rows whose length or strides are no multiple of 16 bytes but that have runs of 16 bytes or
more: the kernels move them in 16-byte pieces at any address, the last piece of a run moved
back to end with it.  Byte for byte against the CPU oracle, at the lengths where that can go
wrong: one piece exactly, one byte more, one byte less than two, whole pieces on a stride that
is none, rows that cross tiles of 256 pieces, per-head runs."""
import zlib

import numpy as np
import pytest

import oracle
from paper_2510_09665_amd import workloads as W

pytestmark = pytest.mark.gpu

# name: geometry, and by how many bytes the layers are moved off their allocation (a multiple
# of what the geometry's sizes and strides are multiples of)
SHAPES = {
    "run16_stride_18": (dict(L=3, P=2, H=1, D=8, e=2, BS=4, NB=40, CT=32, block_pad=2), 2),
    "run17": (dict(L=2, P=1, H=1, D=17, e=1, BS=3, NB=70, CT=24, block_pad=1), 1),
    "run31": (dict(L=2, P=2, H=1, D=31, e=1, BS=4, NB=40, CT=32), 3),
    "run33_hnd": (dict(L=2, P=2, H=3, D=33, e=1, BS=4, NB=40, CT=32, layout="HND"), 1),
    "row216_fp8": (dict(L=5, P=2, H=3, D=72, e=1, BS=16, NB=56, CT=256), 8),
    "row360_bs12": (dict(L=3, P=2, H=5, D=36, e=2, BS=12, NB=40, CT=84), 8),
    "whole_pieces_of_8_byte_heads": (dict(L=3, P=2, H=4, D=36, e=2, BS=4, NB=40, CT=32), 8),
    "run16_only": (dict(L=2, P=1, H=1, D=16, e=1, BS=4, NB=40, CT=17, block_pad=8), 8),
    "run17_whole_planes": (dict(L=2, P=2, H=1, D=17, e=1, BS=4, NB=40, CT=32), 1),
    "run30_hnd_tiles": (dict(L=2, P=2, H=3, D=15, e=2, BS=4, NB=80, CT=96, layout="HND"), 2),
    "hnd_run72_blocks_outer": (dict(L=3, P=2, H=3, D=36, e=2, BS=4, NB=64, CT=32, order="NP", layout="HND",
                                    block_pad=8), 24),
}


def _shifted(layers, off):
    """The same bytes at an address `off` bytes into an allocation."""
    import torch
    out = []
    for d in layers:
        room = torch.full((d.numel() + off,), 0x77, dtype=torch.uint8, device="cuda")
        room[off:] = d
        out.append(room[off:])
    return out


@pytest.mark.parametrize("name", list(SHAPES))
@pytest.mark.parametrize("ordered,at", [(False, None), (True, None), (False, 0), (False, 16), (False, 128)])
def test_both_kernels_match_oracle(name, ordered, at):
    """at: by how many bytes the buffer is off its allocation (None: as the layers).  Inside HBM both
    kernels go row by row wherever the buffer lies; gathers into the pool, which put whole pieces
    of 16 bytes together, are in test_gpu_pool_rows.py."""
    import torch
    from gpu_util import PagedKV, assert_layers_equal, slots_to_device
    from paper_2510_09665_amd import lmc
    kw, off = SHAPES[name]
    g = W.KVGeometry(**kw)
    rng = np.random.default_rng(zlib.crc32(name.encode()))
    n, n_tok = 3, 3 * g.CT
    slots, tau = (rng.permutation(g.n_slots)[:n_tok].astype(np.int64) for _ in range(2))
    slots[rng.integers(0, n_tok, 3)] = -1
    tau[rng.integers(0, n_tok, 3)] = -2
    src, dst = PagedKV(g, np.arange(g.NB), rng), PagedKV(g, np.arange(g.NB), fill="sentinel")
    src_dev, dst.dev = _shifted(src.dev, off), _shifted(dst.dev, off)
    want = oracle.gather(g, src.host, slots)
    with lmc.Context(g, 4 * g.chunk_bytes) as c:
        if ordered:
            c.tune("scatter_order", 2)
        off = off if at is None else at
        buf = torch.full((off + n * g.chunk_bytes + 64,), 0xCD, dtype=torch.uint8, device="cuda")
        c.gather(src_dev, slots_to_device(slots), n, buf[off:], torch.cuda.current_stream())
        torch.cuda.synchronize()
        got = buf.cpu().numpy()
        assert np.array_equal(got[off:-64].reshape(n, -1), want)
        assert (got[:off] == 0xCD).all() and (got[-64:] == 0xCD).all()
        c.scatter(buf[off:], slots_to_device(tau), n, dst.dev, torch.cuda.current_stream())
        torch.cuda.synchronize()
        c.wait()
    oracle.scatter(g, want, tau, dst.host)
    assert_layers_equal([d.cpu().numpy() for d in dst.dev], dst.host, name)


@pytest.mark.parametrize("name", ["run17", "run33_hnd", "row216_fp8"])
@pytest.mark.parametrize("mode", ["by_size", "staged", "layers"])
def test_store_and_retrieve_match_oracle(name, mode):
    """The same rows through the pool: by the kernel across the link, through staging, layer by layer."""
    from gpu_util import PagedKV, assert_layers_equal, slots_to_device
    from paper_2510_09665_amd import lmc
    kw, off = SHAPES[name]
    g = W.KVGeometry(**kw)
    rng = np.random.default_rng(zlib.crc32(name.encode()) + 1)
    n, n_tok = 3, 3 * g.CT
    slots, tau = (rng.permutation(g.n_slots)[:n_tok].astype(np.int64) for _ in range(2))
    src, dst = PagedKV(g, np.arange(g.NB), rng), PagedKV(g, np.arange(g.NB), fill="sentinel")
    src_dev, dst.dev = _shifted(src.dev, off), _shifted(dst.dev, off)
    want = oracle.gather(g, src.host, slots)
    ids = np.arange(7, 7 + n, dtype=np.uint64)
    with lmc.Context(g, (n + 1) * g.chunk_bytes, staging_chunks=2) as c:
        if mode == "staged":
            c.tune("direct_store_below", 0)
            c.tune("direct_retrieve_below", 0)
        d_slots, d_tau = slots_to_device(slots), slots_to_device(tau)
        if mode == "layers":
            t = c.store_begin(d_slots, ids)
            for l in range(g.L):
                c.store_layers(t, l, 1, src_dev)
        else:
            c.store(src_dev, d_slots, ids)
        c.wait()
        for i in range(n):
            assert np.array_equal(c.get_host(ids[i]), want[i])
        if mode == "layers":
            c.retrieve_layerwise(ids, d_tau, dst.dev, 1)
        else:
            c.retrieve(ids, d_tau, dst.dev)
        c.wait()
    oracle.scatter(g, want, tau, dst.host)
    assert_layers_equal([d.cpu().numpy() for d in dst.dev], dst.host, name)
