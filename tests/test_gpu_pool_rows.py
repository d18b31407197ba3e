"""Rows of every kind on their way into the pinned pool and out of it again without staging, byte
for byte against the CPU oracle.

Packed rows: runs of 16 bytes and more that are no multiple of 16, in planes that are.  The
kernel that gathers them puts every 16 bytes of a chunk together from the one or two runs they
hold.  Tokens without a page and slots outside the pages stand on either side of such pieces,
pool slots are consecutive or not, planes are whole lines of 128 bytes or not, and launches
have fewer and more tiles than the 512 from which the grid is doubled.

Narrow rows: runs of less than 16 bytes, in lanes of 8, 4, 2 and 1 bytes, also between the pages
and a buffer in HBM, and scattered in the order of the destination."""
import zlib

import numpy as np
import pytest

import oracle
from paper_2510_09665_amd import workloads as W
from test_gpu_listed_chunks import _fragment

pytestmark = pytest.mark.gpu

# name: geometry, bytes by which the layers are off their allocation, chunks
PACKED = {
    "run16_stride_18": (dict(L=3, P=2, H=1, D=8, e=2, BS=4, NB=64, CT=32, block_pad=2), 2, 6),
    "run17": (dict(L=2, P=2, H=1, D=17, e=1, BS=4, NB=64, CT=32), 1, 6),
    "run17_whole_lines": (dict(L=2, P=2, H=1, D=17, e=1, BS=4, NB=192, CT=128), 1, 5),
    "run30_hnd": (dict(L=2, P=2, H=3, D=15, e=2, BS=4, NB=160, CT=96, layout="HND"), 2, 5),
    "run31_one_token_pages": (dict(L=2, P=1, H=1, D=31, e=1, BS=1, NB=200, CT=16, order="NP"), 3, 9),
    "row216_whole_lines": (dict(L=5, P=2, H=3, D=72, e=1, BS=16, NB=88, CT=256), 8, 4),     # 140 tiles a chunk
    "row360_many_tiles": (dict(L=19, P=2, H=5, D=36, e=2, BS=12, NB=40, CT=84), 8, 5),      # 304 tiles a chunk
}
NARROW = {
    "run8_lanes8": (dict(L=3, P=2, H=1, D=4, e=2, BS=4, NB=64, CT=32), 8, 6),
    "run8_hnd_lanes8": (dict(L=2, P=2, H=3, D=4, e=2, BS=4, NB=96, CT=48, layout="HND"), 8, 5),
    "run12_hnd_lanes4": (dict(L=2, P=2, H=3, D=6, e=2, BS=4, NB=64, CT=32, layout="HND"), 4, 5),
    "run14_hnd_lanes2": (dict(L=2, P=2, H=3, D=7, e=2, BS=4, NB=64, CT=32, layout="HND"), 2, 5),
    "run10_lanes2": (dict(L=2, P=1, H=1, D=5, e=2, BS=4, NB=128, CT=72, order="NP"), 6, 5),
    "run15_lanes1": (dict(L=2, P=2, H=1, D=15, e=1, BS=3, NB=70, CT=24), 1, 6),
}
ROWS = {**PACKED, **NARROW}


def _lanes(g):
    """Bytes that run and strides are multiples of, at most 16, and the run's length."""
    run = g.R if g.H == 1 or g.head_stride == g.D * g.e else g.D * g.e
    strides = [g.plane_stride, g.block_stride, g.token_stride] + ([g.head_stride] if run != g.R else [])
    return int(np.gcd.reduce([g.D * g.e, 16] + strides)), run


def test_the_rows_are_of_the_kind_they_stand_for():
    for name, (kw, off, _) in ROWS.items():
        g = W.KVGeometry(**kw)
        align, run = _lanes(g)
        assert off % align == 0
        if name in PACKED:
            assert align < 16 <= run and g.CT * g.R % 16 == 0
            assert (g.CT * g.R % 128 == 0) == ("whole_lines" in name or name == "run16_stride_18")
        else:
            assert run < 16 and "lanes%d" % align in name


def _setup(name):
    """Pages off their allocation, mappings with tokens that have no page: one by one, in pairs, at
    both ends of a chunk, and some slots outside the pages."""
    import torch
    from gpu_util import PagedKV
    kw, off, n = ROWS[name]
    g = W.KVGeometry(**kw)
    rng = np.random.default_rng(zlib.crc32(name.encode()))
    assert n * g.CT <= g.n_slots
    slots, tau = (rng.permutation(g.n_slots)[:n * g.CT].astype(np.int64) for _ in range(2))
    for m in (slots, tau):
        gone = rng.random(m.size) < 0.25
        gone[[0, g.CT - 1, g.CT, -1]] = True
        m[gone] = rng.choice([-1, -(2**40), -(2**63)], int(gone.sum()))
    outside = rng.permutation(n * g.CT)[:max(2, n * g.CT // 16)]
    src, dst = PagedKV(g, np.arange(g.NB), rng), PagedKV(g, np.arange(g.NB), fill="sentinel")

    def shifted(layers):
        out = []
        for d in layers:
            room = torch.full((d.numel() + off,), 0x77, dtype=torch.uint8, device="cuda")
            room[off:] = d
            out.append(room[off:])
        return out

    src_dev, dst.dev = shifted(src.dev), shifted(dst.dev)
    return g, n, rng, src, src_dev, dst, slots, tau, outside


@pytest.mark.parametrize("name", list(ROWS))
@pytest.mark.parametrize("mode", ["in_a_row", "scattered", "layers", "layers_scattered", "few_groups"])
def test_store_and_retrieve_match_oracle(name, mode):
    from gpu_util import assert_layers_equal, slots_to_device
    from paper_2510_09665_amd import lmc
    g, n, rng, src, src_dev, dst, slots, tau, outside = _setup(name)
    ids = 5 + rng.permutation(1 << 20)[:n].astype(np.uint64)
    want = oracle.gather(g, src.host, slots)
    with lmc.Context(g, (2 * n + 3) * g.chunk_bytes, staging_chunks=2, flags=lmc.LMC_FLAG_DIRECT) as c:
        if mode == "few_groups":
            c.tune("link_groups", 3)
        if "scattered" in mode:
            _fragment(c, g, n, rng, 2)
        else:
            c.put_host([1], np.full(g.chunk_bytes, 0xCD, dtype=np.uint8))       # in front of the chunks
        for bad in (False, True):                                               # the second time some slots are outside
            want_now, use = want, slots
            if bad:
                use, holes = slots.copy(), slots.copy()
                use[outside], holes[outside] = rng.choice([g.n_slots, g.n_slots + 7, 2**31, 2**62], outside.size), -1
                want_now = oracle.gather(g, src.host, holes)
            d_slots = slots_to_device(use)
            if mode.startswith("layers"):
                t = c.store_begin(d_slots, ids)
                for l in range(g.L):
                    c.store_layers(t, l, 1, src_dev)
            else:
                t = c.store(src_dev, d_slots, ids)
            if bad:
                with pytest.raises(lmc.LMCError) as e:
                    c.wait(t)
                assert e.value.status == lmc.LMC_ERR_BADSLOT
            else:
                c.wait(t)
            for i in range(n):
                assert np.array_equal(c.get_host(ids[i]), want_now[i]), (bad, i)
            if "scattered" not in mode:
                assert (c.get_host(1) == 0xCD).all()
            if not bad:
                d_tau = slots_to_device(tau)
                if mode.startswith("layers"):
                    c.retrieve_layerwise(ids, d_tau, dst.dev, 1)
                else:
                    c.retrieve(ids, d_tau, dst.dev)
                c.wait()
                c.clear(ids)
    oracle.scatter(g, want, tau, dst.host)
    assert_layers_equal([d.cpu().numpy() for d in dst.dev], dst.host, name)


@pytest.mark.parametrize("name", list(NARROW))
@pytest.mark.parametrize("ordered", [False, True])
def test_narrow_rows_inside_hbm(name, ordered):
    import torch
    from gpu_util import assert_layers_equal, slots_to_device
    from paper_2510_09665_amd import lmc
    g, n, rng, src, src_dev, dst, slots, tau, _ = _setup(name)
    align, _ = _lanes(g)
    want = oracle.gather(g, src.host, slots)
    with lmc.Context(g, 2 * g.chunk_bytes) as c:
        if ordered:
            c.tune("scatter_order", 2)
        buf = torch.full((align + n * g.chunk_bytes + 64,), 0xCD, dtype=torch.uint8, device="cuda")
        c.gather(src_dev, slots_to_device(slots), n, buf[align:], torch.cuda.current_stream())
        torch.cuda.synchronize()
        got = buf.cpu().numpy()
        assert np.array_equal(got[align:-64].reshape(n, -1), want)
        assert (got[:align] == 0xCD).all() and (got[-64:] == 0xCD).all()
        c.scatter(buf[align:], slots_to_device(tau), n, dst.dev, torch.cuda.current_stream())
        torch.cuda.synchronize()
        c.wait()
    oracle.scatter(g, want, tau, dst.host)
    assert_layers_equal([d.cpu().numpy() for d in dst.dev], dst.host, name)
