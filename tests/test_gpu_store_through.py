"""A gather into the pinned pool writes at system scope where every wavefront writes whole cache
lines (16-byte lanes, planes that begin on a multiple of 128 bytes), with the non-temporal hint
elsewhere; long launches use more workgroups.  Byte for byte against the CPU oracle on both
sides of these lines.  Gathers into buffers in HBM keep the hint wherever the buffer lies."""
import numpy as np
import pytest

import oracle
from paper_2510_09665_amd import workloads as W

pytestmark = pytest.mark.gpu


SHAPES = [dict(L=3, P=2, H=4, D=64, e=2, BS=16, NB=48, CT=256),      # planes of whole lines
          dict(L=3, P=2, H=1, D=24, e=2, BS=4, NB=96, CT=27),       # 48-byte rows, planes are not
          dict(L=3, P=2, H=1, D=8, e=2, BS=4, NB=96, CT=8)]         # planes of one line


@pytest.mark.parametrize("kw", SHAPES)
def test_store_of_planes_on_and_off_a_line(kw):
    from gpu_util import PagedKV, slots_to_device
    from paper_2510_09665_amd import lmc
    g = W.KVGeometry(**kw)
    rng = np.random.default_rng(g.CT)
    src = PagedKV(g, np.arange(g.NB), rng)
    slots = rng.permutation(g.n_slots)[:2 * g.CT].astype(np.int64)
    slots[rng.integers(0, slots.size, 2)] = -1
    with lmc.Context(g, 3 * g.chunk_bytes, staging_chunks=2) as c:
        c.put_host([9], np.full(g.chunk_bytes, 0xCD, dtype=np.uint8))      # the chunks lie behind it
        c.wait(c.store(src.dev, slots_to_device(slots), [1, 2]))
        for i, w in zip((1, 2), oracle.gather(g, src.host, slots)):
            assert np.array_equal(c.get_host(i), w)
        assert (c.get_host(9) == 0xCD).all()


@pytest.mark.parametrize("off", [0, 16, 64, 112, 128])
@pytest.mark.parametrize("kw", SHAPES)
def test_gather_into_buffers_on_and_off_a_line(kw, off):
    import torch
    from gpu_util import PagedKV, slots_to_device
    from paper_2510_09665_amd import lmc
    g = W.KVGeometry(**kw)
    rng = np.random.default_rng(off + g.CT)
    src = PagedKV(g, np.arange(g.NB), rng)
    slots = rng.permutation(g.n_slots)[:2 * g.CT].astype(np.int64)
    slots[rng.integers(0, slots.size, 2)] = -1
    with lmc.Context(g, 2 * g.chunk_bytes, staging_chunks=2) as c:
        buf = torch.full((off + 2 * g.chunk_bytes + 160,), 0xCD, dtype=torch.uint8, device="cuda")
        c.gather(src.dev, slots_to_device(slots), 2, buf[off:], torch.cuda.current_stream())
        torch.cuda.synchronize()
        got = buf.cpu().numpy()
    assert np.array_equal(got[off:-160].reshape(2, -1), oracle.gather(g, src.host, slots))
    assert (got[:off] == 0xCD).all() and (got[-160:] == 0xCD).all()


@pytest.mark.parametrize("n", [1, 31, 32, 33])              # 128 tiles a chunk: 4096 with 32 of them
def test_store_without_staging_is_in_the_pool_when_waited_for(n):
    from gpu_util import PagedKV, slots_to_device
    from paper_2510_09665_amd import lmc
    g = W.geometry("tiny", NB=640)
    rng = np.random.default_rng(n)
    ids = np.arange(1, n + 1, dtype=np.uint64)
    with lmc.Context(g, n * g.chunk_bytes, staging_chunks=2) as c:
        for again in range(3):
            src = PagedKV(g, np.arange(g.NB), rng)
            slots = rng.permutation(g.n_slots)[:n * g.CT].astype(np.int64)
            slots[0] = g.n_slots + 5 if again == 2 else slots[0]       # outside the pages: reported, zeros stored
            d_slots = slots_to_device(slots)
            t = c.store(src.dev, d_slots, ids)
            if again == 2:
                with pytest.raises(lmc.LMCError) as e:
                    c.wait(t)
                assert e.value.status == lmc.LMC_ERR_BADSLOT
                slots[0] = -1
            else:
                c.wait(t)
            for i, w in zip(ids, oracle.gather(g, src.host, slots)):
                assert np.array_equal(c.get_host(i), w)
            c.clear(ids)
