"""Gathers whose runs are multiples of 64 vectors of 16 bytes find token, slot and addresses once
per wavefront.  Byte for byte against the CPU oracle: runs of one, two and three wavefronts, per-head
runs, planes that end inside a tile of four, one-token pages, tokens without a page, slots
outside the pages (reported, zeros), and a slot mapping that is not aligned to its elements."""
import numpy as np
import pytest

import oracle
from paper_2510_09665_amd import workloads as W

pytestmark = pytest.mark.gpu

SHAPES = {
    "one_wave": dict(L=3, P=2, H=8, D=64, e=2, BS=4, NB=24, CT=5),
    "two_waves_ragged": dict(L=2, P=2, H=8, D=128, e=2, BS=16, NB=8, CT=3),
    "three_waves_fp8": dict(L=2, P=1, H=3, D=1024, e=1, BS=3, NB=30, CT=7),
    "heads_apart": dict(L=2, P=2, H=3, D=512, e=2, BS=4, NB=20, CT=5, layout="HND", block_pad=16),
    "one_token_pages": dict(L=2, P=2, H=8, D=64, e=2, BS=1, NB=200, CT=33, order="NP"),
}


@pytest.mark.parametrize("name", list(SHAPES))
@pytest.mark.parametrize("off", [0, 4])
def test_gather_matches_oracle(name, off):
    import torch
    from gpu_util import PagedKV
    from paper_2510_09665_amd import lmc
    g = W.KVGeometry(**SHAPES[name])
    rng = np.random.default_rng(len(name) + off)
    n = 3
    src = PagedKV(g, np.arange(g.NB), rng)
    slots = rng.permutation(g.n_slots)[:n * g.CT].astype(np.int64)
    slots[1], slots[2], slots[-1] = -1, -(2**40), g.n_slots        # the last one is outside the pages
    room = torch.zeros(slots.nbytes + off, dtype=torch.uint8, device="cuda")
    room[off:] = torch.from_numpy(slots.view(np.uint8)).cuda()
    with lmc.Context(g, n * g.chunk_bytes, staging_chunks=2) as c:
        buf = torch.full((n * g.chunk_bytes + 64,), 0xCD, dtype=torch.uint8, device="cuda")
        c.gather(src.dev, room[off:], n, buf, torch.cuda.current_stream())
        torch.cuda.synchronize()
        with pytest.raises(lmc.LMCError) as e:
            c.wait()
        assert e.value.status == lmc.LMC_ERR_BADSLOT
        got = buf.cpu().numpy()
    slots[-1] = -1
    assert np.array_equal(got[:-64].reshape(n, -1), oracle.gather(g, src.host, slots))
    assert (got[-64:] == 0xCD).all()
