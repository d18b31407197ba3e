"""Gathers hand each XCD longer runs of tiles than scatters once a launch has enough of them: the sizes
at which the run grows, one tile less and one more, against the CPU oracle."""
import numpy as np
import pytest

import oracle
from paper_2510_09665_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("row", [2048, 72])
@pytest.mark.parametrize("tiles", [255, 256, 257, 2047, 2048, 2049, 4095, 4096, 8191, 8192, 8199])
def test_sizes_at_which_the_run_grows(row, tiles):
    import torch
    from gpu_util import slots_to_device
    from paper_2510_09665_amd import lmc
    # a chunk is one tile: two rows of 2 KiB, or two of 72 bytes
    g = W.KVGeometry(L=1, P=1, H=1, D=row, e=1, BS=2, NB=512, CT=2)
    rng = np.random.default_rng(tiles)
    pages = rng.integers(0, 256, g.layer_bytes, dtype=np.uint8)
    slots = rng.integers(-1, g.n_slots, tiles * g.CT).astype(np.int64)
    want = oracle.gather(g, [pages], slots)
    dev = torch.from_numpy(pages).cuda()
    with lmc.Context(g, g.chunk_bytes) as c:
        buf = torch.full((tiles * g.chunk_bytes,), 0xCD, dtype=torch.uint8, device="cuda")
        c.gather([dev], slots_to_device(slots), tiles, buf, torch.cuda.current_stream())
        torch.cuda.synchronize()
    assert np.array_equal(buf.cpu().numpy().reshape(tiles, -1), want)
