"""lmc_tune "link_lds_kib": how much LDS the kernels across the link claim.  The same bytes with any value;
with 0 they start and end beside a kernel that holds most of the LDS of every compute unit."""
import numpy as np
import pytest

import oracle
from paper_2510_09665_amd import workloads as W

pytestmark = pytest.mark.gpu

# ends by itself: 64 lanes to a workgroup that look at the 100 MHz clock
STAYS = r"""
extern "C" __global__ void stays(long long ticks, int *out) {
    __shared__ volatile char held[100 << 10];
    if (threadIdx.x == 0) held[blockIdx.x] = 1;
    const long long begin = wall_clock64();
    while (wall_clock64() - begin < ticks) __builtin_amdgcn_s_sleep(64);
    if (threadIdx.x == 0) out[blockIdx.x] = held[blockIdx.x];
}
"""


def _moves(c, g, n, src, dst, d_slots, d_tau, ids, stream, layers):
    if layers:
        t = c.store_begin(d_slots, ids, stream)
        for l in range(g.L):
            c.store_layers(t, l, 1, src.dev, stream)
        c.wait(t)
        t = c.retrieve_layerwise(ids, d_tau, dst.dev, 2, stream)
        for l in range(g.L):
            c.wait_layer(t, l, stream)
    else:
        c.wait(c.store(src.dev, d_slots, ids, stream))
        t = c.retrieve(ids, d_tau, dst.dev, stream)
    c.wait(t)


def _request(L=4, n=3):
    import torch
    from gpu_util import PagedKV, slots_to_device
    g = W.KVGeometry(L=L, P=2, H=8, D=128, e=2, BS=16, NB=160, CT=256)
    rng = np.random.default_rng(51)
    slots, tau = (rng.permutation(g.n_slots)[:n * g.CT].astype(np.int64) for _ in range(2))
    src, dst = PagedKV(g, np.arange(g.NB), rng), PagedKV(g, np.arange(g.NB), fill="sentinel")
    want = oracle.gather(g, src.host, slots)
    host = [h.copy() for h in dst.host]
    oracle.scatter(g, want, tau, host)
    torch.cuda.synchronize()
    return g, src, dst, slots_to_device(slots), slots_to_device(tau), host


@pytest.mark.parametrize("kib", [0, 1, 64, 96, 128, 160])
@pytest.mark.parametrize("how", ["bulk", "listed", "layers", "staged_copies"])
def test_same_bytes_with_any_claim(kib, how):
    from gpu_util import assert_layers_equal
    from paper_2510_09665_amd import lmc
    n = 3
    g, src, dst, d_slots, d_tau, host = _request(n=n)
    ids = np.arange(1, n + 1, dtype=np.uint64)
    with lmc.Context(g, 3 * n * g.chunk_bytes, staging_chunks=2) as c:
        c.tune("link_lds_kib", kib)
        if how in ("listed", "staged_copies"):
            other = (1 << 40) + np.arange(2 * n, dtype=np.uint64)
            c.put_host(other, np.zeros((2 * n, g.chunk_bytes), dtype=np.uint8))
            c.clear(other[::2])
        if how == "staged_copies":
            for key, value in (("direct_store_below", 0), ("direct_retrieve_below", 0), ("copy_kernel", 3)):
                c.tune(key, value)
        _moves(c, g, n, src, dst, d_slots, d_tau, ids, None, how == "layers")
        assert_layers_equal([d.cpu().numpy() for d in dst.dev], host)


def test_values_that_no_compute_unit_has():
    from paper_2510_09665_amd import lmc
    g = W.KVGeometry(L=2, P=1, H=1, D=16, e=2, BS=4, NB=8, CT=4)
    with lmc.Context(g, g.chunk_bytes) as c:
        for bad in (161, 1 << 40):
            with pytest.raises(lmc.LMCError) as e:
                c.tune("link_lds_kib", bad)
            assert e.value.status == lmc.LMC_ERR_INVAL


@pytest.mark.parametrize("layers", [False, True])
def test_beside_a_kernel_that_holds_the_lds_of_every_compute_unit(layers):
    import torch
    from gpu_util import assert_layers_equal, sentinel_byte
    from paper_2510_09665_amd import lmc
    stays = torch.cuda._compile_kernel(STAYS, "stays")
    units, ms = torch.cuda.get_device_properties(0).multi_processor_count, 150
    out = torch.zeros(units, dtype=torch.int32, device="cuda")
    n = 2                                  # 2 MiB a layer: the steps of the store go without staging too
    g, src, dst, d_slots, d_tau, host = _request(n=n)
    ids = np.arange(1, n + 1, dtype=np.uint64)
    with lmc.Context(g, 2 * n * g.chunk_bytes, staging_chunks=3) as c:
        c.tune("link_lds_kib", 0)
        streams = [torch.cuda.Stream() for _ in range(8)]
        masks = [c.probe_stream(s) for s in streams]
        # the kernel's stream shares no hardware queue with the library's kernel streams, nor the caller's with it
        resident = next(i for i, m in enumerate(masks) if m & 0x30 == 0)
        caller = next(i for i, m in enumerate(masks) if m & masks[resident] == 0 and i != resident)
        _moves(c, g, n, src, dst, d_slots, d_tau, ids, streams[caller], layers)      # everything loaded and warm
        c.clear(ids)
        for l, d in enumerate(dst.dev):
            d.fill_(sentinel_byte(l))
        torch.cuda.synchronize()
        with torch.cuda.stream(streams[resident]):
            stays(grid=(units, 1, 1), block=(64, 1, 1), args=[ms * 100000, out])
            ended = torch.cuda.Event()
            ended.record()
        _moves(c, g, n, src, dst, d_slots, d_tau, ids, streams[caller], layers)
        beside = not ended.query()
        torch.cuda.synchronize()
    assert out.cpu().tolist() == [1] * units
    assert beside, (masks, resident, caller)
    assert_layers_equal([d.cpu().numpy() for d in dst.dev], host)
