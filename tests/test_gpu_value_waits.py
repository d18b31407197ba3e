"""lmc_tune "value_waits": retrieves of every kind with the streams' waits by value and by event, the
same bytes, switched between calls; and whether streams are made to wait for values at all: not
with 0, nor where a profiler collects counters, which lets one kernel run at a time and would start the
waiting one first."""
import json
import os
import subprocess
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

HERE = os.path.dirname(os.path.abspath(__file__))


def _retrieves(values, collecting=False):
    """One pass of every kind of retrieve for each value of the knob; True if the pages were right."""
    import torch
    import oracle
    from gpu_util import slots_to_device
    from paper_2510_09665_amd import lmc
    from paper_2510_09665_amd import workloads as W
    if collecting:
        os.environ["ROCPROF_COUNTER_COLLECTION"] = "1"
    g = W.KVGeometry(L=5, P=2, H=2, D=64, e=2, BS=16, NB=64, CT=64)
    rng = np.random.default_rng(11)
    n = 4
    tau = rng.permutation(g.n_slots)[:n * g.CT].astype(np.int64)
    tau[3] = -1
    want = rng.integers(0, 256, (n, g.chunk_bytes), dtype=np.uint8)
    host = [W.sentinel_layer(g, l) for l in range(g.L)]
    oracle.scatter(g, want, tau, host)
    d_tau = slots_to_device(tau)
    ids = np.arange(1, n + 1, dtype=np.uint64)
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    right = True
    with lmc.Context(g, n * g.chunk_bytes, staging_chunks=1) as c:
        c.put_host(ids, want)
        for value in values:
            if value is not None:
                c.tune("value_waits", value)
            for kind in ("bulk", "bulk_behind_another", "layers", "staged", "staged_layers", "switched"):
                c.tune("direct_retrieve_below", 0 if kind.startswith("staged") else 1 << 26)
                dev = [torch.from_numpy(W.sentinel_layer(g, l)).cuda() for l in range(g.L)]
                torch.cuda.synchronize()
                seen = []
                if kind.endswith("layers") or kind == "switched":
                    t = c.retrieve_layerwise(ids, d_tau, dev, 2, a)
                    if kind == "switched" and value is not None:
                        c.tune("value_waits", 1 - value)
                    for l in range(g.L):
                        c.wait_layer(t, l, a)
                        with torch.cuda.stream(a):
                            seen.append(dev[l].clone())
                    if kind == "switched" and value is not None:
                        c.tune("value_waits", value)
                else:
                    if kind == "bulk_behind_another":
                        c.retrieve(ids, d_tau, dev, b)
                    c.retrieve(ids, d_tau, dev, a)
                    with torch.cuda.stream(a):
                        seen = [d.clone() for d in dev]
                torch.cuda.synchronize()
                c.wait()
                right = right and all(np.array_equal(s.cpu().numpy(), h) for s, h in zip(seen, host))
    return right


@pytest.mark.parametrize("values", [[1], [0], [1, 0, 1]], ids=str)
def test_same_bytes_with_either(values):
    assert _retrieves(values)


@pytest.mark.parametrize("value,collecting,waits", [(1, False, True), (0, False, False), (None, False, True),
                                                    (None, True, False)])
def test_calls_that_wait_for_values(value, collecting, waits):
    res = subprocess.run([sys.executable, os.path.abspath(__file__), json.dumps([value, collecting])], capture_output=True,
                         text=True, timeout=110, cwd=os.path.dirname(HERE))
    assert res.returncode == 0, res.stderr[-2000:]
    right, names = json.loads(res.stdout.strip().splitlines()[-1])
    assert right
    assert any("scatter_paced" in n for n in names), names      # the profile does see kernels
    # "switched" flips a set knob for its waits: with 0 nothing was launched that they could wait for by value
    calls = [n for n in names if "hipStreamWaitValue" in n or "hipStreamWriteValue" in n]
    assert bool(calls) == waits, names


def test_a_store_that_arrives_in_the_middle_of_a_staged_retrieve():
    """The retrieve was alone when it was enqueued, so its streams write and wait for words; the store's
    groups go beside them.  Both are right, and so is what the caller's stream reads behind the retrieve."""
    import torch
    import oracle
    from gpu_util import PagedKV, assert_layers_equal, slots_to_device
    from paper_2510_09665_amd import lmc
    from paper_2510_09665_amd import workloads as W
    g = W.KVGeometry(L=6, P=2, H=8, D=128, e=2, BS=16, NB=300, CT=256)      # 6 MiB a chunk
    rng = np.random.default_rng(31)
    n = 6
    tau, slots = (rng.permutation(g.n_slots)[:n * g.CT].astype(np.int64) for _ in range(2))
    src = PagedKV(g, np.arange(g.NB), rng)
    stored = oracle.gather(g, src.host, slots)
    want = rng.integers(0, 256, (n, g.chunk_bytes), dtype=np.uint8)
    host = [W.sentinel_layer(g, l) for l in range(g.L)]
    oracle.scatter(g, want, tau, host)
    d_tau, d_slots = slots_to_device(tau), slots_to_device(slots)
    ids = np.arange(1, n + 1, dtype=np.uint64)
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    with lmc.Context(g, 2 * n * g.chunk_bytes, staging_chunks=2) as c:
        for key in ("direct_store_below", "direct_retrieve_below"):
            c.tune(key, 0)
        c.put_host(ids, want)
        for _ in range(4):
            dev = [torch.from_numpy(W.sentinel_layer(g, l)).cuda() for l in range(g.L)]
            torch.cuda.synchronize()
            c.retrieve(ids, d_tau, dev, a)
            c.store(src.dev, d_slots, ids + 100, b)
            with torch.cuda.stream(a):
                seen = [d.clone() for d in dev]
            a.synchronize()
            assert_layers_equal([d.cpu().numpy() for d in seen], host)
            c.wait()
            for i in range(n):
                assert np.array_equal(c.get_host(ids[i] + 100), stored[i])
            c.clear(ids + 100)


@pytest.mark.parametrize("kind", ["bulk", "layers", "staged"])
def test_words_keep_step_with_calls_that_fail(kind):
    """A HIP call that fails anywhere in a retrieve, then one that succeeds: its waits let nobody through
    early."""
    import torch
    import oracle
    from gpu_util import assert_layers_equal, slots_to_device
    from paper_2510_09665_amd import lmc
    from paper_2510_09665_amd import workloads as W
    g = W.KVGeometry(L=4, P=2, H=8, D=128, e=2, BS=16, NB=80, CT=256)       # 4 MiB a chunk
    rng = np.random.default_rng(37)
    n = 3
    tau = rng.permutation(g.n_slots)[:n * g.CT].astype(np.int64)
    want = rng.integers(0, 256, (n, g.chunk_bytes), dtype=np.uint8)
    host = [W.sentinel_layer(g, l) for l in range(g.L)]
    oracle.scatter(g, want, tau, host)
    d_tau = slots_to_device(tau)
    ids = np.arange(1, n + 1, dtype=np.uint64)
    a = torch.cuda.Stream()
    with lmc.Context(g, n * g.chunk_bytes, staging_chunks=1) as c:
        c.tune("direct_retrieve_below", 0 if kind == "staged" else 1 << 26)
        c.put_host(ids, want)
        failures = 0
        for nth in range(1, 60):
            for fails in (True, False):
                dev = [torch.from_numpy(W.sentinel_layer(g, l)).cuda() for l in range(g.L)]
                torch.cuda.synchronize()
                seen = []
                c.tune("fail_hip_after", nth if fails else 0)
                try:
                    if kind == "layers":
                        t = c.retrieve_layerwise(ids, d_tau, dev, 1, a)
                    else:
                        c.retrieve(ids, d_tau, dev, a)
                except lmc.LMCError as e:
                    assert fails and e.status == lmc.LMC_ERR_HIP
                    failures += 1
                    c.wait()
                    torch.cuda.synchronize()
                    continue
                c.tune("fail_hip_after", 0)
                for l in range(g.L):
                    if kind == "layers":
                        c.wait_layer(t, l, a)
                    with torch.cuda.stream(a):
                        seen.append(dev[l].clone())
                a.synchronize()
                assert_layers_equal([d.cpu().numpy() for d in seen], host, "call %d" % nth)
                c.wait()
            if failures < nth:
                break
        assert failures >= 2


if __name__ == "__main__":
    sys.path[:0] = [os.path.dirname(HERE), HERE]
    import torch
    from torch.profiler import ProfilerActivity, profile
    value, collecting = json.loads(sys.argv[1])
    with profile(activities=[ProfilerActivity.CUDA]) as prof:
        ok = _retrieves([value], collecting)
        torch.cuda.synchronize()
    print(json.dumps([ok, sorted({e.key for e in prof.key_averages()})]))
