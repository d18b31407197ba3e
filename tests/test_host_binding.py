"""The extension module behind Context's hot calls takes what the calls took through ctypes: arrays of
the right type as they are, everything else as numpy.ascontiguousarray converts it, tensors or
addresses, stream objects, handles or None; and refuses what they refused."""
import numpy as np
import pytest

import oracle
from paper_2510_09665_amd import lmc
from paper_2510_09665_amd import workloads as W

G = W.KVGeometry(L=3, P=2, H=2, D=8, e=2, BS=4, NB=8, CT=8)


def _ctx(slots=6):
    return lmc.Context(G, slots * G.chunk_bytes, device=lmc.LMC_DEVICE_NONE)


class Tensor:
    def __init__(self, address, error=None):
        self.address, self.error = address, error

    def data_ptr(self):
        if self.error:
            raise self.error
        return self.address


class Stream:
    cuda_stream = 0x1234


TOKENS = np.arange(100, 100 + 5 * G.CT + 3, dtype=np.int32)
WIDE = np.repeat(TOKENS, 2)


@pytest.mark.parametrize("form", [
    TOKENS, TOKENS.tolist(), tuple(TOKENS.tolist()), TOKENS.astype(np.int64), TOKENS.astype(">i4"), WIDE[::2],
    TOKENS.astype(np.uint32), TOKENS.astype(np.float64), np.frombuffer(TOKENS.tobytes(), dtype=np.int32),
    TOKENS[:5 * G.CT].reshape(5, G.CT)], ids=str)
def test_tokens_of_every_form(form):
    with _ctx() as c:
        ids = c.hash_chunks(form)
    assert isinstance(ids, np.ndarray) and ids.dtype == np.uint64
    assert np.array_equal(ids, oracle.hash_chunks(TOKENS[:5 * G.CT], G.CT, 0))


def test_no_tokens_and_fewer_than_a_chunk():
    with _ctx() as c:
        assert c.hash_chunks([]).size == 0 and c.hash_chunks(TOKENS[:G.CT - 1]).size == 0


@pytest.mark.parametrize("form", [lambda a: a, lambda a: a.tolist(), lambda a: np.repeat(a, 3)[::3], lambda a: a.astype(">u8"),
                                  lambda a: a.astype(np.int64), lambda a: a.reshape(2, 2), lambda a: a[:1][0], lambda a: a[:0]])
def test_ids_of_every_form(form):
    ids = np.array([1, 2 ** 63 - 5, 7, 12], dtype=np.uint64)
    with _ctx() as c:
        data = np.random.default_rng(1).integers(0, 256, (4, G.chunk_bytes), dtype=np.uint8)
        c.put_host(ids, data)
        given = form(ids)
        n = np.size(given)
        assert c.lookup(given) == n
        c.clear(given)
        assert c.lookup(ids) == (0 if n else 4)
        assert c.get_stats()["pool_slots_used"] == 4 - n


def test_ids_that_are_no_integers_are_refused():
    with _ctx() as c:
        for bad in ("text", [object()], None):
            with pytest.raises((TypeError, ValueError)):
                c.lookup(bad)
        with pytest.raises(TypeError):
            c.wait("1")
        with pytest.raises(TypeError):
            c.wait(1.0)
        with pytest.raises(TypeError):
            c.chunk_release(None)


def test_a_chunk_is_lent_read_only_and_counted():
    with _ctx() as c:
        data = np.random.default_rng(2).integers(0, 256, (1, G.chunk_bytes), dtype=np.uint8)
        ids = np.array([2 ** 64 - 3], dtype=np.uint64)
        c.put_host(ids, data)
        for given in (ids[0], int(ids[0])):
            view = c.chunk_acquire(given)
            assert view.dtype == np.uint8 and view.shape == (G.chunk_bytes,) and not view.flags.writeable
            assert np.array_equal(view, data[0])
            assert view.view(np.int64).size * 8 == G.chunk_bytes
            with pytest.raises(lmc.LMCError) as e:
                c.clear(ids)
            assert e.value.status == lmc.LMC_ERR_BUSY
            c.chunk_release(given)
        c.clear(ids)
        for f in (c.chunk_acquire, c.chunk_release):
            with pytest.raises(lmc.LMCError) as e:
                f(ids[0])
            assert e.value.status == lmc.LMC_ERR_MISS and "lmc_chunk" in str(e.value)


@pytest.mark.parametrize("stream", [None, 0, 77, Stream()], ids=["none", "zero", "handle", "object"])
@pytest.mark.parametrize("layers", [[Tensor(4096)] * 3, (4096, 8192, np.int64(12288)), [Tensor(2 ** 40), 64, Tensor(128)]],
                         ids=["tensors", "addresses", "mixed"])
def test_device_arguments_reach_the_library(stream, layers):
    """There is no GPU behind the context: every call of the path is turned down by the library itself."""
    with _ctx() as c:
        ids = np.array([1, 2], dtype=np.uint64)
        calls = [lambda: c.store(layers, Tensor(64), ids, stream), lambda: c.retrieve(ids, 64, layers, stream),
                 lambda: c.retrieve_batch([0, 1, 2], ids, Tensor(64), layers, stream),
                 lambda: c.retrieve_layerwise(ids, Tensor(64), layers, 1, stream), lambda: c.store_begin(Tensor(64), ids, stream),
                 lambda: c.store_layers(1, 0, 1, layers, stream), lambda: c.wait_layer(1, 0, stream),
                 lambda: c.gather(layers, Tensor(64), 1, Tensor(64), stream), lambda: c.scatter(64, Tensor(64), 1, layers, stream)]
        for call in calls:
            with pytest.raises(lmc.LMCError) as e:
                call()
            assert e.value.status == lmc.LMC_ERR_NODEVICE
        c.wait()


def test_layer_tables_that_are_wrong():
    with _ctx() as c:
        ids = np.array([1], dtype=np.uint64)
        for bad in ([4096] * 2, [4096] * 4, []):
            with pytest.raises(ValueError, match="expected 3 layer pointers"):
                c.store(bad, 64, ids)
        with pytest.raises(TypeError):
            c.store(iter([4096] * 3), 64, ids)          # has no length
        with pytest.raises(TypeError):
            c.store([4096, None, 4096], 64, ids)
        with pytest.raises(KeyError):
            c.store([4096, Tensor(0, KeyError("gone")), 4096], 64, ids)
        with pytest.raises(AttributeError):
            c.store([4096, Tensor(0, AttributeError("inside")), 4096], 64, ids)
        with pytest.raises(lmc.LMCError) as e:          # a missing slot mapping is the library's to refuse
            c.store([4096] * 3, None, ids)
        assert e.value.status == lmc.LMC_ERR_INVAL


def test_a_list_that_changes_while_it_is_read():
    """data_ptr() is Python code and may empty the very list that is being read: the layers are those of
    the moment of the call."""
    class Emptying(Tensor):
        def data_ptr(self):
            layers.clear()
            self.filler = [bytearray(64) for _ in range(1000)]     # memory of what was freed is in use again
            return self.address
    with _ctx() as c:
        for call in (lambda: c.store(layers, 64, [1]), lambda: c.retrieve([1], 64, layers),
                     lambda: c.store_layers(1, 0, 1, layers), lambda: c.gather(layers, 64, 1, 64)):
            layers = [Emptying(4096), Tensor(8192), Tensor(12288)]
            with pytest.raises(lmc.LMCError) as e:
                call()
            assert e.value.status == lmc.LMC_ERR_NODEVICE and layers == []


def test_an_extension_that_does_not_bind_is_refused_every_time(monkeypatch):
    import paper_2510_09665_amd
    lmc._lib()

    class Other:
        @staticmethod
        def bind(path, failed):
            raise ImportError("liblmc.so has no lmc_store")
    with monkeypatch.context() as m:
        m.setattr(lmc, "_LIB", None)
        m.setattr(lmc, "_native", None)
        m.setattr(paper_2510_09665_amd, "_lmc_native", Other)
        for _ in range(2):
            with pytest.raises(ImportError, match="paper_2510_09665_amd.build"):
                _ctx()
    with _ctx() as c:
        assert c.lookup([1]) == 0


def test_a_destroyed_context_is_refused():
    c = _ctx()
    c.destroy()
    for call in (lambda: c.lookup([1]), lambda: c.clear([1]), lambda: c.hash_chunks(TOKENS), lambda: c.wait(),
                 lambda: c.chunk_acquire(1), lambda: c.chunk_release(1), lambda: c.test(1)):
        with pytest.raises(lmc.LMCError) as e:
            call()
        assert e.value.status == lmc.LMC_ERR_INVAL
