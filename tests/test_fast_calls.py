"""The native way of Cache's per-layer calls: the same bits and the same refusals as the way through ctypes."""
import ctypes
import importlib.machinery
import importlib.util
import os

import pytest
import torch

import paper_2604_16734_amd as K
from paper_2604_16734_amd import binding as B
from paper_2604_16734_amd import build as build_module

BF16 = torch.bfloat16


def test_module_is_built():
    assert B._fast_call() is not B._not_taken, "build the library: paper_2604_16734_amd.build builds the module, too"


def test_library_is_linked_without_the_module(monkeypatch, tmp_path, capsys):
    """hipcc alone makes the library: what the module needs besides may be missing."""
    commands = []
    monkeypatch.setattr(build_module, "ROOT", str(tmp_path))
    monkeypatch.setattr(build_module, "FAST_CALLS", str(tmp_path / "module.so"))
    monkeypatch.setattr(build_module, "_run", lambda cmd: commands.append(cmd) or "")

    def no_headers():
        raise RuntimeError("Python.h: No such file or directory")
    monkeypatch.setattr(build_module, "build_fast_calls", no_headers)
    (tmp_path / "module.so").write_bytes(b"of older sources")
    assert build_module.build() == build_module.LIB
    assert commands[-1][commands[-1].index("-o") + 1] == build_module.LIB and len(commands) == len(build_module.SOURCES) + 1
    assert "Python.h" in capsys.readouterr().err and not (tmp_path / "module.so").exists()


def test_module_of_another_torch_is_not_called(monkeypatch):
    """It links against any torch that has the symbols, but the layout of a tensor is compiled into it."""
    monkeypatch.setattr(torch, "__version__", torch.__version__ + ".another")
    assert B._fast_call() is B._not_taken
    assert build_module.FAST_CALLS.endswith(importlib.machinery.EXTENSION_SUFFIXES[0])      # (a name that another Python does not look for)


@pytest.fixture(scope="module")
def cpu_call(tmp_path_factory):
    """The module's call, built for tensors on the CPU."""
    path = build_module.build_fast_calls(os.path.join(str(tmp_path_factory.mktemp("fast_calls")), "_fast_calls.so"),
                                         ["KVP_TENSOR_DEVICE=c10::DeviceType::CPU"])
    spec = importlib.util.spec_from_file_location("_fast_calls", path)
    module = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(module)
    return module.call


STEP = ctypes.CFUNCTYPE(ctypes.c_int, ctypes.c_void_p, ctypes.c_int32, ctypes.c_void_p, ctypes.c_void_p, ctypes.c_void_p, ctypes.c_int32,
                        ctypes.c_void_p, ctypes.c_void_p)


def test_what_is_not_plain_is_left(cpu_call):
    """One argument at a time of a call that is taken."""
    taken = []
    entry = STEP(lambda *args: taken.append(args) or 7)
    q, k, out = torch.zeros(4, 64, dtype=BF16), torch.zeros(3, 2, 64, dtype=BF16), torch.zeros(4, 64, dtype=BF16)
    good = [ctypes.cast(entry, ctypes.c_void_p).value, 11, 5, (q, k, k, out), (4, 64), (2, 64), -1, 13, None]
    assert cpu_call(*good) == 7
    assert taken == [(11, 5, q.data_ptr(), k.data_ptr(), k.data_ptr(), 3, out.data_ptr(), 13)]
    wide = torch.zeros(3, 2, 128, dtype=BF16)
    for at, others in [
            (0, [None, 0, "1", -1]), (1, [None, 0, "1", -1, 1 << 64]), (2, [None, 1.0, "1", True, 1 << 40, -(1 << 40)]),
            (3, [[q, k, k, out], (q, k, k), (q, k, k, None), (q, k, k, out, q), (q.float(), k, k, out), (q[:3], k, k, out), (q[None], k, k, out),
                 (q, k[:2], k, out), (q, k, k[:2], out), (q, k[0], k[0], out), (q, wide[..., :64], k, out), (q, k, wide[..., ::2], out),
                 (q, k.transpose(1, 2), k, out), (q, k, k, out[:3]), (q, k, k, out[None]), (q, k.to_sparse(), k, out), (q.numpy, k, k, out),
                 (torch.nn.Parameter(q).to("meta"), k, k, out)]),
            (4, [(4,), None, [4, 64], (4, 64, 1), (4.0, 64), (1 << 40, 64), (5, 64), (4, 32)]), (5, [(2,), None, [2, 64], (3, 64), (2, 128)]),
            (6, [None, 0, "0", 1 << 40]), (7, [None, -1, "0", 1 << 64]), (8, ["0", 1.0, 1 << 40, 0])]:
        for other in others:
            assert cpu_call(*(good[:at] + [other] + good[at + 1:])) is None, (at, other)
    assert len(taken) == 1
    for n in (8, 10):
        with pytest.raises(TypeError):
            cpu_call(*(good + [None])[:n])


def test_blocks_that_are_not_plain_are_left(cpu_call):
    taken = []
    block = ctypes.CFUNCTYPE(ctypes.c_int, ctypes.c_void_p, ctypes.c_int32, ctypes.c_int32, ctypes.c_int32, *[ctypes.c_void_p] * 5)
    proxy = ctypes.CFUNCTYPE(ctypes.c_int, ctypes.c_void_p, ctypes.c_int32, ctypes.c_int32, ctypes.c_int32, *[ctypes.c_void_p] * 5, ctypes.c_int32,
                             ctypes.c_void_p)
    q, k, obs = torch.zeros(3, 4, 64, dtype=BF16), torch.zeros(3, 2, 64, dtype=BF16), torch.zeros(9, 4, 64, dtype=BF16)
    p = [t.data_ptr() for t in (q, k, k, q, obs)]
    for kind, more in [(block, ()), (proxy, (obs,))]:
        entry = kind(lambda *args: taken.append(args) or -5)
        args = lambda *tensors, begin=17: (ctypes.cast(entry, ctypes.c_void_p).value, 11, 5, tensors, (4, 64), (2, 64), -1, 13, begin)
        assert cpu_call(*args(q, k, k, q, *more)) == -5
        assert taken.pop() == (11, 5, 17, 3) + tuple(p[:4]) + ((p[4], 9) if more else ()) + (13,)
        for bad in [(q[:2], k, k, q), (q, k[:2], k, q), (q, k, k[:2], q), (q, k, k, q[:2]), (q, k, k, q.float())]:
            assert cpu_call(*args(*bad, *more)) is None
        for begin in ("17", 1.0, 1 << 40):
            assert cpu_call(*args(q, k, k, q, *more, begin=begin)) is None
    for bad in (obs[0], obs[:, :3], obs.float(), obs.transpose(0, 1)):
        assert cpu_call(*args(q, k, k, q, bad)) is None
    assert not taken


@pytest.mark.filterwarnings("ignore:The PyTorch API of nested tensors")
@pytest.mark.parametrize("rows", [(2, 2, 2), (2, 3, 4)])
def test_nested_tensors_are_left(cpu_call, rows):
    """A list of rows that may differ in length is no tensor of the cache, whatever its address; and asking for its sizes throws."""
    entry = STEP(lambda *_: 7)
    q = torch.zeros(4, 64, dtype=BF16)
    k = torch.nested.nested_tensor([torch.zeros(r, 64, dtype=BF16) for r in rows])
    args = lambda k: (ctypes.cast(entry, ctypes.c_void_p).value, 1, 0, (q, k, k, q), (4, 64), (2, 64), -1, 0, None)
    assert cpu_call(*args(torch.zeros(3, 2, 64, dtype=BF16))) == 7
    assert cpu_call(*args(k)) is None


def _cache(**more):
    cache = K.Cache(2, 8, 2, 64, 96, 64, [K.KvpSegment(0, 4000, K.KVP_TEXT, 0, 0, 0, 0)], scratch_sets=2, device="cuda:0", **more)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)
    for layer in range(2):
        k, v, token, weight, _, _ = cache.decode_ready(layer)
        k.copy_(torch.randn(k.shape, generator=gen, device="cuda"))
        v.copy_(torch.randn(v.shape, generator=gen, device="cuda"))
        token.copy_(torch.arange(96, device="cuda", dtype=torch.int32).expand(2, 96))
        weight.fill_(1.0)
        cache.set_state(layer, 96, 200)
    return cache


def _tensors(n, heads):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n + heads)
    return torch.randn((n, heads, 64), generator=gen, device="cuda", dtype=BF16)


CALLS = {
    "prefill_chunk": lambda c, out: c.prefill_chunk(1, 200, _tensors(40, 8), _tensors(40, 2), _tensors(41, 2)[:40], out),
    "keydiff": lambda c, out: c.prefill_chunk_keydiff(1, 200, _tensors(40, 8), _tensors(40, 2), _tensors(41, 2)[1:], out),
    "proxy": lambda c, out: c.prefill_chunk_proxy(1, 200, _tensors(40, 8), _tensors(40, 2), _tensors(41, 2)[1:], _tensors(9, 8), out),
    "decode": lambda c, out: c.decode_step(1, _tensors(3, 8)[1], _tensors(5, 2), _tensors(6, 2)[1:], None if out is None else out[0]),
    "decode_static": lambda c, out: c.decode_step_static(1, _tensors(3, 8)[1], _tensors(5, 2), _tensors(6, 2)[1:],
                                                         torch.empty_like(_tensors(1, 8)[0]) if out is None else out[0]),
}


@pytest.mark.gpu
@pytest.mark.parametrize("name", CALLS)
@pytest.mark.parametrize("given", [False, True])
def test_same_bits_as_through_ctypes(name, given):
    got = []
    for native in (True, False):
        cache = _cache()
        taken = []
        fast = cache._call
        assert fast is not B._not_taken
        cache._call = (lambda *a: taken.append(fast(*a)) or taken[-1]) if native else B._not_taken
        out = CALLS[name](cache, torch.zeros((40, 8, 64), device="cuda", dtype=BF16) if given else None)
        assert not native or taken == [0]
        if not name.startswith("decode"):
            cache.compact(1)
            got.append([out] + list(cache.decode_ready(1)[:4]))
        else:
            got.append([out])
        cache.close()
    for a, b in zip(*got):
        assert torch.equal(a.view(torch.uint8), b.view(torch.uint8))


@pytest.mark.gpu
@pytest.mark.parametrize("native", [True, False])
def test_refusals(native):
    cache = _cache()
    if not native:
        cache._call = B._not_taken
    q, k, out = _tensors(3, 8)[0], _tensors(5, 2), torch.empty((8, 64), device="cuda", dtype=BF16)
    cache.decode_step(0, q, k, k, out)
    for bad in [(q.float(), k, k, out), (q.cpu(), k, k, out), (q, k, k[1:], out), (q, k.transpose(0, 1), k, out), (q[:4], k, k, out),
                (q, k, k, out.t().contiguous().t()), (q, k, k, _tensors(3, 8)[:1]), (q, _tensors(5, 3), _tensors(5, 3), out)]:
        with pytest.raises(AssertionError):
            cache.decode_step(0, *bad)
    for layer, tail in [(2, k), (-1, k), (0, k[:0])]:
        with pytest.raises(K.KvpError) as e:
            cache.decode_step(layer, q, tail, tail, out)
        assert e.value.code == B.KVP_EINVAL
    block_q, block_k = _tensors(40, 8), _tensors(40, 2)
    with pytest.raises(K.KvpError) as e:
        cache.prefill_chunk(0, 199, block_q, block_k, block_k)      # not the next token
    first = e.value.code
    with pytest.raises(AssertionError):
        cache.prefill_chunk_proxy(0, 200, block_q, block_k, block_k, _tensors(9, 4))
    with pytest.raises(AssertionError):
        cache.prefill_chunk(0, 200, block_q, block_k[1:], block_k[1:])
    assert first == B.KVP_ESTATE or first == B.KVP_EINVAL
    cache.close()
    with pytest.raises(K.KvpError):
        cache.decode_step(0, q, k, k, out)
