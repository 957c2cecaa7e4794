"""The binding's native calls (csrc/calls.cpp): taken for plain arguments, with the general path's results; everything else is left to
the general path, with its answers and errors."""
import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def m():
    import paper_1911_02150_amd.binding as lib
    lib.load_library()
    return lib


def _t(seed, *shape, dtype=torch.float32):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return torch.empty(shape, dtype=torch.float32, device=DEV).normal_(generator=g).mul_(0.3).to(dtype)


def _cases(m, dtype):
    """name, a call with fresh buffers (returns everything it wrote), by an argument for the output or None"""
    b, h, d, k, cap, n, e = 3, 4, 64, 128, 48, 40, 2
    lens = torch.tensor([5, 0, 40], dtype=torch.int32, device=DEV)
    K, V, Km, Vm = (_t(i, *s, k, dtype=dtype) for i, s in enumerate([(b, cap)] * 2 + [(b, h, cap)] * 2))
    Pq, Pk, Pv, Pkm, Pvm, Po = _t(5, h, d, k), _t(6, d, k), _t(7, d, k), _t(8, h, d, k), _t(9, h, d, k), _t(10, h, d, k)
    x, q, o3 = _t(11, b, d), _t(12, b, h, k), _t(13, b, h, k)
    ws = torch.empty(1 << 22, dtype=torch.uint8, device=DEV)
    new = lambda *s: torch.zeros(s, device=DEV)  # noqa: E731
    full = torch.full((b,), cap, dtype=torch.int32, device=DEV)

    def append(multi_head, out):
        Kc, Vc, after = (Km if multi_head else K).clone(), (Vm if multi_head else V).clone(), torch.zeros_like(lens)
        got = m.mqa_project_append_qkv(x, Pq, Pkm if multi_head else Pk, Pvm if multi_head else Pv, Kc, Vc, lens, after, q=new(b, h, k) if out else None)
        return got, Kc, Vc, after

    def memory(multi_head, valid):
        Kc, Vc, got = torch.zeros_like(Km if multi_head else K), torch.zeros_like(Vm if multi_head else V), torch.zeros_like(lens)
        m.mqa_project_memory_kv(_t(14, b, n, d), Pkm if multi_head else Pk, Pvm if multi_head else Pv, Kc, Vc, got, mem_lens=valid)
        return Kc, Vc, got

    def reorder(Ks, Vs):
        out = torch.zeros_like(Ks), torch.zeros_like(Vs), torch.zeros_like(lens)
        m.mqa_beam_reorder_kv(Ks, Vs, lens, torch.tensor([2, 2, 0], dtype=torch.int32, device=DEV), *out)
        return out

    def norm(mode, src, P):
        acc = _t(15, b, 64)
        return m.mqa_project_add_layernorm(mode, src, P, acc, workspace=ws), acc

    yield from [
        ("decode", lambda: m.mqa_decode_step(q, K, V, lens, workspace=ws)), ("decode", lambda: m.mha_decode_step(q, Km, Vm, lens, o=new(b, h, k), scale=0.5, workspace=ws)),
        ("decode", lambda: m.mqa_decode_step_window(q, K, V, lens, 7, workspace=ws)),
        ("decode", lambda: m.mha_decode_step_window(q, Km, Vm, lens, 7, o=new(b, h, k), workspace=ws)),
        ("append_qkv", lambda: append(False, True)), ("append_qkv", lambda: append(True, False)),
        ("memory_kv", lambda: memory(False, None)), ("memory_kv", lambda: memory(True, lens)),
        ("attend_rows", lambda: m.mqa_memory_decode_step(_t(16, b, e, h, k), K, V, lens, workspace=ws)),
        ("beams", lambda: m.mqa_decode_step_beams(_t(17, b, e, h, k), K, V, lens, _t(18, b, e, 9, k, dtype=dtype), _t(19, b, e, 9, k, dtype=dtype),
                                                  torch.full((b * e,), 9, dtype=torch.int32, device=DEV), workspace=torch.empty(1 << 22, dtype=torch.uint8, device=DEV))),
        ("reorder", lambda: reorder(K, V)), ("reorder", lambda: reorder(Km, Vm)),
        ("project", lambda: m.mqa_project_qkvo(m.MQA_PROJ_Q, x, Pq)), ("project", lambda: m.mqa_project_qkvo(m.MQA_PROJ_O, o3, Po, out=new(b, d))),
        ("project", lambda: m.mqa_project_qkvo(m.MQA_PROJ_KV, x, Pk)), ("project", lambda: m.mqa_project_qkvo(m.MQA_PROJ_KV_MH, x, Pkm)),
        ("project", lambda: m.mqa_project_qkvo_ex(m.MQA_PROJ_LINEAR, x, Pk, epilogue=m.MQA_EPI_RELU)),
        ("project", lambda: m.mqa_project_qkvo_ex(m.MQA_PROJ_LINEAR, x, Pk, out=_t(20, b, k), epilogue=m.MQA_EPI_ADD)),
        ("add_layernorm", lambda: norm(m.MQA_PROJ_O, o3, Po)), ("add_layernorm", lambda: norm(m.MQA_PROJ_LINEAR, x, _t(21, d, 64))),
    ]
    if dtype == torch.bfloat16:
        yield "attend_rows", lambda: m.mqa_prefill_attention(_t(22, b, n, h, k), K, V, full, workspace=ws)
        yield "attend_rows", lambda: m.mha_prefill_attention(_t(23, b, h, n, k), Km, Vm, full, o=new(b, h, n, k), workspace=ws)


class _Watch:
    """The native module, with what its functions returned; or (off) one that takes nothing."""

    def __init__(self, native, on):
        self.native, self.on, self.took = native, on, []

    def __getattr__(self, name):
        def call(*args):
            done = getattr(self.native, name)(*args) if self.on else None
            self.took.append((name, done is not None))
            return done
        return call


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_same_as_the_general_path(m, dtype, monkeypatch):
    native = m._native
    for name, call in _cases(m, dtype):
        got = []
        for on in (True, False):
            watch = _Watch(native, on)
            monkeypatch.setattr(m, "_native", watch)
            got.append(call())
            assert watch.took == [(name, on)], name
        a, b = ((g if isinstance(g, tuple) else (g,)) for g in got)
        assert len(a) == len(b) and all(torch.equal(x, y) and x.dtype == y.dtype and x.shape == y.shape for x, y in zip(a, b)), name


def test_left_to_the_general_path(m, monkeypatch):
    b, h, k, cap = 2, 4, 128, 32
    q, K, V = _t(1, b, h, k), _t(2, b, cap, k, dtype=torch.bfloat16), _t(3, b, cap, k, dtype=torch.bfloat16)
    lens, ws = torch.full((b,), cap, dtype=torch.int32, device=DEV), torch.empty(1 << 20, dtype=torch.uint8, device=DEV)
    ref = m.mqa_decode_step(q, K, V, lens, workspace=ws)
    watch = _Watch(m._native, True)
    monkeypatch.setattr(m, "_native", watch)

    class Sub(torch.Tensor):
        pass

    def left(call):
        watch.took.clear()
        try:
            return call()
        finally:
            assert all(not taken for _, taken in watch.took)

    assert torch.equal(left(lambda: m.mqa_decode_step(q.as_subclass(Sub), K, V, lens, workspace=ws)), ref)
    assert torch.equal(left(lambda: m.mqa_decode_step(q, K, V, lens)), ref) and torch.equal(left(lambda: m.mqa_decode_step(q, K, V, lens, stream=torch.cuda.current_stream(), workspace=ws)), ref)
    strided = torch.empty(2 << 20, dtype=torch.uint8, device=DEV)[::2]
    assert torch.equal(left(lambda: m.mqa_decode_step(q, K, V, lens, workspace=strided)), ref)
    assert torch.equal(m.mqa_project_qkvo(m.MQA_PROJ_LINEAR, q.view(b, h * k), _t(4, h * k, 64), out=torch.empty(64 * b, device=DEV)).view(b, 64),
                       m.mqa_project_qkvo(m.MQA_PROJ_LINEAR, q.view(b, h * k), _t(4, h * k, 64)))
    for error, call in ((ValueError, lambda: m.mqa_decode_step(q.transpose(0, 1), K, V, lens, workspace=ws)), (TypeError, lambda: m.mqa_decode_step(q.double(), K, V, lens, workspace=ws)),
                        (ValueError, lambda: m.mqa_decode_step(q, K[:, :16].contiguous(), V, lens, workspace=ws)), (TypeError, lambda: m.mqa_decode_step(q, K, V, lens.long(), workspace=ws)),
                        (ValueError, lambda: m.mqa_decode_step(q.cpu(), K, V, lens, workspace=ws)), (TypeError, lambda: m.mqa_decode_step(q, K.half(), V.half(), lens, workspace=ws)),
                        (ValueError, lambda: m.mqa_decode_step(q, K, V, lens, o=torch.empty(b, h, 64, device=DEV), workspace=ws)),
                        (ValueError, lambda: m.mqa_project_qkvo_ex(m.MQA_PROJ_LINEAR, q.view(b, h * k), _t(4, h * k, 64), epilogue=m.MQA_EPI_ADD))):
        with pytest.raises(error):
            left(call)
    with pytest.raises(RuntimeError):              # (a transform's tensor has no address)
        left(lambda: torch.func.vmap(lambda row: m.mqa_decode_step(row, K, V, lens, workspace=ws))(q.unsqueeze(0)))
    # the library's own refusal, with its status, from either path
    with pytest.raises(m.MqaError) as refused:
        m.mqa_decode_step(torch.empty(q.numel() + 1, device=DEV)[1:].view(q.shape), K, V, lens, workspace=ws)
    assert refused.value.status == 3 and "mqa_decode_step failed" in str(refused.value)


def test_modes_see_what_they_saw(m, monkeypatch):
    """A function mode and a dispatch mode are told of the output, as by the general path."""
    from torch.overrides import TorchFunctionMode
    from torch.utils._python_dispatch import TorchDispatchMode
    x, P = _t(1, 3, 64), _t(2, 64, 128)
    ref = m.mqa_project_qkvo(m.MQA_PROJ_LINEAR, x, P)
    watch = _Watch(m._native, True)
    monkeypatch.setattr(m, "_native", watch)
    seen = []

    class Functions(TorchFunctionMode):
        def __torch_function__(self, func, types, args=(), kwargs=None):
            seen.append(func)
            return func(*args, **(kwargs or {}))

    class Dispatches(TorchDispatchMode):
        def __torch_dispatch__(self, func, types, args=(), kwargs=None):
            seen.append(func)
            return func(*args, **(kwargs or {}))

    for mode, what in ((Functions, torch.empty), (Dispatches, torch.ops.aten.empty.memory_format)):
        seen.clear()
        with mode():
            got = m.mqa_project_qkvo(m.MQA_PROJ_LINEAR, x, P)
        assert what in seen and torch.equal(got, ref) and watch.took.pop() == ("project", False)
    assert torch.equal(m.mqa_project_qkvo(m.MQA_PROJ_LINEAR, x, P), ref) and watch.took.pop() == ("project", True)


def test_parameters_threads_and_streams(m):
    """Weights as Parameters, calls from threads on streams of their own, buffers that are new every time."""
    import threading
    d, k, rows = 64, 128, 40
    P = torch.nn.Parameter(_t(1, d, k))
    xs = [_t(10 + i, rows, d) for i in range(4)]
    refs = [m.mqa_project_qkvo(m.MQA_PROJ_LINEAR, x, P) for x in xs]
    assert not refs[0].requires_grad and m._native.project(m.MQA_PROJ_LINEAR, xs[0], P, None, None) is not None
    torch.cuda.synchronize()
    bad = []

    def work(i):
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream):
            for _ in range(50):
                if not torch.equal(m.mqa_project_qkvo(m.MQA_PROJ_LINEAR, xs[i], P), refs[i]):
                    bad.append(i)

    threads = [threading.Thread(target=work, args=(i,)) for i in range(4)]
    [t.start() for t in threads], [t.join() for t in threads]
    assert not bad
