"""The decoder stack and its weights: every pass multiplies by what the weights hold when it runs, however they came to hold it and whether the
pass is called or replayed, by the products that the same sizes get from a call of their own."""
import math

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def m():
    import paper_1911_02150_amd.binding as lib
    lib.load_library()
    return lib


def _weights(seed, layers, d, h, ff, vocab, cap):
    g = np.random.default_rng(seed)
    draw = lambda fan, *s: (g.standard_normal(s, dtype=np.float32) / np.float32(math.sqrt(fan)))  # noqa: E731
    return dict(E=draw(1, vocab, d), pos=draw(1, cap, d),
                layers=[dict(P_q=draw(d, h, d, 128), P_k=draw(d, d, 128), P_v=draw(d, d, 128), P_o=draw(h * 128, h, d, 128), W1=draw(d, d, ff),
                             W2=draw(ff, ff, d)) for _ in range(layers)])


def _prompts(seed, b, n, vocab):
    return torch.from_numpy(np.random.default_rng(seed).integers(0, vocab, (b, n)).astype(np.int32)).to(DEV)


def _tensors(stack):
    """Every weight: (where it is kept, its name)."""
    for layer in stack.layers:
        yield from ((layer, name) for name in layer)
    yield from ((stack.__dict__, name) for name in ("E", "pos"))


def _now(stack, b, cap):
    """A new stack of the weights as they are."""
    from paper_1911_02150_amd.decoder_stack import DecoderStack
    host = lambda t: t.detach().cpu().numpy().copy()  # noqa: E731
    return DecoderStack(dict(E=host(stack.E), pos=host(stack.pos), layers=[{k: host(v) for k, v in layer.items()} for layer in stack.layers]), b, cap, False, DEV)


def _pass(stack, prompts, n):
    for lens in stack.lens:
        lens.zero_()
    return stack.prefill(prompts), stack.step(prompts[:, 0].contiguous(), n)


def _same(stack, logits, fresh, prompts, n):
    ref = _pass(fresh, prompts, n)
    for got, want in zip(logits, ref):
        assert torch.equal(got, want)
    for l in range(len(stack.layers)):
        assert torch.equal(stack.K[l], fresh.K[l]) and torch.equal(stack.V[l], fresh.V[l]) and torch.equal(stack.lens[l], fresh.lens[l])


# prompts of some hundred and of some thousand rows (whose feed-forward packs its weights), steps of few and of many sequences
SIZES = [(4, 100, 2, 1024, 8, 64, 264), (20, 40, 2, 512, 4, 2048, 9000), (600, 1, 2, 512, 4, 1024, 32768), (64, 128, 3, 1024, 2, 2048, 520)]


@pytest.mark.parametrize("b, n, layers, d, h, ff, vocab", SIZES)
def test_weights_changed_between_passes(m, b, n, layers, d, h, ff, vocab):
    """In place, behind torch's version counter, by another tensor's memory, replaced: the next pass is that of a stack made from them."""
    from paper_1911_02150_amd.decoder_stack import DecoderStack
    stack, prompts = DecoderStack(_weights(b, layers, d, h, ff, vocab, n + 1), b, n + 1, False, DEV), _prompts(1, b, n, vocab)
    first = [t.clone() for t in _pass(stack, prompts, n)]
    for was, again in zip(first, _pass(stack, prompts, n)):
        assert torch.equal(was, again)                       # (a pass repeats itself)

    def changed(how):
        for at, name in _tensors(stack):
            how(at, name, at[name])
        return _now(stack, b, n + 1)

    def replace(at, name, t):
        at[name] = t.flip(0).contiguous()

    def move(at, name, t):
        t.data = t.data.clone().mul_(-0.5)                  # (the same tensor, other memory)

    for how in (lambda at, name, t: t.mul_(-1.5), lambda at, name, t: t.data.mul_(0.75), lambda at, name, t: torch.from_dlpack(t.detach()).neg_(), replace, move):
        fresh = changed(how)
        _same(stack, _pass(stack, prompts, n), fresh, prompts, n)


@pytest.mark.parametrize("b, n, layers, d, h, ff, vocab", SIZES)
def test_weights_changed_between_replays(m, b, n, layers, d, h, ff, vocab):
    """A captured prompt and step, replayed after the weights have changed: also to values that two fp16 terms do not hold, and back."""
    from paper_1911_02150_amd.decoder_stack import DecoderStack
    stack, prompts = DecoderStack(_weights(b, layers, d, h, ff, vocab, n + 1), b, n + 1, False, DEV), _prompts(1, b, n, vocab)
    token = prompts[:, 0].contiguous()
    _pass(stack, prompts, n)
    for lens in stack.lens:
        lens.zero_()
    places = list(stack.lens), list(stack._lens_next)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        logits = stack.prefill(prompts), stack.step(token, n)
    spread = torch.logspace(0, -9, ff, device=DEV)

    def scale(layer, by):
        layer["W1"].mul_(by), layer["W2"].div_(by[:, None])

    for how in (lambda: None, lambda: [at[name].mul_(-0.75) for at, name in _tensors(stack)], lambda: [at[name].data.add_(0.001) for at, name in _tensors(stack)],
                lambda: [scale(layer, spread) for layer in stack.layers], lambda: [scale(layer, 1 / spread) for layer in stack.layers],
                lambda: stack.layers[0]["W1"].view(-1)[::7].mul_(1e-9), lambda: stack.layers[0]["W2"].view(-1)[::7].mul_(1e-9)):
        how()
        for lens in places[0]:
            lens.zero_()
        graph.replay()
        torch.cuda.synchronize()
        ref = _pass(_now(stack, b, n + 1), prompts, n)
        assert torch.isfinite(ref[0]).all()
        for got, want in zip(logits, ref):
            assert torch.equal(got, want)


def _by_calls(m, stack, prompts):
    """prefill by the library's public calls on the float32 weights: logits, K, V."""
    (b, n), d, h, layers = prompts.shape, stack.d, stack.h, stack.layers
    x = m.mqa_stack_embed(prompts.reshape(-1), torch.arange(n, dtype=torch.int32, device=DEV).repeat(b), stack.E, stack.pos)
    hx, caches = m.mqa_stack_layernorm(x), []
    for l, w in enumerate(layers):
        K, V, lens, now = torch.zeros_like(stack.K[l]), torch.zeros_like(stack.V[l]), torch.zeros_like(stack.lens[l]), torch.zeros_like(stack.lens[l])
        m.mqa_project_append_kv_rows(hx.view(b, n, d), w["P_k"], w["P_v"], K, V, lens, now)
        caches.append((K, V))
        if l + 1 == len(layers):
            x, hx = (t.view(b, n, d)[:, -1].contiguous() for t in (x, hx))
        rows = x.shape[0]
        q = m.mqa_project_qkvo(m.MQA_PROJ_Q, hx, w["P_q"]).view(b, rows // b, h, 128)
        o = m.mqa_prefill_attention(q, K, V, now)
        hx = m.mqa_project_add_layernorm(m.MQA_PROJ_O, o.view(rows, h, 128), w["P_o"], x)
        u = m.mqa_project_qkvo_ex(m.MQA_PROJ_LINEAR, hx, w["W1"], epilogue=m.MQA_EPI_RELU)
        if l + 1 == len(layers):
            m.mqa_project_qkvo_ex(m.MQA_PROJ_LINEAR, u, w["W2"], out=x, epilogue=m.MQA_EPI_ADD)
        else:
            hx = m.mqa_project_add_layernorm(m.MQA_PROJ_LINEAR, u, w["W2"], x)
    return _logits(m, stack, x), caches


def _logits(m, stack, x):
    return m.mqa_project_qkvo(m.MQA_PROJ_O, m.mqa_stack_layernorm(x).view(-1, 1, stack.d), stack.E.view(1, -1, stack.d))


@pytest.mark.parametrize("b, n, d, h, ff, vocab", [(4, 100, 1024, 8, 64, 264), (3, 200, 1024, 8, 1024, 9000), (20, 40, 512, 2, 2048, 400), (1, 50, 1024, 8, 512, 32768), (2, 5, 64, 40, 128, 264)])
def test_prompt_is_its_calls(m, b, n, d, h, ff, vocab):
    """Up to some thousand rows a prompt is what the public calls make of the float32 weights, bit for bit: every product in their precision."""
    from paper_1911_02150_amd.decoder_stack import DecoderStack
    stack, prompts = DecoderStack(_weights(n, 2, d, h, ff, vocab, n + 1), b, n + 1, False, DEV), _prompts(1, b, n, vocab)
    want, caches = _by_calls(m, stack, prompts)
    assert torch.equal(stack.prefill(prompts), want)
    for l, (K, V) in enumerate(caches):
        assert torch.equal(stack.K[l], K) and torch.equal(stack.V[l], V)


@pytest.mark.parametrize("b", [1, 8, 16, 128, 300])
def test_logits_are_their_call(m, b):
    """So are the logits, of however few rows: of 1 to 16 the products of float32 instructions."""
    from paper_1911_02150_amd.decoder_stack import DecoderStack
    stack = DecoderStack(_weights(b, 1, 1024, 2, 64, 32768, 4), b, 4, False, DEV)
    x = torch.from_numpy(np.random.default_rng(b).standard_normal((b, 1024), dtype=np.float32)).to(DEV)
    assert torch.equal(stack.logits(x), _logits(m, stack, x))


def test_long_prompt_is_near_its_calls(m, monkeypatch):
    """With the feed-forward in one call: the same but for float32 sums in another order and the cache elements that these round the other way;
    without memory for its workspace: the same bits."""
    from paper_1911_02150_amd.decoder_stack import DecoderStack
    b, n, d, h, ff, vocab = 40, 128, 1024, 2, 2560, 264
    assert m.mqa_stack_feed_forward_plan(b * n, d, ff)[0] & 1
    stack, prompts = DecoderStack(_weights(n, 3, d, h, ff, vocab, n), b, n, False, DEV), _prompts(1, b, n, vocab)
    want, caches = _by_calls(m, stack, prompts)
    for close in (lambda x, y: float((x.float() - y.float()).abs().max()) <= (2e-3 if x.dtype == torch.float32 else 2.0 ** -7) * float(y.float().abs().max()), torch.equal):
        for lens in stack.lens:
            lens.zero_()
        assert close(stack.prefill(prompts), want)
        for l, (K, V) in enumerate(caches):
            assert close(stack.K[l], K) and close(stack.V[l], V)
        whole = stack._workspace

        def no_room(rows, nbytes=0):
            if nbytes > 4 * rows * (d + ff):
                raise torch.OutOfMemoryError
            return whole(rows, nbytes)

        monkeypatch.setattr(stack, "_workspace", no_room)


@pytest.mark.parametrize("multi_head", [False, True])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_other_caches(m, multi_head, dtype):
    """A program may put larger caches in, or of the other type: a step's attention takes what it needs."""
    from paper_1911_02150_amd.decoder_stack import DecoderStack
    w = _weights(1, 2, 64, 2, 64, 72, 9000)
    if multi_head:
        for layer in w["layers"]:
            layer["P_k"], layer["P_v"] = (np.stack([layer[name], -layer[name]]) for name in ("P_k", "P_v"))
    small, large = (DecoderStack(w, 1, cap, multi_head, DEV, cache_dtype=kind) for cap, kind in ((40, torch.bfloat16), (8200, dtype)))
    token = torch.tensor([5], dtype=torch.int32, device=DEV)
    small.step(token, 0)
    for l in range(2):
        small.K[l], small.V[l] = torch.zeros_like(large.K[l]), torch.zeros_like(large.V[l])
        small.lens[l].fill_(8000), large.lens[l].fill_(8000)
    assert torch.equal(small.step(token, 8000), large.step(token, 8000))
