"""Products of packed operands (csrc/packed.hip): every tile form at its edges against float64, the packing's verdict and
scales, the layernorm that packs, and the decoder stack with and without them."""
import math

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
EPS = 2.0 ** -24
# columns, rows of the forms' tiles (form = 16 x the place here + parts)
TILES = [(256, 256), (256, 128), (128, 128), (128, 64), (64, 64), (128, 32)]


@pytest.fixture(scope="module")
def m():
    import paper_1911_02150_amd.binding as lib
    lib.load_library()
    return lib


def _normal(seed, *shape, std=1.0):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return torch.empty(shape, dtype=torch.float32, device=DEV).normal_(generator=g).mul_(std)


def _pack_rows(m, x):
    """layernorm(x) as float32 and packed."""
    y, packed = torch.empty_like(x), torch.empty(4 * x.numel(), dtype=torch.uint8, device=DEV)
    m.mqa_stack_layernorm_packed(x, packed, out=y)
    return y, packed


def _terms(packed, lines, C):
    """A packed matrix as float64 [lines, C], by the layout that mqa.h leaves to the library."""
    t = packed[:4 * lines * C].view(torch.float16).view(C // 32, 2, lines, 32).double()
    return (t[:, 0] + t[:, 1]).permute(1, 0, 2).reshape(lines, C)


def _bound(x, w, C):
    """Two terms of each operand (2^-22, the small times the small left out) and float32 sums of 3 C products in any order."""
    size = x.double().abs() @ w.double().abs()
    return (4 * 2.0 ** -22 + 2 * math.sqrt(3 * C) * EPS) * size + 1e-30


@pytest.mark.parametrize("C", [32, 96, 352])
@pytest.mark.parametrize("form", range(6))
def test_tiles(m, form, C):
    TN, TM = TILES[form]
    e = m.load_library().mqa_stack_layernorm_exponent(C)
    for rows, N in ((1, 8), (TM - 1, TN - 8), (TM + 1, TN + 8), (2 * TM + 17, 40)):
        x = _normal(rows, rows, C)
        W = _normal(N, C, N, std=C ** -0.5)
        y, packed = _pack_rows(m, x)
        w = m.PackedWeights(m.MQA_PROJ_LINEAR, W)
        assert w.verdict.item() == 0
        ref, bound = y.double() @ W.double(), _bound(y, W, C)
        out = torch.full((rows + 1, N), 7.0, device=DEV)
        m.mqa_stack_product(packed, w, 2.0 ** -e, out[:rows], rows, 16 * form + 1)
        assert ((out[:rows] - ref).abs() <= bound).all() and (out[rows] == 7).all(), (rows, N)
        m.mqa_stack_product(packed, w, 2.0 ** -e, out[:rows], rows, 16 * form + 1, m.MQA_EPI_ADD)
        assert ((out[:rows] - 2 * ref).abs() <= 2 * bound + 4 * EPS * ref.abs()).all()
        m.mqa_stack_product(packed, w, 2.0 ** -e, out[:rows], rows, 16 * form + 1, m.MQA_EPI_RELU)
        assert ((out[:rows] - ref.clamp(min=0)).abs() <= bound).all()
        S = {32: 1, 96: 3, 352: 2}[C]
        parts = torch.full((S * rows + 1, N), 7.0, device=DEV)
        m.mqa_stack_product(packed, w, 2.0 ** -e, parts[:S * rows], rows, 16 * form + S)
        assert ((parts[:-1].view(S, rows, N).double().sum(0) - ref).abs() <= bound).all() and (parts[-1] == 7).all()


@pytest.mark.parametrize("rows, d, S", [(1, 32, 0), (3, 1024, 1), (2, 1056, 3), (5, 2048, 2), (3, 2080, 0), (7, 4096, 8)])
def test_layernorm(m, rows, d, S):
    x, parts = _normal(1, rows, d, std=3.0) + 0.5, _normal(2, max(S, 1), rows, d)
    full = x.double() + (parts[:S].double().sum(0) if S else 0)
    y, packed, kept = torch.empty_like(x), torch.zeros(4 * x.numel() + 64, dtype=torch.uint8, device=DEV), x.clone()
    m.mqa_stack_layernorm_packed(x, packed[:-64], out=y, parts=parts if S else None, S=S)
    ref = full - full.mean(1, keepdim=True)
    ref = ref / torch.sqrt((ref * ref).mean(1, keepdim=True) + 1e-6)
    assert ((x - full).abs() <= (S + 1) * EPS * (kept.abs() + parts.abs().sum(0))).all()
    assert (y - ref).abs().max() <= 1e-5 and (packed[-64:] == 0).all()
    e = m.load_library().mqa_stack_layernorm_exponent(d)
    assert math.sqrt(d) * 2.0 ** e <= 2.0 ** 15 and e >= 8
    got = _terms(packed, rows, d) * 2.0 ** -e
    assert ((got - y.double()).abs() <= 2.0 ** -22 * y.double().abs() + 2.0 ** (-25 - e)).all()
    again = torch.zeros_like(packed)
    m.mqa_stack_layernorm_packed(kept, again[:-64], parts=parts if S else None, S=S)         # without y
    assert torch.equal(again, packed) and torch.equal(kept, x)


@pytest.mark.parametrize("mode, shape", [("LINEAR", (96, 40)), ("LINEAR", (544, 264)), ("Q", (3, 64, 40)), ("O", (1, 72, 288)), ("O", (2, 48, 16))])
def test_packing(m, mode, shape):
    mode = getattr(m, "MQA_PROJ_" + mode)
    P = _normal(5, *shape, std=0.05)
    if mode == m.MQA_PROJ_LINEAR:
        flat = P
    else:
        flat = (P.permute(1, 0, 2) if mode == m.MQA_PROJ_Q else P.permute(0, 2, 1)).reshape(-1, shape[0] * shape[2] if mode == m.MQA_PROJ_Q else shape[1])
    C, N = flat.shape
    first = m.PackedWeights(mode, P)
    row_scale = None
    if mode == m.MQA_PROJ_LINEAR:                  # behind the columns of another one
        row_scale = m.PackedWeights(mode, _normal(6, 64, C) * torch.logspace(-1, 1, C, device=DEV))
        flat = flat * row_scale.data[4 * 64 * C:].view(torch.float32)[None, :].t()
        first = m.PackedWeights(mode, P, row_scale)
    scales = first.data[4 * N * C:].view(torch.float32).double()
    largest = flat.abs().amax(0).double() / scales
    assert first.verdict.item() == 0 and (largest >= 2.0 ** 14).all() and (largest < 2.0 ** 15).all()
    got = _terms(first.data, N, C) * scales[:, None]
    assert ((got - flat.t().double()).abs() <= 2.0 ** -22 * flat.t().double().abs() + 2.0 ** -25 * scales[:, None]).all()


@pytest.mark.parametrize("what, verdict", [("zeros", 0), ("column of zeros", 0), ("six small", 0), ("seven small", 1), ("one large", 0), ("large", 1), ("nan", 1),
                                           ("inf", 1), ("huge", 1), ("tiny", 1)])
def test_verdict(m, what, verdict):
    W = _normal(9, 512, 72)
    W += W.sign() * 0.01
    if what == "zeros":
        W[::2] = 0
    elif what == "column of zeros":
        W[:, 70] = 0
    elif what.endswith("small"):
        W[256:256 + (6 if what[0] == "s" and what[1] == "i" else 7), 3] = 1e-6
    elif what == "one large":
        W[7, 3] = 100.0
    elif what == "large":
        W[7, 71] = 1e6
    else:
        W[500, 71] = dict(nan=float("nan"), inf=float("-inf"), huge=2.0 ** 100, tiny=1.0)[what]
        if what == "tiny":
            W[:, 71] = 2.0 ** -101
    assert m.PackedWeights(m.MQA_PROJ_LINEAR, W).verdict.item() == verdict


def _weights(seed, layers, d, h, ff, vocab, cap):
    g = np.random.default_rng(seed)
    draw = lambda fan, *s: (g.standard_normal(s) / math.sqrt(fan)).astype(np.float32)  # noqa: E731
    return dict(E=draw(1, vocab, d), pos=draw(1, cap, d),
                layers=[dict(P_q=draw(d, h, d, 128), P_k=draw(d, d, 128), P_v=draw(d, d, 128), P_o=draw(h * 128, h, d, 128), W1=draw(d, d, ff),
                             W2=draw(ff, ff, d)) for _ in range(layers)])


# prompts whose products are packed whole, in part and not at all, a step of each kind, and widths that have no packed form
@pytest.mark.parametrize("b, n, d, ff, vocab", [(20, 40, 512, 2048, 9000), (3, 100, 512, 1024, 16400), (640, 4, 256, 1024, 520), (4, 9, 72, 160, 400), (3, 50, 96, 200, 1008)])
def test_stack_with_and_without(m, b, n, d, ff, vocab):
    from paper_1911_02150_amd.decoder_stack import DecoderStack
    w = _weights(b, 2, d, 2, ff, vocab, n + 1)
    prompts = torch.from_numpy(np.random.default_rng(1).integers(0, vocab, (b, n)).astype(np.int32)).to(DEV)
    packed, plain = (DecoderStack(w, b, n + 1, False, DEV) for _ in range(2))
    plain._packs = {}
    used = packed._plan(b * n)
    print(b, n, used, packed._plan(b))
    assert not packed._packs or not packed._unheld
    assert plain._plan(b * n) == [(0, 0, 0)] * 2 and (d % 32 == 0 or not packed._packs)
    for got, ref in ((packed.prefill(prompts), plain.prefill(prompts)), (packed.step(prompts[:, 0].contiguous(), n), plain.step(prompts[:, 0].contiguous(), n))):
        scale = float(ref.abs().max())
        assert float((got - ref).abs().max()) <= 2e-3 * scale      # (cache elements that round the other way, as between prompt and steps)
    for l in range(2):
        assert torch.equal(packed.lens[l], plain.lens[l])
        assert float(((packed.K[l].float() - plain.K[l].float()).abs() > 0).float().mean()) < 2e-2


def test_stack_follows_its_weights(m):
    """Weights that are changed in place or replaced count from the next pass on, and those that two terms do not hold are not packed."""
    from paper_1911_02150_amd.decoder_stack import DecoderStack
    b, n, d, ff, vocab = 20, 40, 512, 2048, 16400
    w = _weights(3, 1, d, 2, ff, vocab, n)
    prompts = torch.from_numpy(np.random.default_rng(2).integers(0, vocab, (b, n)).astype(np.int32)).to(DEV)
    stack = DecoderStack(w, b, n, False, DEV)
    assert stack._plan(b * n)[0][0], "this size is to run packed"
    stack.prefill(prompts)
    place = stack._packs[0, "W1"][0].data.data_ptr()

    def check():
        now = dict(E=stack.E.cpu().numpy(), pos=w["pos"], layers=[{k: v.cpu().numpy() for k, v in stack.layers[0].items()}])
        plain = DecoderStack(now, b, n, False, DEV)
        plain._packs = {}
        for lens in stack.lens:
            lens.zero_()
        got, ref = stack.prefill(prompts), plain.prefill(prompts)
        assert float((got - ref).abs().max()) <= 2e-3 * float(ref.abs().max())

    stack.layers[0]["W1"].mul_(-1.5)
    check()
    assert stack._packs[0, "W1"][0].data.data_ptr() == place
    stack.layers[0]["W2"] = stack.layers[0]["W2"].clone().neg_()
    check()
    stack.E = stack.E.flip(0).contiguous()
    check()
    stack.layers[0]["W1"].data.mul_(2.0)          # (unseen)
    stack.pack()
    check()
    stack.layers[0]["W1"][:20, 5] = 1e-9
    check()
    assert (0, "W1") in stack._unheld and stack._plan(b * n)[0] == (0, 0, 0)


def test_two_layers_follow_their_weights(m):
    """The same of the layer whose every row counts: all rows of a prompt's last layer but the last positions' stop at its caches."""
    from paper_1911_02150_amd.decoder_stack import DecoderStack
    b, n, d, ff, vocab = 20, 40, 512, 2048, 400
    w = _weights(4, 2, d, 2, ff, vocab, n)
    prompts = torch.from_numpy(np.random.default_rng(3).integers(0, vocab, (b, n)).astype(np.int32)).to(DEV)
    stack = DecoderStack(w, b, n, False, DEV)
    assert all(stack._plan(b * n)[0][:2]), "this size is to run packed"
    for name in ("P_q", "W1", "W2"):
        if name == "W1":
            stack.layers[0][name].mul_(-1.5)
        else:
            stack.layers[0][name] = stack.layers[0][name].clone().neg_()
        now = dict(E=w["E"], pos=w["pos"], layers=[{k: v.cpu().numpy() for k, v in layer.items()} for layer in stack.layers])
        plain = DecoderStack(now, b, n, False, DEV)
        plain._packs = {}
        for lens in stack.lens:
            lens.zero_()
        got, ref = stack.prefill(prompts), plain.prefill(prompts)
        assert float((got - ref).abs().max()) <= 2e-3 * float(ref.abs().max())
        assert float((stack.K[1] - plain.K[1]).abs().max()) <= 0.05 * float(plain.K[1].abs().max())      # (bf16 near-ties of the layer before)
