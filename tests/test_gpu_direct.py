"""The float32 matrix-instruction kernel (csrc/decode_direct.hip) against 64-bit attention: every cache type and width it
covers, head counts around its blocks of 16 and 32, lengths around its tiles of 16, ranges, windows and the beam step."""
import pytest
import torch

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
TYPES = [(torch.float32, 64), (torch.float32, 128), (torch.bfloat16, 64)]
# a float32 logit of k products is off by at most k 2^-24 |q||k|, at most 6 here (5e-5 for k = 128), which moves a
# weight by that share; the weighted sum and the exponentials add a few 2^-24 of values up to 5
TOL = 4e-4


@pytest.fixture(scope="module")
def m():
    import paper_1911_02150_amd as lib
    lib.load_library()
    return lib


def attend(q, K, V, lens, lo=None):
    """q [n,G,k]; K, V [n,cap,k]."""
    out = torch.zeros(q.shape, dtype=torch.float64, device=DEV)
    for i, L in enumerate(lens):
        a = 0 if lo is None else max(0, L - lo)
        if L > a:
            w = torch.softmax(q[i].double() @ K[i, a:L].double().t(), -1)
            out[i] = w @ V[i, a:L].double()
    return out


def inputs(n, G, cap, k, dtype, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    q = torch.randn(n, G, k, generator=g, device=DEV) * k ** -0.5 * 2
    K = torch.randn(n, cap, k, generator=g, device=DEV).to(dtype)
    V = torch.randn(n, cap, k, generator=g, device=DEV).to(dtype)
    return q, K, V


@pytest.mark.parametrize("dtype,k", TYPES)
@pytest.mark.parametrize("G,cap,lens", [
    (1, 40, [0, 1, 15, 16, 17, 40]),
    (8, 64, [64, 63, 33, 2, 0, 48]),              # 4 waves
    (16, 65, [65, 64, 0, 1, 16, 31]),             # 8 waves
    (17, 130, [130, 129, 128, 127, 3, 0]),        # two blocks of 16 heads in a wave
    (33, 96, [96, 95, 1, 0, 80, 17]),             # two head groups
    (5, 1500, [1500, 1499, 256, 257, 0, 31]),     # several ranges and a merge
])
def test_direct(m, dtype, k, G, cap, lens):
    q, K, V = inputs(len(lens), G, cap, k, dtype, 3)
    for i, L in enumerate(lens):                  # what lies beyond a length is never used
        K[i, L:], V[i, L:] = float("nan"), float("inf")
    L = torch.tensor(lens, dtype=torch.int32, device=DEV)
    got = m.mqa_decode_step(q, K, V, L)
    assert float((got.double() - attend(q, K, V, lens)).abs().max()) < TOL
    got = m.mqa_decode_step(q, K, V, L, tuning=dict(splits=2))
    assert float((got.double() - attend(q, K, V, lens)).abs().max()) < TOL
    got = m.mqa_decode_step_window(q, K, V, L, 20)
    assert float((got.double() - attend(q, K, V, lens, 20)).abs().max()) < TOL


@pytest.mark.parametrize("dtype,k", TYPES)
def test_direct_multi_head(m, dtype, k):
    b, h, cap, lens = 3, 5, 70, [70, 0, 33]
    q, K, V = inputs(b * h, 1, cap, k, dtype, 4)
    L = torch.tensor(lens, dtype=torch.int32, device=DEV)
    got = m.mha_decode_step(q.view(b, h, k), K.view(b, h, cap, k), V.view(b, h, cap, k), L)
    want = attend(q, K, V, [lens[i // h] for i in range(b * h)]).view(b, h, k)
    assert float((got.double() - want).abs().max()) < TOL


@pytest.mark.parametrize("dtype,k", TYPES)
def test_direct_sharp_and_wide(m, dtype, k):
    """Logits that rise along the sequence by more than the rescaling slack, and one that takes all the weight."""
    q, K, V = inputs(2, 3, 200, k, dtype, 5)
    K[0] = (torch.linspace(0, 6, 200, device=DEV)[:, None] * q[0, 0] / q[0, 0].norm()).to(dtype)
    K[1, 77] = (60 * q[1, 1] / q[1, 1].norm()).to(dtype)
    lens = [200, 200]
    got = m.mqa_decode_step(q, K, V, torch.tensor(lens, dtype=torch.int32, device=DEV))
    assert float((got.double() - attend(q, K, V, lens)).abs().max()) < 10 * TOL      # logits up to 60


@pytest.mark.parametrize("dtype,k", TYPES)
def test_direct_beams(m, dtype, k):
    b, beam, h, cs, co = 2, 3, 4, 300, 40
    q, K, V = inputs(b * beam, h, co, k, dtype, 6)
    _, Ks, Vs = inputs(b, 1, cs, k, dtype, 7)
    ls, lo = [300, 17], [40, 1, 16, 33, 0, 5]
    got = m.mqa_decode_step_beams(q.view(b, beam, h, k), Ks, Vs, torch.tensor(ls, dtype=torch.int32, device=DEV),
                                  K.view(b, beam, co, k), V.view(b, beam, co, k), torch.tensor(lo, dtype=torch.int32, device=DEV))
    for r in range(b * beam):
        Kc, Vc = (torch.cat([s[r // beam, :ls[r // beam]], own[r, :lo[r]]])[None] for s, own in ((Ks, K), (Vs, V)))
        want = attend(q[r:r + 1], Kc, Vc, [Kc.shape[1]])
        assert float((got.view(b * beam, h, k)[r].double() - want[0]).abs().max()) < TOL
