"""The prompt kernel (csrc/prompt_mfma.hip) against 64-bit attention: rows around its blocks of 32 and 128, lengths around its
tiles of 64, sequence counts that do and do not divide over the XCDs."""
import pytest
import torch

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
# q and the weights carry 16 bits (hi + lo bf16 terms): 2^-16 of logits up to 12 moves a weight by 2e-4, of values up to 4.5
TOL = 1e-3


@pytest.fixture(scope="module")
def m():
    import paper_1911_02150_amd as lib
    lib.load_library()
    return lib


def causal(q, K, V, L):
    """q [n,128] of consecutive positions ending at L - 1."""
    n = q.shape[0]
    z = q.double() @ K[:max(L, 0)].double().t()
    at, last = torch.arange(max(L, 0), device=DEV), torch.arange(L - n, L, device=DEV)
    z.masked_fill_(at[None, :] > last[:, None], float("-inf"))
    return torch.nan_to_num(torch.softmax(z, -1), nan=0.0) @ V[:max(L, 0)].double()


@pytest.mark.parametrize("b,n,h,prefix", [
    (1, 33, 1, 0),         # one row past 32
    (2, 16, 8, 0),         # a whole block of 128 rows
    (3, 43, 3, 20),        # 129 rows: one in the second block; 63 positions
    (2, 64, 5, 0),         # positions fill a tile
    (8, 65, 2, 63),        # one sequence per XCD; rows that straddle tiles
    (5, 150, 8, 107),
    (1, 700, 12, 1),
])
def test_prompt(m, b, n, h, prefix):
    g = torch.Generator(device=DEV)
    g.manual_seed(n + h)
    cap = n + prefix + 5
    q = torch.randn(b, n, h, 128, generator=g, device=DEV) * 0.25
    K = torch.randn(b, cap, 128, generator=g, device=DEV).to(torch.bfloat16)
    V = torch.randn(b, cap, 128, generator=g, device=DEV).to(torch.bfloat16)
    lens = [n + prefix] * b
    lens[-1] = n + prefix + 5
    if b > 2:
        lens[1] = n // 2          # shorter than the prompt: the first rows see nothing
        lens[2] = 0
    for i, L in enumerate(lens):
        K[i, L:], V[i, L:] = float("nan"), float("inf")
    got = m.mqa_prefill_attention(q, K, V, torch.tensor(lens, dtype=torch.int32, device=DEV))
    for i, L in enumerate(lens):
        for j in range(h):
            assert float((got[i, :, j].double() - causal(q[i, :, j], K[i], V[i], L)).abs().max()) < TOL


@pytest.mark.parametrize("b,n,h,prefix", [(1, 33, 3, 0), (2, 128, 4, 64), (3, 129, 3, 0), (1, 513, 2, 30)])
def test_prompt_multi_head(m, b, n, h, prefix):
    g = torch.Generator(device=DEV)
    g.manual_seed(n)
    cap = n + prefix
    q = torch.randn(b, h, n, 128, generator=g, device=DEV) * 0.25
    K = torch.randn(b, h, cap, 128, generator=g, device=DEV).to(torch.bfloat16)
    V = torch.randn(b, h, cap, 128, generator=g, device=DEV).to(torch.bfloat16)
    got = m.mha_prefill_attention(q, K, V, torch.full((b,), cap, dtype=torch.int32, device=DEV))
    for i in range(b):
        for j in range(h):
            assert float((got[i, j].double() - causal(q[i, j], K[i, j], V[i, j], cap)).abs().max()) < TOL


def test_prompt_rescaling(m):
    """Logits that rise along the sequence by far more than the rescaling slack."""
    n, cap = 200, 200
    g = torch.Generator(device=DEV)
    g.manual_seed(1)
    q = torch.randn(1, n, 2, 128, generator=g, device=DEV)
    d = torch.randn(128, generator=g, device=DEV)
    q += d
    K = (torch.linspace(-1, 1, cap, device=DEV)[:, None] * d + 0.05 * torch.randn(cap, 128, generator=g, device=DEV)).to(torch.bfloat16)[None]
    V = torch.randn(1, cap, 128, generator=g, device=DEV).to(torch.bfloat16)
    got = m.mqa_prefill_attention(q, K, V, torch.tensor([cap], dtype=torch.int32, device=DEV))
    for j in range(2):      # logits up to 150
        assert float((got[0, :, j].double() - causal(q[0, :, j], K[0], V[0], cap)).abs().max()) < 1e-2


@pytest.mark.parametrize("multi_head", [False, True])
@pytest.mark.parametrize("n,h,prefix,at", [
    (200, 8, 0, 23),       # inside a wave's 32 rows
    (200, 8, 30, 200),
    (150, 3, 5, 154),      # the last position
    (300, 1, 0, 40),
    (300, 1, 17, 129),
])
@pytest.mark.parametrize("value", [float("inf"), float("nan")])
def test_prompt_values_that_are_not_finite(m, multi_head, n, h, prefix, at, value):
    """A V row that is not finite reaches the rows that see its position and no others, also inside a block of rows."""
    g = torch.Generator(device=DEV)
    g.manual_seed(n + h + at)
    cap = n + prefix
    if multi_head:
        q = torch.randn(1, h, n, 128, generator=g, device=DEV) * 0.25
        K = torch.randn(1, h, cap, 128, generator=g, device=DEV).to(torch.bfloat16)
        V = torch.randn(1, h, cap, 128, generator=g, device=DEV).to(torch.bfloat16)
    else:
        q = torch.randn(1, n, h, 128, generator=g, device=DEV) * 0.25
        K = torch.randn(1, cap, 128, generator=g, device=DEV).to(torch.bfloat16)
        V = torch.randn(1, cap, 128, generator=g, device=DEV).to(torch.bfloat16)
    V[..., at, :] = value
    attend = m.mha_prefill_attention if multi_head else m.mqa_prefill_attention
    got = attend(q, K, V, torch.tensor([cap], dtype=torch.int32, device=DEV))
    clean = V.clone()
    clean[..., at, :] = 0
    first = at - prefix                       # the first query that sees position `at`
    for j in range(h):
        o = got[0, j] if multi_head else got[0, :, j]
        Kj, Vj = (K[0, j], clean[0, j]) if multi_head else (K[0], clean[0])
        qj = q[0, j] if multi_head else q[0, :, j]
        want = causal(qj, Kj, Vj, cap)
        assert float((o[:first].double() - want[:first]).abs().max()) < TOL
        assert not torch.isfinite(o[first:]).any()


@pytest.mark.parametrize("multi_head", [False, True])
@pytest.mark.parametrize("n,h,prefix,cap", [
    (300, 1, 0, 300),      # the first rows see one team's tile only
    (40, 3, 217, 257),     # five tiles, the last of one position: one team's
    (40, 3, 280, 320),     # five whole tiles
    (33, 5, 352, 400),     # six, and one past the length
    (260, 2, 125, 385),
    (128, 8, 0, 1000),     # few tiles of a large cache: one team's
    (40, 3, 216, 1000),    # four tiles, the last one full
    (130, 3, 127, 1000),   # of the first row blocks four, of the last one five
])
def test_prompt_in_two_teams(m, multi_head, n, h, prefix, cap):
    """Few workgroups and more than 256 positions: every second tile is another team's."""
    g = torch.Generator(device=DEV)
    g.manual_seed(n + cap)
    b, one = 3, (h,) if multi_head else ()
    q = torch.randn(b, *((h, n) if multi_head else (n, h)), 128, generator=g, device=DEV) * 0.25
    K = torch.randn(b, *one, cap, 128, generator=g, device=DEV)
    q += 0.5 * K[0].reshape(-1, 128)[0]       # logits that differ between the teams' tiles
    K = (K * (1 + torch.arange(cap, device=DEV)[:, None] // 64 % 2)).to(torch.bfloat16)
    V = torch.randn(b, *one, cap, 128, generator=g, device=DEV).to(torch.bfloat16)
    lens = [n + prefix, n // 2, 0]
    for i, L in enumerate(lens):
        K[i, ..., L:, :], V[i, ..., L:, :] = float("nan"), float("inf")
    attend = m.mha_prefill_attention if multi_head else m.mqa_prefill_attention
    got = attend(q, K, V, torch.tensor(lens, dtype=torch.int32, device=DEV))
    for i, L in enumerate(lens):
        for j in range(h):
            o, qj = (got[i, j], q[i, j]) if multi_head else (got[i, :, j], q[i, :, j])
            Kj, Vj = (K[i, j], V[i, j]) if multi_head else (K[i], V[i])
            assert float((o.double() - causal(qj, Kj, Vj, L)).abs().max()) < 5 * TOL      # (logits up to 60)


@pytest.mark.parametrize("b,h,cap", [(1, 8, 4000), (3, 40, 700), (2, 64, 2000), (5, 1, 33), (20, 8, 129)])
@pytest.mark.parametrize("multi_head", [False, True])
def test_single_query(m, b, h, cap, multi_head):
    """One query per sequence is a prompt like any other: two-term weights of however many heads, and no memory but its output's."""
    g = torch.Generator(device=DEV)
    g.manual_seed(cap)
    of = (b, h) if multi_head else (b,)
    K, V = (torch.randn(*of, cap, 128, generator=g, device=DEV).bfloat16() for _ in range(2))
    q = torch.randn(*((b, h, 1) if multi_head else (b, 1, h)), 128, generator=g, device=DEV) * 0.1
    lens = (torch.arange(b, device=DEV, dtype=torch.int32) * 37 + cap) % (cap + 1)
    lens[1:2] = 0                                  # (nothing to attend to: zeros)
    ws = torch.full((1 << 24,), 7, dtype=torch.uint8, device=DEV)
    attend = m.mha_prefill_attention if multi_head else m.mqa_prefill_attention
    got = attend(q, K, V, lens, workspace=ws)
    assert (ws == 7).all()
    for i in range(b):
        for j in range(h):
            qj, o = (q[i, j], got[i, j]) if multi_head else (q[i, :, j], got[i, :, j])
            want = causal(qj, K[i, j] if multi_head else K[i], V[i, j] if multi_head else V[i], int(lens[i]))
            assert (o - want).norm() <= 5e-5 * want.norm()      # (16 bits of the logits and of the weights)
