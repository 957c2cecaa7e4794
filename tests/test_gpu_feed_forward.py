"""mqa_stack_feed_forward (csrc/packed.hip): its products from packed operands at the edges of their tiles against float64, and the values that
two fp16 terms do not hold, which it multiplies as the calls it stands for do."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
EPS = 2.0 ** -24


@pytest.fixture(scope="module")
def m():
    import paper_1911_02150_amd.binding as lib
    lib.load_library()
    return lib


def _normal(seed, *shape, std=1.0):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return torch.empty(shape, dtype=torch.float32, device=DEV).normal_(generator=g).mul_(std)


def _inputs(rows, d, ff):
    return _normal(rows, rows, d), _normal(d, d, ff, std=d ** -0.5), _normal(ff, ff, d, std=ff ** -0.5)


def _call(m, x, W1, W2):
    """What the call makes of x, from a workspace of just its size and full of NaN."""
    nbytes = m.mqa_stack_feed_forward_plan(*x.shape, W1.shape[1])[1]
    room = torch.full((nbytes + 64,), 255, dtype=torch.uint8, device=DEV)
    out = m.mqa_stack_feed_forward(x.clone(), W1, W2, room[:nbytes])
    assert (room[nbytes:] == 255).all()
    return out


def _calls(m, x, W1, W2):
    """... and the three calls."""
    x, hx = x.clone(), m.mqa_stack_layernorm(x)
    u = m.mqa_project_qkvo_ex(m.MQA_PROJ_LINEAR, hx, W1, epilogue=m.MQA_EPI_RELU)
    return m.mqa_project_qkvo_ex(m.MQA_PROJ_LINEAR, u, W2, out=x, epilogue=m.MQA_EPI_ADD)


def _reference(m, x, W1, W2):
    """float64 of the float32 layernorm, and how far sums may be from it: two terms of each operand (2^-22, the small times the small
    left out) and float32 sums of 3 C products in any order, of the hidden values and then of the outputs; two terms of the hidden values, cut off
    at 2^-25 of what they are scaled to, and the residual's rounding."""
    d, ff = W1.shape
    y, w1, w2 = m.mqa_stack_layernorm(x).double(), W1.double(), W2.double()
    term = lambda C: 4 * 2.0 ** -22 + 2 * math.sqrt(3 * C) * EPS  # noqa: E731
    u, off = torch.relu(y @ w1), term(d) * (y.abs() @ w1.abs())
    s = next(s for s in range(15, -1, -1) if math.sqrt(d) * 2.0 ** s <= 2.0 ** 15)
    scale = 2.0 ** (14 - torch.floor(torch.log2(w1.abs().amax(0).clamp(min=2.0 ** -126))) + 2 * s - 27)
    off += 2.0 ** -22 * u + 2.0 ** -25 / scale
    return x.double() + u @ w2, (term(ff) * u + off) @ w2.abs() + 2 * EPS * (x.double().abs() + (u @ w2).abs())


# tiles of the first and second product, whose rows, columns and blocks of the contraction end inside one
@pytest.mark.parametrize("rows, d, ff, forms", [
    (7937, 1312, 2048, (1, 1)), (8191, 608, 3104, (1, 2)), (2305, 1280, 5120, (1, 3)), (20001, 96, 3072, (1, 3)), (6145, 1024, 1056, (2, 2)), (2177, 1280, 2048, (2, 3)),
    (3000, 4096, 1024, (3, 1)), (20001, 480, 96, (3, 1)), (4751, 1024, 4096, (3, 2)), (1751, 1312, 2080, (3, 3)), (9001, 288, 288, (3, 3)),
])
def test_tiles(m, rows, d, ff, forms):
    plan, nbytes = m.mqa_stack_feed_forward_plan(rows, d, ff)
    assert (plan >> 4 & 15, plan >> 8 & 15) == forms and nbytes > 0
    x, W1, W2 = _inputs(rows, d, ff)
    x += 3 * x[:, :1]                              # (rows with a mean)
    got = _call(m, x, W1, W2)
    for at in (slice(0, 600), slice(rows - 600, rows)):
        ref, bound = _reference(m, x[at], W1, W2)
        assert ((got[at] - ref).abs() <= bound).all(), (at, float(((got[at] - ref).abs() / bound).max()))
    assert torch.equal(got, _call(m, x, W1, W2))


@pytest.mark.parametrize("what, packed", [("zeros", True), ("columns of zeros", True), ("scaled columns", True), ("six small", True), ("seven small", False), ("one large", True),
                                          ("large", False), ("nan", False), ("inf", False), ("huge", False), ("tiny", False)])
@pytest.mark.parametrize("second", [False, True])
def test_weights_that_two_terms_hold_or_not(m, what, packed, second):
    """Where they do not, the bits of the three calls; where they do, products of the packed operands."""
    x, W1, W2 = _inputs(4100, 1024, 1024)
    W = W2 if second else W1
    W += W.sign() * 0.01
    if what == "zeros":
        W[::2] = 0
    elif what == "columns of zeros":
        W[:, 70] = W[:, 1023] = 0
    elif what == "scaled columns":
        by = torch.logspace(-12, 12, 1024, device=DEV)
        W1.mul_(by), W2.div_(by[:, None])
    elif what.endswith("small"):
        W[256:256 + (6 if what == "six small" else 7), 3] = 1e-7
    elif what == "one large":
        W[7, 3] = 100.0
        packed = second                            # (a hidden column so much larger takes W2's other rows below what its columns hold)
    elif what == "large":
        W[7, 71] = 1e7
    else:
        W[500, 71] = dict(nan=float("nan"), inf=float("-inf"), huge=2.0 ** 101, tiny=1.0)[what]
        if what == "tiny":
            W[:, 71] = 2.0 ** -115
    got, want = _call(m, x, W1, W2), _calls(m, x, W1, W2)
    assert torch.equal(got.isnan(), want.isnan())
    assert torch.equal(got.nan_to_num(), want.nan_to_num()) != packed
    if packed:
        ref, bound = _reference(m, x[:500], W1, W2)
        assert ((got[:500] - ref).abs() <= bound).all()


def test_rows_that_are_not_finite(m):
    """Their layernorm is NaN and their hidden values zeros, as by the three calls; the others are what they are without them."""
    x, W1, W2 = _inputs(4100, 1024, 1024)
    clean = _call(m, x, W1, W2)
    rows = torch.tensor([0, 255, 256, 4099], device=DEV)
    x[rows, 5] = torch.tensor([float("nan"), float("inf"), float("-inf"), 3e38], device=DEV)
    x[4099, 6] = 3e38
    got, want, others = _call(m, x, W1, W2), _calls(m, x, W1, W2), torch.ones(4100, dtype=torch.bool, device=DEV)
    others[rows] = False
    assert torch.equal(got[others], clean[others]) and torch.equal(got[rows].nan_to_num(), want[rows].nan_to_num()) and torch.equal(got[rows].isnan(), want[rows].isnan())


def _spread(decades):
    """1024 values, each beside its negative: 1 down to 10^decades."""
    return torch.logspace(0, decades, 512, device=DEV).repeat_interleave(2) * torch.tensor([1.0, -1.0], device=DEV).repeat(512)


@pytest.mark.parametrize("what, packed", [("spread", False), ("one far above", False), ("nearly equal", False), ("few", True), ("some small", True), ("hidden spread", False),
                                          ("hidden far above", False)])
def test_rows_that_two_terms_hold_or_not(m, what, packed):
    """One row that they do not hold: the 256 around it are those of the three calls, bit for bit, all others what they are without it."""
    x, W1, W2 = _inputs(4100, 1024, 1024)
    row, sign = torch.randn(1024, device=DEV), x[7].sign()
    if what.startswith("hidden"):                  # columns of one value each, or of one size
        W1 = torch.diag(torch.full((1024,), 1.0, device=DEV)) if what == "hidden spread" else W1.index_fill(1, torch.tensor([5], device=DEV), 0).add_(
            torch.nn.functional.pad(0.1 * sign[:, None], (5, 1018)))
    clean = _call(m, x, W1, W2)
    if what.endswith("spread"):
        row = _spread(-9 if what == "spread" else -4.8)      # (of the hidden spread the layernorm's values lie between 1e-4 and 10)
    elif what == "one far above":
        row[7], row[8] = 1e6, -1e6
    elif what == "nearly equal":                   # (the layernorm's eps)
        row = row * 1e-9 + 1e-9
    elif what == "few":
        row = torch.zeros_like(row)
        row[3], row[900] = 1.0, -1.0
    elif what == "some small":
        row[::100] = row.mean() + 1e-5
    else:
        row = sign
    x[2100] = row
    got, want, block = _call(m, x, W1, W2), _calls(m, x, W1, W2), slice(2048, 2304)
    others = torch.ones(4100, dtype=torch.bool, device=DEV)
    others[2100 if packed else block] = False
    assert torch.equal(got[others], clean[others])
    assert torch.equal(got[block], want[block]) != packed
    if packed:
        ref, bound = _reference(m, x[block], W1, W2)
        assert ((got[block] - ref).abs() <= bound).all()


def test_small_values_that_alone_count(m):
    """Hidden values far below the largest of their row, each the only one in its output: as good as products of float32 numbers."""
    x = _spread(-4.8).expand(4100, 1024).contiguous()
    y = m.mqa_stack_layernorm(x)
    W1, W2 = torch.eye(1024, device=DEV), torch.diag(1e3 / y[0].abs())
    got, want = _call(m, x, W1, W2), x.double() + torch.relu(y.double()) @ W2.double()
    assert ((got - want).abs() <= 2.0 ** -20 * want.abs()).all()
