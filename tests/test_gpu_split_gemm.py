"""The large float32 products made of fp16 terms (csrc/gemm.hip): edges of both tile sizes, both weight
layouts, the epilogues, and values that have no split."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.fixture(scope="module")
def m():
    import paper_1911_02150_amd as lib
    lib.load_library()
    return lib


def product(m, layout, x, W, out=None, epilogue=None):
    """x [rows,C] . W [C,N] through the entry point whose weights are laid out n-contiguous or c-contiguous."""
    rows, C = x.shape
    if layout == "n":
        return m.mqa_project_qkvo_ex(m.MQA_PROJ_LINEAR, x, W, out=out, epilogue=epilogue or m.MQA_EPI_STORE)
    kv = 128 if C % 128 == 0 else C
    P = W.t().contiguous().view(-1, C // kv, kv).permute(1, 0, 2).contiguous()      # [h, N, kv]
    return m.mqa_project_qkvo_ex(m.MQA_PROJ_O, x.view(rows, C // kv, kv), P, out=out, epilogue=epilogue or m.MQA_EPI_STORE)


def cut_off(a):
    """Per line of a [lines, C]: where the terms may begin to hold its values in fewer bits.  Few octets may hold such a value
    (none of up to 7 that are not all zeros, 2 and an eighth of more), so it is no more than the smallest
    value of the octet that is next."""
    least = torch.nn.functional.pad(a, (0, -a.shape[1] % 8)).view(a.shape[0], -1, 8)
    least = torch.where(least > 0, least, float("inf")).amin(2).sort(1).values
    octets = torch.isfinite(least).sum(1)
    allowed = torch.where(octets < 8, 0, 2 + octets // 8)
    return least.gather(1, allowed[:, None].clamp(max=least.shape[1] - 1))


def bound(x, W):
    # three products per 16 contraction indices round the running sum once each (2^-24 of it); two terms hold an operand
    # from its cut-off on to 2^-21 (2^-23 from four times the cut-off on) and the product of the second terms, at most
    # 2^-22 |a||b|, is dropped (together 20 . 2^-24); the scaling back and the last store round once more each; and the few
    # values below a line's cut-off are off by 2^-21 of it
    a, b = x.double().abs(), W.double().abs()
    ta, tb = cut_off(a), cut_off(b.t().contiguous()).t()
    small = 2.0 ** -21 * (torch.where(a < ta, ta, 0.0) @ b + a @ torch.where(b < tb, tb, 0.0))
    return (0.1875 * x.shape[1] + 24) * 2.0 ** -24 * (a @ b) + torch.nan_to_num(small, nan=0.0)


def tiles_of(m, layout, rows, C, N):
    """The edge of the tiles that `product` takes for these sizes; 0: another kernel."""
    if layout == "n":
        return m.mqa_project_plan(m.MQA_PROJ_LINEAR, rows, C, 1, N)
    kv = 128 if C % 128 == 0 else C
    return m.mqa_project_plan(m.MQA_PROJ_O, rows, N, C // kv, kv)


SIZES = [
    # tiles, rows, C, N
    (128, 128, 1024, 24584),     # one tile row, 8 columns in the last tile column
    (128, 1601, 136, 2056),      # one row, eight columns in the last tiles, tail of 8 in a stage of 32
    (256, 12000, 8, 4104),       # fewer indices than a stage of 16, a last tile of 8 columns (shorter products of the other edges
                                 # are left to the split-contraction kernel)
    (256, 4096, 1024, 4096),     # whole tiles only
    (256, 4097, 136, 4104),      # one row, eight columns in the last tiles, tail of 8 in a stage of 16
    (256, 16000, 40, 1024),      # tile rows that do not fill a band of eight
    (32, 500, 1000, 1000),       # last tiles of 20 rows and 8 columns, 104 indices in the last stage
    (32, 225, 1000, 2024),       # one row, eight columns in the last tiles
    (64, 129, 1024, 4104),       # one row, eight columns in the last tiles
    (64, 1001, 1000, 1000),      # 41 rows, 40 columns, 40 indices in the last stage
    (64, 768, 4096, 1024),       # whole tiles only
]
EDGES = [(128, 1601, 136, 2056), (256, 4097, 136, 4104), (32, 500, 1000, 1000), (64, 1001, 1000, 1000)]


def kept_in_terms(a, top, known):
    """Do the fp16 terms hold all lines of a [lines, C], scaled such that `known` (per line) comes to 2^top?"""
    x = torch.nn.functional.pad(a.abs() * (2.0 ** top / known)[:, None], (0, -a.shape[1] % 8)).view(a.shape[0], -1, 8)
    octets = (x > 0).any(2).sum(1)
    short = ((x > 0) & (x < 2.0 ** -4)).any(2).sum(1)
    return bool(((short <= torch.where(octets < 8, 0, 2 + octets // 8)) & (x.amax((1, 2)) < 65520)).all())


@pytest.mark.parametrize("spread", [0, 4])
@pytest.mark.parametrize("layout", ["n", "c"])
@pytest.mark.parametrize("tiles,rows,C,N", SIZES)
def test_split_gemm(m, layout, tiles, rows, C, N, spread):
    """spread 0: fp16 terms throughout; 4: columns of W too wide for them, float32 instructions."""
    assert tiles_of(m, layout, rows, C, N) == tiles
    g = torch.Generator(device=DEV)
    g.manual_seed(rows + C + N)
    x = torch.randn(rows, C, generator=g, device=DEV) * torch.exp(3 * torch.randn(rows, 1, generator=g, device=DEV))
    W = torch.randn(C, N, generator=g, device=DEV) * torch.exp(spread * torch.randn(C, 1, generator=g, device=DEV))
    if C >= 64:                                # (shorter ones are not tried in terms)
        for a in (x, W.t()):
            # at the smallest scale that the first 32 to 128 indices lead to / the largest that the line allows
            if spread == 0:
                assert kept_in_terms(a, 9, a[:, :128].abs().amax(1))
        assert spread == 0 or not kept_in_terms(W.t(), 15, W.abs().amax(0))
    ref, most = x.double() @ W.double(), bound(x, W)
    assert ((product(m, layout, x, W).double() - ref).abs() <= most).all()
    got = product(m, layout, x, W, epilogue=m.MQA_EPI_RELU)
    assert ((got.double() - ref.clamp(min=0)).abs() <= most).all() and float(got.min()) >= 0
    held = torch.randn(rows, N, generator=g, device=DEV)
    got = product(m, layout, x, W, out=held.clone(), epilogue=m.MQA_EPI_ADD)
    assert ((got.double() - (ref + held.double())).abs() <= most + 2.0 ** -23 * (ref.abs() + held.double().abs())).all()


@pytest.mark.parametrize("layout", ["n", "c"])
@pytest.mark.parametrize("tiles,rows,C,N", EDGES)
def test_split_gemm_scales(m, layout, tiles, rows, C, N):
    """Lines that begin with zeros or with values far from those that follow: the scales are set a second time."""
    assert tiles_of(m, layout, rows, C, N) == tiles
    g = torch.Generator(device=DEV)
    g.manual_seed(7)
    x = torch.randn(rows, C, generator=g, device=DEV)
    W = torch.randn(C, N, generator=g, device=DEV)
    x[:, :40] *= torch.where(torch.rand(rows, 1, generator=g, device=DEV) < 0.02, 0.0, 1.0)
    x[5, :40], x[6, :40], x[rows - 1, :40] = 1e-6, 1e-30, 0
    x[8] *= 1e-30
    x[17] *= 1e25
    W[:40, 3], W[:40, 300], W[:40, N - 1] = 0, 1e-20, 1e-3
    W[40:, 301] *= 1e-12
    W[:, 302] *= 1e-30
    x[20] = 0
    W[:, 40] = 0
    ref, got = x.double() @ W.double(), product(m, layout, x, W).double()
    assert ((got - ref).abs() <= bound(x, W) + 2.0 ** -149).all()


@pytest.mark.parametrize("layout", ["n", "c"])
@pytest.mark.parametrize("tiles,rows,C,N", EDGES)
def test_split_gemm_values_without_a_split(m, layout, tiles, rows, C, N):
    """Infinities, NaN, the largest floats (their first term would round to infinity) and overflowing outputs."""
    assert tiles_of(m, layout, rows, C, N) == tiles
    g = torch.Generator(device=DEV)
    g.manual_seed(5)
    x = torch.randn(rows, C, generator=g, device=DEV)
    W = torch.randn(C, N, generator=g, device=DEV) / 16
    big = float(np.finfo(np.float32).max)
    x[3, 5], x[rows - 1, 0], x[13, C - 1] = float("inf"), float("-inf"), float("inf")
    x[7], x[130, C - 1] = float("nan"), float("nan")
    x[9, :] = 0
    x[9, 11] = big                           # one product of the largest float per output of the row
    x[11, :8] = 1e30
    W[:8, 2] = 1e30                          # that output overflows
    W[:, N - 1] = 0                          # inf . 0
    ref = (x.double() @ W.double()).float()
    got = product(m, layout, x, W)
    assert torch.equal(torch.isnan(got), torch.isnan(ref))
    assert torch.equal(torch.isposinf(got), torch.isposinf(ref)) and torch.equal(torch.isneginf(got), torch.isneginf(ref))
    fine = torch.isfinite(ref)
    lim = torch.nan_to_num(bound(x, W), nan=0.0, posinf=0.0)
    assert ((got.double() - ref.double()).abs()[fine] <= lim[fine] + 2.0 ** -23 * ref.double().abs()[fine]).all()


def off(got, x, W):
    """The largest error of a row and of a column, 2-norm over 2-norm."""
    ref = x.double() @ W.double()
    e = (got.double() - ref).square()
    one = lambda dim: float((e.sum(dim) / ref.square().sum(dim).clamp(min=1e-300)).max()) ** 0.5
    return max(one(0), one(1))


@pytest.mark.parametrize("layout", ["n", "c"])
@pytest.mark.parametrize("tiles,rows,C,N", EDGES)
@pytest.mark.parametrize("ratio", [2.0 ** 6, 2.0 ** 10, 2.0 ** 14, 2.0 ** 17, 2.0 ** 20, 2.0 ** 24, 2.0 ** 40])
def test_split_gemm_wide_lines(m, layout, tiles, rows, C, N, ratio):
    """Values far above the rest of their row or column that meet zeros, or weights as far below: what float32 products
    keep of the rest is kept.  float32 instructions are off by 5.7e-7 at C = 1024, as the root of C; four times that."""
    assert tiles_of(m, layout, rows, C, N) == tiles
    g = torch.Generator(device=DEV)
    g.manual_seed(int(ratio) % 1000 + C)
    most = 2.3e-6 * max(0.5, (C / 1024) ** 0.5)
    x0 = torch.randn(rows, C, generator=g, device=DEV)
    W0 = torch.randn(C, N, generator=g, device=DEV)
    for at in ([3], [C // 2], [C - 1], list(range(C // 2, C))):
        x, W = x0.clone(), W0.clone()
        x[:, at] *= ratio                    # a channel of every row
        W[at] = 0
        assert off(product(m, layout, x, W), x, W) < most, ("rows", at[0])
        x, W = x0.clone(), W0.clone()
        W[at] *= ratio                       # of every column
        x[:, at] = 0
        assert off(product(m, layout, x, W), x, W) < most, ("columns", at[0])
        x, W = x0.clone(), W0.clone()
        x[5, at] *= ratio                    # of one row, one column
        W[at, 7] = 0
        W[C // 3, 9] *= ratio
        x[11, C // 3] = 0
        got, ref = product(m, layout, x, W).double(), x.double() @ W.double()
        for r, n in ((5, 7), (11, 9)):
            assert abs(float(got[r, n] - ref[r, n])) < 4 * most * float((x[r].double() * W[:, n].double()).norm())
    x, W = x0.clone(), W0.clone()
    x[:, C // 2] *= ratio
    W[C // 2] /= ratio
    assert off(product(m, layout, x, W), x, W) < most


@pytest.mark.parametrize("layout", ["n", "c"])
@pytest.mark.parametrize("tiles,rows,C,N", EDGES)
def test_split_gemm_sparse_lines(m, layout, tiles, rows, C, N):
    """Rows of mostly zeros: few values, some of them far below the other rows', and rows whose only values come late."""
    assert tiles_of(m, layout, rows, C, N) == tiles
    g = torch.Generator(device=DEV)
    g.manual_seed(3)
    x = torch.randn(rows, C, generator=g, device=DEV).clamp(min=0)
    W = torch.randn(C, N, generator=g, device=DEV)
    x[::3] *= (torch.rand(rows, C, generator=g, device=DEV) < 0.05)[::3]
    for r, (c, v) in enumerate([(2, 1e-9), (C - 2, 1e-9), (C // 2, 1e-20), (40, 1e-6), (C - 9, 1e12)]):
        x[7 + r] = 0
        x[7 + r, c] = v
    x[rows - 1, :C - 8] = 0
    x[rows - 1, C - 8:] *= 1e-8
    most = 2.3e-6 * max(0.5, (C / 1024) ** 0.5)
    assert off(product(m, layout, x, W), x, W) < most


@pytest.mark.parametrize("kv", [8, 24, 72])
@pytest.mark.parametrize("tiles,rows,width", [(32, 512, 1024), (64, 1001, 1000), (128, 4096, 1024), (256, 4096, 4096)])
def test_split_gemm_small_heads(m, kv, tiles, rows, width):
    """Column tiles (q) and stages of the contraction (output) that reach over several heads, in every tile size."""
    g = torch.Generator(device=DEV)
    g.manual_seed(kv + rows)
    h = width // kv
    assert m.mqa_project_plan(m.MQA_PROJ_Q, rows, width, h, kv) == m.mqa_project_plan(m.MQA_PROJ_O, rows, width, h, kv) == tiles
    x = torch.randn(rows, width, generator=g, device=DEV)
    P = torch.randn(h, width, kv, generator=g, device=DEV)
    W = P.permute(1, 0, 2).reshape(width, h * kv)
    got = m.mqa_project_qkvo(m.MQA_PROJ_Q, x, P).view(rows, h * kv)
    assert ((got.double() - x.double() @ W.double()).abs() <= bound(x, W)).all()
    o = torch.randn(rows, h, kv, generator=g, device=DEV)
    W = P.permute(0, 2, 1).reshape(h * kv, width)
    got = m.mqa_project_qkvo(m.MQA_PROJ_O, o, P)
    assert ((got.double() - o.view(rows, -1).double() @ W.double()).abs() <= bound(o.view(rows, -1), W)).all()
