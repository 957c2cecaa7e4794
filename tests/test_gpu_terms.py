"""Decode-sized products from three bfloat16 terms (csrc/project_terms.hip), alone and in parts with the residual and the layernorm:
every tile and split, both weight layouts, last tiles and steps that are not full, values without terms and at the ends of the range, and
the error against 64 bits."""
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


def weights(layout, W, kv):
    """W [C,N] as the library's operand: (mode, P, shape of a row of the input)."""
    import paper_1911_02150_amd as m
    C, N = W.shape
    if layout == "n":
        return m.MQA_PROJ_LINEAR, W, (C,)
    return m.MQA_PROJ_O, W.t().contiguous().view(N, C // kv, kv).permute(1, 0, 2).contiguous(), (C // kv, kv)


def bound(x, W):
    # the tiles of 128 x 128 round the running sum three times for every 16 indices (2^-24 of it), the terms and the float32 instructions
    # less often; the sums of up to 8 waves and 16 parts and the small products' another 32 times; the products of terms that are
    # left out are below 2^-24 |a||b|.  (What the terms hold shows in test_relative_error.)
    return (0.1875 * x.shape[1] + 32) * 2.0 ** -24 * (x.double().abs() @ W.double().abs())


# rows, C, N, kv (c contiguous): rows and columns past whole tiles, a last step of 8, 16 and 24 indices, heads inside a step
ALONE = [(65, 2056, 1032, 8), (190, 1024, 1000, 128), (65, 2048, 2048, 512), (250, 512, 648, 64), (129, 4072, 1024, 8)]
PARTS = [(1, 4096, 1024, 128), (16, 264, 40, 24), (17, 1048, 1032, 8), (31, 272, 4096, 16), (64, 4096, 1024, 128), (128, 2072, 512, 56),
         (129, 1024, 1024, 128), (190, 2048, 1288, 64), (224, 520, 136, 40), (3, 256, 8, 8),
         (385, 4072, 1024, 8), (513, 5120, 1288, 40), (1000, 4096, 1024, 128), (1300, 4104, 1016, 24)]      # (parts in tiles of 128 x 128)


@pytest.mark.parametrize("layout,rows,C,N,kv", [(layout, *s) for layout in "nc" for s in ALONE] + [("n", 120, 1048, 4088, 8)])
def test_product(m, layout, rows, C, N, kv):
    g = torch.Generator(device=DEV)
    g.manual_seed(rows + C + N)
    x = torch.randn(rows, C, generator=g, device=DEV) * torch.exp(5 * torch.randn(rows, 1, generator=g, device=DEV))
    x[1], x[2, ::3] = 0, 1e-30
    W = torch.randn(C, N, generator=g, device=DEV) * torch.exp(4 * torch.randn(C, 1, generator=g, device=DEV))
    mode, P, row = weights(layout, W, kv)
    sizes = (1, N) if layout == "n" else (C // kv, kv)
    assert m.mqa_project_plan(mode, rows, C if layout == "n" else N, *sizes) == 1
    ref, most = x.double() @ W.double(), bound(x, W)
    for epilogue, want, slack in ((m.MQA_EPI_STORE, ref, 0), (m.MQA_EPI_RELU, ref.clamp(min=0), 0), (m.MQA_EPI_ADD, ref + 3, 2.0 ** -23 * (ref.abs() + 3))):
        out = torch.full((rows, N), 3.0, device=DEV)
        got = m.mqa_project_qkvo_ex(mode, x.view(rows, *row), P, out=out, epilogue=epilogue)
        assert ((got.double() - want).abs() <= most + slack).all()


@pytest.mark.parametrize("layout", ["n", "c"])
def test_values_without_terms(m, layout):
    """Infinities, NaN, the largest floats (their first term would be an infinity) and overflowing sums."""
    rows, C, N = 65, 2048, 2048
    g = torch.Generator(device=DEV)
    g.manual_seed(5)
    x = torch.randn(rows, C, generator=g, device=DEV)
    W = torch.randn(C, N, generator=g, device=DEV) / 16
    big = float(np.finfo(np.float32).max)
    x[3, 5], x[rows - 1, 0], x[13, C - 1] = float("inf"), float("-inf"), float("inf")
    x[7], x[60, C - 1] = float("nan"), float("nan")
    x[9] = 0
    x[9, 11] = big
    x[11, :8] = 1e30
    W[:8, 2] = 1e30
    W[:, N - 1] = 0
    mode, P, row = weights(layout, W, 128)
    ref = (x.double() @ W.double()).float()
    got = m.mqa_project_qkvo_ex(mode, x.view(rows, *row), P)
    assert torch.equal(torch.isnan(got), torch.isnan(ref))
    assert torch.equal(torch.isposinf(got), torch.isposinf(ref)) and torch.equal(torch.isneginf(got), torch.isneginf(ref))
    fine = torch.isfinite(ref)
    lim = torch.nan_to_num(bound(x, W), nan=0.0, posinf=0.0)
    assert ((got.double() - ref.double()).abs()[fine] <= lim[fine] + 2.0 ** -23 * ref.double().abs()[fine]).all()


# one size of every tile, alone and in parts
FORMS = [(65, 2056, 1032, 8, False), (65, 2048, 2048, 512, False), (129, 4072, 1024, 8, False), (1, 4096, 1024, 128, True), (16, 264, 40, 24, True),
         (64, 4096, 1024, 128, True), (129, 1024, 1024, 128, True), (190, 2048, 1288, 64, True), (385, 4072, 1024, 8, True)]


def results(m, layout, x, W, kv, parts):
    """(the sums, what they should be) for every epilogue, or of the call with the layernorm."""
    rows, C, N = x.shape[0], x.shape[1], W.shape[1]
    mode, P, row = weights(layout, W, kv)
    sizes = (C, 1, N) if layout == "n" else (N, C // kv, kv)
    ref = x.double() @ W.double()
    acc = torch.zeros(rows, N, device=DEV)
    if parts:
        assert m.mqa_project_add_layernorm_workspace_bytes(mode, rows, *sizes) > 0
        m.mqa_project_add_layernorm(mode, x.view(rows, *row), P, acc)
        return [(acc, ref)]
    assert m.mqa_project_plan(mode, rows, *sizes) == 1
    product = lambda e, out=None: m.mqa_project_qkvo_ex(mode, x.view(rows, *row), P, out=out, epilogue=e)  # noqa: E731
    return [(product(m.MQA_EPI_STORE), ref), (product(m.MQA_EPI_RELU), ref.clamp(min=0)), (product(m.MQA_EPI_ADD, acc), ref)]


def agree(got, want, most):
    """Infinities where the float32 result has them, no NaN, and the rest within `most` and a rounding of the result."""
    ref = want.float()
    assert not torch.isnan(got).any()
    assert torch.equal(torch.isposinf(got), torch.isposinf(ref)) and torch.equal(torch.isneginf(got), torch.isneginf(ref))
    fine = torch.isfinite(ref)
    assert ((got.double() - want).abs()[fine] <= (most + 2.0 ** -23 * want.abs())[fine]).all()


@pytest.mark.parametrize("values", ["normal", "relu"])
@pytest.mark.parametrize("layout", ["n", "c"])
@pytest.mark.parametrize("rows,C,N,kv,parts", FORMS + [(65, 512, 1032, 8, True), (128, 1280, 1024, 128, True), (300, 1280, 1024, 128, True)])
def test_relative_error(m, layout, rows, C, N, kv, parts, values):
    """What the terms hold shows in the root mean square: a product of terms left out is 2^-18 of the result (1.5e-6 at the
    least).  The float32 instructions come to 0.8 to 4.1e-7 here (normal deviates) and 0.6 to 2.9e-7 (relu), the tiles of 128 x 128 to
    2.1e-7 of their two terms, the three terms to 0.5 to 1.4e-7."""
    g = torch.Generator(device=DEV)
    g.manual_seed(rows + C)
    x, W = torch.randn(rows, C, generator=g, device=DEV), torch.randn(C, N, generator=g, device=DEV) * C ** -0.5
    if values == "relu":
        x.clamp_(min=0)
    for got, want in results(m, layout, x, W, kv, parts):
        assert float((got.double() - want).norm() / want.norm()) < (2.4e-7 if rows > 256 else 1.5e-7 if values == "normal" else 1.2e-7)


@pytest.mark.parametrize("layout", ["n", "c"])
@pytest.mark.parametrize("rows,C,N,kv,parts", FORMS)
def test_products_past_the_largest_float(m, layout, rows, C, N, kv, parts):
    """Finite operands whose products are past the largest float, or just below it (where the product of the first terms is not)."""
    g = torch.Generator(device=DEV)
    g.manual_seed(rows + N)
    x, W = torch.randn(rows, C, generator=g, device=DEV), torch.randn(C, N, generator=g, device=DEV) / 16
    at = [C // 5, C // 2, C - 3]               # in steps of their own, and rows of their own where there are as many
    near = 1.997 * 2.0 ** 63
    for i, r in zip(range(3), (rows - 1, rows // 2, 0)):
        if i and rows < 3:
            break
        x[r, at[i]] = (1e30, -1e30, near)[i]
        W[at[i], 3 * i] = (1e30, 1e30, near)[i]
    if rows >= 3:
        x[0, :at[2]], x[0, at[2] + 1:] = 0, 0
    most = torch.nan_to_num(bound(x, W), posinf=0.0)
    for got, want in results(m, layout, x, W, kv, parts):
        assert torch.isposinf(got[rows - 1, 0])
        agree(got, want, most)


@pytest.mark.parametrize("layout", ["n", "c"])
@pytest.mark.parametrize("rows,C,N,kv,parts", FORMS)
def test_nan_beside_overflow(m, layout, rows, C, N, kv, parts):
    """Rows with a NaN among rows whose products overflow, in the same step and tile: NaN is NaN, the others keep their infinities."""
    g = torch.Generator(device=DEV)
    g.manual_seed(rows + N)
    x, W = torch.randn(rows, C, generator=g, device=DEV), torch.randn(C, N, generator=g, device=DEV) / 16
    x[::3, C // 3] = float("nan")
    x[1::3, C // 3], W[C // 3, N - 2] = 1e30, 1e30
    W[C // 7, N // 2] = float("nan")
    for k, (got, want) in enumerate(results(m, layout, x, W, kv, parts)):
        ref = want.float()
        if k == 1:                             # relu: max(NaN, 0) is 0
            ref = torch.nan_to_num(ref, nan=0.0, posinf=float("inf"))
        assert torch.equal(torch.isnan(got), torch.isnan(ref)) and torch.equal(torch.isposinf(got), torch.isposinf(ref))
        fine = torch.isfinite(ref) & torch.isfinite(want)
        lim = torch.nan_to_num(bound(x, W), nan=0.0, posinf=0.0) + 2.0 ** -23 * torch.nan_to_num(want, posinf=0.0).abs()
        assert ((got.double() - want).abs()[fine] <= lim[fine]).all()


@pytest.mark.parametrize("small", ["rows", "columns"])
@pytest.mark.parametrize("layout", ["n", "c"])
@pytest.mark.parametrize("rows,C,N,kv,parts", FORMS)
def test_operands_near_the_smallest_float(m, layout, rows, C, N, kv, parts, small):
    """Rows (columns) down to subnormal values against columns (rows) that bring the sums back into range, among zeros."""
    g = torch.Generator(device=DEV)
    g.manual_seed(rows + N)
    x, W = torch.randn(rows, C, generator=g, device=DEV), torch.randn(C, N, generator=g, device=DEV)
    x[:, 1::7], W[2::5] = 0, 0
    lines, others = (x, W.t()) if small == "rows" else (W.t(), x)
    for i, e in {i * lines.shape[0] // 5: e for i, e in enumerate((-111, -116, -124, -132, -146))}.items():
        lines[i] *= 2.0 ** e
    others[others.shape[0] // 2:] *= 2.0 ** 70
    # the products and their sums are rounded to whole subnormals besides
    for got, want in results(m, layout, x, W, kv, parts):
        agree(got, want, bound(x, W) + C * 2.0 ** -149)


@pytest.mark.parametrize("with_workspace", [True, False])
@pytest.mark.parametrize("layout", ["n", "c"])
@pytest.mark.parametrize("rows,C,N,kv", PARTS)
def test_add_layernorm(m, layout, rows, C, N, kv, with_workspace):
    """In parts (given the workspace) and as the two calls it stands for; nothing behind x, y and the workspace is written."""
    g = torch.Generator(device=DEV)
    g.manual_seed(rows + C + N)
    x = torch.randn(rows, C, generator=g, device=DEV)
    W = torch.randn(C, N, generator=g, device=DEV) * C ** -0.5
    mode, P, row = weights(layout, W, kv)
    nbytes = m.mqa_project_add_layernorm_workspace_bytes(mode, rows, *((C, 1, N) if layout == "n" else (N, C // kv, kv)))
    assert nbytes > 0 and nbytes % (4 * rows * N) == 0
    buffers = torch.full((2, rows + 1, N), 7.0, device=DEV)
    acc, y = buffers[0, :rows], buffers[1, :rows]
    acc.copy_(torch.randn(rows, N, generator=g, device=DEV))
    was = acc.double()
    ws = torch.full((nbytes + 64,), 255, dtype=torch.uint8, device=DEV)      # (NaN, should a part be read that was not written)
    assert m.mqa_project_add_layernorm(mode, x.view(rows, *row), P, acc, out=y, workspace=ws[:nbytes if with_workspace else nbytes - 16]) is y
    want = was + x.double() @ W.double()
    off = bound(x, W) + 2.0 ** -23 * (want.abs() + was.abs())
    assert ((acc.double() - want).abs() <= off).all()
    c = want - want.mean(1, keepdim=True)
    std = (c.square().mean(1, keepdim=True) + 1e-6).sqrt()
    # an error e of the row is (e + mean |e| + |y| rms e) / std of the result; the sums and the root are off by some 2^-20 of it
    e = off / std
    norm = c / std
    assert ((y.double() - norm).abs() <= e + e.mean(1, keepdim=True) + norm.abs() * e.square().mean(1, keepdim=True).sqrt() + 2.0 ** -20 * (1 + norm.abs())).all()
    assert (buffers[:, rows] == 7).all() and (ws[nbytes:] == 255).all()
    if with_workspace:
        again, y2 = was.float(), torch.empty_like(y)
        m.mqa_project_add_layernorm(mode, x.view(rows, *row), P, again, out=y2)
        assert torch.equal(again, acc) and torch.equal(y2, y)                # (the same every time)


def test_add_layernorm_refuses(m):
    x, W, acc = torch.zeros(4, 64, device=DEV), torch.zeros(64, 32, device=DEV), torch.zeros(4, 32, device=DEV)
    with pytest.raises(ValueError):
        m.mqa_project_add_layernorm(m.MQA_PROJ_Q, x, W.view(1, 64, 32), acc)
    with pytest.raises(ValueError):
        m.mqa_project_add_layernorm(m.MQA_PROJ_LINEAR, x, W, acc[:3])
    with pytest.raises(m.MqaError, match="status 2"):
        m.mqa_project_add_layernorm(m.MQA_PROJ_LINEAR, torch.zeros(4, 60, device=DEV), torch.zeros(60, 32, device=DEV), acc)
