"""New K / V rows of many positions (csrc/project_kv_rows.hip with a workspace, csrc/project_kv.hip without, and the float64 kernel
they stand in for): the cache holds the correctly rounded product, bit for bit, whatever the values."""
import pytest
import torch

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.fixture(scope="module")
def m():
    import paper_1911_02150_amd as lib
    lib.load_library()
    return lib


def rounded(X, W):
    """float64 products and sums, rounded to float32 and then to bfloat16."""
    return (X.double() @ W.double()).float().to(torch.bfloat16)


def same(got, want):
    nan = torch.isnan(want)
    return torch.equal(torch.isnan(got), nan) and torch.equal(got[~nan], want[~nan])


def inputs(b, n, d, heads, k, v, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    one = (heads,) if heads else ()
    x = torch.randn(b, n, d, generator=g, device=DEV)
    return x, torch.randn(*one, d, k, generator=g, device=DEV) * d ** -0.5, torch.randn(*one, d, v, generator=g, device=DEV) * d ** -0.5


def expected(x, P, heads):
    b, n, d = x.shape
    X = x.reshape(b * n, d)
    if not heads:
        return rounded(X, P).view(b, n, -1)
    return torch.stack([rounded(X, P[j]).view(b, n, -1) for j in range(heads)], 1)


def caches(b, heads, cap, k, v, dtype=torch.bfloat16):
    one = (heads,) if heads else ()
    return torch.full((b, *one, cap, k), 7.0, dtype=dtype, device=DEV), torch.full((b, *one, cap, v), 7.0, dtype=dtype, device=DEV)


ROUTES = ["with", "without"]                   # a workspace: kv_rows_kernel and project_kv_exact_kernel where integers pay


def scratch(m, route, b, n, d, heads, k, v, dtype=torch.bfloat16, integers=True):
    """The workspace to hand over: the one the sizes ask for, or one that is too small for any."""
    nbytes = m.mqa_project_kv_workspace_bytes(b, n, d, heads or 1, k, v, m.MQA_BF16 if dtype == torch.bfloat16 else m.MQA_F32)
    assert (nbytes > 0) == (integers and dtype == torch.bfloat16)
    return torch.full((nbytes if route == "with" and nbytes else 16,), 255, dtype=torch.uint8, device=DEV)


# rows and columns past whole tiles of 128, contraction tails of 8 and of 24 in a stage of 32, heads inside a column tile;
# the last two are too small for the integer kernel
SHAPES = [(64, 300, 1000, 0, 128, 128), (46, 811, 72, 0, 128, 64), (40, 500, 88, 5, 48, 80), (70, 257, 520, 2, 256, 16),
          (3, 40, 512, 0, 128, 128), (2, 9, 72, 3, 16, 32)]


def test_shapes_take_the_kernel_they_are_for(m):
    taken = [m.mqa_project_kv_plan(b * n, d, 0, heads or 1, k, v, m.MQA_BF16) for b, n, d, heads, k, v in SHAPES]
    assert taken == [1, 1, 1, 1, 0, 0]
    asked = [m.mqa_project_kv_workspace_bytes(b, n, d, heads or 1, k, v, m.MQA_BF16) > 0 for b, n, d, heads, k, v in SHAPES]
    assert asked == [True] * 4 + [False] * 2
    assert m.mqa_project_kv_plan(64 * 300, 1000, 0, 1, 128, 128, m.MQA_F32) == 0


@pytest.mark.parametrize("route", ROUTES)
@pytest.mark.parametrize("b,n,d,heads,k,v", SHAPES)
def test_memory_rows(m, b, n, d, heads, k, v, route):
    x, P_k, P_v = inputs(b, n, d, heads, k, v, n)
    K, V = caches(b, heads, n + 3, k, v)
    lens = torch.zeros(b, dtype=torch.int32, device=DEV)
    m.mqa_project_memory_kv(x, P_k, P_v, K, V, lens, workspace=scratch(m, route, b, n, d, heads, k, v, integers=b > 3))
    assert torch.equal(K[..., :n, :], expected(x, P_k, heads)) and torch.equal(V[..., :n, :], expected(x, P_v, heads))
    assert (K[..., n:, :] == 7).all() and (V[..., n:, :] == 7).all() and (lens == n).all()


@pytest.mark.parametrize("route", ROUTES)
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("b,n,d,heads,k,v", SHAPES)
def test_append_rows(m, b, n, d, heads, k, v, dtype, route):
    """Behind what is there; a sequence without room (or with a negative length) stays as it is."""
    x, P_k, P_v = inputs(b, n, d, heads, k, v, n + 1)
    cap = n + 10
    K, V = caches(b, heads, cap, k, v, dtype)
    lens = torch.arange(b, dtype=torch.int32, device=DEV) % 11
    lens[b - 1] = 11
    lens[0] = -2
    after = torch.zeros_like(lens)
    m.mqa_project_append_kv_rows(x, P_k, P_v, K, V, lens, after, workspace=scratch(m, route, b, n, d, heads, k, v, dtype, b > 3))
    wk, wv = caches(b, heads, cap, k, v, dtype)
    for i, L in enumerate(lens.tolist()):
        if 0 <= L <= 10:
            for w, P in ((wk, P_k), (wv, P_v)):
                if dtype == torch.bfloat16:
                    w[i, ..., L:L + n, :] = expected(x[i:i + 1], P, heads)[0]
                else:
                    w[i, ..., L:L + n, :] = (x[i].double() @ P.double()).float()
    if dtype == torch.bfloat16:
        assert torch.equal(K, wk) and torch.equal(V, wv)
    else:      # (the order of the float64 sum may show in the last place)
        assert torch.allclose(K, wk, rtol=2.0 ** -23, atol=1e-12) and torch.allclose(V, wv, rtol=2.0 ** -23, atol=1e-12)
    assert after.tolist() == [L + n if 0 <= L <= 10 else L for L in lens.tolist()]


@pytest.mark.parametrize("route", ROUTES)
@pytest.mark.parametrize("ratio", [2.0 ** 6, 2.0 ** 8, 2.0 ** 9, 2.0 ** 12, 2.0 ** 40])
@pytest.mark.parametrize("b,n,d,heads,k,v", [s for s in SHAPES if s[0] > 3])
def test_one_large_channel(m, b, n, d, heads, k, v, ratio, route):
    """One channel far above the others, its weights as far below: the bounds leave from a few elements of a tile to all of
    it open."""
    x, P_k, P_v = inputs(b, n, d, heads, k, v, n + 2)
    assert m.mqa_project_kv_plan(b * n, d, 0, heads or 1, k, v, m.MQA_BF16) == 1
    x[..., d // 3] *= ratio
    P_k[..., d // 3, :] /= ratio
    P_v[..., d // 3, :] /= ratio
    K, V = caches(b, heads, n + 3, k, v)
    lens = torch.zeros(b, dtype=torch.int32, device=DEV)
    m.mqa_project_memory_kv(x, P_k, P_v, K, V, lens, workspace=scratch(m, route, b, n, d, heads, k, v))
    assert torch.equal(K[..., :n, :], expected(x, P_k, heads)) and torch.equal(V[..., :n, :], expected(x, P_v, heads))
    assert (K[..., n:, :] == 7).all() and (V[..., n:, :] == 7).all()


@pytest.mark.parametrize("append", [False, True])
@pytest.mark.parametrize("route", ROUTES)
def test_rows_of_any_values(m, route, append):
    """Zeros, ties, wide ranges inside a row and a column, sums that cancel, subnormals, infinities and NaN."""
    b, n, d = 64, 300, 200
    assert m.mqa_project_kv_plan(b * n, d, 0, 1, 128, 128, m.MQA_BF16) == 1
    x, P_k, P_v = inputs(b, n, d, 0, 128, 128, 9)
    x[0, :40] = 0
    x[1, 3], x[1, 4] = x[1, 3].abs() * 1e30, x[1, 4] * 1e-30
    x[2] *= torch.exp(4 * torch.randn(n, d, device=DEV))
    x[3, :, 100:] = -x[3, :, :100]
    x[4, 5] = 1e-42
    x[5, 7, 9], x[5, 8, 9], x[6, 0, 0] = float("inf"), float("nan"), float("-inf")
    x[7] = torch.randint(-4, 5, (n, d), device=DEV).float()
    P_k[100:, 16:64] = P_k[:100, 16:64]       # x[3]: sums that cancel
    P_k[:, 3] = 0
    P_k[:, 5] = torch.randint(-2, 3, (d,), device=DEV).float() * 2.0 ** -9      # with x[7]: sums that are exact ties
    P_k[:, 6] *= torch.exp(4 * torch.randn(d, device=DEV))
    P_k[17, 8], P_k[18, 9] = float("inf"), float("nan")
    P_k[:, 10] *= 1e-35
    K, V = caches(b, 0, n, 128, 128)
    lens = torch.zeros(b, dtype=torch.int32, device=DEV)
    ws = scratch(m, route, b, n, d, 0, 128, 128)
    if append:
        m.mqa_project_append_kv_rows(x, P_k, P_v, K, V, torch.zeros_like(lens), lens, workspace=ws)
    else:
        m.mqa_project_memory_kv(x, P_k, P_v, K, V, lens, workspace=ws)
    want = expected(x, P_k, 0)
    # sums that cancel to nothing are what the order of the 64-bit sum leaves: 200 roundings of sums below 100
    assert float(K[3, :, 16:64].abs().max()) < 200 * 100 * 2.0 ** -53
    K[3, :, 16:64] = want[3, :, 16:64]
    assert same(K, want) and same(V, expected(x, P_v, 0))


@pytest.mark.parametrize("with_workspace", [True, False])
def test_lines_with_a_nan(m, with_workspace):
    """A NaN (of either sign) makes its row or column the quiet NaN that the integer kernels store, without summing: as many as open a
    whole tile to the float64 sums otherwise.  So does an infinity against a row of zeros."""
    from paper_1911_02150_amd import binding
    lib = binding.load_library()
    b, n, d = 64, 300, 200
    x, P_k, P_v = inputs(b, n, d, 0, 128, 128, 11)
    nan = torch.tensor([0x7fc00000, -0x400000], dtype=torch.int32, device=DEV).view(torch.float32)
    x[::2, ::20, 7] = nan[0]
    x[1::2, ::20, d - 1] = nan[1]
    P_k[5, 3], P_v[d - 1, 127] = nan[1], nan[0]
    P_v[0, 5], x[4, 10] = float("inf"), 0
    K, V = caches(b, 0, n, 128, 128)
    lens = torch.zeros(b, dtype=torch.int32, device=DEV)
    nbytes = lib.mqa_project_kv_workspace_bytes(b, n, d, 1, 128, 128, m.MQA_BF16) if with_workspace else 0
    assert m.mqa_project_kv_plan(b * n, d, 0, 1, 128, 128, m.MQA_BF16) == 1 and (nbytes > 0) == with_workspace
    ws = torch.empty(max(16, nbytes), dtype=torch.uint8, device=DEV)
    assert lib.mqa_project_memory_kv_ws(x.data_ptr(), P_k.data_ptr(), P_v.data_ptr(), K.data_ptr(), V.data_ptr(), None, lens.data_ptr(), b, n, d, 1, n,
                                        128, 128, m.MQA_BF16, ws.data_ptr(), nbytes, torch.cuda.current_stream().cuda_stream) == 0
    for got, P in ((K, P_k), (V, P_v)):
        want = expected(x, P, 0)
        assert same(got, want) and (got.view(torch.int16)[torch.isnan(want)] == 0x7fc0).all()


@pytest.mark.parametrize("route,d", [("without", 8), ("without", 64), ("with", 64)])       # (zeros behind the first eight)
@pytest.mark.parametrize("sign", [1, -1])
def test_sums_around_a_power_of_two(m, sign, route, d):
    """Sums that end just above and just below 2^42, whose error bound (what the fixed point drops of the values beside one
    of 1.25 . 2^30) reaches the nearest tie: below the power of two the ties lie half as far apart."""
    b, n, big = 64, 512, 1.25 * 2.0 ** 30
    assert m.mqa_project_kv_plan(b * n, d, 0, 1, 128, 128, m.MQA_BF16) == 1
    x = torch.tensor([big] * 4 + [-0.99] * 3 + [0.0] * (d - 7), device=DEV).repeat(b, n, 1)
    x[..., 7] = torch.linspace(3262, 3302, b * n, device=DEV).view(b, n)
    x[::2, :, 7] = x[::2, :, 7].floor()
    w = sign * torch.tensor([-0.99] * 4 + [big] * 4 + [0.0] * (d - 8), device=DEV)
    P = w[:, None] * 2.0 ** torch.arange(-64, 64, device=DEV)
    K, V = caches(b, 0, n, 128, 128)
    lens = torch.zeros(b, dtype=torch.int32, device=DEV)
    m.mqa_project_memory_kv(x, P, P * 2, K, V, lens, workspace=scratch(m, route, b, n, d, 0, 128, 128, integers=d >= 64))
    want = expected(x, P, 0)
    assert (want[..., 64].abs() < 2.0 ** 42).any() and (want[..., 64].abs() > 2.0 ** 42).any()
    assert torch.equal(K, want) and torch.equal(V, expected(x, P * 2, 0))


FULL = [2 ** 31 - 1, 2 ** 31 - 2, 2 ** 31 - 5, 2 ** 30, -1, -2 ** 31]      # lengths no cache has room behind


@pytest.mark.parametrize("route", ROUTES)
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("b,n,d,heads,k,v", [(64, 300, 1000, 0, 128, 128), (6, 9, 72, 3, 16, 32)])
def test_append_to_any_length(m, b, n, d, heads, k, v, dtype, route):
    """Lengths up to the largest integer: the cache and the length stay as they are."""
    x, P_k, P_v = inputs(b, n, d, heads, k, v, 3)
    lens = torch.zeros(b, dtype=torch.int32, device=DEV)
    lens[:6] = torch.tensor(FULL, dtype=torch.int32, device=DEV)
    K, V = caches(b, heads, n, k, v, dtype)
    after = torch.zeros_like(lens)
    m.mqa_project_append_kv_rows(x, P_k, P_v, K, V, lens, after, workspace=scratch(m, route, b, n, d, heads, k, v, dtype, b > 6))
    assert after.tolist() == FULL + [n] * (b - 6) and (K[:6] == 7).all() and (V[:6] == 7).all()
    K2, V2 = caches(b, heads, n, k, v, dtype)
    one = (b, n, heads) if heads else (b, n)
    held = lens.clone()
    m.mqa_append_kv_rows(K2, V2, torch.ones(*one, k, device=DEV), torch.ones(*one, v, device=DEV), held)
    assert held.tolist() == FULL + [n] * (b - 6) and (K2[:6] == 7).all() and (V2[:6] == 7).all()


@pytest.mark.parametrize("b,d,h,k,v,integer", [(1300, 1024, 8, 128, 128, 1), (40, 72, 3, 16, 32, 0)])
def test_decode_step_to_any_length(m, b, d, h, k, v, integer):
    """The fused projection of one position per sequence, multi-head: enough rows and columns for the integer kernel, and few."""
    cap = 3
    assert m.mqa_project_kv_plan(b, d, h, h, k, v, m.MQA_BF16) == integer
    x, P_k, P_v = inputs(b, 1, d, h, k, v, 4)
    x = x.view(b, d)
    P_q = torch.randn(h, d, k, device=DEV) * d ** -0.5
    lens = torch.arange(b, dtype=torch.int32, device=DEV) % (cap + 1)
    lens[:6] = torch.tensor(FULL, dtype=torch.int32, device=DEV)
    K, V = caches(b, h, cap, k, v)
    after = torch.zeros_like(lens)
    q = m.mqa_project_append_qkv(x, P_q, P_k, P_v, K, V, lens, after)
    wk, wv = caches(b, h, cap, k, v)
    new_k, new_v = expected(x.view(b, 1, d), P_k, h)[:, :, 0], expected(x.view(b, 1, d), P_v, h)[:, :, 0]
    for i, L in enumerate(lens.tolist()):
        if 0 <= L < cap:
            wk[i, :, L], wv[i, :, L] = new_k[i], new_v[i]
    assert torch.equal(K, wk) and torch.equal(V, wv)
    assert after.tolist() == [L + 1 if 0 <= L < cap else L for L in lens.tolist()]
    want = torch.stack([x.double() @ P_q[j].double() for j in range(h)], 1)
    assert float((q.double() - want).abs().max()) < 1e-5


@pytest.mark.parametrize("share", [0, 0.5, 1])
@pytest.mark.parametrize("b,n,d,heads,k,v", [s for s in SHAPES if s[0] > 3] + [(33, 129, 1032, 0, 32, 16), (9, 1000, 64, 0, 128, 128)])
def test_rows_with_and_without_a_workspace(m, b, n, d, heads, k, v, share):
    """The call without a workspace (or with less than it asks for) and the one with: the same rows and lengths, nothing beside
    them.  One row and one column past tiles of 64 x 128, a contraction that ends in the first octet of a stage of 64."""
    from paper_1911_02150_amd import binding
    lib = binding.load_library()
    x, P_k, P_v = inputs(b, n, d, heads, k, v, n + 5)
    K, V = caches(b, heads, n + 3, k, v)
    lens, valid = torch.zeros(b, dtype=torch.int32, device=DEV), torch.arange(b, dtype=torch.int32, device=DEV)
    nbytes = int(share * lib.mqa_project_kv_workspace_bytes(b, n, d, heads or 1, k, v, m.MQA_BF16))
    assert share == 0 or nbytes > 0 or (b, n) == (33, 129) or (b, n) == (9, 1000)
    ws = torch.full((max(16, nbytes),), 255, dtype=torch.uint8, device=DEV)
    rc = lib.mqa_project_memory_kv_ws(x.data_ptr(), P_k.data_ptr(), P_v.data_ptr(), K.data_ptr(), V.data_ptr(), valid.data_ptr(),
                                      lens.data_ptr(), b, n, d, heads or 1, n + 3, k, v, m.MQA_BF16, ws.data_ptr() if share else None,
                                      nbytes, torch.cuda.current_stream().cuda_stream)
    assert rc == 0
    assert torch.equal(K[..., :n, :], expected(x, P_k, heads)) and torch.equal(V[..., :n, :], expected(x, P_v, heads))
    assert (K[..., n:, :] == 7).all() and (V[..., n:, :] == 7).all() and torch.equal(lens, valid.clamp(max=n))


@pytest.mark.parametrize("own_workspace", [True, False])
@pytest.mark.parametrize("append", [True, False])
def test_captured_rows(m, append, own_workspace):
    """The call in a graph that torch captures, with the program's workspace and without: every replay gives the eager rows of the inputs
    it finds, with other work on the same sizes of memory between the replays."""
    b, n, d = 64, 300, 520
    x, P_k, P_v = inputs(b, n, d, 0, 128, 128, 21)
    nbytes = m.mqa_project_kv_workspace_bytes(b, n, d, 1, 128, 128, m.MQA_BF16)
    assert nbytes > 0
    K, V = caches(b, 0, n, 128, 128)
    lens, after = torch.zeros(b, dtype=torch.int32, device=DEV), torch.empty(b, dtype=torch.int32, device=DEV)
    ws = torch.empty(nbytes, dtype=torch.uint8, device=DEV) if own_workspace else None

    def call():
        if append:
            m.mqa_project_append_kv_rows(x, P_k, P_v, K, V, lens, after, workspace=ws)
        else:
            m.mqa_project_memory_kv(x, P_k, P_v, K, V, after, workspace=ws)

    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        call()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call()
    for k in range(3):
        x.copy_(torch.randn(b, n, d, device=DEV))
        P_k.mul_(-1.5)
        K.fill_(7), V.fill_(7), after.fill_(-1)
        others = [torch.full((nbytes,), k, dtype=torch.uint8, device=DEV) for _ in range(3)]
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(K, expected(x, P_k, 0)) and torch.equal(V, expected(x, P_v, 0)) and (after == n).all()
        assert all((o == k).all() for o in others)


def test_rows_in_a_graph_of_the_program(m):
    """A capture that torch knows nothing of: no block of its allocator is the graph's, so the call takes none."""
    import ctypes
    from paper_1911_02150_amd import binding
    hip = binding.load_library()               # (the runtime's functions are found through the library that uses it)
    vp = ctypes.c_void_p
    b, n, d = 64, 300, 520
    x, P_k, P_v = inputs(b, n, d, 0, 128, 128, 23)
    K, V = caches(b, 0, n, 128, 128)
    after = torch.empty(b, dtype=torch.int32, device=DEV)
    nbytes = m.mqa_project_kv_workspace_bytes(b, n, d, 1, 128, 128, m.MQA_BF16)
    side = torch.cuda.Stream()
    ws = torch.empty(nbytes, dtype=torch.uint8, device=DEV)
    for w in (ws, torch.empty(16, dtype=torch.uint8, device=DEV)):      # (both routes, before anything is captured)
        m.mqa_project_memory_kv(x, P_k, P_v, K, V, after, workspace=w)
    with torch.cuda.stream(side):
        spare = torch.empty(nbytes, dtype=torch.uint8, device=DEV)
    del spare                                  # a block that an allocation on that stream would get
    torch.cuda.synchronize()
    graph, run = vp(), vp()
    assert hip.hipStreamBeginCapture(vp(side.cuda_stream), 2) == 0       # (relaxed)
    m.mqa_project_memory_kv(x, P_k, P_v, K, V, after, stream=side)
    assert hip.hipStreamEndCapture(vp(side.cuda_stream), ctypes.byref(graph)) == 0
    count = ctypes.c_size_t()
    assert hip.hipGraphGetNodes(graph, None, ctypes.byref(count)) == 0 and count.value == 1
    assert hip.hipGraphInstantiate(ctypes.byref(run), graph, None, None, ctypes.c_size_t(0)) == 0
    with torch.cuda.stream(side):
        others = [torch.full((nbytes,), 5, dtype=torch.uint8, device=DEV) for _ in range(2)]
    for _ in range(3):
        x.copy_(torch.randn(b, n, d, device=DEV))
        K.fill_(7), V.fill_(7), after.fill_(-1)
        torch.cuda.synchronize()
        assert hip.hipGraphLaunch(run, vp(side.cuda_stream)) == 0
        torch.cuda.synchronize()
        assert torch.equal(K, expected(x, P_k, 0)) and torch.equal(V, expected(x, P_v, 0)) and (after == n).all()
        assert all((o == 5).all() for o in others)
    assert hip.hipGraphExecDestroy(run) == 0 and hip.hipGraphDestroy(graph) == 0


def test_rows_on_any_stream(m):
    """A stream given as an object with a `cuda_stream`, as torch's, and as the default one."""
    import types
    b, n, d = 64, 300, 520
    side = torch.cuda.Stream()
    for stream in (side, types.SimpleNamespace(cuda_stream=side.cuda_stream), types.SimpleNamespace(cuda_stream=0), torch.cuda.ExternalStream(side.cuda_stream)):
        x, P_k, P_v = inputs(b, n, d, 0, 128, 128, 22)
        K, V = caches(b, 0, n, 128, 128)
        lens, after = torch.zeros(b, dtype=torch.int32, device=DEV), torch.empty(b, dtype=torch.int32, device=DEV)
        torch.cuda.synchronize()
        m.mqa_project_append_kv_rows(x, P_k, P_v, K, V, lens, after, stream=stream)
        torch.cuda.synchronize()
        assert torch.equal(K, expected(x, P_k, 0)) and torch.equal(V, expected(x, P_v, 0)) and (after == n).all()
        K.fill_(7), V.fill_(7)
        torch.cuda.synchronize()
        m.mqa_project_memory_kv(x, P_k, P_v, K, V, after, stream=stream)
        torch.cuda.synchronize()
        assert torch.equal(K, expected(x, P_k, 0)) and torch.equal(V, expected(x, P_v, 0)) and (after == n).all()


def test_refused_sizes_keep_their_error(m):
    """A size that the library refuses (a head of 20 columns) raises the library's error with its status, from both calls."""
    x = torch.zeros(2, 3, 64, device=DEV)
    P = torch.zeros(64, 20, device=DEV)
    K, V = caches(2, 0, 3, 20, 20)
    a, b = torch.zeros(2, dtype=torch.int32, device=DEV), torch.zeros(2, dtype=torch.int32, device=DEV)
    with pytest.raises(m.MqaError, match="mqa_project_memory_kv failed"):
        m.mqa_project_memory_kv(x, P, P, K, V, a)
    with pytest.raises(m.MqaError, match="mqa_project_append_kv_rows failed"):
        m.mqa_project_append_kv_rows(x, P, P, K, V, a, b)
