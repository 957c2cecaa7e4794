"""The fused q / K / V kernel and the memory rows (csrc/project.hip) in every tile width that their rule takes.  Operands are small
whole numbers, so that every sum is exact in float32 in any order and only the caches' rounding is left: results are compared bit by bit."""
import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def m():
    import paper_1911_02150_amd.binding as lib
    lib.load_library()
    return lib


def _whole(g, *shape):
    return torch.randint(-15, 16, shape, generator=g, device=DEV).float()


def _operands(heads, d, h, k, v, dtype, b, cap):
    g = torch.Generator(device=DEV)
    g.manual_seed(b * d + h)
    of = (h,) if heads == "multihead" else ()
    Pq, Pk, Pv = _whole(g, h, d, k), _whole(g, *of, d, k), _whole(g, *of, d, v)
    K, V = torch.full((b, *of, cap, k), 3.0, device=DEV, dtype=dtype), torch.full((b, *of, cap, v), 3.0, device=DEV, dtype=dtype)
    return g, Pq, Pk, Pv, K, V


def _rows(x, P):
    """[rows, d] by [d, k] or [h, d, k], exact."""
    return (x.double() @ P.double()).float() if P.dim() == 2 else torch.stack([x.double() @ p.double() for p in P], 1).float()


# blocks of columns: one (narrow caches; few rows), two, four; a round of tiles and more than one; a last chunk of 8 indices; rows past a tile
STEPS = [("multiquery", 17, 24, 2, 16, 32), ("multihead", 24, 1032, 8, 64, 64), ("multihead", 64, 1032, 8, 128, 128), ("multihead", 81, 1032, 8, 128, 128),
         ("multihead", 129, 1032, 8, 128, 128), ("multihead", 250, 1000, 8, 128, 128), ("multiquery", 65, 1032, 8, 128, 128), ("multiquery", 130, 1032, 8, 128, 128),
         ("multiquery", 161, 1032, 8, 128, 128), ("multiquery", 513, 520, 3, 128, 64), ("multiquery", 100, 2056, 16, 128, 128), ("multihead", 700, 1000, 8, 128, 128)]


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("heads,b,d,h,k,v", STEPS)
def test_step(m, heads, b, d, h, k, v, dtype):
    cap = 5
    g, Pq, Pk, Pv, K, V = _operands(heads, d, h, k, v, dtype, b, cap)
    x = _whole(g, b, d)
    lens = torch.arange(b, device=DEV, dtype=torch.int32) % (cap + 1)          # every sixth is full and keeps its rows
    after, q = torch.zeros_like(lens), torch.full((b + 1, h, k), 7.0, device=DEV)
    K0, V0 = K.clone(), V.clone()
    m.mqa_project_append_qkv(x, Pq, Pk, Pv, K, V, lens, after, q=q[:b])
    assert torch.equal(q[:b], _rows(x, Pq)) and (q[b:] == 7.0).all()
    assert torch.equal(after, (lens + 1).clamp(max=cap))
    open_ = (lens < cap).nonzero()[:, 0]
    at = lens[open_].long()
    for cache, P in ((K0, Pk), (V0, Pv)):
        new = _rows(x, P)[open_].to(dtype)
        if heads == "multihead":
            cache[open_, :, at] = new
        else:
            cache[open_, at] = new
    assert torch.equal(K, K0) and torch.equal(V, V0)


MEMORIES = [("multiquery", 1, 16, 24, 16, 16), ("multiquery", 4, 100, 1032, 128, 128), ("multiquery", 8, 128, 1000, 128, 128), ("multihead", 3, 43, 1032, 64, 128),
            ("multihead", 4, 64, 648, 128, 128), ("multiquery", 16, 512, 520, 64, 64), ("multiquery", 3, 349541, 8, 16, 16)]     # the last: 65539 tiles of rows


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("heads,b,n,d,k,v", MEMORIES)
def test_memory(m, heads, b, n, d, k, v, dtype):
    g, _, Pk, Pv, K, V = _operands(heads, d, 5, k, v, dtype, b, n)
    x = _whole(g, b, n, d)
    lens = torch.zeros(b, dtype=torch.int32, device=DEV)
    m.mqa_project_memory_kv(x, Pk, Pv, K, V, lens)
    assert (lens == n).all()
    for cache, P in ((K, Pk), (V, Pv)):
        ref = _rows(x.view(b * n, d), P).to(dtype).view(b, n, *cache.shape[1:-2], cache.shape[-1])
        assert torch.equal(cache, ref.transpose(1, 2) if heads == "multihead" else ref)
