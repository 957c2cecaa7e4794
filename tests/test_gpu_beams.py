"""Beam search decoding through the C ABI against the float64 oracle: the step
over a shared source memory plus per-hypothesis rows, the cache reorder by
parent index (bit-exact), and a short search loop that uses both with the
append.  Tolerances as in test_gpu_parity (float32 cache 1e-5; bf16 cache 2e-2
absolute and 1e-2 relative)."""
import numpy as np
import pytest
import torch

import mqa_inputs as mi
from oracle import mqa_oracle as orc

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def m():
    import paper_1911_02150_amd as lib
    lib.load_library()
    return lib


def dev_cache(a):
    return mi.bits_to_torch_bf16(a).to(DEV) if a.dtype == np.uint16 else torch.from_numpy(a).to(DEV)


def check(got, ref, cache, what):
    got = got.detach().cpu().numpy().astype(np.float64)
    assert np.isfinite(got).all(), f"{what}: non-finite output"
    err = float(np.max(np.abs(got - ref)))
    if cache == "f32":
        assert err <= 1e-5, f"{what}: max abs err {err:.3e} > 1e-5"
    else:
        assert err <= 2e-2 and err <= 1e-2 * float(np.max(np.abs(ref))), f"{what}: max abs err {err:.3e}"
    return err


def run_beams(m, c, scale=1.0):
    t = {n: (dev_cache(a) if n[0] in "KV" else torch.from_numpy(a).to(DEV)) for n, a in c.items()}
    o = m.mqa_decode_step_beams(t["q"], t["K_src"], t["V_src"], t["lens_src"], t["K_own"], t["V_own"], t["lens_own"],
                                scale=scale)
    torch.cuda.synchronize()
    ref = orc.mqa_decode_beams(c["q"], mi.cache_as_f64(c["K_src"]), mi.cache_as_f64(c["V_src"]), c["lens_src"],
                               mi.cache_as_f64(c["K_own"]), mi.cache_as_f64(c["V_own"]), c["lens_own"], scale)
    return o, ref


BEAM_CASES = [
    # (seed, b, beam, h, cap_src, cap_own, k, v, cache, lens_src, lens_own)
    (1, 3, 4, 8, 300, 70, 128, 128, "bf16", "ragged", "ragged"),      # MFMA: 32 rows share a source, 8 an own part
    (2, 2, 4, 8, 128, 128, 128, 128, "bf16", "full", "full"),          # the paper's shape: 128 source + 128 target
    (3, 8, 4, 8, 4096, 128, 128, 128, "bf16", "ragged", "ragged"),     # long prompts: the source pass is split
    (4, 2, 3, 5, 90, 40, 64, 32, "f32", "ragged", "ragged"),           # generic kernel, odd sizes
    (5, 2, 4, 8, 64, 32, 128, 128, "f32", "ragged", "ragged"),
    (6, 1, 1, 8, 200, 50, 128, 128, "bf16", "full", "ragged"),         # one hypothesis
    (7, 2, 8, 16, 500, 33, 128, 128, "bf16", "ragged", "ragged"),      # 128 rows per source: four head groups
    (8, 2, 4, 8, 100, 20, 128, 128, "bf16", "ragged", [0] * 8),        # first step: nothing generated yet
    (9, 2, 4, 8, 100, 20, 128, 128, "bf16", [0, 0], "full"),           # no shared rows at all
    (10, 2, 2, 8, 100, 20, 128, 128, "bf16", [0, 37], [0, 5, 0, 0]),   # a hypothesis with nothing to see: zeros
    (11, 2, 2, 40, 200, 40, 128, 128, "bf16", "ragged", "ragged"),     # more than 32 heads: head groups in both parts
]


@pytest.mark.parametrize("seed,b,beam,h,cap_src,cap_own,k,v,cache,ls,lo", BEAM_CASES)
def test_decode_step_beams(m, seed, b, beam, h, cap_src, cap_own, k, v, cache, ls, lo):
    c = mi.beam_case(seed, b, beam, h, cap_src, cap_own, k, v, cache=cache, lens_src=ls, lens_own=lo)
    o, ref = run_beams(m, c, scale=1.0 if seed % 2 else 0.5)
    check(o, ref, cache, f"beams case {seed}")
    if seed == 10:
        assert float(o[0, 0].abs().max()) == 0.0      # source 0, hypothesis 0: no valid row anywhere


def test_beams_equal_plain_steps_on_gpu(m):
    """The same outputs from the plain step over per-hypothesis copies of the memory (GPU vs GPU,
    both within tolerance of the oracle; here the two GPU paths are compared directly)."""
    b, beam, h, cs, co = 2, 4, 8, 160, 40
    c = mi.beam_case(21, b, beam, h, cs, co, 128, 128, lens_src="ragged", lens_own="ragged", poison=False)
    o, ref = run_beams(m, c)
    K = np.zeros((b * beam, cs + co, 128), dtype=np.uint16)
    V = np.zeros_like(K)
    lens = np.zeros(b * beam, dtype=np.int32)
    for i in range(b):
        for e in range(beam):
            r, a, n = i * beam + e, int(c["lens_src"][i]), int(c["lens_own"][i * beam + e])
            K[r, :a], V[r, :a] = c["K_src"][i, :a], c["V_src"][i, :a]
            K[r, a:a + n], V[r, a:a + n] = c["K_own"][i, e, :n], c["V_own"][i, e, :n]
            lens[r] = a + n
    flat = m.mqa_decode_step(torch.from_numpy(c["q"]).to(DEV).view(b * beam, h, 128), dev_cache(K), dev_cache(V),
                             torch.from_numpy(lens).to(DEV))
    assert float((flat.view_as(o) - o).abs().max()) <= 1e-3
    check(flat.view_as(o), ref, "bf16", "materialised memories")


@pytest.mark.parametrize("cache,h_kv", [("bf16", 1), ("f32", 1), ("bf16", 3), ("f32", 2)])
def test_beam_reorder_bit_exact(m, cache, h_kv):
    g = mi.rng(2100, h_kv)
    n, cap, k, v = 12, 530, 128, 64
    shape_k = (n, cap, k) if h_kv == 1 else (n, h_kv, cap, k)
    shape_v = shape_k[:-1] + (v,)
    K = g.standard_normal(shape_k, dtype=np.float32)
    V = g.standard_normal(shape_v, dtype=np.float32)
    if cache == "bf16":
        K, V = mi.f32_to_bf16_bits(K), mi.f32_to_bf16_bits(V)
    lens = g.integers(0, cap + 1, size=n).astype(np.int32)
    lens[0], lens[1] = cap, 0
    parent = g.integers(0, n, size=n).astype(np.int32)
    parent[:3] = [1, 0, 0]
    K2, V2, lens2 = orc.beam_reorder_kv(K, V, lens, parent)
    dK, dV = dev_cache(K), dev_cache(V)
    oK, oV = torch.full_like(dK, 7.0), torch.full_like(dV, 7.0)
    olens = torch.full((n,), -5, dtype=torch.int32, device=DEV)
    m.mqa_beam_reorder_kv(dK, dV, torch.from_numpy(lens).to(DEV), torch.from_numpy(parent).to(DEV), oK, oV, olens)
    torch.cuda.synchronize()
    assert np.array_equal(olens.cpu().numpy(), lens2)
    as_np = (lambda t: t.view(torch.int16).cpu().numpy().view(np.uint16)) if cache == "bf16" else (lambda t: t.cpu().numpy())
    gK, gV = as_np(oK), as_np(oV)
    seven = as_np(torch.full((1,), 7.0, dtype=dK.dtype))[0]
    for r in range(n):
        L = int(lens2[r])
        assert np.array_equal(gK[r, ..., :L, :], K2[r, ..., :L, :]) and np.array_equal(gV[r, ..., :L, :], V2[r, ..., :L, :])
        assert (gK[r, ..., L:, :] == seven).all() and (gV[r, ..., L:, :] == seven).all()   # beyond the length: untouched
    # the source is unchanged
    assert np.array_equal(as_np(dK), K) and np.array_equal(as_np(dV), V)


def test_beam_search_loop(m):
    """A short search: every step appends a row to each hypothesis' own cache, attends, and
    re-orders the caches by seeded parent choices (double-buffered).  The oracle does the same
    with numpy; rows are given float32 inputs, so both caches hold identical bf16 rows and the
    step outputs are held to the bf16 tolerance at every step."""
    b, beam, h, k, v, cs, co, steps = 3, 4, 8, 128, 128, 96, 16, 12
    c = mi.beam_case(31, b, beam, h, cs, co, k, v, lens_src="ragged", lens_own=[0] * (b * beam), poison=False)
    g = mi.rng(2200, 0)
    n = b * beam
    Ksrc, Vsrc = dev_cache(c["K_src"]), dev_cache(c["V_src"])
    lsrc = torch.from_numpy(c["lens_src"]).to(DEV)
    bufs = [[torch.zeros((n, co, k), dtype=torch.bfloat16, device=DEV), torch.zeros((n, co, v), dtype=torch.bfloat16, device=DEV),
             torch.zeros((n,), dtype=torch.int32, device=DEV)] for _ in range(2)]
    rK, rV = np.zeros((n, co, k)), np.zeros((n, co, v))
    rlens = np.zeros(n, dtype=np.int64)
    cur = 0
    for t in range(steps):
        q = g.standard_normal((b, beam, h, k), dtype=np.float32) * np.float32(k ** -0.5)
        kn = g.standard_normal((n, k), dtype=np.float32)
        vn = g.standard_normal((n, v), dtype=np.float32)
        K, V, lens = bufs[cur]
        m.mqa_append_kv(K, V, torch.from_numpy(kn).to(DEV), torch.from_numpy(vn).to(DEV), lens)
        orc.append_kv(rK, rV, kn, vn, rlens, cache="bf16")
        o = m.mqa_decode_step_beams(torch.from_numpy(q).to(DEV), Ksrc, Vsrc, lsrc, K.view(b, beam, co, k),
                                    V.view(b, beam, co, v), lens)
        ref = orc.mqa_decode_beams(q, mi.cache_as_f64(c["K_src"]), mi.cache_as_f64(c["V_src"]), c["lens_src"],
                                   rK.reshape(b, beam, co, k), rV.reshape(b, beam, co, v), rlens)
        check(o, ref, "bf16", f"search step {t}")
        # hypotheses continue parents within their own source
        parent = (np.arange(n) // beam) * beam + g.integers(0, beam, size=n)
        nK, nV, nlens = bufs[1 - cur]
        m.mqa_beam_reorder_kv(K, V, lens, torch.from_numpy(parent.astype(np.int32)).to(DEV), nK, nV, nlens)
        rK, rV, rlens = orc.beam_reorder_kv(rK, rV, rlens, parent)
        cur = 1 - cur
    torch.cuda.synchronize()
    K, V, lens = bufs[cur]
    assert np.array_equal(lens.cpu().numpy(), rlens) and int(rlens[0]) == steps
    for r in range(n):
        assert np.array_equal(K[r, :steps].double().cpu().numpy(), rK[r, :steps])


def test_encoder_decoder_memory_with_beams(m):
    """Encoder-decoder attention (Section 3 `MultiqueryAttention`: queries against a static memory M)
    under beam search: the memory rows of a source are projected once, its `beam` hypotheses are
    beam*h rows of one multi-query call over that fixed cache.  The cache holds the oracle's
    bf16-rounded K/V rows (oracle -> GPU), so the stated tolerance applies to y."""
    b, beam, h, d, k, v, cap = 6, 4, 8, 256, 128, 128, 100
    g = mi.rng(2300, 0)
    s = np.float32(d ** -0.5)
    x = g.standard_normal((b, beam, d), dtype=np.float32)
    M = g.standard_normal((b, cap, d), dtype=np.float32)
    P_q = g.standard_normal((h, d, k), dtype=np.float32) * s
    P_k = g.standard_normal((d, k), dtype=np.float32) * s
    P_v = g.standard_normal((d, v), dtype=np.float32) * s
    P_o = g.standard_normal((h, d, v), dtype=np.float32) * np.float32((h * v) ** -0.5)
    mlen = g.integers(1, cap + 1, size=b).astype(np.int32)
    Kr = orc.round_to_bf16(orc.project_kv(M.reshape(b * cap, d), P_k)).reshape(b, cap, k)
    Vr = orc.round_to_bf16(orc.project_kv(M.reshape(b * cap, d), P_v)).reshape(b, cap, v)
    ref = np.zeros((b, beam, d))
    for i in range(b):
        for e in range(beam):
            qi = orc.project_q(x[i, e][None], P_q)[0]
            o = orc.mqa_decode(qi[None], Kr[i][None], Vr[i][None], [mlen[i]])
            ref[i, e] = orc.project_o(o, P_o)[0]
    dx = torch.from_numpy(x).to(DEV).view(b * beam, d)
    q = m.mqa_project_qkvo(m.MQA_PROJ_Q, dx, torch.from_numpy(P_q).to(DEV))               # [b*beam, h, k]
    K = torch.from_numpy(Kr).to(torch.bfloat16).to(DEV)
    V = torch.from_numpy(Vr).to(torch.bfloat16).to(DEV)
    o = m.mqa_decode_step(q.view(b, beam * h, k), K, V, torch.from_numpy(mlen).to(DEV))     # beam*h rows per source
    y = m.mqa_project_qkvo(m.MQA_PROJ_O, o.view(b * beam, h, v), torch.from_numpy(P_o).to(DEV))
    torch.cuda.synchronize()
    check(y.view(b, beam, d), ref, "bf16", "encoder-decoder attention, beam 4")
    # the GPU's own projection of the memory, appended in bulk, gives valid roundings of the same rows
    kn = m.mqa_project_qkvo(m.MQA_PROJ_KV, torch.from_numpy(M).to(DEV).view(b * cap, d), torch.from_numpy(P_k).to(DEV))
    vn = m.mqa_project_qkvo(m.MQA_PROJ_KV, torch.from_numpy(M).to(DEV).view(b * cap, d), torch.from_numpy(P_v).to(DEV))
    K2, V2 = torch.zeros_like(K), torch.zeros_like(V)
    l2 = torch.zeros(b, dtype=torch.int32, device=DEV)
    m.mqa_append_kv_rows(K2, V2, kn.view(b, cap, k), vn.view(b, cap, v), l2)
    assert int(l2.min()) == cap and float((K2.float() - K.float()).abs().max()) <= 2.0 ** -6
    assert float((K2 != K).float().mean()) < 1e-2


# one, two and four words a thread, words in turn (also of a slot alone); rows of K and V of different length, a last piece that is not full, empty and full slots
@pytest.mark.parametrize("n,h,cap,k,v,dtype", [(3, 1, 5, 8, 24, torch.bfloat16), (64, 1, 129, 128, 128, torch.bfloat16), (40, 2, 1001, 64, 128, torch.bfloat16),
                                               (9, 1, 30011, 128, 64, torch.bfloat16), (5, 3, 24000, 128, 128, torch.bfloat16), (7, 1, 40003, 104, 128, torch.float32),
                                               (60, 2, 1501, 128, 64, torch.bfloat16), (5, 1, 4097, 8, 256, torch.float32), (300, 1, 1029, 128, 120, torch.bfloat16)])
def test_beam_reorder_of_any_size(m, n, h, cap, k, v, dtype):
    g = torch.Generator(device=DEV)
    g.manual_seed(cap)
    shape = (n, h, cap) if h > 1 else (n, cap)
    K, V = (torch.randn(*shape, w, generator=g, device=DEV).to(dtype) for w in (k, v))
    lens = torch.randint(0, cap + 1, (n,), generator=g, device=DEV, dtype=torch.int32)
    lens[0], lens[1] = cap, 0
    parent = torch.randint(0, n, (n,), generator=g, device=DEV, dtype=torch.int32)
    parent[0], parent[1] = 1, 0
    out = [torch.full_like(K, 7.0), torch.full_like(V, 7.0), torch.full_like(lens, -1)]
    m.mqa_beam_reorder_kv(K, V, lens, parent, *out)
    assert torch.equal(out[2], lens[parent.long()])
    for new, old in zip(out, (K, V)):
        there = torch.arange(cap, device=DEV) < out[2][:, None]
        there = (there[:, None] if h > 1 else there).unsqueeze(-1)
        assert torch.equal(new, torch.where(there, old[parent.long()], torch.full_like(old, 7.0)))


def test_beam_reorder_of_a_deep_grid(m):
    """Sixteen words a thread: where pieces of eight would be more than 65535 (K rows of 2 GiB)."""
    cap = 65535 * 256 * 8 // 64 + 9
    K, V = torch.empty(1, cap, 256, device=DEV).normal_(), torch.empty(1, cap, 8, device=DEV).normal_()
    lens, parent = torch.tensor([cap - 2], dtype=torch.int32, device=DEV), torch.zeros(1, dtype=torch.int32, device=DEV)
    out = [torch.zeros_like(K), torch.zeros_like(V), torch.zeros_like(lens)]
    m.mqa_beam_reorder_kv(K, V, lens, parent, *out)
    assert out[2].item() == cap - 2
    for new, old in zip(out, (K, V)):
        assert torch.equal(new[:, :-2], old[:, :-2]) and not new[:, -2:].any()
