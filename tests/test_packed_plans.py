"""mqa_stack_product_plan on the host: what it says is what mqa_stack_product takes, and products of three exact terms stay what they are."""
import random

import pytest
import torch


@pytest.fixture(scope="module")
def m():
    import paper_1911_02150_amd.binding as lib
    lib.load_library()
    return lib


def test_forms_are_valid(m):
    lib, rng, packed, parts_seen = m.load_library(), random.Random(5), 0, set()
    for _ in range(20000):
        mode = rng.choice([m.MQA_PROJ_Q, m.MQA_PROJ_O, m.MQA_PROJ_LINEAR])
        h = rng.choice([1, 1, 2, 8])
        d, kv, rows = 8 * rng.randint(1, 640), 8 * rng.randint(1, 640), int(2 ** rng.uniform(0, 15))
        residual = rng.random() < 0.5
        form = lib.mqa_stack_product_plan(mode, rows, d, h, kv, int(residual))
        h = 1 if mode == m.MQA_PROJ_LINEAR else h
        N, C = (d, h * kv) if mode == m.MQA_PROJ_O else (h * kv, d)
        assert form >= 0
        if form == 0:
            continue
        packed += 1
        S, blocks = form & 15, C // 32
        assert C % 32 == 0 and form >> 4 <= 5 and 1 <= S <= 8 and (residual or S == 1) and (N <= 4096 or not residual)
        per = -(-blocks // S)
        assert -(-blocks // per) == S                                # no empty parts
        if not residual:
            assert lib.mqa_project_plan(mode, rows, d, h, kv) != 1     # not one of three terms
        parts_seen.add(S)
    assert packed > 1000 and parts_seen == {1, 2, 4, 8}


def test_sizes_without_a_form(m):
    lib = m.load_library()
    plan = lib.mqa_stack_product_plan
    assert plan(m.MQA_PROJ_LINEAR, 16384, 1024, 1, 4096, 0) >> 4 == 0 and plan(m.MQA_PROJ_LINEAR, 16384, 4096, 1, 1024, 1) & 15 == 1
    assert plan(m.MQA_PROJ_LINEAR, 128, 1024, 1, 4096, 0) == 0 and plan(m.MQA_PROJ_LINEAR, 128, 4096, 1, 1024, 1) == 0      # three terms
    assert plan(m.MQA_PROJ_LINEAR, 16384, 1000, 1, 4096, 0) == 0 and plan(m.MQA_PROJ_LINEAR, 16384, 1024, 1, 4100, 0) == 0
    assert plan(m.MQA_PROJ_KV, 16384, 1024, 1, 4096, 0) == 0 and plan(m.MQA_PROJ_Q, 0, 1024, 8, 128, 0) == 0
    assert plan(m.MQA_PROJ_O, 4096, 4128, 8, 128, 1) == 0                                        # rows too long for the layernorm that packs
    for lines, C, nbytes in ((4096, 1024, 4 * 4096 * 1024), (8, 40, 0), (0, 32, 0), (1 << 26, 32, 0), (8, 0, 0)):
        assert lib.mqa_stack_packed_bytes(lines, C, 0) == nbytes and lib.mqa_stack_packed_bytes(lines, C, 1) == (nbytes + 4 * lines if nbytes else 0)


@pytest.mark.skipif(torch.cuda.is_available(), reason="addresses that are not there: only where nothing can be launched")
def test_refused(m):
    lib, A = m.load_library(), 0x10000
    ok = dict(rows=4, N=32, C=96, epi=0, form=1)
    for change, status in ((dict(C=40), 2), (dict(N=12), 2), (dict(rows=0), 2), (dict(form=16 * 6 + 1), 2), (dict(form=0), 2), (dict(form=4), 2),
                           (dict(form=3, epi=2), 2), (dict(N=40, epi=3), 2), (dict(epi=4), 5), (dict(form=-1), 2), ({}, 6)):
        c = dict(ok, **change)
        assert lib.mqa_stack_product(A, A, 1.0, A, c["rows"], c["N"], c["C"], c["epi"], c["form"], 0) == status, change
    assert lib.mqa_stack_product(A + 8, A, 1.0, A, 4, 32, 96, 0, 1, 0) == 3 and lib.mqa_stack_product(None, A, 1.0, A, 4, 32, 96, 0, 1, 0) == 1
    assert lib.mqa_stack_layernorm_packed(None, 0, A, None, A, 4, 40, 1e-6, 0) == 2 and lib.mqa_stack_layernorm_packed(None, 0, A, None, A, 4, 4128, 1e-6, 0) == 2
    assert lib.mqa_stack_layernorm_packed(None, 1, A, A, None, 4, 64, 1e-6, 0) == 1 and lib.mqa_stack_layernorm_packed(None, 0, A, None, None, 4, 64, 1e-6, 0) == 1
    assert lib.mqa_stack_pack(m.MQA_PROJ_KV, A, None, 64, 1, 64, A, A, 0) == 5 and lib.mqa_stack_pack(m.MQA_PROJ_LINEAR, A, None, 40, 1, 64, A, A, 0) == 2
    assert lib.mqa_stack_add_layernorm_packed(m.MQA_PROJ_LINEAR, A, A, A, None, A, 4, 64, 1, 40, 1e-6, None, 0, 0) == 2
    assert lib.mqa_stack_add_layernorm_packed(m.MQA_PROJ_LINEAR, A, A, A, None, None, 4, 64, 1, 64, 1e-6, None, 0, 0) == 1
