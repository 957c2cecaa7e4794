"""mqa_stack_feed_forward on the host: the plan says what the call takes, and what is refused is refused before anything is launched."""
import ctypes
import random

import pytest
import torch


@pytest.fixture(scope="module")
def m():
    import paper_1911_02150_amd.binding as lib
    lib.load_library()
    return lib


def test_plans(m):
    rng, forms = random.Random(5), set()
    for _ in range(20000):
        rows, d, ff = int(2 ** rng.uniform(0, 16)), rng.choice([8, 32, 32]) * rng.randint(1, 40), rng.choice([8, 32, 32]) * rng.randint(1, 160)
        plan, nbytes = m.mqa_stack_feed_forward_plan(rows, d, ff)
        assert (plan == 0) == (nbytes == 0)
        if plan == 0:
            continue
        assert d % 32 == 0 and ff % 32 == 0 and nbytes == 16 + 4 * (d + ff) + 16 * -(-rows // 1024) + 8 * d * ff + 4 * rows * (d + ff + -(-ff // 128))
        assert plan & 1 == (rows >= 4096 and rows * d * ff >= 12e9)
        forms.add((plan >> 4 & 15, plan >> 8 & 15))
        if plan & 1:                               # the layernorm and the two products are those that the call stands for, or none are faster in parts
            assert m.load_library().mqa_project_plan(m.MQA_PROJ_LINEAR, rows, d, 1, ff) in (128, 256)
            assert m.load_library().mqa_project_plan(m.MQA_PROJ_LINEAR, rows, ff, 1, d) in (128, 256)
            assert m.mqa_project_add_layernorm_workspace_bytes(m.MQA_PROJ_LINEAR, rows, ff, 1, d) == 0
    assert {f for f, _ in forms} == {f for _, f in forms} == {1, 2, 3}


def test_sizes_without_a_form(m):
    for rows, d, ff in ((0, 1024, 4096), (16384, 1000, 4096), (16384, 1024, 4104), (16384, 4128, 4096), (16384, 0, 32), (128, 1024, 4096), (1 << 26, 32, 32), (-5, 32, 32)):
        assert m.mqa_stack_feed_forward_plan(rows, d, ff) == (0, 0)
    assert m.load_library().mqa_stack_feed_forward_plan(16384, 1024, 4096, None) & 1


@pytest.mark.skipif(torch.cuda.is_available(), reason="addresses that are not there: only where nothing can be launched")
def test_refused(m):
    lib, A, nbytes = m.load_library(), 0x10000, ctypes.c_size_t(0)
    lib.mqa_stack_feed_forward_plan(16384, 1024, 4096, ctypes.byref(nbytes))

    def status(W1=A, W2=A, x=A, rows=16384, d=1024, ff=4096, ws=A, n=nbytes.value, eps=1e-6):
        return lib.mqa_stack_feed_forward(W1, W2, x, rows, d, ff, eps, ws, n, None)

    for change, want in ((dict(W1=None), 1), (dict(W2=None), 1), (dict(x=None), 1), (dict(d=1000), 2), (dict(rows=0), 2), (dict(rows=128), 2), (dict(eps=-1e-3), 2), (dict(eps=float("nan")), 2), (dict(x=A + 4), 3), (dict(ws=A + 8), 3),
                         (dict(W2=A + 8), 3), (dict(ws=None), 4), (dict(n=nbytes.value - 1), 4), ({}, 6)):
        assert status(**change) == want, change
