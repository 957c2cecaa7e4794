"""How many ranges the default plan cuts a sequence into: never more than fill the compute units, fewer where the last round
of workgroups would be nearly empty or the merge would cost more than it spreads; what fits a plan's workspace fits it still."""
import os

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_1911_02150_amd", "libmqa_decode.so")
pytestmark = pytest.mark.skipif(not os.path.exists(LIB), reason="library not built (run __graft_entry__.build())")


@pytest.mark.parametrize("b,h,cap,k,f32,mh,want", [
    (128, 8, 256, 128, False, False, 1),      # a merge launch for 128 positions per range
    (64, 8, 256, 128, False, False, 1),
    (64, 8, 512, 128, False, False, 4),       # worth it: 9.3 us against 10.4
    (200, 8, 512, 128, False, False, 1),      # 400 workgroups on 256 compute units
    (200, 8, 512, 128, True, False, 1),
    (100, 8, 8192, 128, False, False, 2),     # 200 instead of 300
    (64, 32, 8192, 128, False, False, 4),
    (32, 8, 2048, 128, True, False, 8),
    (130, 20, 512, 64, False, False, 1),
    (1, 8, 1 << 17, 128, False, False, 256),
    (512, 64, 4096, 128, False, False, 1),
    (100, 64, 4096, 128, False, False, 3),    # 64 heads per workgroup: as many as fill the chip
    (25, 8, 512, 128, False, True, 1),
])
def test_default_ranges(b, h, cap, k, f32, mh, want):
    import paper_1911_02150_amd as m
    dt = m.MQA_F32 if f32 else m.MQA_BF16
    assert m.mqa_decode_num_splits(b, h, cap, k, k, dt, multi_head=mh) == want


def test_ranges_stay_within_what_filled_the_chip():
    import paper_1911_02150_amd as m
    for k, dt in ((128, m.MQA_BF16), (128, m.MQA_F32), (64, m.MQA_BF16), (48, m.MQA_F32)):
        for b in (1, 3, 17, 64, 100, 129, 255, 256, 700):
            for cap in (1, 31, 128, 129, 300, 1000, 5000, 40000):
                S, chunk, _ = m.mqa_decode_plan(b, 8, cap, k, k, dt)
                least = 128 if (k, dt) == (128, m.MQA_BF16) else 256
                most = max(1, min(-(-256 // b), -(-cap // least)))
                assert 1 <= S <= most and chunk % 32 == 0 and (S - 1) * chunk < cap <= S * chunk
                assert m.mqa_decode_workspace_bytes_default(b, 8, cap, k, k, dt) <= most * b * 8 * (k + 2) * 4 + 16 + 4 * b


def test_projection_plans():
    """Which kernel a projection takes: refused sizes as the calls refuse them, small products and new K / V rows not in the
    split-operand kernel, larger ones in larger tiles, offsets past 32 bits not."""
    import paper_1911_02150_amd as m
    plan, kv = m.mqa_project_plan, m.mqa_project_kv_plan
    assert plan(9, 4, 64, 2, 16) == -5 and plan(m.MQA_PROJ_Q, 4, 60, 2, 16) == -2 and plan(m.MQA_PROJ_O, 0, 64, 2, 16) == -2
    assert plan(m.MQA_PROJ_LINEAR, 4, 64, 0, 16) == 0                     # h is ignored
    assert plan(m.MQA_PROJ_Q, 128, 1024, 8, 128) == plan(m.MQA_PROJ_O, 128, 1024, 8, 128) == 0
    assert plan(m.MQA_PROJ_KV, 1 << 15, 1024, 1, 4096) == plan(m.MQA_PROJ_KV_MH, 1 << 15, 1024, 8, 128) == 0
    assert [plan(m.MQA_PROJ_LINEAR, rows, 1024, 1, N) for rows, N in ((512, 1024), (1024, 1024), (4096, 1024), (16384, 4096))] == [32, 64, 128, 256]
    assert plan(m.MQA_PROJ_LINEAR, 512, 1 << 24, 1, 4096) == 0            # 64 rows of a tile reach over 4 GiB
    assert kv(4, 64, 0, 1, 20, 16, m.MQA_BF16) == -2 and kv(4, 64, 0, 1, 16, 16, 7) == -5 and kv(4, 64, -1, 1, 16, 16, m.MQA_BF16) == -2
    assert kv(1 << 15, 1024, 0, 1, 128, 128, m.MQA_BF16) == 1 and kv(1 << 15, 1024, 0, 1, 128, 128, m.MQA_F32) == 0
    assert kv(128, 1024, 8, 8, 128, 128, m.MQA_BF16) == 0 and kv(128, 1024, 0, 1, 128, 128, m.MQA_BF16) == 0
    assert kv(1 << 15, 1 << 15, 0, 1, 128, 128, m.MQA_BF16) == 0          # sums of digit products past 32 bits
