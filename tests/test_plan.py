"""Regression guard for the cost model that lays out the two matrix products of a pass (tile sizes, k
split of the g_w product, dispatch order).  Its constants were fitted to a sweep of every plan over
these layer shapes on MI355X, where the picked plan measured within 2 % of the best one; a change
to the model that moves any of these picks has to come with a new sweep.  Host arithmetic only."""
import pytest

import paper_2406_15102_amd as hlq
from paper_2406_15102_amd import workloads as wl

# workload -> (tile edge of the g_x product, of the g_w product, k splits of the g_w product, g_w first)
MEASURED_PICKS = {
    "c2": (128, 128, 1, 1), "c3": (128, 128, 2, 1),
    "c4": (256, 256, 1, 0), "c4_b32": (256, 256, 1, 0), "c4_b64": (256, 256, 1, 0),
    "c5_r4": (256, 256, 1, 0), "c5_r8": (256, 256, 1, 0), "c5_r16": (256, 256, 1, 0),
    "p01": (128, 128, 6, 1), "p02": (128, 128, 4, 0), "p05": (128, 128, 12, 1), "p07": (128, 128, 12, 1),
    "p08": (128, 128, 6, 1), "p09": (128, 128, 16, 0), "p10": (128, 128, 6, 0), "p12": (128, 128, 1, 0),
}


@pytest.mark.parametrize("name", sorted(MEASURED_PICKS))
def test_pair_plan_picks_the_measured_plan(name):
    w = wl.WORKLOADS[name]
    Kc = w.N // w.B * w.r
    bits = hlq.HLQ_BITS_4_PACKED if w.d_out % 32 == 0 else hlq.HLQ_BITS_4
    plan = hlq.hlq_backward_products_plan(w.N, w.d_in, w.d_out, Kc, bits, False, 1 << 28)
    assert plan[:4] == MEASURED_PICKS[name], plan


def test_plan_properties():
    # without scratch the g_w product is never split; the split never exceeds its k steps
    for name in ("c3", "p05", "p09"):
        w = wl.WORKLOADS[name]
        Kc = w.N // w.B * w.r
        assert hlq.hlq_backward_products_plan(w.N, w.d_in, w.d_out, Kc, hlq.HLQ_BITS_4_PACKED, False, 0)[2] == 1
        s = hlq.hlq_backward_products_plan(w.N, w.d_in, w.d_out, Kc, hlq.HLQ_BITS_4_PACKED, False, 1 << 28)[2]
        assert 1 <= s <= (2 * Kc + 127) // 128
        assert s * w.d_out * w.d_in * 4 <= 1 << 28
    with pytest.raises(hlq.HlqError):
        hlq.hlq_backward_products_plan(4096, 4096, 11000, 2048, hlq.HLQ_BITS_4_PACKED)   # d_out % 32 for packed codes


F6, NIBBLES, BYTES = 2, 1, 0


def test_how_codes_are_kept():
    """The route of the g_x codes: the 6-bit layout unless its rows are mostly padding, and for weight codes that are handed over
    where the tokens pay for bringing them into it."""
    def kept(N, I, O, codes=False, flags=0):
        return hlq.hlq_linear_backward_plan(N, I, O, 16, 8, w_is_codes=codes, flags=flags)[5]

    assert kept(4096, 4096, 11008) == F6 and kept(4096, 4096, 11008, True) == F6
    assert kept(1024, 432, 96) == NIBBLES and kept(1024, 432, 80) == BYTES
    for flag in (hlq.HLQ_FLAG_GX_8BIT, hlq.HLQ_FLAG_GX_UNPACKED):
        assert kept(4096, 4096, 11008, flags=flag) == BYTES
    # 235 million codes: read, written and read again by every call
    assert kept(256, 28672, 8192) == F6
    for N in (256, 512, 1024):
        assert kept(N, 28672, 8192, True) == NIBBLES
        assert kept(N, 28672, 8208, True) == BYTES
    assert kept(1040, 28672, 8192, True) == F6
    assert kept(1056, 28672, 8192, True, hlq.HLQ_FLAG_GW_INT8) == NIBBLES and kept(2048, 28672, 8192, True, hlq.HLQ_FLAG_GW_INT8) == F6
    assert kept(512, 8192, 28672, True) == NIBBLES and kept(1024, 8192, 28672, True) == F6
    # long reductions, and few codes
    assert kept(256, 4096, 11008, True) == F6 and kept(256, 8192, 8192, True) == NIBBLES and kept(256, 4096, 8192, True) == F6


def test_pass_plan_checks_like_the_pass():
    N, I, O = 4096, 512, 768
    need = hlq.hlq_workspace_bytes_mode(N, I, O, 16, 8, False, 0)
    assert hlq.hlq_linear_backward_plan(N, I, O, 16, 8, workspace_bytes=need)[6] == N // 2
    assert hlq.hlq_linear_backward_plan(N + 16, I, O, 16, 8)[6] == (N + 16) // 2 + 56      # whole steps of 64 values
    for bad in ((N + 8, I, O, 16, 8), (N, I, O, 24, 8), (N, I, O, 16, 17)):
        with pytest.raises(hlq.HlqError):
            hlq.hlq_linear_backward_plan(*bad, workspace_bytes=need)
    with pytest.raises(hlq.HlqError):
        hlq.hlq_linear_backward_plan(N, I, O, 16, 8, workspace_bytes=1 << 20)
    with pytest.raises(hlq.HlqError):
        hlq.hlq_linear_backward_plan(N, I, O, 16, 8, flags=1 << 20, workspace_bytes=need)


# (N, d_in, d_out, B, r) -> tile edges, k splits, g_w first, of passes whose codes are kept in the 6-bit layout: the pick is the best plan that
# was timed, or within 2 % of it; the last three are wide layers of few tokens (kManyRoundsMore), before them one that is not
MEASURED_PICKS_OF_PASSES = {
    (12608, 768, 3072, 16, 8): (256, 128, 1, 1), (9200, 1160, 3120, 16, 8): (256, 128, 1, 0), (4096, 4096, 11008, 16, 8): (256, 256, 1, 0),
    (512, 28672, 8192, 16, 8): (128, 128, 1, 0), (1024, 28672, 8192, 16, 8): (256, 256, 1, 0), (1024, 8192, 8192, 16, 8): (256, 256, 1, 0),
    (2048, 11008, 4096, 16, 8): (256, 256, 1, 0),
}


@pytest.mark.parametrize("shape", sorted(MEASURED_PICKS_OF_PASSES))
def test_pass_plan_picks_the_measured_plan(shape):
    plan = hlq.hlq_linear_backward_plan(*shape)
    assert plan[:4] == MEASURED_PICKS_OF_PASSES[shape] and plan[5] == F6, plan
