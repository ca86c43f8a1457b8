"""Workspaces smaller than the size the library names: what was once enough for the fewest partials is accepted still."""
import pytest

import launch_record as rec
from test_decode_plan import _params


# batch, q heads, kv heads, head_dim, prompt, bound, block size, blocks, bytes that were enough
@pytest.mark.parametrize("B,Hq,Hkv,d,s,bound,block,blocks,size", [
    (5, 112, 16, 128, 3992, 4928, 8, 280, 6068224),        # chunks as long as a span of the contexts takes
    (1, 128, 32, 128, 1988, 11288, 8, 14, 2575872),
    (3, 16, 4, 64, 8260, 18233, 16, 3, 1896960),           # chunks that save no turn
    (136, 16, 4, 64, 506, 400, 8, 149, 2828800),           # many-rows items that only the cache speaks for
])
def test_decode_with_the_fewest_partials(B, Hq, Hkv, d, s, bound, block, blocks, size):
    p = _params(B, Hq, Hkv, s, bound, bs=block, d=d, num_blocks=blocks)
    assert size < rec.workspace_bytes(p)
    assert rec.decode(p, workspace=size)


def test_prompt_phase_as_a_whole_where_the_cut_does_not_fit():
    """A close estimate of both forms keeps the cut, which needs three partials here; the whole form needs none."""
    p = _params(9, 16, 8, 701, 128, bs=128, d=64, num_blocks=9)
    assert rec.prefill(p, 972, 216, workspace=8087040)[0]["whole"]
    assert not rec.prefill(p, 972, 216)[0]["whole"]


def test_several_prompts_as_a_whole_where_the_cut_does_not_fit():
    """By the rows that share a prompt the cut is the shorter form, by the mean over the prompts the whole one."""
    p = _params(12, 128, 32, 565, 17, d=64)
    call = (p, [565, 182, 145, 9], [1, 1, 6, 4], [7, 7, 42, 28], 14)
    assert rec.prefill_multi(*call, workspace=5591040)[0]["whole"]
    assert not rec.prefill_multi(*call)[0]["whole"]
