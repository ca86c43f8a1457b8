"""Several prompts of which one has most of the requests, or that no request uses: the forms go by the rows of a step and not
by the list of prompts."""
import pytest

import launch_record as rec
from test_decode_plan import _params


# q heads, kv heads, head_dim, prompts, requests, new tokens of each, context before them; us whole and cut
@pytest.mark.parametrize("Hq,Hkv,d,lens,counts,m,ctx", [
    (40, 40, 128, [57, 201, 57, 57, 57], [15, 1, 1, 1, 1], 9, 0),              # 47.0, 22.1
    (40, 40, 128, [530, 65, 65, 65, 65, 65], [16, 1, 1, 1, 1, 1], 9, 0),       # 59.7, 26.8
    (16, 16, 64, [7540, 1254, 1254], [22, 1, 1], 113, 0),                      # 194, 159
    (40, 40, 128, [6150, 518, 518, 518], [15, 1, 1, 1], 84, 2499),             # 577, 451
])
def test_prompt_phase_of_one_large_application_and_some_small_ones(Hq, Hkv, d, lens, counts, m, ctx):
    B = sum(counts)
    p = _params(B, Hq, Hkv, max(lens), ctx + m, d=d, num_blocks=B * ((ctx + m) * 11 // 160 + 1))
    launches = rec.prefill_multi(p, lens, counts, [c * m for c in counts], m)
    assert [x["launch"] for x in launches] == ["rows", "fuse"] and launches[0]["whole"] == 0
    # (the workspace is sized without the groups and serves the same requests in even ones as well)
    even = [B // len(lens) + (1 if i < B % len(lens) else 0) for i in range(len(lens))]
    rec.prefill_multi(p, lens, even, [c * m for c in even], m)


@pytest.mark.parametrize("B,Hq,Hkv,d,s,bound,blocks", [
    (4, 8, 8, 128, 323, 250, 49),
    (12, 32, 8, 64, 300, 100, 120),
    (48, 28, 4, 128, 1200, 700, 1500),
])
@pytest.mark.parametrize("unused", [[16000] * 3, [0] * 20])
def test_prompts_that_no_request_of_the_step_uses(B, Hq, Hkv, d, s, bound, blocks, unused):
    p = _params(B, Hq, Hkv, s, bound, d=d, num_blocks=blocks)
    half = [B // 2, B - B // 2]
    want = rec.decode_grouped(p, [s, s // 2], half)
    assert rec.decode_grouped(p, [s, s // 2] + unused, half + [0] * len(unused)) == want
