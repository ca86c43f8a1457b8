"""Launches of exactly two workgroups per compute unit with short contexts: equal spans for all context wavefronts, or
light ones next to the system workgroups."""
import pytest

import launch_record as rec
from test_decode_plan import _params


# batch, q heads, kv heads, head_dim, prompts, bound, blocks of 16 in the cache; equal spans?  (us: equal, light and heavy)
@pytest.mark.parametrize("B,Hq,Hkv,d,prompts,bound,blocks,equal", [
    (76, 40, 40, 128, (3128,), 31, 150, True),           # 32.2, 48.1
    (65, 8, 8, 128, (13815,), 688, 160, True),           # 26.7, 32.7
    (58, 52, 52, 128, (215,), 672, 128, True),           # 20.8, 23.9: spans below the floor otherwise
    (122, 52, 52, 128, (190,), 128, 270, False),         # 34.9, 32.0
    (93, 52, 52, 128, (234,), 192, 144, False),          # 26.4, 24.3
    (166, 52, 52, 128, (4759,), 30, 366, False),         # 85.9, 80.7: many-rows items, the bound at the lengths
    (161, 40, 40, 128, (3558,), 304, 354, True),         # 54.1, 60.2: many-rows items by the cache
    (84, 40, 40, 128, (100, 117, 135, 153), 96, 214, False),   # 26.7, 24.1
])
def test_equal_spans_where_they_pay(B, Hq, Hkv, d, prompts, bound, blocks, equal):
    p = _params(B, Hq, Hkv, max(prompts), bound, d=d, num_blocks=blocks)
    if len(prompts) == 1:
        tiles = rec.decode(p)[0]
    else:
        tiles = rec.decode_grouped(p, prompts, [B // len(prompts)] * len(prompts))[0]
    assert tiles["sys_items"] + tiles["ctx_waves"] // 4 == 512
    assert (tiles["light"] == 0) == equal
