"""The form of prompt-phase calls whose two estimates lie close together: calls that were timed in both."""
import pytest

import launch_record as rec
from test_decode_plan import _params


# batch, q heads, kv heads, head_dim, prompt, bound, blocks of 16 in the cache, new tokens and the most of a request; whole?
CASES = [
    (4, 8, 8, 128, 277, 11808, 208, 2042, 917, 0),           # 67.2 us whole, 52.0 cut
    (11, 32, 8, 64, 463, 832, 1 << 21, 659, 76, 1),          # 21.7, 27.1: the cache says nothing
    (8, 28, 4, 128, 170, 192, 36, 111, 15, 0),               # 21.0, 16.5: many requests in a block
    (9, 28, 4, 128, 342, 384, 208, 386, 49, 0),              # 39.5, 26.8
]


@pytest.mark.parametrize("B,Hq,Hkv,d,s,bound,blocks,total,most,whole", CASES)
def test_form(B, Hq, Hkv, d, s, bound, blocks, total, most, whole):
    p = _params(B, Hq, Hkv, s, bound, d=d, num_blocks=blocks)
    launches = rec.prefill(p, total, most)
    assert launches[0]["whole"] == whole and len(launches) == 2 - whole
