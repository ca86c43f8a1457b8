"""The kind of a decode step's system items where what the cache holds and the bound would choose differently."""
import pytest

import launch_record as rec
from test_decode_plan import _params


# batch, q heads, kv heads, head_dim, prompt, bound, blocks of 16 in the cache; many-rows items?  (us: many-rows, streaming)
@pytest.mark.parametrize("B,Hq,Hkv,d,s,bound,blocks,rows", [
    (135, 32, 32, 128, 5122, 688, 347, True),        # 55, 65
    (124, 32, 8, 64, 8754, 2752, 504, True),         # 33, 39
    (99, 40, 40, 128, 8655, 1760, 654, True),        # 83, 122
    (84, 32, 8, 64, 272, 128, 173, False),           # 11.7, 9.8: short chunks
    (132, 28, 4, 128, 1716, 3280, 239, False),       # 52, 36: long spans
    (173, 32, 8, 128, 1363, 3424, 480, False),       # 108, 53
    (135, 28, 4, 128, 12708, 9744, 911, False),      # 110, 81
    (132, 28, 4, 128, 1716, 26, 1 << 20, True),      # by the bound as well
])
def test_kind_of_the_system_items(B, Hq, Hkv, d, s, bound, blocks, rows):
    p = _params(B, Hq, Hkv, s, bound, d=d, num_blocks=blocks)
    tiles = rec.decode(p)[0]
    assert tiles["rows_sys"] == rows
    assert (tiles["slots"] - 1) * tiles["floor"] >= -(-bound // 32)       # any length up to the bound has its slots
