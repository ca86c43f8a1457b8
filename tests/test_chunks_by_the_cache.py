"""System chunks of decode steps that are planned for what the cache holds: no shorter than the bound's where that saves no
turn of the four wavefronts, or where the launch waits for the contexts anyway."""
import pytest

import launch_record as rec
from test_decode_plan import _params


# batch, q heads, kv heads, head_dim, prompt, bound, blocks of 16 in the cache; tiles of a chunk, least slots
@pytest.mark.parametrize("B,Hq,Hkv,d,s,bound,blocks,tiles,slots", [
    (25, 40, 40, 128, 645, 80, 48, 7, 3),                # 6 take as many turns
    (6, 52, 52, 128, 768, 437, 126, 12, 6),              # 8: shorter than the spans of the contexts
    (7, 32, 32, 128, 1732, 20512, 167, 55, 66),          # 10
    (132, 28, 4, 128, 1716, 3280, 239, 54, 16),          # 27: contexts of one tile, each begun anew
    (6, 16, 16, 64, 12650, 27600, 361, 44, 80),          # 25, and no longer than the spans
    (18, 32, 32, 128, 1008, 1500, 24, 8, 40),            # 6 take as many turns
])
def test_chunk_of_a_plan_by_the_cache(B, Hq, Hkv, d, s, bound, blocks, tiles, slots):
    p = _params(B, Hq, Hkv, s, bound, d=d, num_blocks=blocks)
    launch = rec.decode(p)[0]
    assert launch["chunk"] == 32 * tiles and launch["slots"] >= slots
    assert (launch["slots"] - 1) * launch["floor"] >= -(-bound // 32)     # any length up to the bound has its slots
