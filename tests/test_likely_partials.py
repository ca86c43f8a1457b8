"""The partials that the fusion expects of a row: those of the contexts a decode step is planned for, whatever the bound."""
import pytest

import launch_record as rec
from test_decode_plan import _params


# batch, q heads, kv heads, head_dim, prompt, bound, blocks of 16 in the cache; late payloads?
@pytest.mark.parametrize("B,Hq,Hkv,d,s,bound,blocks,late", [
    (225, 32, 8, 128, 400, 2048, 648, True),         # two tiles a context: one or two slots of seven
    (225, 56, 8, 64, 400, 2048, 648, True),
    (225, 32, 8, 128, 400, 2048, 1 << 20, True),     # contexts up to the bound: no likelier than that
    (225, 32, 8, 128, 400, 70, 1125, False),         # a bound at the lengths
    (200, 32, 32, 128, 300, 4096, 900, True),
    (20, 2, 2, 128, 1500, 1024, 1 << 20, False),     # little to load either way
])
def test_slots_that_short_contexts_leave_empty_are_not_likely(B, Hq, Hkv, d, s, bound, blocks, late):
    p = _params(B, Hq, Hkv, s, bound, d=d, num_blocks=blocks)
    tiles, fuse = rec.decode(p)
    assert (tiles["launch"], fuse["launch"]) == ("tiles", "fuse")
    held = min(-(-bound // 32), blocks // 2 / B + 0.5)                    # tiles of a context, in the mean
    assert fuse["likely"] <= tiles["sys_chunks"] + -(-held // tiles["floor"]) + 1
    assert rec.late_payloads(fuse, d) == late
