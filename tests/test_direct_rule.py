"""Which decode steps are one launch: steps whose two forms were timed, on either side of the line."""
import pytest

import launch_record as rec
from test_decode_plan import _params


# batch, q heads, kv heads, head_dim, prompt, bound, blocks of 16 in the cache; one launch?
STEPS = [
    (1, 32, 8, 128, 512, 90, 7, True),               # 6.8 us in one launch, 10.2 in two
    (16, 16, 16, 64, 1000, 255, 160, True),          # 7.8, 10.8
    (10, 8, 8, 128, 641, 1600, 634, False),          # 19.3, 14.8: long contexts
    (3, 32, 8, 128, 46, 1188, 225, False),           # 13.1, 11.2
    (4, 32, 8, 128, 372, 871, 218, False),           # 12.7, 11.4
    (4, 16, 16, 64, 369, 2496, 625, False),          # 13.7, 12.8
    (50, 16, 16, 64, 42, 31, 100, False),            # 10.6, 7.9: many workgroups
    (11, 32, 32, 128, 412, 128, 42, False),          # 11.5, 10.8
    (4, 4, 2, 128, 100, 700, 176, True),             # 8.6, 10.9
    (3, 8, 8, 128, 100, 1000, 189, False),           # 11.8, 11.0
    (8, 4, 4, 64, 100, 1000, 504, True),             # 7.3, 9.3
    (34, 4, 4, 64, 34, 2336, 4964, True),            # 15.6, 20.8: five rounds, but 81 MB
    (4, 32, 8, 128, 1024, 163, 34, True),            # 10.2, 12.0
    (4, 32, 32, 128, 488, 1072, 109, True),          # 11.1, 15.0: six rounds and more by the bound only
    (4, 8, 8, 128, 323, 784, 49, True),              # 9.1, 12.2
    # the last row of four rounds of 256 with a context of more than three, and the one behind it
    (1, 32, 32, 128, 255, 769, 49, True), (1, 32, 32, 128, 256, 769, 49, False),
    (1, 32, 32, 64, 511, 1537, 97, True), (1, 32, 32, 64, 512, 1537, 97, False),
    # and of six with one of three
    (1, 32, 32, 128, 768, 768, 48, True), (1, 32, 32, 128, 769, 768, 48, False),
]


@pytest.mark.parametrize("B,Hq,Hkv,d,s,bound,blocks,one", STEPS)
def test_line_between_one_launch_and_two(B, Hq, Hkv, d, s, bound, blocks, one):
    p = _params(B, Hq, Hkv, s, bound, d=d, num_blocks=blocks)
    assert [x["launch"] for x in rec.decode(p)] == (["direct"] if one else ["tiles", "fuse"])
    p.sys_chunk_tokens = 128
    assert [x["launch"] for x in rec.decode(p)] == ["tiles", "fuse"]
