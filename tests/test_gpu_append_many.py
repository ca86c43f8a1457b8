"""relay_attn_cache_append over many tokens and requests: the place of every row, byte for byte."""
import numpy as np
import pytest
import torch

import paper_2402_14808_amd as ra

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,Hkv,d,bs,lo,hi", [
    (1, 1, 64, 16, 1, 1),
    (70, 1, 64, 16, 0, 40),        # more than 64 requests, some without new tokens, 16 tokens per workgroup
    (130, 5, 128, 32, 3, 30),      # 80 pieces per token: rounds that end inside a token
    (3, 40, 128, 16, 200, 700),    # 640 pieces per token
    (2, 70, 128, 1, 1, 9),         # more pieces per token than one round moves
])
@pytest.mark.parametrize("offset", [0, 37])
def test_rows_land_where_the_tables_say(B, Hkv, d, bs, lo, hi, offset):
    rng = np.random.default_rng(B * 100 + Hkv)
    m = rng.integers(lo, hi + 1, B)
    m[-1] = max(1, m[-1])
    lens = m + offset * rng.integers(0, 2, B)
    n_blocks = -(-lens // bs)
    pool = int(n_blocks.sum()) + 3
    perm, width = rng.permutation(pool), int(n_blocks.max()) + 1
    table, at = np.full((B, width), 0x7FFFFFF0, np.int32), 0
    for i, k in enumerate(n_blocks):
        table[i, :k] = perm[at:at + k]
        at += k
    cu = np.concatenate([[0], np.cumsum(m)]).astype(np.int32)
    total = int(cu[-1])
    new = [torch.randn(total, Hkv, d, device="cuda").to(torch.bfloat16) for _ in range(2)]
    cache = [torch.zeros(pool, Hkv, bs, d, device="cuda", dtype=torch.bfloat16) for _ in range(2)]
    want = [c.clone() for c in cache]
    token_req = np.repeat(np.arange(B), m)
    pos = lens[token_req] - m[token_req] + np.arange(total) - cu[token_req]
    blk, row = torch.from_numpy(table[token_req, pos // bs]).long(), torch.from_numpy(pos % bs).long()
    for w, x in zip(want, new):
        w[blk.cuda(), :, row.cuda()] = x
    q = torch.empty(total, Hkv, d, device="cuda", dtype=torch.bfloat16)
    tables = torch.from_numpy(table).cuda()
    p = ra.make_params(q, q, None, cache[0], tables, batch=B, softmax_scale=1.0)
    ra.relay_attn_cache_append(p, new[0], new[1], torch.from_numpy(cu).cuda(), total, cache[0], cache[1], tables,
                               torch.from_numpy(lens.astype(np.int32)).cuda())
    torch.cuda.synchronize()
    assert all(torch.equal(c, w) for c, w in zip(cache, want))
