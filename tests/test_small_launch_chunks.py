"""System chunks of small decode launches: multiples of four 32-position tiles where the rule asks for it."""
import numpy as np
import pytest

import oracle
import paper_2402_14808_amd as ra
import workloads as W
from gpu_util import DeviceCase
from test_decode_plan import _params

# batch, q heads, kv heads, head_dim, prompt, bound, tiles of a chunk
CASES = [
    (1, 16, 16, 64, 1625, 8140, 11),       # not one workgroup per unit either way: stays (8, a turn less, was no faster)
    (2, 32, 32, 128, 3221, 188, 16),       # 13: one workgroup per unit instead of a few more
    (12, 32, 8, 128, 6612, 46, 16),        # 13, stacked rows of a grouped model
    (88, 16, 16, 64, 787, 35, 9),          # half of the units would hold a system workgroup: stays
    (1, 4, 4, 64, 96, 64, 3),              # up to four tiles: stays
    # either side of a limit: workgroups without the rule, 256 per launch of one per unit
    (8, 32, 32, 128, 185, 201, 6),         # 256: fits as it is
    (1, 16, 16, 64, 7646, 20, 16),         # 257, 241 with a chunk of 16
    (12, 32, 8, 128, 4119, 308, 12),       # 320, a quarter more: 256
    (1, 32, 32, 128, 477, 1531, 8),        # 288: 256
    (22, 32, 8, 64, 2616, 171, 9),         # 328, more than a quarter: stays
    (1, 32, 8, 128, 6159, 1820, 7),        # 281: 257 with a chunk of 8
    # 2.5 tiles per wavefront, and a little more
    (4, 40, 40, 128, 3140, 206, 20),
    (1, 16, 16, 64, 10363, 22, 21),
]


@pytest.mark.parametrize("B,Hq,Hkv,d,s,bound,tiles", CASES)
def test_chunk_of_small_launches(B, Hq, Hkv, d, s, bound, tiles):
    p = _params(B, Hq, Hkv, s, bound, d=d)
    plan = ra.relay_attn_decode_plan(p)
    if plan.compute_units != 256:
        pytest.skip("the numbers are those of 256 compute units")
    assert plan.sys_chunk_tokens == 32 * tiles and plan.num_sys_chunks == -(-s // (32 * tiles))
    need = (plan.num_sys_chunks + plan.num_ctx_slots) * B * Hq * (d + 1) * 4
    assert ra.relay_attn_workspace_bytes(p, B) >= need


@pytest.mark.gpu
@pytest.mark.parametrize("B,Hq,Hkv,d,s,bound,tiles", CASES[:3])
def test_decode_matches_oracle(B, Hq, Hkv, d, s, bound, tiles):
    cfg = W.AttnConfig(name="sc", batch=B, num_q_heads=Hq, num_kv_heads=Hkv, head_dim=d, sys_len=s, ctx_lo=1,
                       ctx_hi=bound, block_size=16)
    case = W.make_case(cfg, 60 + B)
    print("[case] %s" % cfg, flush=True)
    want, wlse, _ = oracle.decode_attention(case.q, case.k_sys, case.v_sys, case.k_cache, case.v_cache,
                                            case.block_tables, case.context_lens, case.scale)
    pad = np.full((B, -(-bound // 16) - case.block_tables.shape[1]), W.POISON_BLOCK, np.int32)
    case.block_tables = np.ascontiguousarray(np.concatenate([case.block_tables, pad], 1))
    dc = DeviceCase(case)
    got, lse = dc.decode(max_context_len=bound, num_blocks=1 << 20)          # the plan that is checked above
    assert dc.last_plan.compute_units != 256 or dc.last_plan.sys_chunk_tokens == 32 * tiles
    assert np.isfinite(got).all() and np.abs(got - want).max() <= 2e-3 and np.abs(lse - wlse).max() <= 1e-3
