"""Context wavefronts next to a system workgroup that take a span in some of their four only: the spans the
header's rule gives cover the tiles once, within the slots; on the GPU against the oracle."""
import numpy as np
import pytest

import oracle
import paper_2402_14808_amd as ra
import workloads as W
from gpu_util import DeviceCase
from test_decode_plan import _check_cover, _params, spans


# batch, heads, prompt, bound, contexts, and the q they give
CASES = [
    (12, 40, 16326, 800, (50, 145), 1),
    (32, 52, 16384, 127, (127, 127), 1),
    (16, 40, 16326, 800, (150, 250), 3),
    (8, 52, 9000, 300, (1, 40), 0),
]


@pytest.mark.parametrize("B,H,s,bound,ctx,want", CASES)
def test_spans_cover_every_item_within_its_slots(B, H, s, bound, ctx, want):
    plan = ra.relay_attn_decode_plan(_params(B, H, H, s, bound))
    if plan.compute_units != 256:
        pytest.skip("light wavefronts exist on 256 compute units only")
    lens = np.random.default_rng(B).integers(ctx[0], ctx[1] + 1, B)
    _, q, dropped = spans(plan, int(np.maximum(1, (lens + 31) // 32).sum()) * H, 16)
    assert q == want and not dropped
    _check_cover(plan, lens, H, 16)


@pytest.mark.gpu
@pytest.mark.parametrize("B,H,s,bound,ctx,want", [c for c in CASES if c[2] != 16384])
def test_decode_matches_oracle(B, H, s, bound, ctx, want):
    cfg = W.AttnConfig(name="ls", batch=B, num_q_heads=H, num_kv_heads=H, head_dim=128, sys_len=s, ctx_lo=ctx[0],
                       ctx_hi=ctx[1], block_size=16)
    case = W.make_case(cfg, 40 + B)
    pad = np.full((B, bound // 16 + 1 - case.block_tables.shape[1]), W.POISON_BLOCK, np.int32)
    case.block_tables = np.ascontiguousarray(np.concatenate([case.block_tables, pad], 1))
    print("[case] %s" % cfg, flush=True)
    rows = np.array([(t, h) for t in range(B) for h in (0, H // 2, H - 1)])
    want_o, want_l, _ = oracle.decode_attention(case.q, case.k_sys, case.v_sys, case.k_cache, case.v_cache,
                                                case.block_tables, case.context_lens, case.scale, rows=rows)
    dc = DeviceCase(case)
    got, lse = dc.decode(max_context_len=bound)
    _, q, _ = spans(dc.last_plan, int(np.maximum(1, (case.context_lens + 31) // 32).sum()) * H, 16)
    assert dc.last_plan.compute_units != 256 or (dc.last_plan.num_light_ctx_wavefronts > 0 and q == want)
    r = (rows[:, 0], rows[:, 1])
    assert np.isfinite(got).all() and np.abs(got[r] - want_o).max() <= 2e-3 and np.abs(lse[r] - want_l).max() <= 1e-3


# batch, q heads, kv heads, head_dim, prompt, bound, contexts
LARGER = [
    (58, 16, 4, 64, 101, 438, (200, 400)),       # spans of one item on both sides of the gap
    (17, 64, 16, 128, 117, 378, (180, 378)),
    (60, 8, 4, 64, 1000, 40000, (0, 400)),       # all work in front of the gap
]

# contexts whose items run from heavy wavefronts into light ones, out of them, or through all of them, and q
ACROSS = [
    (32, 4, 19422, 33674, [28, 30846], 1),
    (32, 4, 15810, 8167, [28, 18, 7112, 13, 7], 1),
    (32, 8, 18073, 10567, [9016, 32], 2),
    (64, 8, 19480, 22586, [13103], 3),
    (64, 8, 15593, 18944, [16444], 4),
    (32, 8, 756, 30778, [28363], None),          # an even share
]


def _larger_case(B, Hq, Hkv, d, s, bound, ctx):
    cfg = W.AttnConfig(name="lo", batch=B, num_q_heads=Hq, num_kv_heads=Hkv, head_dim=d, sys_len=s, ctx_lo=ctx[0],
                       ctx_hi=ctx[1], block_size=16)
    return W.make_case(cfg, 90 + d)


@pytest.mark.parametrize("B,Hq,Hkv,d,s,bound,ctx", LARGER)
def test_larger_launches_leave_the_light_ones_out(B, Hq, Hkv, d, s, bound, ctx):
    plan = ra.relay_attn_decode_plan(_params(B, Hq, Hkv, s, bound, d=d))
    if plan.compute_units != 256:
        pytest.skip("light wavefronts exist on 256 compute units only")
    lens = _larger_case(B, Hq, Hkv, d, s, bound, ctx).context_lens
    n_tiles = int(np.maximum(1, (lens + 31) // 32).sum()) * Hkv
    length, q, _ = spans(plan, n_tiles, 16)
    assert q == "spare" and (sum(length[:plan.first_light_ctx_wavefront]) < n_tiles) == (bound < 1000)
    _check_cover(plan, lens, Hkv, 16)


@pytest.mark.parametrize("Hq,Hkv,s,bound,lens,want", ACROSS)
def test_contexts_across_both_classes_are_covered(Hq, Hkv, s, bound, lens, want):
    plan = ra.relay_attn_decode_plan(_params(len(lens), Hq, Hkv, s, bound, d=64))
    if plan.compute_units != 256:
        pytest.skip("light wavefronts exist on 256 compute units only")
    tiles = np.maximum(1, (np.array(lens) + 31) // 32)
    length, q, dropped = spans(plan, int(tiles.sum()) * Hkv, 16)
    assert q == want and not dropped
    at = np.concatenate([[0], np.cumsum(length)])
    inner = {at[plan.first_light_ctx_wavefront], at[plan.first_light_ctx_wavefront + plan.num_light_ctx_wavefronts]}
    assert inner - set(np.cumsum(np.repeat(tiles, Hkv)))               # a border inside an item
    _check_cover(plan, np.array(lens), Hkv, 16)


def _decode_matches_oracle(case, bound):
    columns = -(-bound // case.cfg.block_size) - case.block_tables.shape[1]
    pad = np.full((case.cfg.batch, columns), W.POISON_BLOCK, np.int32)
    case.block_tables = np.ascontiguousarray(np.concatenate([case.block_tables, pad], 1))
    print("[case] %s" % case.cfg, flush=True)
    want_o, want_l, _ = oracle.decode_attention(case.q, case.k_sys, case.v_sys, case.k_cache, case.v_cache,
                                                case.block_tables, case.context_lens, case.scale)
    dc = DeviceCase(case)
    got, lse = dc.decode(max_context_len=bound, num_blocks=1 << 20)          # the plan that the replay above checks
    assert dc.last_plan.compute_units != 256 or dc.last_plan.num_light_ctx_wavefronts > 0
    assert np.isfinite(got).all() and np.abs(got - want_o).max() <= 2e-3 and np.abs(lse - want_l).max() <= 1e-3


@pytest.mark.gpu
@pytest.mark.parametrize("B,Hq,Hkv,d,s,bound,ctx", LARGER)
def test_larger_launches_match_oracle(B, Hq, Hkv, d, s, bound, ctx):
    _decode_matches_oracle(_larger_case(B, Hq, Hkv, d, s, bound, ctx), bound)


@pytest.mark.gpu
@pytest.mark.parametrize("Hq,Hkv,s,bound,lens,want", ACROSS)
def test_contexts_across_both_classes_match_oracle(Hq, Hkv, s, bound, lens, want):
    cfg = W.AttnConfig(name="lc", batch=len(lens), num_q_heads=Hq, num_kv_heads=Hkv, head_dim=64, sys_len=s,
                       ctx_lo=max(lens), ctx_hi=max(lens), block_size=16)
    case = W.make_case(cfg, 80 + s)
    case.context_lens[:] = lens
    _decode_matches_oracle(case, bound)
