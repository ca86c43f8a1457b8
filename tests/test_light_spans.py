"""Context wavefronts next to a system workgroup that take a span in some of their four only: the spans the
header's rule gives cover the tiles once, within the slots; on the GPU against the oracle."""
import bisect

import numpy as np
import pytest

import oracle
import paper_2402_14808_amd as ra
import workloads as W
from gpu_util import DeviceCase
from test_decode_plan import _params


def _spans(plan, n_tiles):
    """(first tile, tiles) per wavefront that takes any, in order; and q."""
    w, floor = plan.num_ctx_wavefronts, plan.min_tiles_per_ctx_wavefront
    lb, nl = plan.first_light_ctx_wavefront, plan.num_light_ctx_wavefronts
    heavy = (w - nl) // 4
    light_l = max(0, (plan.sys_tiles_total + n_tiles) // 256 - plan.sys_workgroup_tiles)
    assert nl and light_l // 4 < floor
    step = floor * (nl // 4)
    fullest = {q: max(plan.sys_workgroup_tiles + q * floor, 2 * ((n_tiles - q * step) // heavy))
               for q in range(5) if q * step <= n_tiles}
    q = min(fullest, key=lambda k: (fullest[k], k))
    rest = n_tiles - q * step
    per = rest // heavy
    extra = rest - per * heavy if per // 4 >= floor else 0

    def length(i):                              # of heavy wavefront i
        if per // 4 < floor:
            return floor
        t = per + (1 if i // 4 < extra else 0)
        return t // 4 + (1 if i % 4 < t % 4 else 0)
    spans, at = [], 0
    for i in range(w):
        inside = lb <= i < lb + nl
        n = (floor if (i - lb) % 4 < q else 0) if inside else length(i if i < lb else i - nl)
        if n:
            spans.append((at, n))
            at += n
    assert at >= n_tiles
    return spans, q


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
    tiles = np.repeat(np.maximum(1, (lens + 31) // 32), H)
    spans, q = _spans(plan, int(tiles.sum()))
    assert q == want
    begins, ends = [b for b, _ in spans], np.cumsum(tiles)
    for first, last in zip(ends - tiles, ends - 1):
        assert bisect.bisect_right(begins, last) - bisect.bisect_right(begins, first) + 1 <= plan.num_ctx_slots


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
    got, lse = DeviceCase(case).decode(max_context_len=bound)
    r = (rows[:, 0], rows[:, 1])
    assert np.isfinite(got).all() and np.abs(got[r] - want_o).max() <= 2e-3 and np.abs(lse[r] - want_l).max() <= 1e-3
