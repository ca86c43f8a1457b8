"""The prompt phase where the library cuts system prompt and contexts itself: launches with few blocks of
rows and long contexts, parts that no row of a block can see, wavefronts without a live row."""
import numpy as np
import pytest

import oracle
import workloads as W
from gpu_util import DeviceCase

pytestmark = pytest.mark.gpu
TOL = 2e-3         # as in the other parity tests: fp32 output, error about 1e-6
LSE_TOL = 1e-3


# bound: factor on the longest context that the call gives as its bound (parts behind the real end).
@pytest.mark.parametrize("B,Hq,Hkv,d,s,q,ctx,bs,bound", [
    (1, 2, 2, 128, 3000, (1, 1), (2500, 2500), 16, 1),       # one row per block: three idle wavefronts
    (3, 4, 1, 128, 700, (9, 40), (0, 3000), 16, 1),          # one context far shorter than the others
    (2, 8, 2, 64, 129, (31, 33), (2100, 2200), 32, 3),       # rows around one block of 128, parts behind the end
    (2, 3, 1, 64, 0, (60, 130), (2300, 4200), 16, 1),        # no system prompt, blocks across a causal edge
    (2, 2, 1, 128, 600, (5, 70), (1500, 1700), 1, 1),        # block size 1: parts of 256 positions at most
    (5, 4, 4, 64, 6000, (3, 20), (0, 10), 16, 40),           # chunks of the prompt; every part but one is empty
])
def test_cut_prompt_phase(B, Hq, Hkv, d, s, q, ctx, bs, bound):
    cfg = W.AttnConfig(name="ps", batch=B, num_q_heads=Hq, num_kv_heads=Hkv, head_dim=d, sys_len=s, ctx_lo=ctx[0],
                       ctx_hi=ctx[1], block_size=bs, q_lo=q[0], q_hi=q[1])
    case = W.make_case(cfg, 700 + B + s, prefill=True, extra_context=True)
    longest = int(case.context_lens.max()) * bound
    if bound > 1:
        pad = np.full((B, -(-longest // bs) - case.block_tables.shape[1]), W.POISON_BLOCK, np.int32)
        case.block_tables = np.ascontiguousarray(np.concatenate([case.block_tables, pad], 1))
    print("[case] %s m=%s c=%s" % (cfg, np.diff(case.cu_seqlens_q), case.context_lens), flush=True)
    want, wlse, _ = oracle.prefill_attention(case.q, case.cu_seqlens_q, case.k_sys, case.v_sys, case.k_cache, case.v_cache,
                                             case.block_tables, case.context_lens, case.scale)
    dc = DeviceCase(case, sys_layout="padded")
    got, lse = dc.prefill(max_context_len=longest)
    assert not bool((dc.last_workspace == 0xFF).all()), "the cut form was expected (partials in the workspace)"
    assert np.isfinite(got).all() and np.abs(got - want).max() <= TOL and np.abs(lse - wlse).max() <= LSE_TOL


@pytest.mark.parametrize("bound", [0, 8192, 65536])        # 0: exactly the longest context
def test_new_conversations_under_a_loose_bound_stay_one_launch(bound):
    """Contexts that are the new tokens only, a bound that is the capacity of the block table: how the launch
    is cut goes by the lengths the cache can hold, not by the bound alone."""
    cfg = W.AttnConfig(name="nc", batch=2, num_q_heads=32, num_kv_heads=8, head_dim=128, sys_len=300, ctx_lo=0, ctx_hi=0,
                       block_size=16, q_lo=300, q_hi=900)
    case = W.make_case(cfg, 750, prefill=True)
    if bound:
        pad = np.full((2, bound // 16 - case.block_tables.shape[1]), W.POISON_BLOCK, np.int32)
        case.block_tables = np.ascontiguousarray(np.concatenate([case.block_tables, pad], 1))
    total = int(case.cu_seqlens_q[-1])
    print("[case] %s tokens %d bound %d" % (cfg, total, bound), flush=True)
    rows = np.array([(t, h) for t in (0, 1, total // 2, total - 1) for h in (0, 31)])
    want, wlse, _ = oracle.prefill_attention(case.q, case.cu_seqlens_q, case.k_sys, case.v_sys, case.k_cache, case.v_cache,
                                             case.block_tables, case.context_lens, case.scale, rows=rows)
    dc = DeviceCase(case)
    got, lse = dc.prefill(max_context_len=bound or None)
    untouched = bool((dc.last_workspace == 0xFF).all())     # (a comparison inside the assertion would be unpacked)
    assert untouched, "the one-launch form was expected (workspace untouched)"
    r = (rows[:, 0], rows[:, 1])
    assert np.isfinite(got).all() and np.abs(got[r] - want).max() <= TOL and np.abs(lse[r] - wlse).max() <= LSE_TOL



def test_few_tokens_of_several_requests_in_a_block_are_cut():
    """Eight blocks of rows that would go through five requests each, one after the other, under a loose bound."""
    cfg = W.AttnConfig(name="ft", batch=5, num_q_heads=8, num_kv_heads=8, head_dim=128, sys_len=281, ctx_lo=0, ctx_hi=0,
                       block_size=16, q_lo=15, q_hi=28)
    case = W.make_case(cfg, 760, prefill=True)
    pad = np.full((5, 42 - case.block_tables.shape[1]), W.POISON_BLOCK, np.int32)
    case.block_tables = np.ascontiguousarray(np.concatenate([case.block_tables, pad], 1))
    print("[case] %s m=%s" % (cfg, np.diff(case.cu_seqlens_q)), flush=True)
    want, wlse, _ = oracle.prefill_attention(case.q, case.cu_seqlens_q, case.k_sys, case.v_sys, case.k_cache, case.v_cache,
                                             case.block_tables, case.context_lens, case.scale)
    dc = DeviceCase(case)
    got, lse = dc.prefill(max_context_len=672)
    untouched = bool((dc.last_workspace == 0xFF).all())
    assert not untouched, "the cut form was expected (partials in the workspace)"
    assert np.isfinite(got).all() and np.abs(got - want).max() <= TOL and np.abs(lse - wlse).max() <= LSE_TOL
