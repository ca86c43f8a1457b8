"""Prompt-phase calls of few tokens per request, or of one long context, whose walk is short by the bound: they are cut
(partials in the workspace), where going through one request after the other in one launch took up to four times as long."""
import numpy as np
import pytest

import oracle
import workloads as W
from gpu_util import DeviceCase

pytestmark = pytest.mark.gpu
TOL, LSE_TOL = 2e-3, 1e-3          # as in the other parity tests: fp32 output, error about 1e-6


@pytest.mark.parametrize("B,Hq,Hkv,d,s,q,ctx", [
    (17, 8, 8, 128, 324, (10, 13), (77, 82)),
    (12, 4, 4, 64, 272, (3, 15), (0, 0)),
    (1, 28, 4, 128, 155, (57, 57), (1600, 1600)),
])
def test_short_walks_past_many_requests_are_cut(B, Hq, Hkv, d, s, q, ctx):
    cfg = W.AttnConfig(name="pf", batch=B, num_q_heads=Hq, num_kv_heads=Hkv, head_dim=d, sys_len=s, ctx_lo=ctx[0],
                       ctx_hi=ctx[1], block_size=16, q_lo=q[0], q_hi=q[1])
    case = W.make_case(cfg, 780 + B, prefill=True, extra_context=ctx[1] > 0)
    print("[case] %s m=%s c=%s" % (cfg, np.diff(case.cu_seqlens_q), case.context_lens), flush=True)
    want, wlse, _ = oracle.prefill_attention(case.q, case.cu_seqlens_q, case.k_sys, case.v_sys, case.k_cache, case.v_cache,
                                             case.block_tables, case.context_lens, case.scale)
    dc = DeviceCase(case, sys_layout="padded")
    got, lse = dc.prefill()
    untouched = bool((dc.last_workspace == 0xFF).all())
    assert not untouched, "the cut form was expected (partials in the workspace)"
    assert np.isfinite(got).all() and np.abs(got - want).max() <= TOL and np.abs(lse - wlse).max() <= LSE_TOL
