"""Rows whose result comes from many partials: the number of context partials of a row against the
slots its launch has room for, and the fusion of more than two batches of eight of them."""
import numpy as np
import pytest

import oracle
import workloads as W
from gpu_util import DeviceCase

pytestmark = pytest.mark.gpu
TOL = 2e-3         # as in the other parity tests: fp32 output, error about 1e-6
LSE_TOL = 1e-3


# spread: the bound on the lengths over the longest of them (1: the bound is met).
@pytest.mark.parametrize("B,Hq,Hkv,d,s,lo,hi,spread", [
    (1, 1, 1, 128, 0, 9000, 9000, 1),        # a slot per span, several rounds of 64 partials
    (1, 4, 1, 64, 40, 9000, 9000, 2),
    (2, 2, 2, 128, 300, 1, 4000, 1),         # from one partial to many in one launch
    (3, 8, 2, 64, 33, 0, 2000, 8),
    (12, 16, 4, 128, 500, 100, 3000, 1),
    (5, 4, 4, 128, 64, 31, 33, 40),          # every row leaves almost all slots unused
])
def test_rows_of_many_partials(B, Hq, Hkv, d, s, lo, hi, spread):
    cfg = W.AttnConfig(name="mp", batch=B, num_q_heads=Hq, num_kv_heads=Hkv, head_dim=d, sys_len=s,
                       ctx_lo=lo, ctx_hi=hi, block_size=16)
    case = W.make_case(cfg, 900 + B)
    bound = min(case.max_blocks * 16, int(case.context_lens.max()) * spread)
    if spread > 1:
        pad = np.full((B, case.max_blocks * (spread - 1)), 0x7FFFFFF0, case.block_tables.dtype)
        case.block_tables = np.ascontiguousarray(np.concatenate([case.block_tables, pad], 1))
        bound = case.block_tables.shape[1] * 16
    want, wlse, _ = oracle.decode_attention(case.q, case.k_sys, case.v_sys, case.k_cache, case.v_cache,
                                            case.block_tables, case.context_lens, case.scale)
    dc = DeviceCase(case)
    got, lse = dc.decode(max_context_len=bound)
    print("[case] %s slots %d chunks %d" % (cfg, dc.last_plan.num_ctx_slots, dc.last_plan.num_sys_chunks), flush=True)
    assert np.isfinite(got).all() and np.abs(got - want).max() <= TOL
    some = np.isfinite(wlse)
    assert (some == np.isfinite(lse)).all() and np.abs(lse[some] - wlse[some]).max() <= LSE_TOL
    again, _ = dc.decode(max_context_len=bound)
    assert (again == got).all()
