"""Workspaces below the size the library asks for: one that was made for a larger batch serves a smaller one whose
size is larger, one that the fewest partials do not fit is refused, and nothing is written behind its end."""
import numpy as np
import pytest
import torch

import oracle
import paper_2402_14808_amd as ra
import workloads as W
from gpu_util import DeviceCase

pytestmark = pytest.mark.gpu
TOL = 2e-3         # as in the other parity tests: fp32 output, error about 1e-6
LSE_TOL = 1e-3
GUARD = 4096


def _workspace(dc, nbytes):
    return torch.full((nbytes + GUARD,), 0xFF, dtype=torch.uint8, device=dc.dev)


def _guard_intact(ws, nbytes):
    return bool((ws[nbytes:] == 0xFF).all())


def _pad_tables(case, bound):
    pad = np.full((case.cfg.batch, bound // 16 - case.block_tables.shape[1]), W.POISON_BLOCK, np.int32)
    case.block_tables = np.ascontiguousarray(np.concatenate([case.block_tables, pad], 1))


@pytest.mark.parametrize("d", [128, 64])
def test_decode_with_the_workspace_of_a_larger_batch(d):
    bound, large, B = 16416, 16, 15
    cfg = W.AttnConfig(name="sw", batch=B, num_q_heads=32, num_kv_heads=8, head_dim=d, sys_len=777, ctx_lo=1, ctx_hi=2000,
                       block_size=16)
    case = W.make_case(cfg, 31 + d)
    _pad_tables(case, bound)
    dc = DeviceCase(case)
    out, lse = dc._outputs(True)
    p = ra.make_params(dc.q, out, dc.k_sys, dc.k_cache, dc.block_tables, batch=large, softmax_scale=case.scale,
                       max_context_len=bound)
    held = ra.relay_attn_workspace_bytes(p, large)
    p.batch = B
    if d == 128:
        assert ra.relay_attn_workspace_bytes(p, B) > held       # the size does not only rise with the batch
    print("[case] %s workspace %d of %d" % (cfg, held, ra.relay_attn_workspace_bytes(p, B)), flush=True)
    rows = np.array([(t, h) for t in (0, 1, 7, 14) for h in (0, 13, 31)])
    want, wlse, _ = oracle.decode_attention(case.q, case.k_sys, case.v_sys, case.k_cache, case.v_cache,
                                            case.block_tables, case.context_lens, case.scale, rows=rows)
    r = (rows[:, 0], rows[:, 1])
    least = 3 * B * 32 * (d + 1) * 4                            # no cut of this call gets by with three partials
    for nbytes in (held, held // 2):
        ws = _workspace(dc, nbytes)
        out.fill_(float("nan"))
        ra.relay_attn_decode(p, dc.q, dc.k_sys, dc.v_sys, dc.k_cache, dc.v_cache, dc.block_tables, dc.context_lens,
                             out, lse, ws[:nbytes])
        torch.cuda.synchronize()
        got, got_lse = out.cpu().numpy(), lse.cpu().numpy()
        assert np.isfinite(got).all() and np.abs(got[r] - want).max() <= TOL and np.abs(got_lse[r] - wlse).max() <= LSE_TOL
        assert _guard_intact(ws, nbytes)
    ws = _workspace(dc, least)
    with pytest.raises(ra.RelayAttnError) as e:
        ra.relay_attn_decode(p, dc.q, dc.k_sys, dc.v_sys, dc.k_cache, dc.v_cache, dc.block_tables, dc.context_lens,
                             out, lse, ws[:least])
    assert e.value.status == ra.binding.RA_ERR_WORKSPACE_TOO_SMALL
    torch.cuda.synchronize()


@pytest.mark.parametrize("B,Hq,Hkv,d,s,q,ctx", [
    (3, 8, 2, 128, 1500, (20, 60), (500, 3000)),
    (2, 4, 4, 64, 3000, (3, 9), (0, 2000)),
])
def test_prompt_phase_with_room_for_the_coarsest_cut(B, Hq, Hkv, d, s, q, ctx):
    cfg = W.AttnConfig(name="sp", batch=B, num_q_heads=Hq, num_kv_heads=Hkv, head_dim=d, sys_len=s, ctx_lo=ctx[0],
                       ctx_hi=ctx[1], block_size=16, q_lo=q[0], q_hi=q[1])
    case = W.make_case(cfg, 77 + B, prefill=True, extra_context=True)
    dc = DeviceCase(case)
    out, lse = dc._outputs(True)
    total, longest = int(case.cu_seqlens_q[-1]), int(case.context_lens.max())
    p = ra.make_params(dc.q, out, dc.k_sys, dc.k_cache, dc.block_tables, batch=B, softmax_scale=case.scale,
                       max_context_len=longest)
    # chunks of 512 system positions, context parts of 4096
    partials = -(-s // 512) + -(-longest // 4096)
    nbytes = -(-partials * total * Hq * (d + 1) * 4 // 256) * 256 + 512
    print("[case] %s workspace %d of %d" % (cfg, nbytes, ra.relay_attn_workspace_bytes(p, total)), flush=True)
    assert nbytes < ra.relay_attn_workspace_bytes(p, total)
    want, wlse, _ = oracle.prefill_attention(case.q, case.cu_seqlens_q, case.k_sys, case.v_sys, case.k_cache, case.v_cache,
                                             case.block_tables, case.context_lens, case.scale)
    ws = _workspace(dc, nbytes)
    ra.relay_attn_prefill(p, dc.q, dc.cu_seqlens_q, total, int(np.diff(case.cu_seqlens_q).max()), dc.k_sys, dc.v_sys,
                          dc.k_cache, dc.v_cache, dc.block_tables, dc.context_lens, out, lse, ws[:nbytes])
    torch.cuda.synchronize()
    got, got_lse = out.cpu().numpy(), lse.cpu().numpy()
    assert np.isfinite(got).all() and np.abs(got - want).max() <= TOL and np.abs(got_lse - wlse).max() <= LSE_TOL
    assert _guard_intact(ws, nbytes)
