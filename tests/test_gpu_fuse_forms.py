"""The forms of the fusion: one thread group per row or a workgroup per row, payloads with the log-sum-exps or
after them, one shared prompt or several of unequal length; rows that end in any of a round's batches."""
import numpy as np
import pytest
import torch

import oracle
import launch_record as rec
import paper_2402_14808_amd as ra
import workloads as W
from gpu_util import DeviceCase, _bf16
from test_decode_plan import _params

pytestmark = pytest.mark.gpu
TOL = 2e-3         # as in the other parity tests: fp32 output, error about 1e-6
LSE_TOL = 1e-3


def _pad_tables(case, bound):
    columns = bound // case.cfg.block_size - case.block_tables.shape[1]
    pad = np.full((case.cfg.batch, columns), W.POISON_BLOCK, np.int32)
    case.block_tables = np.ascontiguousarray(np.concatenate([case.block_tables, pad], 1))


def _lens(case, lens):
    """Other context lengths than the ones drawn, the first `lens` of them; none longer than its own."""
    case.context_lens[:len(lens)] = np.minimum(case.context_lens[:len(lens)], lens)


# batch, q heads, kv heads, head_dim, longest context, bound; prompts (one or several); late payloads?
DECODE = [
    (20, 2, 2, 128, 700, 1024, (300, 0, 1500), False),
    (20, 2, 1, 64, 3000, 8192, (300, 0, 1500), False),
    (64, 32, 8, 128, 300, 16384, (500,), True),              # a workgroup per row
    (64, 32, 8, 128, 3000, 16384, (600, 40, 1200), True),
    (96, 20, 4, 64, 3000, 16384, (600, 0, 1200), True),
    (225, 32, 8, 128, 70, 2048, (400,), True),               # a thread group per row
    (225, 56, 8, 64, 70, 2048, (200, 0, 400), True),
]


@pytest.mark.parametrize("B,Hq,Hkv,d,longest,bound,prompts,late", DECODE)
def test_decode(B, Hq, Hkv, d, longest, bound, prompts, late):
    cfg = W.AttnConfig(name="ff", batch=B, num_q_heads=Hq, num_kv_heads=Hkv, head_dim=d, sys_len=max(prompts),
                       ctx_lo=1, ctx_hi=longest, block_size=16)
    case = W.make_case(cfg, 500 + B + d)
    _lens(case, [1, 31, 32, 33, longest // 2])
    _pad_tables(case, bound)
    sizes = [B // len(prompts)] * (len(prompts) - 1)
    sizes.append(B - sum(sizes))
    groups = W.make_prefix_groups(case, 900 + B, tuple(sizes), prompts) if len(prompts) > 1 else \
        [(0, B, case.k_sys, case.v_sys)]
    p = _params(B, Hq, Hkv, max(prompts), bound, d=d, num_blocks=case.k_cache.shape[0])       # as the call below
    fuse = (rec.decode_multi(p, prompts, sizes) if len(prompts) > 1 else rec.decode(p))[-1]
    print("[case] %s prompts %s %s" % (cfg, prompts, fuse), flush=True)
    if ra.relay_attn_decode_plan(p).compute_units == 256:
        assert rec.late_payloads(fuse, d) == late
    dc = DeviceCase(case)
    out, lse = dc._outputs(True)
    device = [(_bf16(k, dc.dev) if len(k) else None, _bf16(v, dc.dev) if len(v) else None, at, m) for at, m, k, v in groups]
    p = ra.make_params(dc.q, out, max((g[0] for g in device if g[0] is not None), key=len), dc.k_cache, dc.block_tables,
                       batch=B, softmax_scale=case.scale, max_context_len=bound)
    ws = dc._workspace(p, B)
    if len(prompts) > 1:
        ra.relay_attn_decode_multi(p, device, dc.q, dc.k_cache, dc.v_cache, dc.block_tables, dc.context_lens, out, lse, ws)
    else:
        ra.relay_attn_decode(p, dc.q, device[0][0], device[0][1], dc.k_cache, dc.v_cache, dc.block_tables,
                             dc.context_lens, out, lse, ws)
    torch.cuda.synchronize()
    got, got_lse = out.cpu().numpy(), lse.cpu().numpy()
    assert np.isfinite(got).all()
    for at, m, k, v in groups:
        sl = slice(at, at + m)
        some = sorted({0, 1, 2, 3, 4, m // 2, m - 1})
        rows_of = np.array([(t, h) for t in some for h in sorted({0, Hq // 2, Hq - 1})])
        want, wlse, _ = oracle.decode_attention(case.q[sl], k, v, case.k_cache, case.v_cache, case.block_tables[sl],
                                                case.context_lens[sl], case.scale, rows=rows_of)
        r = (rows_of[:, 0] + at, rows_of[:, 1])
        assert np.abs(got[r] - want).max() <= TOL and np.abs(got_lse[r] - wlse).max() <= LSE_TOL


@pytest.mark.parametrize("B,Hq,Hkv,d,s,q,ctx,bound", [
    (6, 16, 4, 128, 2000, (40, 60), (0, 3000), 32768),       # one thread group per row, 8 parts or more
    (40, 32, 8, 64, 600, (4, 9), (100, 1500), 65536),
])
def test_prompt_phase(B, Hq, Hkv, d, s, q, ctx, bound):
    cfg = W.AttnConfig(name="fp", batch=B, num_q_heads=Hq, num_kv_heads=Hkv, head_dim=d, sys_len=s, ctx_lo=ctx[0],
                       ctx_hi=ctx[1], block_size=16, q_lo=q[0], q_hi=q[1])
    case = W.make_case(cfg, 800 + B, prefill=True, extra_context=True)
    _pad_tables(case, bound)
    total = int(case.cu_seqlens_q[-1])
    print("[case] %s tokens %d" % (cfg, total), flush=True)
    rows = np.array([(t, h) for t in sorted({0, 1, total // 3, total // 2, total - 2, total - 1}) for h in (0, Hq - 1)])
    want, wlse, _ = oracle.prefill_attention(case.q, case.cu_seqlens_q, case.k_sys, case.v_sys, case.k_cache, case.v_cache,
                                             case.block_tables, case.context_lens, case.scale, rows=rows)
    dc = DeviceCase(case)
    got, lse = dc.prefill(max_context_len=bound, ctx_part_tokens=4096)
    untouched = bool((dc.last_workspace == 0xFF).all())     # (a comparison inside the assertion would be unpacked)
    assert not untouched, "partials in the workspace were expected"
    r = (rows[:, 0], rows[:, 1])
    assert np.isfinite(got).all() and np.abs(got[r] - want).max() <= TOL and np.abs(lse[r] - wlse).max() <= LSE_TOL
