"""The one-launch form of a small decode step, and the two-launch form at the same sizes (which the measurement entry
point with its phases one by one always takes): both against the oracle."""
import re

import numpy as np
import pytest
import torch

import oracle
import paper_2402_14808_amd as ra
import workloads as W
from gpu_util import DeviceCase
from test_codegen import _device_asm

TOL, LSE_TOL = 2e-3, 1e-3          # as in the other parity tests: fp32 output, error about 1e-6

# 16 wavefronts of 16 (head_dim 128) or 32 (head_dim 64) rows a batch: sizes around one batch, one round of
# 256 / 512 rows and two; the border of prompt and context inside a batch; nothing on one side or on both.
SIZES = [
    (1, 4, 1, 128, 512, (90, 90), 16), (2, 8, 1, 128, 0, (15, 17), 16), (3, 3, 3, 64, 31, (0, 2), 1),
    (2, 7, 1, 64, 480, (31, 34), 32), (2, 2, 2, 128, 255, (1, 1), 8), (2, 2, 2, 128, 256, (0, 1), 2),
    (1, 6, 2, 64, 1000, (25, 25), 128), (5, 5, 5, 64, 1, (0, 0), 16), (2, 4, 4, 128, 0, (0, 0), 16),
    (4, 4, 2, 128, 100, (500, 700), 4),
]


def _case(B, Hq, Hkv, d, s, ctx, bs, seed=800):
    cfg = W.AttnConfig(name="dd", batch=B, num_q_heads=Hq, num_kv_heads=Hkv, head_dim=d, sys_len=s, ctx_lo=ctx[0],
                       ctx_hi=ctx[1], block_size=bs)
    print("[case] %s" % (cfg,), flush=True)
    return W.make_case(cfg, seed + B)


def _decode(dc, fp32_out=True, max_context_len=None, phases=None):
    """(out, lse, whether the workspace was left alone)"""
    c = dc.case
    out, lse = dc._outputs(fp32_out)
    bound = int(c.context_lens.max()) if max_context_len is None else max_context_len
    p = ra.make_params(dc.q, out, dc.k_sys, dc.k_cache, dc.block_tables, batch=c.cfg.batch, softmax_scale=c.scale,
                       max_context_len=bound)
    ws = dc._workspace(p, c.cfg.batch)
    args = (dc.q, dc.k_sys, dc.v_sys, dc.k_cache, dc.v_cache, dc.block_tables, dc.context_lens, out, lse, ws)
    if phases is None:
        ra.relay_attn_decode(p, *args)
    else:
        for phase in phases:
            ra.relay_attn_debug_decode_phases(p, phase, *args)
    torch.cuda.synchronize()
    return out.float().cpu().numpy(), lse.cpu().numpy(), bool((ws == 0xFF).all())


def _check(got, lse, want, wlse):
    assert np.isfinite(got).all() and np.abs(got - want).max() <= TOL
    some = np.isfinite(wlse)
    assert (np.isfinite(lse) == some).all() and (not some.any() or np.abs(lse[some] - wlse[some]).max() <= LSE_TOL)


@pytest.mark.gpu
@pytest.mark.parametrize("B,Hq,Hkv,d,s,ctx,bs", SIZES)
def test_small_steps_in_one_launch_and_in_two(B, Hq, Hkv, d, s, ctx, bs):
    case = _case(B, Hq, Hkv, d, s, ctx, bs)
    want, wlse, _ = oracle.decode_attention(case.q, case.k_sys, case.v_sys, case.k_cache, case.v_cache, case.block_tables,
                                            case.context_lens, case.scale)
    dc = DeviceCase(case, sys_layout="padded")
    got, lse, untouched = _decode(dc)
    assert untouched, "the one-launch form was expected (workspace untouched)"
    _check(got, lse, want, wlse)
    b16, _, _ = _decode(dc, fp32_out=False)
    assert np.array_equal(W.bf16_round(got), b16)
    got, lse, untouched = _decode(dc, phases=(1, 2))
    assert not untouched
    _check(got, lse, want, wlse)


@pytest.mark.gpu
@pytest.mark.parametrize("B,Hq,Hkv,d,s,ctx,bs", [c for c in SIZES if c[5][0] > 0])
@pytest.mark.parametrize("chunk", [0, 128])               # a hand-set chunk keeps the two-launch form
def test_append_in_both_forms(B, Hq, Hkv, d, s, ctx, bs, chunk):
    case = _case(B, Hq, Hkv, d, s, ctx, bs, 820)
    rng = np.random.Generator(np.random.PCG64(821 + B))
    k_new, v_new = (W.bf16_round(rng.standard_normal((B, Hkv, d), dtype=np.float32)) for _ in range(2))
    want_k, want_v = oracle.cache_append(case.k_cache, case.v_cache, case.block_tables, case.context_lens, k_new, v_new)
    want, wlse, _ = oracle.decode_attention(case.q, case.k_sys, case.v_sys, want_k, want_v, case.block_tables,
                                            case.context_lens, case.scale)
    dc = DeviceCase(case)
    out, lse = dc._outputs(True)
    p = ra.make_params(dc.q, out, dc.k_sys, dc.k_cache, dc.block_tables, batch=B, softmax_scale=case.scale,
                       max_context_len=int(case.context_lens.max()), sys_chunk_tokens=chunk)
    ws = dc._workspace(p, B)
    kd, vd = (torch.from_numpy(x).to(dc.dev).to(torch.bfloat16) for x in (k_new, v_new))
    ra.relay_attn_decode_append(p, dc.q, kd, vd, dc.k_sys, dc.v_sys, dc.k_cache, dc.v_cache, dc.block_tables,
                                dc.context_lens, out, lse, ws)
    torch.cuda.synchronize()
    untouched = bool((ws == 0xFF).all())
    assert untouched == (chunk == 0)
    _check(out.cpu().numpy(), lse.cpu().numpy(), want, wlse)
    got_k, got_v = dc.k_cache.float().cpu().numpy(), dc.v_cache.float().cpu().numpy()
    assert np.array_equal(got_k, want_k, equal_nan=True) and np.array_equal(got_v, want_v, equal_nan=True)


@pytest.mark.gpu
@pytest.mark.parametrize("lens", [(300, 70, 0), (0, 0, 513)])
@pytest.mark.parametrize("chunk", [0, 64])
@pytest.mark.parametrize("d,Hq,Hkv", [(128, 6, 2), (64, 4, 4)])
def test_several_prompts_in_both_forms(lens, chunk, d, Hq, Hkv):
    case = _case(7, Hq, Hkv, d, 0, (0, 40), 16, 840)
    sys_id = [2, 0, 1, 1, 0, 2, 0]
    rng = np.random.Generator(np.random.PCG64(841))
    apps = [tuple(W.bf16_round(rng.standard_normal((n, Hkv, d), dtype=np.float32)) for _ in range(2)) for n in lens]
    order, counts = ra.relay_attn_group_requests(sys_id, 3)
    dc = DeviceCase(case)
    dev = [tuple(torch.from_numpy(x).to(dc.dev).to(torch.bfloat16) if len(x) else None for x in kv) for kv in apps]
    out, lse = dc._outputs(True)
    p = ra.make_params(dc.q, out, dev[int(np.argmax(lens))][0], dc.k_cache, dc.block_tables, batch=7,
                       softmax_scale=case.scale, max_context_len=int(case.context_lens.max()), sys_chunk_tokens=chunk)
    ws = dc._workspace(p, 7)
    ids, runs = (torch.tensor(x, dtype=torch.int32, device=dc.dev) for x in (sys_id, order))
    ra.relay_attn_decode_grouped(p, [(k, v, n) for (k, v), n in zip(dev, counts)], ids, runs, dc.q, dc.k_cache, dc.v_cache,
                                 dc.block_tables, dc.context_lens, out, lse, ws)
    torch.cuda.synchronize()
    untouched = bool((ws == 0xFF).all())
    assert untouched == (chunk == 0)
    got, glse = out.cpu().numpy(), lse.cpu().numpy()
    for app, (k, v) in enumerate(apps):
        idx = np.array([i for i, a in enumerate(sys_id) if a == app])
        want, wlse, _ = oracle.decode_attention(case.q[idx], k, v, case.k_cache, case.v_cache, case.block_tables[idx],
                                                case.context_lens[idx], case.scale)
        _check(got[idx], glse[idx], want, wlse)


@pytest.mark.gpu
def test_large_steps_stay_two_launches():
    """By the bound alone: contexts that may be long keep the form that spreads a context over the machine."""
    case = _case(2, 4, 1, 128, 300, (40, 60), 16)
    pad = np.full((2, 1024), W.POISON_BLOCK, np.int32)
    case.block_tables = np.ascontiguousarray(np.concatenate([case.block_tables, pad], 1))
    dc = DeviceCase(case)
    dc.k_cache = torch.cat([dc.k_cache, torch.zeros(1024, *dc.k_cache.shape[1:], dtype=torch.bfloat16, device=dc.dev)])
    dc.v_cache = torch.cat([dc.v_cache, torch.zeros_like(dc.k_cache[:1024])])
    untouched = _decode(dc, max_context_len=0)[2]
    assert not untouched, "the two-launch form was expected (partials in the workspace)"


def test_no_scratch_memory():
    text = _device_asm("decode_direct")
    assert set(re.findall(r"\.vgpr_spill_count:\s*(\d+)", text)) == {"0"}
    assert set(re.findall(r"\.private_segment_fixed_size:\s*(\d+)", text)) == {"0"}
