"""Decode plans where the cache holds fewer positions than the bound allows, and where contexts are short: the slots
serve every length up to the bound, and the results are the oracle's for lengths and workspaces on either side."""
import numpy as np
import pytest
import torch

import oracle
import paper_2402_14808_amd as ra
import workloads as W
import launch_record as rec
from gpu_util import DeviceCase, _bf16
from test_decode_plan import _check_cover, _params

TOL, LSE_TOL = 2e-3, 1e-3          # as in the other parity tests: fp32 output, error about 1e-6

# batch, q heads, kv heads, head_dim, prompt, contexts, bound
CASES = [
    (7, 32, 32, 128, 5429, (5, 17), 17),         # fewer tiles a wavefront than a system workgroup has turns
    (18, 32, 32, 128, 1008, (3, 21), 1500),      # the bound's tiles are not there
    (40, 28, 4, 128, 1400, (37, 310), 960),      # many rows, contexts of several tiles: by the bound
    (60, 28, 4, 128, 700, (2, 18), 640),         # many rows, short contexts
    (50, 40, 40, 128, 1792, (9, 56), 56),        # equal spans instead of light and heavy ones
    (12, 8, 8, 64, 813, (8, 76), 900),           # spans of one tile
    (10, 8, 8, 128, 641, (287, 1540), 1664),     # longer contexts: the bound's floor
]


@pytest.mark.parametrize("B,Hq,Hkv,d,s,ctx,bound", CASES)
@pytest.mark.parametrize("blocks", [0, 1, 7, 100, 5000, 1 << 20])
def test_slots_serve_the_bound(B, Hq, Hkv, d, s, ctx, bound, blocks):
    p = _params(B, Hq, Hkv, s, bound, d=d, num_blocks=blocks * B if blocks < 5000 else blocks)
    plan, t_max = ra.relay_attn_decode_plan(p), -(-bound // 32)
    assert (plan.num_ctx_slots - 1) * plan.min_tiles_per_ctx_wavefront >= t_max
    assert (plan.num_sys_chunks + plan.num_ctx_slots) * B * Hq * (d + 1) * 4 <= ra.relay_attn_workspace_bytes(p, B)
    # longest contexts everywhere: no wavefront has more blocks than its table holds
    span = max(plan.min_tiles_per_ctx_wavefront, -(-B * Hkv * t_max // plan.num_ctx_wavefronts))
    if plan.num_light_ctx_wavefronts == 0:
        assert span * 32 // 16 + 1 <= plan.max_blocks_per_span
    rng = np.random.default_rng(B + blocks)
    for lens in (np.full(B, bound), rng.integers(0, bound, B, endpoint=True), rng.integers(0, ctx[1], B, endpoint=True)):
        _check_cover(plan, lens, Hkv, 16)


# plans for a full cache that are larger than the workspace for one with room to spare
@pytest.mark.parametrize("B,Hq,Hkv,d,s,bound,blocks", [
    (38, 28, 4, 128, 3988, 300, 38), (46, 40, 40, 128, 2575, 300, 46), (25, 4, 4, 64, 3412, 1000, 50),
])
def test_workspaces_serve_caches_of_another_size(B, Hq, Hkv, d, s, bound, blocks):
    small, large = (_params(B, Hq, Hkv, s, bound, d=d, num_blocks=n) for n in (blocks, 1 << 20))
    sizes = rec.workspace_bytes(small), rec.workspace_bytes(large)
    assert sizes[0] > sizes[1]
    for p in (small, large):
        for size in sizes:
            launches = rec.decode(p, workspace=size)
            partials = (launches[-1]["partials"]) * B * Hq * (d + 1) * 4
            assert partials <= size and (launches[0]["slots"] - 1) * launches[0]["floor"] >= -(-bound // 32)


# (a workspace is sized without the grouping)
FALL_BACK = [
    (8, 8, 128, (2037, 1323), (9, 9), 300, 720),
    (8, 8, 128, (852, 3715, 3132), (11, 9, 6), 5000, 1040),
    (40, 40, 128, (1207, 3991), (2, 4), 300, 48),
]


@pytest.mark.parametrize("Hq,Hkv,d,lens,counts,bound,blocks", FALL_BACK)
def test_grouped_plans_that_outgrow_the_workspace_are_planned_within_it(Hq, Hkv, d, lens, counts, bound, blocks):
    B = sum(counts)
    p = _params(B, Hq, Hkv, max(lens), bound, d=d, num_blocks=blocks)
    size = rec.workspace_bytes(p)
    within, beyond = rec.decode_grouped(p, lens, counts), rec.decode_grouped(p, lens, counts, workspace=1 << 34)
    taken = [x[-1]["partials"] * B * Hq * (d + 1) * 4 for x in (within, beyond)]
    assert taken[0] <= size < taken[1]
    # still the plan that counts the groups' workgroups: a row tile for each prefix
    assert within[0]["sys_items"] == sum(Hkv * -(-n // 32) * -(-s // within[0]["chunk"]) for s, n in
                                         zip(lens, [c * Hq // Hkv for c in counts]))


@pytest.mark.gpu
@pytest.mark.parametrize("B,Hq,Hkv,d,s,ctx,bound", CASES)
@pytest.mark.parametrize("held", ["batch", "large", "sized for large"])
def test_results(B, Hq, Hkv, d, s, ctx, bound, held):
    cfg = W.AttnConfig(name="hb", batch=B, num_q_heads=Hq, num_kv_heads=Hkv, head_dim=d, sys_len=s, ctx_lo=ctx[0],
                       ctx_hi=ctx[1], block_size=16)
    case = W.make_case(cfg, 700 + B)
    pad = np.full((B, max(0, -(-bound // 16) - case.block_tables.shape[1])), W.POISON_BLOCK, np.int32)
    case.block_tables = np.ascontiguousarray(np.concatenate([case.block_tables, pad], 1))
    print("[case] %s bound %d held %s" % (cfg, bound, held), flush=True)
    rows = np.array([(t, h) for t in {0, B // 2, B - 1} for h in {0, Hq // 2, Hq - 1}])
    want, wlse, _ = oracle.decode_attention(case.q, case.k_sys, case.v_sys, case.k_cache, case.v_cache,
                                            case.block_tables, case.context_lens, case.scale, rows=rows)
    dc = DeviceCase(case)
    out, lse = dc._outputs(True)
    p = ra.make_params(dc.q, out, dc.k_sys, dc.k_cache, dc.block_tables, batch=B, softmax_scale=case.scale,
                       max_context_len=bound)
    small = ra.relay_attn_workspace_bytes(p, B)                 # of the cache as it is
    blocks, p.num_blocks = p.num_blocks, 1 << 20                # what a cache with room to spare would say
    nbytes = ra.relay_attn_workspace_bytes(p, B)
    if held != "large":
        p.num_blocks = blocks
    if held == "batch":
        nbytes = small
    r = (rows[:, 0], rows[:, 1])
    for size in {nbytes, small}:                                # either one serves the call
        ws = torch.full((size + 4096,), 0xFF, dtype=torch.uint8, device=dc.dev)
        out.fill_(float("nan"))
        ra.relay_attn_decode(p, dc.q, dc.k_sys, dc.v_sys, dc.k_cache, dc.v_cache, dc.block_tables, dc.context_lens,
                             out, lse, ws[:size])
        torch.cuda.synchronize()
        got, got_lse = out.cpu().numpy(), lse.cpu().numpy()
        assert np.isfinite(got).all() and np.abs(got[r] - want).max() <= TOL and np.abs(got_lse[r] - wlse).max() <= LSE_TOL
        assert bool((ws[size:] == 0xFF).all())


@pytest.mark.gpu
@pytest.mark.parametrize("Hq,Hkv,d,lens,counts,bound,blocks", FALL_BACK)
def test_grouped_plans_within_the_workspace_match_oracle(Hq, Hkv, d, lens, counts, bound, blocks):
    B, per = sum(counts), blocks // sum(counts)
    cfg = W.AttnConfig(name="gw", batch=B, num_q_heads=Hq, num_kv_heads=Hkv, head_dim=d, sys_len=0, ctx_lo=1,
                       ctx_hi=min(bound, 16 * per), block_size=16)
    case = W.make_case(cfg, 760 + B)
    pad = np.full((B, max(0, -(-bound // 16) - case.block_tables.shape[1])), W.POISON_BLOCK, np.int32)
    case.block_tables = np.ascontiguousarray(np.concatenate([case.block_tables, pad], 1))
    rng = np.random.Generator(np.random.PCG64(761))
    apps = [tuple(W.bf16_round(rng.standard_normal((n, Hkv, d), dtype=np.float32)) for _ in range(2)) for n in lens]
    sys_id = rng.permutation(np.repeat(np.arange(len(lens)), counts)).tolist()
    order, got_counts = ra.relay_attn_group_requests(sys_id, len(lens))
    print("[case] %s %s %s" % (cfg, lens, counts), flush=True)
    dc = DeviceCase(case)
    dev = [tuple(_bf16(x, dc.dev) for x in kv) for kv in apps]
    out, lse = dc._outputs(True)
    p = ra.make_params(dc.q, out, dev[int(np.argmax(lens))][0], dc.k_cache, dc.block_tables, batch=B,
                       softmax_scale=case.scale, max_context_len=bound)
    p.num_blocks = blocks
    size = ra.relay_attn_workspace_bytes(p, B)
    ws = torch.full((size + 4096,), 0xFF, dtype=torch.uint8, device=dc.dev)
    ids, runs = (torch.tensor(x, dtype=torch.int32, device=dc.dev) for x in (sys_id, order))
    ra.relay_attn_decode_grouped(p, [(k, v, n) for (k, v), n in zip(dev, got_counts)], ids, runs, dc.q, dc.k_cache, dc.v_cache,
                                 dc.block_tables, dc.context_lens, out, lse, ws[:size])
    torch.cuda.synchronize()
    got, glse = out.cpu().numpy(), lse.cpu().numpy()
    beyond = bool((ws[size:] == 0xFF).all())
    assert beyond and np.isfinite(got).all()
    for app, (k, v) in enumerate(apps):
        idx = np.array([i for i, a in enumerate(sys_id) if a == app])
        want, wlse, _ = oracle.decode_attention(case.q[idx], k, v, case.k_cache, case.v_cache, case.block_tables[idx],
                                                case.context_lens[idx], case.scale)
        assert np.abs(got[idx] - want).max() <= TOL and np.abs(glse[idx] - wlse).max() <= LSE_TOL
