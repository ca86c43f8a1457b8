"""The one-launch prompt phase with several prefixes starts its items with the longest prompt's where they are many: any order of the
lengths, equal and empty ones among them, gives every group its own prompt."""
import numpy as np
import pytest

import launch_record as rec
import workloads as W
from test_decode_plan import _params
from test_gpu_multi_prefix import _prefill_oracle, _run_prefill

pytestmark = pytest.mark.gpu
TOL, LSE_TOL = 2e-3, 1e-3          # as in the other parity tests: fp32 output, error about 1e-6


SHORT = [(40, 90, 200, 200), (200, 0, 90, 40), (90, 200, 0, 90), (1, 64, 65, 129)]


@pytest.mark.parametrize("lens,d,Hq,Hkv", [(lens, *heads) for lens in SHORT for heads in [(128, 4, 1), (64, 3, 3)]] +
                         [(lens, 64, 132, 132) for lens in SHORT] +            # sorted: more than 512 items
                         [((64, 4100, 200, 90), 64, 90, 90)])                  # sorted: a long prompt
def test_any_order_of_prompt_lengths(lens, d, Hq, Hkv):
    cfg = W.AttnConfig(name="po", batch=6, num_q_heads=Hq, num_kv_heads=Hkv, head_dim=d, sys_len=max(lens), ctx_lo=0,
                       ctx_hi=40, block_size=16, q_lo=33, q_hi=70)
    case = W.make_case(cfg, 770 + lens[0], prefill=True, extra_context=True)
    groups = W.make_prefix_groups(case, 771, (1, 2, 2, 1), lens)
    print("[case] %s lens %s m=%s" % (cfg, lens, np.diff(case.cu_seqlens_q)), flush=True)
    p = _params(6, Hq, Hkv, max(lens), int(case.context_lens.max()), d=d, num_blocks=case.k_cache.shape[0])
    toks = [int(case.cu_seqlens_q[at + n] - case.cu_seqlens_q[at]) for at, n in ((0, 1), (1, 2), (3, 2), (5, 1))]
    order = rec.prefill_multi(p, lens, (1, 2, 2, 1), toks, int(np.diff(case.cu_seqlens_q).max()))[0]["prompts"]
    assert order == (sorted(lens, reverse=True) if Hkv >= 90 else list(lens))
    got, lse = _run_prefill(case, groups)
    untouched = bool((_run_prefill.last_workspace == 0xFF).all())
    assert untouched, "the one-launch form was expected"
    want, wlse = _prefill_oracle(case, groups)
    assert np.isfinite(got).all() and np.abs(got - want).max() <= TOL and np.abs(lse - wlse).max() <= LSE_TOL
