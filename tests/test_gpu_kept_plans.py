"""GPU calls one after the other on one thread whose plans take the same bytes but hold
other work (the plan kept from the call before must not serve the next one): each
equals, bit for bit, the same call on a thread of its own, which has kept nothing."""
import threading

import numpy as np
import pytest
import torch

import cw_workloads as cw
import paper_2606_16824_amd as cwlib
from gpu_util import bits, to_gpu

pytestmark = pytest.mark.gpu

CALLS = {
    "extend": [([900, 2000, 300], [130, 70, 200]), ([2000, 900, 300], [130, 70, 200]), ([901, 2000, 300], [130, 70, 200]),
               ([900, 2000, 300], [129, 71, 200])],
    "decode": [([900, 2000, 300], [1, 1, 1]), ([2000, 900, 300], [1, 1, 1]), ([901, 2000, 300], [1, 1, 1])],
    "step": [([900, 2000, 300], [130, 1, 200]), ([2000, 900, 300], [130, 1, 200]), ([900, 2001, 300], [130, 1, 200]),
             ([900, 2000, 300], [1, 130, 200]), ([900, 2000, 300], [129, 1, 201])],
}


def _run(kind, dw, k0, v0):
    s = dw.spec
    out = torch.full_like(dw.q, float("nan"))
    if kind == "step":  # writes the pools
        dw.k_pool.copy_(k0)
        dw.v_pool.copy_(v0)
    args = (dw.q, dw.k_new, dw.v_new, dw.k_pool, dw.v_pool, dw.block_table, s.prefix_lens)
    if kind == "decode":
        cwlib.decode_attention(*args, s.gqa_group, s.softmax_scale, out=out)
    else:
        fn = cwlib.extend_attention if kind == "extend" else cwlib.step_attention
        fn(*args, s.suffix_lens, s.gqa_group, s.softmax_scale, out=out)
    torch.cuda.synchronize()
    return bits(out)


@pytest.mark.parametrize("kind", list(CALLS))
def test_calls_of_equal_plan_size(kind):
    print(f"\n[case] kept plans {kind}", flush=True)
    cases = []
    for i, (lp, ls) in enumerate(CALLS[kind]):
        dw = to_gpu(cw.materialize(cw.custom_spec(lp, ls, num_kv_heads=2, gqa_group=4, head_dim=128, page_size=16,
                                                  kv_dtype="bf16", seed=151 + i)))
        k0, v0 = dw.k_pool.clone(), dw.v_pool.clone()
        got = []
        t = threading.Thread(target=lambda: got.append(_run(kind, dw, k0, v0)))
        t.start()
        t.join()
        cases.append((dw, k0, v0, got[0]))
    for i in list(range(len(cases))) * 2 + np.random.default_rng(157).integers(0, len(cases), 12).tolist():
        dw, k0, v0, want = cases[i]
        assert np.array_equal(_run(kind, dw, k0, v0), want), CALLS[kind][i]
