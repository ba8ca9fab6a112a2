"""GPU extend with a levelled plan: query tiles cut at key ranges of unequal length
so that all workgroups finish together.  Against the same call with whole tiles
(a target of 256 workgroups in the place of the automatic plan), whose parity the
other tests pin: the split-K merge may move a result by up to two bf16 ulps; and, for
tiles that cost the same but differ in shape, against the oracle.  The no-alloc call
and a captured call run the same plan bit for bit."""
import numpy as np
import pytest
import torch

import cw_workloads as cw
import oracle
import paper_2606_16824_amd as cwlib
from conftest import paged_inputs
from gpu_util import BF16_MAX_ABS, BF16_MEAN_ABS, as_f64, assert_close, assert_within_bf16_ulps, bits, run_extend, to_gpu

pytestmark = pytest.mark.gpu

# 33 replies of one query tile each (264 tiles on 256 CUs); replies of 12 to 600
# tokens; one kv head, every CU on the same keys
CASES = {
    "one_more_than_a_round": dict(lp=[6000 + 5 * i for i in range(33)], ls=[64 - i % 3 for i in range(33)], hkv=8, g=4,
                                  d=128, p=16, dt="bf16"),
    "replies_d64": dict(lp=[19000, 31000, 5000, 12000, 27000, 9000, 30000, 8001],
                        ls=[598, 59, 14, 66, 154, 15, 542, 402], hkv=8, g=4, d=64, p=64, dt="bf16"),
    # full tiles and longer ones of 32 rows that cost the same
    "equal_cost": dict(lp=[3632, 5120] * 33, ls=[32, 4] * 33, hkv=4, g=8, d=64, p=16, dt="bf16"),
    "mqa_fp8": dict(lp=[40000, 39990, 40010, 17, 40005], ls=[700, 699, 701, 5, 703], hkv=1, g=16, d=128, p=16, dt="fp8"),
}


@pytest.mark.parametrize("name", list(CASES))
def test_levelled_against_whole_tiles(name):
    c = CASES[name]
    spec = cw.custom_spec(c["lp"], c["ls"], num_kv_heads=c["hkv"], gqa_group=c["g"], head_dim=c["d"],
                          page_size=c["p"], kv_dtype=c["dt"], seed=83)
    print(f"\n[case] levelled {name}: {c}", flush=True)
    items = cwlib.plan_items(spec.prefix_lens, spec.suffix_lens, c["hkv"], c["g"], c["d"], c["p"])
    assert (items[:, 5] >= 0).any()
    w = cw.materialize(spec)
    dw = to_gpu(w)
    out, lse = run_extend(dw)
    if name == "equal_cost":  # small enough for the oracle
        ref, ref_lse = oracle.extend_attention_blocked(paged_inputs(w))
        assert_close(as_f64(out), ref, BF16_MAX_ABS, BF16_MEAN_ABS, "levelled " + name)
        assert_close(lse.cpu().double().numpy(), ref_lse, 1e-2, None, "levelled " + name + " lse")
        cwlib.set_tuning(2, 2)  # the four-wave kernel runs the same plan
        try:
            four, _ = run_extend(dw)
        finally:
            cwlib.set_tuning(2, 0)
        assert_close(as_f64(four), ref, BF16_MAX_ABS, BF16_MEAN_ABS, "levelled four-wave " + name)
    cwlib.set_tuning(1, 256)
    try:
        whole, whole_lse = run_extend(dw)
    finally:
        cwlib.set_tuning(1, 0)
    assert (bits(out) != bits(whole)).any()  # another plan ran
    if name == "equal_cost":
        # the cuts cost no precision: over the cut tiles' rows the error is the whole tiles' (2% is
        # far above its scatter over 10^5 values, partials rounded to bf16 would add 4 to 9%)
        parts = items[items[:, 5] >= 0]
        cut = np.zeros(out.shape[:2], bool)
        cu = np.concatenate([[0], np.cumsum(c["ls"])])
        for seq, kvh in np.unique(parts[:, :2], axis=0):  # (every sequence is one tile per kv head)
            cut[cu[seq]:cu[seq + 1], kvh * c["g"]:(kvh + 1) * c["g"]] = True
        rms = [np.sqrt(np.mean((as_f64(x) - ref)[cut] ** 2)) for x in (out, whole)]
        print(f"rms error over {int(cut.sum())} cut rows: {rms[0]:.4e}, whole tiles {rms[1]:.4e}", flush=True)
        assert rms[0] <= 1.02 * rms[1]
    assert_within_bf16_ulps(as_f64(out), as_f64(whole), 2, f"levelled {name}")
    # the rounded weights of a key range depend on its first tile's max: 2 * 2^-9 in lse
    assert_close(lse.cpu().double().numpy(), whole_lse.cpu().double().numpy(), 2 ** -8, None, f"levelled {name} lse")

    cwlib.init()
    sc = dict(k_scale=dw.k_scale, v_scale=dw.v_scale)
    args = (dw.q, dw.k_new, dw.v_new, dw.k_pool, dw.v_pool, dw.block_table, spec.prefix_lens, spec.suffix_lens,
            spec.gqa_group, spec.softmax_scale)
    again = torch.full_like(dw.q, float("nan"))
    cwlib.extend_attention_noalloc(*args, out=again, **sc)
    torch.cuda.synchronize()
    assert np.array_equal(bits(again), bits(out))
    ws = torch.empty(cwlib.extend_workspace_bytes(spec.prefix_lens, spec.suffix_lens, c["hkv"], c["g"], c["d"],
                                                  c["p"]), dtype=torch.uint8, device=dw.q.device)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        cwlib.extend_attention(*args, out=again, workspace=ws, **sc)
    for _ in range(3):
        again.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(bits(again), bits(out))
