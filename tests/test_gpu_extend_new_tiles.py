"""GPU extend over long runs of new tokens: the loop for key tiles that lie wholly in
the new tokens and are seen by every row of the workgroup starts and ends at every
alignment (prefix ends at, before and past a tile's edge, none at all; suffixes
around whole tiles; query tiles of 16, 64 and 256 tokens; key ranges cut anywhere
among the new tokens).  Against the oracle."""
import pytest

import cw_workloads as cw
import oracle
import paper_2606_16824_amd as cwlib
from conftest import paged_inputs
from gpu_util import BF16_MAX_ABS, BF16_MEAN_ABS, FP8_MAX_ABS, as_f64, assert_close, run_extend, to_gpu

pytestmark = pytest.mark.gpu

LENS = [(0, 64), (0, 517), (1, 320), (63, 193), (64, 192), (65, 191), (127, 385), (128, 448), (130, 511), (200, 700),
        (0, 1), (640, 257)]


@pytest.mark.parametrize("chunk", [0, 1, 3, 5])
@pytest.mark.parametrize("g", [1, 4, 16])
@pytest.mark.parametrize("d,p,dt", [(64, 16, "bf16"), (128, 64, "bf16"), (64, 64, "fp8"), (128, 16, "fp8")])
def test_new_tiles(d, p, dt, g, chunk):
    spec = cw.custom_spec([a for a, _ in LENS], [b for _, b in LENS], num_kv_heads=1, gqa_group=g, head_dim=d,
                          page_size=p, kv_dtype=dt, seed=127 + g)
    what = f"new tiles d={d} p={p} {dt} g={g} chunk={chunk}"
    print(f"\n[case] {what}", flush=True)
    w = cw.materialize(spec)
    cwlib.set_tuning(0, chunk)
    try:
        out, lse = run_extend(to_gpu(w))
    finally:
        cwlib.set_tuning(0, 0)
    ref, ref_lse = oracle.extend_attention_blocked(paged_inputs(w))
    if dt == "bf16":
        assert_close(as_f64(out), ref, BF16_MAX_ABS, BF16_MEAN_ABS, what)
    else:
        assert_close(as_f64(out), ref, FP8_MAX_ABS, None, what)
    assert_close(lse.cpu().double().numpy(), ref_lse, 1e-2, None, what + " lse")
