"""GPU decode at the edges of its tile pipeline: items of one to nine tiles (three in
flight, none issued past the last), a last tile of one key, a new token that starts
a page, one to eight sequences (an item's sequence searched by scalar loads) and more
(by the whole wave), plans in small and large kernel arguments and uploaded; against
the oracle, and the fused page write bit for bit against cw_kv_write_pages."""
import numpy as np
import pytest
import torch

import cw_workloads as cw
import oracle
import paper_2606_16824_amd as cwlib
from conftest import paged_inputs
from gpu_util import BF16_MAX_ABS, BF16_MEAN_ABS, FP8_MAX_ABS, as_f64, assert_close, to_gpu

pytestmark = pytest.mark.gpu

KEYS = {("bf16", 128): 32, ("bf16", 64): 64, ("fp8", 128): 32, ("fp8", 64): 64}  # keys per tile
SHAPES = [(64, 16, "bf16"), (64, 64, "bf16"), (128, 16, "bf16"), (128, 64, "bf16"),
          (64, 16, "fp8"), (64, 64, "fp8"), (128, 16, "fp8"), (128, 64, "fp8")]


def _raw(t):
    return t.view(torch.int16) if t.dtype == torch.bfloat16 else t


def _check(lp, hkv, g, d, p, dt, seed, what):
    spec = cw.custom_spec(lp, [1] * len(lp), num_kv_heads=hkv, gqa_group=g, head_dim=d, page_size=p, kv_dtype=dt,
                          seed=seed)
    w = cw.materialize(spec)
    dw = to_gpu(w)
    ones = np.ones(len(lp), np.int32)
    ref, ref_lse = oracle.extend_attention_rowwise(paged_inputs(w))
    k_w, v_w = dw.k_pool.clone(), dw.v_pool.clone()
    cwlib.kv_write_pages(dw.k_new, dw.v_new, k_w, v_w, dw.block_table, spec.prefix_lens, ones, k_scale=dw.k_scale,
                         v_scale=dw.v_scale)
    out = torch.full_like(dw.q, float("nan"))
    lse = torch.full(dw.q.shape[:2], float("nan"), device=dw.q.device)
    cwlib.step_attention(dw.q, dw.k_new, dw.v_new, dw.k_pool, dw.v_pool, dw.block_table, spec.prefix_lens, ones, g,
                         spec.softmax_scale, k_scale=dw.k_scale, v_scale=dw.v_scale, out=out, lse=lse)
    torch.cuda.synchronize()
    if dt == "bf16":
        assert_close(as_f64(out), ref, BF16_MAX_ABS, BF16_MEAN_ABS, what)
    else:
        assert_close(as_f64(out), ref, FP8_MAX_ABS, None, what)
    assert_close(lse.cpu().double().numpy(), ref_lse, 1e-2, None, what + " lse")
    assert torch.equal(_raw(dw.k_pool), _raw(k_w)) and torch.equal(_raw(dw.v_pool), _raw(v_w))


@pytest.mark.parametrize("chunk", [0, 1, 2, 3, 4, 9])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: f"d{s[0]}p{s[1]}{s[2]}")
def test_tile_edges(shape, chunk):
    d, p, dt = shape
    kpt = KEYS[(dt, d)]
    lp = [0, 1, kpt - 1, kpt, kpt + 1] + [n * kpt + e for n in (2, 3, 4, 5, 6, 9) for e in (-1, 0, 1)]
    print(f"\n[case] decode tiles {shape} chunk {chunk}", flush=True)
    cwlib.set_tuning(0, chunk)
    try:
        _check(lp, 2, 4, d, p, dt, 103 + chunk, f"tiles {shape} {chunk}")
        for n in (1, 7, 8, 9):  # sequences
            _check(lp[-n:], 1, 3, d, p, dt, 107 + n, f"tiles {shape} {chunk} n={n}")
    finally:
        cwlib.set_tuning(0, 0)


@pytest.mark.parametrize("n", [120, 130, 400])
def test_plan_sizes(n):
    """Compact plans of just under and over the small arguments' 4 KB, and one too
    large for any: 30-odd bytes per sequence."""
    lp = [(37 * i) % 200 for i in range(n)]
    print(f"\n[case] decode plan sizes {n}", flush=True)
    _check(lp, 1, 4, 64, 16, "bf16", 109, f"{n} sequences")


@pytest.mark.parametrize("d,p", [(128, 16), (64, 64)])
@pytest.mark.parametrize("parts", [[4, 1, 2], [5, 2], [64, 17, 16, 15], [65, 3, 64], [128, 33], [129, 1, 31], [300, 256, 257]])
def test_merge_counts(d, p, parts):
    """Rows of up to 4, 64, 128 and more partials (another merge kernel or another
    batch size beyond each), with rows of fewer partials in the same call."""
    keys = KEYS[("bf16", d)]
    lp = [n * keys - 1 - (i % 3) for i, n in enumerate(parts)]
    print(f"\n[case] merge of {parts} partials d={d}", flush=True)
    cwlib.set_tuning(0, 1)
    try:
        items, groups = cwlib.decode_plan(lp, 2, 5, d, p)
        assert sorted(set(groups[:, 5].tolist())) == sorted(set(n for n in parts if n > 1))
        _check(lp, 2, 5, d, p, "bf16", 113, f"merge of {parts} partials d={d}")
    finally:
        cwlib.set_tuning(0, 0)


# chunks adjusted to whole rounds, whose partials are fp32: up to 64 partials per row and more
@pytest.mark.parametrize("d,p,dt,hkv,lp,parts", [
    (128, 16, "bf16", 8, [63, 92, 85, 47, 151, 58, 93, 58, 277, 226, 456, 744, 658, 169, 321, 306, 108, 149, 178, 83,
                          320, 66, 826], 9),
    (128, 16, "bf16", 3, [3164, 9422, 3720], 99),
    (64, 16, "bf16", 1, [33655, 31493, 56186, 4413, 21483], 220),
    (64, 64, "fp8", 8, [1216, 490, 955, 85, 1205, 1209, 71, 102, 1291, 771, 164, 783, 222, 748, 1182, 1228, 703, 248, 158,
                        357, 766, 1289], 7),
])
def test_merge_of_fp32_partials(d, p, dt, hkv, lp, parts):
    print(f"\n[case] merge of fp32 partials d={d} {dt} up to {parts}", flush=True)
    items, groups = cwlib.decode_plan(lp, hkv, 4, d, p, dt)
    assert groups[:, 5].max() == parts
    n_parts = int((items[:, 5] >= 0).sum())
    assert cwlib.decode_workspace_bytes(lp, hkv, 4, d, p, dt) >= n_parts * 4 * d * 4
    _check(lp, hkv, 4, d, p, dt, 137, f"merge of fp32 partials d={d} {dt} up to {parts}")
