"""GPU cw_kv_write_pages at the edges of its work split (a wave takes 128 pieces of 8
elements, several tokens when the rows are short, and steps over sequences; up to
1024 sequences travel in the kernel arguments), and its fp8 codes for every bf16
value: bit for bit against the oracle's scatter and codes."""
import numpy as np
import pytest
import torch

import cw_workloads as cw
import oracle
import paper_2606_16824_amd as cwlib
from conftest import paged_inputs
from gpu_util import to_gpu

pytestmark = pytest.mark.gpu


def _raw(t):
    t = t.cpu()
    return t.view(torch.int16).numpy().view(np.uint16) if t.dtype == torch.bfloat16 else t.numpy()


def _check(w, what):
    s = w.spec
    dw = to_gpu(w)
    cwlib.kv_write_pages(dw.k_new, dw.v_new, dw.k_pool, dw.v_pool, dw.block_table, s.prefix_lens, s.suffix_lens,
                         k_scale=dw.k_scale, v_scale=dw.v_scale)
    torch.cuda.synchronize()
    want_k, want_v = oracle.write_pages(paged_inputs(w))
    nk, nv = int((_raw(dw.k_pool) != want_k).sum()), int((_raw(dw.v_pool) != want_v).sum())
    print(f"[{what}] mismatching elements: K {nk}, V {nv}", flush=True)
    assert nk == 0 and nv == 0


# rows of 8 pieces (16 tokens per wave) with empty and one-token sequences between;
# a wave's pieces ending inside a row; one piece more and one less than a wave's
# share; 1024 sequences (kernel arguments) and 1025 (uploaded)
SHAPES = {
    "short_rows": ([5, 0, 33, 2, 0, 70, 1], [3, 0, 1, 0, 0, 40, 1], 1, 64, 16),
    "odd_heads": ([7, 100], [45, 19], 3, 128, 64),
    "one_wave": ([0], [16], 1, 64, 64),
    "one_row_more": ([3], [17], 1, 64, 16),
    "one_row_less": ([20], [15], 1, 64, 16),
    "long_rows": ([1, 9], [3, 2], 40, 128, 16),
    "1024_sequences": ([i % 40 for i in range(1024)], [(i * 7) % 4 for i in range(1024)], 1, 64, 16),
    "1025_sequences": ([i % 40 for i in range(1025)], [(i * 7) % 4 for i in range(1025)], 1, 64, 16),
}


@pytest.mark.parametrize("dt", ["bf16", "fp8"])
@pytest.mark.parametrize("name", list(SHAPES))
def test_split(name, dt):
    lp, ls, hkv, d, p = SHAPES[name]
    print(f"\n[case] pages split {name} {dt}", flush=True)
    _check(cw.materialize(cw.custom_spec(lp, ls, num_kv_heads=hkv, gqa_group=1, head_dim=d, page_size=p, kv_dtype=dt,
                                         seed=89)), name)


def test_every_value_against_many_scales():
    """All 65536 bf16 values (infinities, NaNs, subnormals and both zeros among them),
    each against 128 K scales and 128 V scales, drawn anew for every pass and page:
    exponents drawn from -70 to 69 (half of them from -12 to 2), significands at both
    ends, between, and within 32 of the multiples of 2^20 that the quick quotient's
    proof turns on; some of the scales are ones it does not take."""
    d, p, hkv, tokens = 64, 16, 8, 1024
    spec = cw.custom_spec([0], [tokens], num_kv_heads=hkv, gqa_group=1, head_dim=d, page_size=p, kv_dtype="fp8", seed=97)
    w = cw.materialize(spec)
    vals = torch.arange(65536, dtype=torch.int32).to(torch.int16).view(torch.bfloat16).view(tokens, 1, d)
    w.k_new.copy_(vals.expand(tokens, hkv, d))
    w.v_new.copy_(vals.flip(0).expand(tokens, hkv, d))
    # a NaN quotient clamps to -448
    nan = torch.isnan(w.k_new.float()), torch.isnan(w.v_new.float())
    dw = to_gpu(w)
    bt = w.block_table[0, :tokens // p].long()
    rng = np.random.default_rng(101)
    n = w.k_scale.numel()
    for i in range(16):
        for t in (w.k_scale, w.v_scale):
            tie = rng.integers(8, 16, size=n) * (1 << 20) + rng.integers(-32, 33, size=n)
            kinds = [rng.choice([0, 1, 0x7FFFFF, 0x7FFFFE, 0x400000, 0x555555], size=n), rng.integers(0, 1 << 23, size=n),
                     np.maximum(tie, 1 << 23) - (1 << 23)]
            sig = np.choose(rng.integers(0, 3, size=n), kinds).astype(np.uint32)
            exp = np.where(np.arange(n) % 2 == 0, rng.integers(115, 130, size=n), rng.integers(57, 197, size=n))
            t.copy_(torch.from_numpy(((exp.astype(np.uint32) << 23) | sig).view(np.float32).reshape(t.shape)))
        dw.k_scale.copy_(w.k_scale)
        dw.v_scale.copy_(w.v_scale)
        cwlib.kv_write_pages(dw.k_new, dw.v_new, dw.k_pool, dw.v_pool, dw.block_table, spec.prefix_lens,
                             spec.suffix_lens, k_scale=dw.k_scale, v_scale=dw.v_scale)
        torch.cuda.synchronize()
        for pool, new, scale, bad in ((dw.k_pool, w.k_new, w.k_scale, nan[0]), (dw.v_pool, w.v_new, w.v_scale, nan[1])):
            got = pool.cpu()[bt].transpose(1, 2).reshape(tokens, hkv, d)
            s = scale[bt].repeat_interleave(p, 0)[:, :, None]
            x = torch.where(bad, torch.tensor(-float("inf")), new.float()) / s  # IEEE fp32 on the CPU
            want = x.clamp(-448.0, 448.0).to(torch.float8_e4m3fn).view(torch.uint8)
            diff = int((got != want).sum())
            print(f"pass {i}: differing codes: {diff} of {got.numel()}", flush=True)
            assert diff == 0
