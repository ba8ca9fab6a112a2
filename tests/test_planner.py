"""Properties of the host work planner (runs on the CPU)."""
import numpy as np
import pytest

import paper_2606_16824_amd as cwlib

BN = 64
BM = 256  # packed query rows per work item (both pool dtypes)


def check_plan(lp, ls, hkv, g, d=128, p=16):
    items = cwlib.plan_items(lp, ls, hkv, g, d, p)
    bm = BM
    real = items[items[:, 0] >= 0]
    # every (seq, kv head, query tile) key range [0, kv_len) is covered exactly once
    cover = {}
    for seq, kvh, r0, kb, ke, part, rows, _ in real:
        assert 0 <= kb < ke and kb % BN == 0
        cover.setdefault((seq, kvh, r0), []).append((kb, ke, part, rows))
    for b in range(len(lp)):
        nrows = ls[b] * g
        for r0 in range(0, nrows, bm):
            rows = min(bm, nrows - r0)
            kv_len = lp[b] + (r0 + rows - 1) // g + 1
            for h in range(hkv):
                ch = sorted(cover.pop((b, h, r0)))
                assert ch[0][0] == 0 and ch[-1][1] == kv_len
                for (a0, a1, _, _), (b0, _, _, _) in zip(ch, ch[1:]):
                    assert a1 == b0
                assert all(c[3] == rows for c in ch)
                parts = [c[2] for c in ch]
                if len(ch) == 1:
                    assert parts == [-1]
                else:
                    assert parts == list(range(parts[0], parts[0] + len(ch)))
    assert not cover
    allp = real[:, 5][real[:, 5] >= 0]
    assert len(np.unique(allp)) == len(allp)
    return items


def test_turn_plan_fills_every_cu():
    # 256-row items, one resident per CU
    items = check_plan([16384], [1024], 8, 4)
    assert len(items) == 256
    # XCD-aware: workgroup i runs on XCD i % 8; all work of a kv head on one XCD
    for x in range(8):
        assert len(set(items[x::8, 1].tolist())) == 1


def test_split_boundaries_weight_suffix_tiles():
    """The turn's tiles split into two chunks of equal cost, a key tile past the
    prefix costing 1.25 prefix tiles: tile 15 (272 key tiles, 16 past the
    prefix) splits after 138 tiles (13800 of 27600), not at 136."""
    items = check_plan([16384], [1024], 8, 4)
    t15 = items[(items[:, 1] == 0) & (items[:, 2] == 15 * BM)]
    assert sorted(t15[:, 3:5].tolist()) == [[0, 138 * BN], [138 * BN, 17408]]
    cwlib.set_tuning(5, 100)
    try:
        items = check_plan([16384], [1024], 8, 4)
        t15 = items[(items[:, 1] == 0) & (items[:, 2] == 15 * BM)]
        assert sorted(t15[:, 3:5].tolist()) == [[0, 136 * BN], [136 * BN, 17408]]
    finally:
        cwlib.set_tuning(5, 125)


def test_long_plan_is_dealt_round_by_round():
    """Long: 8 kv heads x 256 tiles, unsplit.  Round r (workgroups 256r ..
    256r + 255, 32 per XCD) is all of kv head r, every XCD streaming it at once;
    XCD x gets the 32 consecutive tiles of block (x + r) % 8, in reverse order
    on odd rounds, so over the eight rounds every XCD does every block once."""
    items = check_plan([131072], [8192], 8, 8, p=64)
    assert len(items) == 2048 and np.all(items[:, 5] == -1)
    keys = np.zeros(8)
    for r in range(8):
        rnd = items[256 * r:256 * (r + 1)]
        assert set(rnd[:, 1].tolist()) == {r}
        for x in range(8):
            tiles = rnd[x::8, 2] // BM  # query tile index, in launch order on XCD x
            blk = (x + r) % 8
            want = np.arange(32 * blk, 32 * blk + 32)
            assert np.array_equal(tiles, want[::-1] if r % 2 else want)
            keys[x] += (rnd[x::8, 4] - rnd[x::8, 3]).sum()
    assert keys.max() == keys.min()  # every XCD streams the same number of keys


def test_long_plan_without_dealing_keeps_a_head_per_xcd():
    cwlib.set_tuning(3, 0)
    try:
        items = check_plan([131072], [8192], 8, 8, p=64)
    finally:
        cwlib.set_tuning(3, 1)
    assert len(items) == 2048
    for x in range(8):
        assert len(set(items[x::8, 1].tolist())) == 1


def test_dealt_rounds_then_bundles():
    """A bundle of 300 tiles deals one round (256 items) and leaves 44 items
    that, with a second sequence's bundles, go to the XCD queues after it."""
    items = check_plan([4000, 500], [300 * 64, 100], 1, 4)
    real = items[items[:, 0] >= 0]
    first = items[:256]
    assert np.all(first[:, 0] == 0) and np.all(first[:, 5] == -1)
    assert len(real) == 300 + 2


@pytest.mark.parametrize("lp,ls,hkv,g", [
    ([256], [64], 1, 4),
    ([0, 37, 200, 64], [70, 1, 129, 33], 2, 1),
    ([40, 10, 0], [0, 20, 0], 1, 4),
    ([5000, 30000, 12000], [1, 1, 1], 8, 4),
    ([100] * 40, [300] * 40, 4, 2),
])
def test_plan_coverage(lp, ls, hkv, g):
    check_plan(np.array(lp), np.array(ls), hkv, g)


def test_forced_chunking():
    cwlib.set_tuning(0, 3)
    try:
        items = check_plan(np.array([700]), np.array([150]), 2, 4)
        real = items[items[:, 0] >= 0]
        assert np.all(real[:, 4] - real[:, 3] <= 3 * BN)
    finally:
        cwlib.set_tuning(0, 0)


RATE = (72, 72, 72, 72, 80, 89, 95, 100)  # cost of a key tile by 32-row waves in use


def finish_times(items, lp):
    """Finishing time of every slot (8 XCDs x 32 CUs, one workgroup each) when the
    items go to their XCD's first free slot, in the planner's cost units."""
    t = np.zeros((8, 32))
    for i, (seq, _, _, kb, ke, _, rows, _) in enumerate(items):
        if seq < 0:
            continue
        k0, k1 = kb // BN, -(-ke // BN)
        pre = max(0, min(k1, lp[seq] // BN) - k0)
        x = t[i % 8]
        x[x.argmin()] += 300 + (pre * 100 + (k1 - k0 - pre) * 125) * RATE[(rows - 1) // 32] / 100
    return t


@pytest.mark.parametrize("lp,ls,hkv,g,cut", [
    # one tile more than fits a round; short replies on long prefixes; turns of all
    # lengths (whole tiles in another order level them); an odd number of heads
    # (bundles spread over XCDs); wide heads; no cached prefix
    ([20000] * 33, [64] * 33, 8, 4, True),
    ([19000, 31000, 5000, 12000, 27000, 9000, 30000, 8000, 22000, 16000],
     [598, 59, 14, 66, 154, 15, 54, 30, 542, 402], 8, 4, True),
    ([18504, 43579, 48305, 23677, 64755, 14911, 24185], [3506, 1864, 3197, 2380, 383, 1686, 2631], 8, 4, False),
    ([70000, 500], [2500, 1], 3, 8, True),
    ([40000] * 5, [700] * 5, 1, 16, True),
    ([0] * 4, [4071, 4153, 3780, 3373], 8, 4, False),
])
def test_levelled_plan(lp, ls, hkv, g, cut):
    """Calls that a plan of whole tiles leaves uneven: every key is still covered
    once, cut pieces hold at least four key tiles, all slots finish within 6% of the
    mean, and the meta stays within 64 KiB of the whole-tile plan's."""
    items = check_plan(np.array(lp), np.array(ls), hkv, g)
    real = items[items[:, 0] >= 0]
    parts = real[real[:, 5] >= 0]
    assert (len(parts) > 0) == cut
    assert np.all(-(-(parts[:, 4] - parts[:, 3]) // BN) >= 4)
    t = finish_times(items, lp)
    assert t.max() <= 1.06 * t.mean()
    cwlib.set_tuning(1, 256)  # a target in the place of the automatic one: whole tiles, or equal chunks
    try:
        whole = check_plan(np.array(lp), np.array(ls), hkv, g)
    finally:
        cwlib.set_tuning(1, 0)
    assert finish_times(whole, lp).max() > 1.04 * t.max()
    n_groups = len(np.unique(parts[:, :3], axis=0))
    assert len(items) * 32 + n_groups * 32 <= len(whole) * 32 + (64 << 10)


def equal_cost_kinds(rng, g, n_kinds):
    """Two to n_kinds sequences (prefix, new tokens) of one query tile each whose tiles cost the same in
    the planner's units but differ in key tiles or rows."""
    by_cost = {}
    for ls in range(1, BM // g + 1):
        for pre in range(40, 260):
            n_kt = -(-(pre * BN + ls) // BN)
            by_cost.setdefault((pre * 100 + (n_kt - pre) * 125) * RATE[(ls * g - 1) // 32] // 100, []).append((pre, ls))
    buckets = [k for cost, k in sorted(by_cost.items()) if cost >= 5000 and len({pre for pre, _ in k}) >= 2]
    kinds = {}
    for pre, ls in rng.permutation(buckets[rng.integers(len(buckets))]).tolist():
        kinds.setdefault(pre, (pre * BN, ls))
    return list(kinds.values())[:n_kinds]


# Tiles of one cost and several shapes: neighbouring queues then look alike by their costs.
@pytest.mark.parametrize("kinds,n,hkv,g", [
    ([(11680, 64), (16320, 8)], 264, 1, 4),
    ([(11704, 16), (16320, 2)], 136, 2, 16),
    ([(11696, 32), (16320, 4)], 66, 4, 8),
    ([(7072, 64), (9920, 32)], 66, 4, 4),
    ([(9920, 32), (7072, 64)], 66, 4, 4),
    ([(3632, 32), (5120, 4)], 66, 4, 8),
])
def test_levelled_plan_tiles_of_equal_cost(kinds, n, hkv, g):
    seqs = [kinds[i % len(kinds)] for i in range(n)]
    items = check_plan(np.array([a for a, _ in seqs]), np.array([b for _, b in seqs]), hkv, g)
    assert (items[:, 5] >= 0).any()  # tiles were cut


@pytest.mark.parametrize("hkv", [1, 2, 3, 4, 5, 8, 16])
def test_levelled_plan_tiles_of_equal_cost_generated(hkv):
    rng = np.random.default_rng(131 + hkv)
    cut = 0
    for _ in range(12):
        g = int(rng.choice([1, 4, 8, 16]))
        kinds = equal_cost_kinds(rng, g, int(rng.integers(2, 4)))
        n = -(-int(rng.integers(257, 420)) // hkv)
        seqs = [kinds[i % len(kinds)] for i in range(n)]
        items = check_plan(np.array([a for a, _ in seqs]), np.array([b for _, b in seqs]), hkv, g)
        cut += bool((items[:, 5] >= 0).any())
    assert cut >= 6


def part_elem_bytes(total, n_seqs, items, n_groups, rows, d):
    """Bytes per element of the partial O in a workspace of `total` bytes."""
    up = lambda x: -(-x // 256) * 256
    n_parts = int((items[:, 5] >= 0).sum())
    meta = up(up(up(n_seqs * 16) + len(items) * 32) + n_groups * 32)
    for e in (2, 4):
        if up(up(meta + n_parts * rows * d * e) + n_parts * rows * 8) == total:
            return e
    raise AssertionError(total)


@pytest.mark.parametrize("lp,ls,hkv,g,d,elem", [
    ([20000] * 33, [64] * 33, 8, 4, 128, 4),  # tiles of one item each without levelling
    ([30000] * 9, [300] * 9, 8, 4, 64, 4),
    ([16384], [1024], 8, 4, 128, 2),  # cut because there are fewer tiles than CUs
])
def test_levelled_partials_are_fp32(lp, ls, hkv, g, d, elem):
    """A sum that one item would hold in fp32 is not rounded to bf16 because levelling
    cuts it."""
    items = check_plan(np.array(lp), np.array(ls), hkv, g, d)
    groups = len(np.unique(items[items[:, 5] >= 0][:, :3], axis=0))
    total = cwlib.extend_workspace_bytes(lp, ls, hkv, g, d, 16)
    assert part_elem_bytes(total, len(lp), items, groups, BM, d) == elem


@pytest.mark.parametrize("lp,hkv,d,dt,elem", [
    ([20000] * 8, 8, 128, "bf16", 4),  # whole rounds: other chunks than the mean's
    ([300] * 30 + [30000] * 6, 8, 64, "fp8", 4),
    ([1700], 8, 128, "bf16", 2), ([30000] * 40, 8, 128, "bf16", 2),  # the chunks they would have anyway
])
def test_decode_partials_of_adjusted_chunks_are_fp32(lp, hkv, d, dt, elem):
    items, groups = cwlib.decode_plan(lp, hkv, 4, d, 16, dt)
    total = cwlib.decode_workspace_bytes(lp, hkv, 4, d, 16, dt)
    assert part_elem_bytes(total, len(lp), items, len(groups), 4, d) == elem


RAGGED = [100 + 9 * i for i in range(100)]
_MEAN = -(-sum((x + 32) // 32 * 8 for x in RAGGED) // 768) * 32  # keys of one of 768 equal shares (below 64 pages)
N_RAGGED = sum((x + _MEAN) // _MEAN * 8 for x in RAGGED)


# (prefix lens, kv heads, pool, items): one round of at most three waves per CU for
# bf16 pools and four for fp8; two and three rounds of the resident waves where the
# longest chunk (64 pages) needs more than one; one sequence a little over a round;
# more than four rounds (the longest chunk); mostly last chunks (chunk of the mean)
@pytest.mark.parametrize("lp,hkv,dt,lo,hi", [
    ([32000], 8, "bf16", 600, 768), ([32000], 8, "fp8", 900, 1024),
    ([40000, 30000, 20000], 8, "fp8", 900, 1024), ([60000, 70000], 2, "bf16", 700, 768),
    ([20000] * 8, 8, "bf16", 1400, 1536), ([20000] * 12, 8, "bf16", 2000, 2304),
    ([16000] * 24, 8, "fp8", 2600, 3072), ([30000] * 6, 8, "fp8", 1400, 1536),
    ([30000] * 40, 8, "bf16", 40 * 8 * 30, 40 * 8 * 30), (RAGGED, 8, "bf16", N_RAGGED, N_RAGGED),
])
def test_decode_chunks_fill_rounds(lp, hkv, dt, lo, hi):
    items, groups = cwlib.decode_plan(lp, hkv, 4, 128, 16, dt)
    assert lo <= len(items) <= hi, len(items)
    keys = items[:, 4] - items[:, 3]
    assert keys.max() <= 64 * 16
    # every chunk but a sequence's last has the same length
    last = {}
    for s, h, _, kb, ke, *_ in items.tolist():
        last[(s, h)] = max(last.get((s, h), 0), ke)
    full = [ke - kb for s, h, _, kb, ke, *_ in items.tolist() if ke != last[(s, h)]]
    assert len(set(full)) <= 1
    rebuilt, rebuilt_groups = cwlib.decode_plan(lp, hkv, 4, 128, 16, dt, rebuilt=True)
    assert np.array_equal(items, rebuilt) and np.array_equal(groups, rebuilt_groups)


def test_decode_chunks_keep_the_plan_in_the_arguments():
    """390 sequences of 4096 keys, all in whole chunks of 1024: 40 bytes per sequence, which
    fit the kernel arguments.  Chunks of 832 would add a last chunk's 4 bytes to each
    and fit no longer, so they are taken only from where neither fits."""
    items, _ = cwlib.decode_plan([4095] * 390, 1, 4, 128, 16)
    assert len(items) == 4 * 390 and np.all(items[:, 4] - items[:, 3] == 1024)
    items, _ = cwlib.decode_plan([4095] * 420, 1, 4, 128, 16)
    assert len(items) == 5 * 420
