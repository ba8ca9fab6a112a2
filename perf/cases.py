"""The work that serving agent sessions asks of this library, as measurable cases.

A case is a dict of plain values: what kind of call it is, the shape of the model
(kv heads, query heads per kv head, head dim), the page size, the pool's data type and
the ranges that its sequence lengths are drawn from (`lens_seed`: the lengths are part
of the case; the data come from the seed given to `prepare`).

Kinds
  step      cw_step_attention: one step of a serving engine, decodes and extends mixed
            (either may be absent), page write fused; workspace and outputs kept
  decode    cw_decode_attention with a log-sum-exp output
  extend    cw_extend_attention with its own output and workspace each call
  write     cw_write_extend_attention (page write and extend in one call)
  pages     cw_kv_write_pages: the new K/V of a batch into their pages
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2606_16824_amd as cw

DEV = "cuda:0"

# Most work a drawn case may ask for, both below what `long_session` needs.
MAX_FLOPS = 3.0e13
MAX_KEYS = 1 << 21  # cached keys (all sequences) of a drawn case


def _case(name, kind, *, hkv=8, g=4, d=128, page=16, dtype="bf16", decodes=0, dec_lo=0, dec_hi=0,
          extends=0, pre_lo=0, pre_hi=0, suf_lo=0, suf_hi=0, log_suffix=False, lens_seed=1):
    return {"name": name, "kind": kind, "hkv": hkv, "g": g, "d": d, "page": page, "dtype": dtype,
            "decodes": decodes, "dec_lo": dec_lo, "dec_hi": dec_hi, "extends": extends, "pre_lo": pre_lo,
            "pre_hi": pre_hi, "suf_lo": suf_lo, "suf_hi": suf_hi, "log_suffix": log_suffix,
            "lens_seed": lens_seed}


def listed():
    return [
        # one session generating alone: the smallest step, latency and launches count
        _case("one_decode", "step", decodes=1, dec_lo=1700, dec_hi=1700),
        # the generating half of a busy node on a model with 64-wide heads, ragged lengths
        _case("decode_d64", "decode", d=64, page=64, decodes=96, dec_lo=200, dec_hi=6000, lens_seed=2),
        # the 48 decodes of a mixed step over an fp8 pool, prefixes of 2k to 32k tokens
        _case("decode_fp8", "step", dtype="fp8", decodes=48, dec_lo=2048, dec_hi=32768, lens_seed=3),
        # one very long session generating: 131072 cached tokens, GQA 8
        _case("decode_long", "step", g=8, page=64, decodes=1, dec_lo=131072, dec_hi=131072),
        # sessions coming back with short tool outputs (tens to hundreds of tokens)
        _case("tool_replies", "step", extends=10, pre_lo=4096, pre_hi=32768, suf_lo=12, suf_hi=600,
              log_suffix=True, lens_seed=5),
        # opening prompts (no cached prefix) of a model with 64-wide heads
        _case("opening_prompts", "write", d=64, extends=4, suf_lo=2000, suf_hi=6000, lens_seed=6),
        # a single agent turn: 1024 new tokens on a 16384-token cached prefix
        _case("turn", "step", extends=1, pre_lo=16384, pre_hi=16384, suf_lo=1024, suf_hi=1024),
        # agent turns of 200 to 4000 new tokens, called without buffers of the caller's
        _case("turns", "extend", extends=7, pre_lo=4096, pre_hi=65536, suf_lo=200, suf_hi=4000, lens_seed=8),
        # chunked prefill: 32 chunks of at most 512 tokens scheduled with 32 decodes
        _case("chunked", "step", decodes=32, dec_lo=2048, dec_hi=32768, extends=32, pre_lo=8192, pre_hi=32768,
              suf_lo=128, suf_hi=512, lens_seed=9),
        # a mixed step over an fp8 pool: 48 decodes and 16 turns
        _case("mixed_fp8", "step", dtype="fp8", decodes=48, dec_lo=2048, dec_hi=32768, extends=16, pre_lo=8192,
              pre_hi=32768, suf_lo=256, suf_hi=2048, lens_seed=10),
        # the longest session: 8192 new tokens on 131072 cached ones, GQA 8
        _case("long_session", "step", g=8, page=64, extends=1, pre_lo=131072, pre_hi=131072, suf_lo=8192,
              suf_hi=8192),
        # a finished prefill's K/V quantised into its fp8 pages
        _case("pages_fp8", "pages", dtype="fp8", extends=12, pre_lo=0, pre_hi=16384, suf_lo=300, suf_hi=4000,
              lens_seed=12),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the ranges above: any kind of call, any supported shape."""
    while True:
        hkv, g = rng.choice([(8, 4), (8, 4), (8, 8), (4, 8), (8, 2), (2, 16), (1, 4), (16, 1), (4, 5)])
        case = _case("", "step", hkv=hkv, g=g, d=rng.choice([128, 128, 64]), page=rng.choice([16, 64]),
                     dtype=rng.choice(["bf16", "bf16", "fp8"]), lens_seed=rng.randrange(1, 1 << 30))
        del case["name"]
        what = rng.choice(["decode", "decode", "extend", "extend", "extend", "mixed", "mixed", "pages"])
        if what in ("decode", "mixed"):
            case["decodes"] = _log_int(rng, 1, 160)
            case["dec_hi"] = _log_int(rng, 300, 131072)
            case["dec_lo"] = max(1, int(case["dec_hi"] * rng.uniform(0.03, 1.0)))
            if what == "decode":
                case["kind"] = rng.choice(["decode", "step"])
        if what in ("extend", "mixed", "pages"):
            case["extends"] = _log_int(rng, 1, 40)
            case["pre_hi"] = rng.choice([0, _log_int(rng, 100, 131072), _log_int(rng, 2000, 65536)])
            case["pre_lo"] = int(case["pre_hi"] * rng.uniform(0.0, 1.0))
            case["suf_hi"] = _log_int(rng, 8, 8192)
            case["suf_lo"] = max(2, int(case["suf_hi"] * rng.uniform(0.03, 1.0)))
            case["suf_hi"] = max(case["suf_hi"], case["suf_lo"])
            case["log_suffix"] = rng.random() < 0.4
            if what == "extend":
                case["kind"] = rng.choice(["step", "extend", "write"])
            if what == "pages":
                case["kind"] = "pages"
        lp, ls = _lens(case)
        if work(case)["flops"] <= MAX_FLOPS and int((lp + ls).sum()) <= MAX_KEYS:
            return case


# ---------------------------------------------------------------------------- sizes


def _lens(case):
    """Prefix and suffix lengths of every sequence, int32, in a mixed order."""
    rng = np.random.default_rng(case["lens_seed"])
    nd, ne = case["decodes"], case["extends"]
    lp = [rng.integers(case["dec_lo"], case["dec_hi"] + 1, size=nd),
          rng.integers(case["pre_lo"], case["pre_hi"] + 1, size=ne)]
    if case["log_suffix"]:
        se = np.exp(rng.uniform(math.log(max(1, case["suf_lo"])), math.log(max(1, case["suf_hi"])), size=ne))
        se = np.clip(np.rint(se), case["suf_lo"], case["suf_hi"])
    else:
        se = rng.integers(case["suf_lo"], case["suf_hi"] + 1, size=ne)
    lp = np.concatenate(lp).astype(np.int32)
    ls = np.concatenate([np.ones(nd), se]).astype(np.int32)
    order = rng.permutation(nd + ne)
    return lp[order], ls[order]


def _elem(case):
    return 1 if case["dtype"] == "fp8" else 2


def work(case):
    hkv, g, d, p, e = case["hkv"], case["g"], case["d"], case["page"], _elem(case)
    fp8 = case["dtype"] == "fp8"
    lp, ls = (x.astype(np.int64) for x in _lens(case))
    new = int(ls.sum())
    pages_new = int(((lp + ls + p - 1) // p - lp // p).sum())
    new_kv = 2 * new * hkv * d * 2  # k_new and v_new
    write = 2 * new * hkv * d * e + (pages_new * (4 + (8 * hkv if fp8 else 0)))
    if case["kind"] == "pages":
        return {"bytes": new_kv + write, "flops": 0}
    pages = int(((lp + p - 1) // p).sum())
    kv = 2 * int(lp.sum()) * hkv * d * e + pages * (4 + (8 * hkv if fp8 else 0))
    rows = new * hkv * g
    byts = kv + new_kv + 2 * rows * d * 2 + rows * 4  # q, out, lse
    if case["kind"] in ("step", "write"):
        byts += write
    pairs = int((ls * lp + ls * (ls + 1) // 2).sum())
    return {"bytes": byts, "flops": 4 * d * hkv * g * pairs}


# ---------------------------------------------------------------------------- inputs


def _normal(gen, *shape):
    return torch.randn(*shape, generator=gen, device=DEV, dtype=torch.bfloat16)


def _pool(gen, case, pages, scale):
    """A page pool of N(0, 1) values: bf16, or e4m3fn codes of value / scale."""
    shape = (pages, case["hkv"], case["page"], case["d"])
    if case["dtype"] != "fp8":
        return _normal(gen, *shape)
    out = torch.empty(shape, dtype=torch.uint8, device=DEV)
    for p0 in range(0, pages, 8192):
        x = torch.randn(min(8192, pages - p0), *shape[1:], generator=gen, device=DEV)
        x = (x / scale[p0:p0 + 8192, :, None, None]).clamp_(-448.0, 448.0)
        out[p0:p0 + 8192] = x.to(torch.float8_e4m3fn).view(torch.uint8)
    return out


class _State:
    pass


def prepare(case, seed):
    gen = torch.Generator(device=DEV).manual_seed(seed)
    hkv, g, d, p = case["hkv"], case["g"], case["d"], case["page"]
    fp8 = case["dtype"] == "fp8"
    s = _State()
    s.kind, s.g, s.scale = case["kind"], g, 1.0 / math.sqrt(d)
    s.lp, s.ls = _lens(case)
    need = (s.lp.astype(np.int64) + s.ls + p - 1) // p
    pages = int(need.sum()) * 5 // 4 + 8
    s.k_scale = s.v_scale = None
    if fp8:
        s.k_scale = torch.rand(pages, hkv, generator=gen, device=DEV) * 0.09 + 0.01
        s.v_scale = torch.rand(pages, hkv, generator=gen, device=DEV) * 0.09 + 0.01
    s.k_pool, s.v_pool = _pool(gen, case, pages, s.k_scale), _pool(gen, case, pages, s.v_scale)
    ids = torch.randperm(pages, generator=gen, device=DEV).to(torch.int32)
    # the pools as whole numbers: their bytes are compared one by one
    s.k_bits = s.k_pool if fp8 else s.k_pool.view(torch.int16)
    s.v_bits = s.v_pool if fp8 else s.v_pool.view(torch.int16)
    n, t = len(s.lp), int(s.ls.sum())
    s.table = torch.zeros(n, max(1, int(need.max())), dtype=torch.int32, device=DEV)
    at = 0
    for b in range(n):
        s.table[b, :int(need[b])] = ids[at:at + int(need[b])]
        at += int(need[b])
    s.k_new, s.v_new = _normal(gen, t, hkv, d), _normal(gen, t, hkv, d)
    if s.kind == "pages":
        return s
    # heads range from nearly uniform attention to sharply peaked
    sharp = torch.rand(1, hkv * g, 1, generator=gen, device=DEV) * 2.0 + 0.5
    s.q = (_normal(gen, t, hkv * g, d) * sharp).to(torch.bfloat16)
    s.out, s.lse, s.ws = torch.empty_like(s.q), torch.empty(t, hkv * g, device=DEV), None
    if s.kind == "step":
        n_ws = cw.step_workspace_bytes(s.lp, s.ls, hkv, g, d, p, case["dtype"])
    elif s.kind == "decode":
        n_ws = cw.decode_workspace_bytes(s.lp, hkv, g, d, p, case["dtype"])
    else:
        n_ws = cw.extend_workspace_bytes(s.lp, s.ls, hkv, g, d, p)
    if s.kind != "extend":
        s.ws = torch.empty(max(256, n_ws), dtype=torch.uint8, device=DEV)
    return s


def run(s):
    sc = {"k_scale": s.k_scale, "v_scale": s.v_scale}
    if s.kind == "step":
        cw.step_attention(s.q, s.k_new, s.v_new, s.k_pool, s.v_pool, s.table, s.lp, s.ls, s.g, s.scale,
                          out=s.out, lse=s.lse, workspace=s.ws, **sc)
        return {"out": s.out, "lse": s.lse, "k": s.k_bits, "v": s.v_bits}
    if s.kind == "decode":
        cw.decode_attention(s.q, s.k_new, s.v_new, s.k_pool, s.v_pool, s.table, s.lp, s.g, s.scale,
                            out=s.out, lse=s.lse, workspace=s.ws, **sc)
        return {"out": s.out, "lse": s.lse}
    if s.kind == "extend":
        out = cw.extend_attention(s.q, s.k_new, s.v_new, s.k_pool, s.v_pool, s.table, s.lp, s.ls, s.g,
                                  s.scale, **sc)
        return {"out": out}
    if s.kind == "write":
        cw.write_extend_attention(s.q, s.k_new, s.v_new, s.k_pool, s.v_pool, s.table, s.lp, s.ls, s.g,
                                  s.scale, out=s.out, workspace=s.ws, **sc)
        return {"out": s.out, "k": s.k_bits, "v": s.v_bits}
    cw.kv_write_pages(s.k_new, s.v_new, s.k_pool, s.v_pool, s.table, s.lp, s.ls, **sc)
    return {"k": s.k_bits, "v": s.v_bits}


# ---------------------------------------------------------------------------- what is right


def tolerance(case):
    """Weights and outputs in bf16 (fp16 weights over fp8 pools), sums in 32 bits: about four
    times the error against 64 bits that these ranges show. Pages are exact."""
    if case["kind"] == "pages":
        return "exact"
    return {"rel": 0.02, "max": 0.3}


def _rows(case, s, b):
    """K and V of sequence b in 64 bits, [keys, hkv, d]: its cached prefix, then its new rows."""
    p, hkv, d = case["page"], case["hkv"], case["d"]
    lp, ls = int(s.lp[b]), int(s.ls[b])
    cu = int(s.ls[:b].sum())
    got = []
    for pool, scale, new in ((s.k_pool, s.k_scale, s.k_new), (s.v_pool, s.v_scale, s.v_new)):
        ids = s.table[b, :(lp + p - 1) // p].long()
        if scale is None:
            old = pool[ids].double()
        else:
            old = pool[ids].view(torch.float8_e4m3fn).float().double() * scale[ids].double()[:, :, None, None]
        old = old.transpose(1, 2).reshape(-1, hkv, d)[:lp]
        got.append(torch.cat([old, new[cu:cu + ls].double()]))
    return got[0], got[1], lp, ls, cu


def exact(case, seed):
    """The attention in 64 bits; page writes only move or round values and have no such value."""
    if case["kind"] == "pages":
        return None
    s = prepare(case, seed)
    g = case["g"]
    out = torch.empty(s.q.shape, dtype=torch.float64, device=DEV)
    lse = torch.empty(s.q.shape[:2], dtype=torch.float64, device=DEV)
    for b in range(len(s.lp)):
        k, v, lp, ls, cu = _rows(case, s, b)
        n = lp + ls
        key = torch.arange(n, device=DEV)
        step = max(1, (1 << 28) // (n * g))
        for h in range(case["hkv"]):
            kt, vh = k[:, h].t().contiguous(), v[:, h].contiguous()
            for t0 in range(0, ls, step):
                t1 = min(ls, t0 + step)
                q = s.q[cu + t0:cu + t1, h * g:(h + 1) * g].double()
                x = torch.mm(q.reshape(-1, case["d"]), kt).mul_(s.scale).view(t1 - t0, g, n)
                hide = key[None, :] > lp + torch.arange(t0, t1, device=DEV)[:, None]
                x.masked_fill_(hide[:, None, :], -math.inf)
                m = x.amax(-1, keepdim=True)
                x.sub_(m).exp_()
                z = x.sum(-1, keepdim=True)
                o = torch.mm(x.view(-1, n), vh).view(t1 - t0, g, -1)
                out[cu + t0:cu + t1, h * g:(h + 1) * g] = o / z
                lse[cu + t0:cu + t1, h * g:(h + 1) * g] = (m + z.log())[..., 0]
    if case["kind"] == "extend":
        return {"out": out}
    if case["kind"] == "write":
        return {"out": out, "k": None, "v": None}
    if case["kind"] == "decode":
        return {"out": out, "lse": lse}
    return {"out": out, "lse": lse, "k": None, "v": None}
