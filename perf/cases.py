"""Timed cases of the attention path, through the package's public calls.

A case is a dict of plain values:

  kind      "attn" (decode, prefill or both) or "append" (KV append)
  hq, hkv, dqk, dv, page    attention geometry; dqk 576 is the latent layout
            (values are the first 512 columns of the key rows)
  decodes, dec_lo, dec_hi   decode sequences (one new token) and the range of
            their context lengths
  prompts, new_lo, new_hi, pre_lo, pre_hi   prompts, their new tokens and the
            tokens already cached before them
  lens      seed of the length draw (lengths belong to the case, so that its
            work is fixed; values and page order come from prepare's seed)
  call      "decode", "prefill", "serial", "corun" or "fused"
  cus_decode   co-run: compute units of the decode share
  lse       whether the log-sum-exp is asked for beside the output

Geometries are the ones of the package's workloads and tests (28/4 heads of
128, latent 576/512 with 128 or 64 heads, split-out heads 192/128) and generic
grouped-query ones with heads of 64.
"""
from __future__ import annotations

import math
import random

import torch

from paper_2606_04415_amd import flexattn as F

QWEN = dict(hq=28, hkv=4, dqk=128, dv=128, page=16)
LATENT = dict(hq=128, hkv=1, dqk=576, dv=512, page=64)
SPLIT = dict(hq=128, hkv=128, dqk=192, dv=128, page=64)


def _attn(name, geo, call, decodes=0, dec=(0, 0), prompts=0, new=(0, 0), pre=(0, 0), lens=1, cus_decode=0, lse=False):
    c = dict(kind="attn", call=call, decodes=decodes, dec_lo=dec[0], dec_hi=dec[1], prompts=prompts, new_lo=new[0],
             new_hi=new[1], pre_lo=pre[0], pre_hi=pre[1], lens=lens, cus_decode=cus_decode, lse=lse, **geo)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # One user's decode step: a single sequence, launch latency and split depth.
        _attn("decode-one", QWEN, "decode", 1, (2000, 2000), lse=True),
        # The decode batch of the package's benchmark.
        _attn("decode-64", QWEN, "decode", 64, (512, 4096)),
        # A large decode batch of a model with 64-wide heads and large pages.
        _attn("decode-d64", dict(hq=32, hkv=8, dqk=64, dv=64, page=64), "decode", 128, (1000, 8000), lse=True),
        # A few short prompts arriving together, ragged.
        _attn("prefill-short", QWEN, "prefill", prompts=5, new=(50, 300), lse=True),
        # The prefill batch of the benchmark.
        _attn("prefill-8x2048", QWEN, "prefill", prompts=8, new=(2048, 2048)),
        # The benchmark's mixed step: a 2048-token chunk beside 128 decodes, co-run.
        _attn("mixed-corun", QWEN, "corun", 128, (1024, 8192), 1, (2048, 2048), (4096, 4096), cus_decode=96),
        # A serving step in one launch: a short chunk beside 48 decodes.
        _attn("mixed-fused", QWEN, "fused", 48, (500, 6000), 2, (200, 600), (0, 1500)),
        # Latent decode of the benchmark: 256 sequences, all 128 heads.
        _attn("latent-decode", LATENT, "decode", 256, (1024, 16384)),
        # One of two devices' heads, small pages: a small mixed latent step, ragged.
        _attn("latent-mixed-64h", dict(LATENT, hq=64, page=16), "serial", 24, (500, 6000), 1, (300, 300), (2000, 2000), lse=True),
        # Absorbed latent prefill of the benchmark's prompt.
        _attn("latent-prefill", LATENT, "prefill", prompts=1, new=(4096, 4096)),
        # The same prompt with the heads split out.
        _attn("split-prefill", SPLIT, "prefill", prompts=1, new=(4096, 4096)),
        # New tokens' rows of the mixed step into the paged pool.
        dict(name="append", kind="append", tokens=2176, pages=2048, **QWEN),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw(rng):
    fam = rng.choice(["decode", "decode", "prefill", "prefill", "mixed", "mixed", "latent", "latent", "split", "append"])
    lens, lse = rng.randrange(1, 1 << 20), rng.random() < 0.5
    d, page = rng.choice([64, 128]), rng.choice([16, 64])
    hq, hkv = rng.choice([(28, 4), (28, 4), (32, 8), (4, 1), (32, 2), (8, 8), (40, 8)])
    geo = dict(hq=hq, hkv=hkv, dqk=d, dv=d, page=page)
    hi = _log(rng, 16, 16384)
    dec = (max(1, hi // rng.choice([1, 4, 16])), hi)
    nhi = _log(rng, 2, 4096)
    new = (max(2, nhi // rng.choice([1, 3, 8])), nhi)
    phi = rng.choice([0, _log(rng, 1, 8192)])
    pre = (phi // 2, phi)
    decodes, prompts = _log(rng, 1, 256), _log(rng, 1, 16)
    if fam == "append":
        return dict(kind="append", tokens=_log(rng, 1, 16384), pages=2048 if page == 16 else 512, **geo)
    if fam == "decode":
        return _attn(None, geo, "decode", decodes, dec, lens=lens, lse=lse)
    if fam == "prefill":
        return _attn(None, geo, "prefill", prompts=prompts, new=new, pre=pre, lens=lens, lse=lse)
    if fam == "split":
        return _attn(None, dict(SPLIT, hq=(h := rng.choice([16, 32, 64, 128])), hkv=h), "prefill", prompts=prompts, new=new,
                     pre=pre, lens=lens, lse=lse)
    if fam == "latent":
        geo = dict(LATENT, hq=rng.choice([64, 128]), page=page)
        call = rng.choice(["decode", "prefill", "serial"])
        return _attn(None, geo, call, 0 if call == "prefill" else decodes, dec, 0 if call == "decode" else 1 + prompts // 4, new,
                     pre, lens, lse=lse)
    call = rng.choice(["serial", "corun", "fused"])
    if call == "fused":   # the shapes that have a one-launch form: 5 or more query heads on 3 to 8 KV heads
        geo = dict(rng.choice([QWEN, dict(QWEN, hq=40, hkv=8)]), page=page)
    return _attn(None, geo, call, decodes, dec, 1 + prompts // 4, new, pre, lens,
                 cus_decode=rng.choice([64, 96, 128]) if call == "corun" else 0, lse=lse)


def draw(rng):
    most = max(_cost(c) for c in listed())
    while True:
        c = _draw(rng)
        if _cost(c) <= most:
            return c


def _cost(case):
    w = work(case)
    return max(w["bytes"], w["flops"] / 250)


def _lengths(case):
    """(new tokens, context) of every sequence, decodes after prompts."""
    r = random.Random(case["lens"])
    ns, ls = [], []
    for _ in range(case["prompts"]):
        n = r.randint(case["new_lo"], case["new_hi"])
        ns.append(n)
        ls.append(n + r.randint(case["pre_lo"], case["pre_hi"]))
    for _ in range(case["decodes"]):
        ns.append(1)
        ls.append(r.randint(case["dec_lo"], case["dec_hi"]))
    return ns, ls


def work(case):
    hq, hkv, dqk, dv = case["hq"], case["hkv"], case["dqk"], case["dv"]
    kv = hkv * (dqk if dqk == 576 else dqk + dv) * 2
    if case["kind"] == "append":
        return {"bytes": case["tokens"] * (2 * kv + 4), "flops": 0}
    b = f = 0
    for n, L in zip(*_lengths(case)):
        b += L * kv + n * hq * (2 * (dqk + dv) + (4 if case["lse"] else 0)) + 4 * -(-L // case["page"])
        f += hq * 2 * (dqk + dv) * (n * (L - n) + n * (n + 1) // 2)
    return {"bytes": b, "flops": f}


def _scale(case):
    return 1.0 / math.sqrt(192.0 if case["dqk"] in (192, 576) else case["dqk"])


def _inputs(case, seed):
    """Device tensors of one batch: standard normal keys and values, queries
    twice that, so that scores spread over several units as a trained
    model's do; pages of the pool in random order."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    hg = torch.Generator().manual_seed(seed)

    def normal(*shape):
        return torch.randn(shape, generator=g, device="cuda", dtype=torch.bfloat16)

    ns, ls = _lengths(case)
    P, hq, hkv = case["page"], case["hq"], case["hkv"]
    pages = [-(-L // P) for L in ls]
    used = sum(pages)
    perm = torch.randperm(used + 1, generator=hg).to(torch.int32)
    bt = torch.full((len(ls), max(pages)), int(perm[used]), dtype=torch.int32)   # entries past a sequence: a spare page
    at = 0
    for s, n in enumerate(pages):
        bt[s, :n] = perm[at:at + n]
        at += n
    qsl = torch.zeros(len(ls) + 1, dtype=torch.int32)
    qsl[1:] = torch.cumsum(torch.tensor(ns), 0)
    k = normal(used + 1, P, hkv, case["dqk"])
    v = None if case["dqk"] == 576 else normal(used + 1, P, hkv, case["dv"])
    q = normal(sum(ns), hq, case["dqk"]) * 2
    return dict(q=q, k=k, v=v, bt=bt, sl=torch.tensor(ls, dtype=torch.int32), qsl=qsl)


def _append_inputs(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)

    def normal(*shape):
        return torch.randn(shape, generator=g, device="cuda", dtype=torch.bfloat16)

    n, P, hkv = case["tokens"], case["page"], case["hkv"]
    slots = torch.randperm(case["pages"] * P, generator=torch.Generator().manual_seed(seed))[:n].to(torch.int32)
    k_new, k = normal(n, hkv, case["dqk"]), normal(case["pages"], P, hkv, case["dqk"])
    v_new, v = normal(n, hkv, case["dv"]), normal(case["pages"], P, hkv, case["dv"])
    return dict(k_new=k_new, v_new=v_new, k=k, v=v, slots=slots)


_stream = None   # the program's own stream: co-run steps are issued from it
_pair = {}       # the one co-run pair a program keeps, by its split


def _corun(cus_prefill, cus_decode):
    key = (cus_prefill, cus_decode)
    if key not in _pair:
        for old in _pair.values():
            old.close()
        _pair.clear()
        _pair[key] = F.Corun(cus_prefill, cus_decode)
    return _pair[key]


def _shape(case):
    return F.make_shape(case["hq"], case["hkv"], case["dqk"], case["dv"], case["page"], _scale(case), case["dqk"] == 576)


def prepare(case, seed):
    global _stream
    if case["kind"] == "append":
        x = _append_inputs(case, seed)
        x["slots"] = x["slots"].cuda()
        return dict(case=case, shape=_shape(case), args=F.make_append_args(x["k_new"], x["v_new"], x["slots"], x["k"], x["v"]),
                    keep=x)
    x = _inputs(case, seed)
    opts = F.make_opts(cus_decode=case["cus_decode"], bm=32 if case["call"] == "fused" else 0)
    pa = F.PagedAttention(_shape(case), opts, x["qsl"], x["sl"], x["bt"].shape[1])
    out, lse = pa.alloc_out(x["q"], with_lse=case["lse"])
    dev = [x[n].cuda() for n in ("bt", "sl", "qsl")]
    if _stream is None:
        _stream = torch.cuda.Stream()
    corun = _corun(pa.plan.info["cus_prefill"], pa.plan.info["cus_decode"]) if case["call"] == "corun" else None
    return dict(case=case, pa=pa, args=pa.args(x["q"], x["k"], x["v"], *dev, out, lse), corun=corun, out=out, lse=lse,
                keep=(x, dev))


MODES = {"serial": F.FLEX_MODE_SERIAL, "corun": F.FLEX_MODE_CORUN, "fused": F.FLEX_MODE_FUSED}


def run(state):
    case = state["case"]
    if case["kind"] == "append":
        F.flex_attn_kv_append(state["shape"], state["args"])
        return state["keep"]["k"], state["keep"]["v"]
    plan, args = state["pa"].plan, state["args"]
    if case["call"] == "decode":
        F.flex_attn_decode(plan, args)
    elif case["call"] == "prefill":
        F.flex_attn_prefill(plan, args)
    elif case["call"] == "corun":
        with torch.cuda.stream(_stream):
            F.flex_attn_mixed(plan, args, F.FLEX_MODE_CORUN, corun=state["corun"])
    else:
        F.flex_attn_mixed(plan, args, MODES[case["call"]])
    return {"out": state["out"], "lse": state["lse"]} if case["lse"] else state["out"]


def tolerance(case):
    """Copies are exact. Attention: probabilities and outputs are rounded to
    bf16 (2^-9 each), so another order of the sums moves outputs by a few
    thousandths of their norm."""
    if case["kind"] == "append":
        return "exact"
    return {"rel": 8e-3, "max": 6e-2}


def exact(case, seed):
    if case["kind"] == "append":
        x = _append_inputs(case, seed)
        at = x["slots"].long().cuda()
        for new, pool in ((x["k_new"], x["k"]), (x["v_new"], x["v"])):
            pool.view(-1, *pool.shape[2:])[at] = new
        return x["k"], x["v"]
    x = _inputs(case, seed)
    ns, ls = _lengths(case)
    hq, hkv, dv, P = case["hq"], case["hkv"], case["dv"], case["page"]
    G = hq // hkv
    T = sum(ns)
    out = torch.empty((T, hq, dv), dtype=torch.float64, device="cuda")
    lse = torch.empty((T, hq), dtype=torch.float64, device="cuda")
    at = 0
    for s, (n, L) in enumerate(zip(ns, ls)):
        pages = x["bt"][s, :-(-L // P)].long().cuda()
        k = x["k"][pages].reshape(-1, hkv, case["dqk"])[:L].transpose(0, 1).double().contiguous()
        v = (k[:, :, :dv] if x["v"] is None else x["v"][pages].reshape(-1, hkv, dv)[:L].transpose(0, 1).double()).contiguous()
        kt = k.transpose(1, 2).contiguous()
        step = max(1, (1 << 27) // (hq * L))          # rows of queries at a time
        for r0 in range(0, n, step):
            r1 = min(n, r0 + step)
            q = x["q"][at + r0:at + r1].double().reshape(r1 - r0, hkv, G, -1).transpose(0, 1).reshape(hkv, (r1 - r0) * G, -1)
            z = torch.matmul(q.contiguous(), kt) * _scale(case)
            seen = L - n + torch.arange(r0, r1, device="cuda").repeat_interleave(G) + 1
            z.masked_fill_(torch.arange(L, device="cuda")[None, :] >= seen[:, None], -math.inf)
            e = torch.logsumexp(z, -1, keepdim=True)
            o = torch.matmul(torch.exp(z - e), v)
            out[at + r0:at + r1] = o.reshape(hkv, r1 - r0, G, dv).transpose(0, 1).reshape(r1 - r0, hq, dv)
            lse[at + r0:at + r1] = e.reshape(hkv, r1 - r0, G).transpose(0, 1).reshape(r1 - r0, hq)
        at += n
    return {"out": out, "lse": lse} if case["lse"] else out
