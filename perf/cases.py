"""What is measured of this framework: calls through the public binding (bsfa_forward, bsfa_calibrate,
bsfa_calibrate_topk) over the range of sizes, types and options that its users call them with.

The listed cases, and what each stands for in use:

* tiny_512             the smallest call: two heads of width 64, 64 x 64 tiles, every statistic; launches count
* prompt_1000          a short prompt through one 32/8-head layer, ragged length, views of a fused QKV projection
* llama_8k             an ordinary prompt, about half of the gateable blocks skipped
* llama_32k            the first headline length at half skip
* llama_32k_dense      the same layer with the gate off: the dense path that every speed-up is quoted against
* llama_128k           the headline workload and the largest call
* ragged_batch_fp16    a batch of prompts of different lengths, fp16, thresholds per query tile, log-sum-exp
* bidirectional_8k     causal = 0, heads-first layout
* fp8_scores_32k       the score product on fp8 copies of Q and K
* heads64_tile64       heads of width 64 on the 64 x 64 gate tile, three query heads to a KV head
* calibrate_32k        per-head thresholds of a calibration sample at five target fractions
* topk_8k              per-query-tile thresholds at three sparsity levels, two samples

Keys of a case: op (forward, calibrate, topk); b, n, hq, hkv, d, bm: batch, tokens, heads, width, query tile;
dtype; causal; skip: share of gateable blocks that the thresholds skip (0: thresholds of -inf);
per_tile: thresholds per query tile; stats: counts, skip mask and log-sum-exp; lengths: batch elements
have lengths of their own; layout: how Q, K and V lie in memory; fp8: fp8 score product; single:
single_head_groups.
"""
import math

import torch

from paper_2512_07011_amd import binding

BN = 64                                     # key block rows (the only ones the library is built for)
FRACTIONS = [0.25, 0.5, 0.75, 0.9, 0.95]    # target skip fractions of a calibration
DTYPES = {"bf16": torch.bfloat16, "fp16": torch.float16}
DEV = "cuda"


def _case(op="forward", b=1, n=1024, hq=32, hkv=8, d=128, bm=128, dtype="bf16", causal=True, skip=0.5, per_tile=False,
          stats=False, lengths=False, layout="bnhd", fp8=False, single=False, **more):
    return dict(op=op, b=b, n=n, hq=hq, hkv=hkv, d=d, bm=bm, dtype=dtype, causal=causal, skip=skip, per_tile=per_tile,
                stats=stats, lengths=lengths, layout=layout, fp8=fp8, single=single, **more)


def listed():
    return [
        _case(name="tiny_512", n=512, hq=2, hkv=2, d=64, bm=64, stats=True),
        _case(name="prompt_1000", n=1000, layout="qkv"),
        _case(name="llama_8k", n=8192),
        _case(name="llama_32k", n=32768),
        _case(name="llama_32k_dense", n=32768, skip=0.0),
        _case(name="llama_128k", n=131072),
        _case(name="ragged_batch_fp16", b=4, n=6001, dtype="fp16", per_tile=True, stats=True, lengths=True),
        _case(name="bidirectional_8k", n=8192, causal=False, layout="bhnd"),
        _case(name="fp8_scores_32k", n=32768, fp8=True),
        _case(name="heads64_tile64", b=2, n=4096, hq=12, hkv=4, d=64, bm=64),
        _case(name="calibrate_32k", op="calibrate", n=32768),
        _case(name="topk_8k", op="topk", n=8192),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: forward calls above all; lengths spread over their logarithm, most of them ragged."""
    op = rng.choices(["forward", "calibrate", "topk"], [10, 1, 1])[0]
    d = rng.choices([128, 64], [3, 1])[0]
    bm = rng.choices([128, 64, 32], [6, 2, 1])[0]
    hq, hkv = rng.choice([(32, 8), (32, 8), (16, 8), (8, 8), (12, 4), (4, 2), (2, 2), (28, 4), (64, 8)])
    causal = rng.random() < 0.85
    n = _log_uniform(rng, 256, 65536 if bm == 128 else 16384)
    if op == "topk":
        n = min(n, _log_uniform(rng, 256, 16384))
    b = rng.choice([1, 1, 1, 2, 3, 4]) if n <= 16384 else 1
    if b * hq * n > 32 * 65536:
        hq, hkv = 32, 8
    if not causal:
        n = max(128, n // 128 * 128)
    elif rng.random() < 0.3:
        n = max(64, n // 64 * 64)
    c = _case(op=op, b=b, n=n, hq=hq, hkv=hkv, d=d, bm=bm, causal=causal, dtype=rng.choices(["bf16", "fp16"], [3, 1])[0],
              layout=rng.choice(["bnhd", "bnhd", "qkv", "bhnd"]))
    if op == "forward":
        c["skip"] = rng.choice([0.0, 0.25, 0.5, 0.5, 0.75, 0.9])
        c["stats"] = rng.random() < 0.3
        c["per_tile"] = causal and c["skip"] > 0 and rng.random() < 0.25
        c["lengths"] = causal and b > 1 and rng.random() < 0.6
        c["fp8"] = d == 128 and bm == 128 and rng.random() < 0.15
        c["single"] = rng.random() < 0.1
    return c


# ---- inputs ------------------------------------------------------------------------------------------
def _gateable(c, i, n):
    """Key blocks that the gate applies to for query tile i: those that need no causal mask."""
    if c["causal"]:
        return (i * c["bm"] + 1) // BN
    return n // BN - (-(-(i * c["bm"] + c["bm"]) // BN) - i * c["bm"] // BN)


def _lay_out(c, q, k, v):
    """The same values as the program's projections leave them: contiguous, as slices of one fused QKV
    tensor, or heads first."""
    if c["layout"] == "qkv":
        return torch.cat([q, k, v], dim=2).split([c["hq"], c["hkv"], c["hkv"]], dim=2)
    if c["layout"] == "bhnd":
        return tuple(t.transpose(1, 2).contiguous().transpose(1, 2) for t in (q, k, v))
    return q, k, v


def _qkv(c, seed):
    """Q, K, V ~ N(0, 1) with an attention sink on the first 64 keys and, for every query tile and head, up
    to eight earlier keys along the tile's mean query: the structure that the method meets in long prompts."""
    b, n, hq, hkv, d, bm = (c[x] for x in ("b", "n", "hq", "hkv", "d", "bm"))
    g = torch.Generator(device=DEV).manual_seed(seed)
    q = torch.randn(b, n, hq, d, generator=g, device=DEV)
    k = torch.randn(b, n, hkv, d, generator=g, device=DEV)
    v = torch.randn(b, n, hkv, d, generator=g, device=DEV)
    u = torch.randn(b, 1, hkv, d, generator=g, device=DEV)
    k[:, :64] += 4.0 * u / u.norm(dim=-1, keepdim=True)
    tiles = n // bm                                                     # whole query tiles
    if tiles > 1:
        mean = q[:, :tiles * bm].view(b, tiles, bm, hq, d).mean(dim=2)[:, 1:]
        mean = mean / mean.norm(dim=-1, keepdim=True)
        at = torch.rand(b, tiles - 1, hq, 8, generator=g, device=DEV, dtype=torch.float64)
        before = (torch.arange(1, tiles, device=DEV) * bm)[None, :, None, None]
        row = torch.floor((torch.arange(8, device=DEV) + at) / 8 * before).long()
        head = (torch.arange(hq, device=DEV) // (hq // hkv))[None, None, :, None]
        flat = ((torch.arange(b, device=DEV)[:, None, None, None] * n + row) * hkv + head).reshape(-1)
        flat, order = torch.sort(flat, stable=True)
        first = torch.ones_like(flat, dtype=torch.bool)                 # one needle to a key row
        first[1:] = flat[1:] != flat[:-1]
        k.view(-1, d)[flat[first]] += math.sqrt(d) * mean.reshape(-1, d)[order[first] // 8]
    return tuple(t.to(DTYPES[c["dtype"]]) for t in (q, k, v))


def _score_operands(c, q, k):
    """Q and K as the score product multiplies them."""
    return (t.to(torch.float8_e4m3fn).to(t.dtype) if c["fp8"] else t for t in (q, k))


def _thresholds(c, q, k):
    """Thresholds as a calibration on other inputs leaves them: quantiles of the block maxima of a few query tiles
    of each head, halfway between two of them, since a held-out threshold is none of these inputs' own maxima."""
    hq, n, bm = c["hq"], c["n"], c["bm"]
    mq = -(-n // bm)
    if not c["skip"]:
        return torch.full((hq,), -math.inf, device=DEV)
    q, k = _score_operands(c, q, k)
    whole = n // bm

    def between(x, at):
        return (x[min(max(at, 1), len(x) - 1)] + x[min(max(at, 1), len(x) - 1) - 1]) / 2

    picks = sorted({int(whole * f) for f in (0.35, 0.5, 0.65, 0.8, 0.9)} | {whole - 1})
    per_head = []
    for h in range(hq):
        kt = k[0, :n // BN * BN, h // (hq // c["hkv"])].double().t()
        vals = []
        for i in picks:
            blocks = i * bm // BN if c["causal"] else n // BN
            if blocks > 0 and i >= 0:
                s = q[0, i * bm:(i + 1) * bm, h].double() @ kt[:, :blocks * BN]
                vals.append(s.view(-1, blocks, BN).amax(dim=(0, 2)))
        per_head.append(torch.sort(torch.cat(vals))[0] / math.sqrt(c["d"]) if vals else torch.zeros(2, dtype=torch.float64, device=DEV))
    if not c["per_tile"]:
        return torch.stack([between(x, int(c["skip"] * len(x))) for x in per_head]).float()
    # a fixed number of retained blocks in every tile, so that about `skip` of all gateable blocks go
    keep = max(1, int((1.0 - c["skip"]) * 0.6 * n / BN))
    tau = torch.empty(hq, mq)
    for h, x in enumerate(per_head):
        x = x.cpu()
        for i in range(mq):
            a = _gateable(c, i, n)
            tau[h, i] = -math.inf if a <= keep else float(between(x, int((1.0 - keep / a) * len(x))))
    return tau.to(DEV)


def _lengths(c, seed):
    """Tokens of each batch element: the first has them all."""
    if not c["lengths"]:
        return [c["n"]] * c["b"]
    r = torch.Generator().manual_seed(seed)
    return [c["n"]] + [max(1, int(c["n"] * f)) for f in (0.15 + 0.8 * torch.rand(c["b"] - 1, generator=r)).tolist()]


def _levels(c):
    """Numbers of retained blocks that a top-k calibration is asked for."""
    blocks = -(-c["n"] // BN)
    return [max(1, blocks // 8), max(1, blocks // 4), max(1, blocks // 2)]


def prepare(case, seed):
    c = case
    q, k, v = _qkv(c, seed)
    if c["op"] == "calibrate":
        q, k, _ = _lay_out(c, q, k, v)
        return {"case": c, "q": q, "k": k}
    if c["op"] == "topk":
        second = _qkv(c, seed + 500009)
        return {"case": c, "samples": [_lay_out(c, q, k, v)[:2], _lay_out(c, *second)[:2]]}
    s = {"case": c, "tau": _thresholds(c, q, k)}
    s["q"], s["k"], s["v"] = _lay_out(c, q, k, v)
    s["out"] = torch.zeros(c["b"], c["n"], c["hq"], c["d"], dtype=DTYPES[c["dtype"]], device=DEV)
    s["seqlens"] = torch.tensor(_lengths(c, seed), dtype=torch.int32, device=DEV) if c["lengths"] else None
    s["stats"] = binding.alloc_stats(s["q"], c["bm"], BN, counts=True, skip_mask=True, lse=True) if c["stats"] else None
    if c["stats"]:
        s["stats"].lse.zero_()
    return s


def run(state):
    c = state["case"]
    if c["op"] == "calibrate":
        return binding.bsfa_calibrate(state["q"], state["k"], FRACTIONS, causal=c["causal"], block_m=c["bm"], block_n=BN)
    if c["op"] == "topk":
        return binding.bsfa_calibrate_topk(state["samples"], _levels(c), causal=c["causal"], block_m=c["bm"], block_n=BN)
    out = binding.bsfa_forward(state["q"], state["k"], state["v"], state["tau"], causal=c["causal"], out=state["out"],
                               skip_stats=state["stats"], block_m=c["bm"], block_n=BN, seqlens=state["seqlens"],
                               single_head_groups=c["single"], qk_fp8=c["fp8"])
    st = state["stats"]
    return out if st is None else {"out": out, "lse": st.lse, "counts": st.counts, "skip_mask": st.skip_mask}


def work(case):
    """Operations: the score product over every reachable block, the second one over the kept share; bytes:
    Q, K, V once, the outputs once."""
    c = case
    lengths = _lengths(c, 1)
    reach = gate = 0
    for n in lengths:
        for i in range(-(-n // c["bm"])):
            reach += min(-(-(i + 1) * c["bm"] // BN), -(-n // BN)) if c["causal"] else n // BN
            gate += _gateable(c, i, n)
    product = 2.0 * c["bm"] * BN * c["d"] * c["hq"]                      # one product on one tile of every head
    rows = float(sum(lengths)) * c["d"] * 2
    samples = 2 if c["op"] == "topk" else 1
    if c["op"] != "forward":
        return {"flops": samples * product * reach, "bytes": samples * rows * (c["hq"] + c["hkv"])}
    return {"flops": product * (2 * reach - c["skip"] * gate), "bytes": rows * (2 * c["hq"] + 2 * c["hkv"])}


def tolerance(case):
    """Forward: rounding of the probabilities and of the result to the element type (a block whose maximum lies
    within rounding of its threshold may fall on either side).  Calibration: 32-bit sums of 128 products."""
    if case["op"] != "forward":
        return {"rel": 1e-5, "max": 1e-4}
    return {"rel": 1e-2 if case["dtype"] == "bf16" else 2e-3, "max": 0.5, "differ": 0.01}


# ---- the same in 64 bits ------------------------------------------------------------------------------
def _maxima(c, q, k, b, h, n):
    """For one head: the query tiles' scores in 64 bits (natural units, masked) with their block maxima and which
    blocks the gate applies to, a group of tiles at a time."""
    bm, mkv = c["bm"], -(-n // BN)
    kt = torch.zeros(c["d"], mkv * BN, dtype=torch.float64, device=DEV)
    kt[:, :n] = k[b, :n, h // (c["hq"] // c["hkv"])].double().t()
    mq = -(-n // bm)
    step = max(1, min(mq, (1 << 26) // (bm * mkv * BN)))
    for i0 in range(0, mq, step):
        i1 = min(mq, i0 + step)
        r0, r1 = i0 * bm, min(n, i1 * bm)
        cols = min(mkv * BN, -(-r1 // BN) * BN) if c["causal"] else mkv * BN
        s = (q[b, r0:r1, h].double() @ kt[:, :cols]) / math.sqrt(c["d"])
        col = torch.arange(cols, device=DEV)
        row = torch.arange(r0, r1, device=DEV)
        s.masked_fill_(col[None] >= n, -math.inf)
        if c["causal"]:
            s.masked_fill_(col[None] > row[:, None], -math.inf)
        by_row = s.view(r1 - r0, cols // BN, BN).amax(dim=2)
        pad = (i1 - i0) * bm - (r1 - r0)
        if pad:
            by_row = torch.cat([by_row, by_row[-1:].expand(pad, -1)])
        mx = by_row.view(i1 - i0, bm, cols // BN).amax(dim=1)
        blk, tile = torch.arange(cols // BN, device=DEV)[None], torch.arange(i0, i1, device=DEV)[:, None]
        if c["causal"]:
            gate = blk < (tile * bm + 1) // BN
        else:
            gate = (blk < tile * bm // BN) | (blk >= -(-(tile * bm + bm) // BN))
        yield i0, i1, r0, r1, s, mx, gate


def exact(case, seed):
    c = case
    if c["b"] * c["hq"] * c["n"] ** 2 > 40 * 65536 ** 2:
        return None
    q, k, v = _qkv(c, seed)
    if c["op"] == "calibrate":
        rows = []
        for h in range(c["hq"]):
            x = torch.cat([mx[gate] for b in range(c["b"]) for _, _, _, _, _, mx, gate in _maxima(c, q, k, b, h, c["n"])])
            x = torch.sort(x)[0]
            at = [math.floor(torch.tensor(f, dtype=torch.float32).double().item() * len(x)) for f in FRACTIONS]
            rows.append([-math.inf if r == 0 else math.inf if r >= len(x) else float(x[r]) for r in at])
        return torch.tensor(rows, dtype=torch.float64).t().contiguous()
    if c["op"] == "topk":
        levels, total, count = _levels(c), 0.0, 0
        for q, k, _ in ((q, k, v), _qkv(c, seed + 500009)):
            for b in range(c["b"]):
                t = torch.empty(len(levels), c["hq"], -(-c["n"] // c["bm"]), dtype=torch.float64, device=DEV)
                for h in range(c["hq"]):
                    for i0, i1, _, _, _, mx, gate in _maxima(c, q, k, b, h, c["n"]):
                        x = torch.sort(mx.masked_fill(~gate, -math.inf), dim=1, descending=True)[0]
                        for j, kk in enumerate(levels):
                            t[j, h, i0:i1] = torch.where(gate.sum(1) > kk, x[:, min(kk, x.shape[1]) - 1], -math.inf)
                total, count = total + t, count + 1
        return total / count
    tau = _thresholds(c, q, k)
    out = torch.zeros(c["b"], c["n"], c["hq"], c["d"], dtype=torch.float64, device=DEV)
    lse = torch.zeros(c["b"], c["n"], c["hq"], dtype=torch.float64, device=DEV)
    qs, ks = _score_operands(c, q, k)
    for b, n in enumerate(_lengths(c, seed)):
        for h in range(c["hq"]):
            vd = v[b, :n, h // (c["hq"] // c["hkv"])].double()
            for i0, i1, r0, r1, s, mx, gate in _maxima(c, qs, ks, b, h, n):
                t = tau[h] if tau.dim() == 1 else tau[h, i0:i1, None]
                skip = (gate & (mx.float() < t)).repeat_interleave(c["bm"], dim=0)[:r1 - r0]
                s.view(r1 - r0, -1, BN).masked_fill_(skip[:, :, None], -math.inf)
                m = s.amax(dim=1, keepdim=True)
                p = s.sub_(m).exp_()
                total = p.sum(dim=1, keepdim=True)
                out[b, r0:r1, h] = (p[:, :n] @ vd[:p.shape[1]]) / total
                lse[b, r0:r1, h] = (m + total.log())[:, 0]
    return {"out": out, "lse": lse, "counts": None, "skip_mask": None} if c["stats"] else out
