"""Timed workloads of the sparse-selection path, one call or one layer each.

Every case is a plain dict: an operation ("op"), a batch of sessions and the
options that the operation takes.  Session lengths follow from the case alone
(log-uniform histories and uniform appends between the stated bounds, drawn
from "lens"); the data follow from the seed.

    scores   janus_index_scores / janus_index_scores_mxfp4 over a prefill
    select   top-k (whole rows or Eq. 3's shards), page demand with its runs,
             and the difference against a predicted page set
    attn     MLA attention over given selections, bf16 or fp8 KV rows
    decode   one decode step: scores, top-k, page demand, the load set and
             the split attention
    layer    one prefill layer: scores, top-k, page demand and attention

Shapes are those of the repository's own workloads and benchmark: 64 indexer
heads x 128 dims, MLA rows of 576/512, 64-token pages behind a permuted page
table, histories of 8K to 160K tokens with 5% of them in eight hot spans, and
the small fp32 layer with MQA attention.
"""
import math
import random

import numpy as np
import torch

import paper_2609_36938_amd as janus

FP8_MAX = 448.0
E2M1 = (0.0, 0.5, 1.0, 1.5, 2.0, 3.0, 4.0, 6.0)
MAX_RUN = 32
KV8_ROW = 592


def _case(name, op, sessions, hist, new, lens=0, shift=0, page=64, k=2048, **more):
    """hist and new are (lowest, highest) tokens of a session."""
    c = {"name": name, "op": op, "sessions": sessions, "hist_lo": hist[0], "hist_hi": hist[1], "new_lo": new[0],
         "new_hi": new[1], "lens": lens, "shift": shift, "page": page, "k": k}
    c.update(more)
    return c


def listed():
    return [
        # the indexer of one long append prefill: the benchmark's layer
        _case("scores_fp8_128k", "scores", 1, (131072, 131072), (8192, 8192), keys="fp8", H=64, d=128),
        # a bf16 indexer at the median append
        _case("scores_bf16_32k", "scores", 1, (32768, 32768), (2048, 2048), keys="bf16", H=64, d=128),
        # several sessions of different lengths prefilled together, FP4 keys
        _case("scores_mxfp4_ragged", "scores", 8, (8192, 65536), (512, 4096), lens=3, keys="mxfp4", H=64, d=128),
        # selection and its page sets after the indexer of a 4096-token append
        _case("select_128k", "select", 1, (131072, 131072), (4096, 4096), shards=0),
        # the lookahead's sharded prediction over a few appended tokens
        _case("select_sharded_128k", "select", 1, (131072, 131072), (64, 64), shards=8),
        # attention of the benchmark's layer, all 128 heads on one GPU
        _case("attn_bf16_128h", "attn", 1, (131072, 131072), (8192, 8192), kv="bf16", heads=128),
        # the heads of one of eight tensor-parallel shards
        _case("attn_bf16_16h", "attn", 1, (65536, 65536), (2048, 2048), kv="bf16", heads=16),
        # ragged sessions over an fp8 KV cache
        _case("attn_fp8_ragged", "attn", 5, (8192, 65536), (200, 900), lens=5, kv="fp8", heads=128),
        # a decode step of a small batch: latency and launches
        _case("decode_2", "decode", 2, (8192, 16384), (1, 1), lens=2, keys="fp8", kv="bf16", heads=128),
        # a decode step of a full batch
        _case("decode_64", "decode", 64, (32768, 163840), (1, 1), lens=6, keys="fp8", kv="bf16", heads=128),
        # the small fp32 layer with 8-head MQA attention
        _case("layer_f32_tiny", "layer", 1, (4096, 4096), (256, 256), k=256, keys="f32", H=4, d=64, kv="mqa",
              heads=8),
        # selection by entries of 128 tokens over a million-token history
        _case("layer_entries_1m", "layer", 1, (1048576, 1048576), (2048, 2048), shift=7, k=512, keys="mxfp4", H=64,
              d=128, kv="fp8", heads=128),
    ]


def _log_int(rng, lo, hi):
    return int(math.floor(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))


def draw(rng: random.Random):
    op = rng.choice(["scores", "scores", "select", "select", "attn", "attn", "decode", "decode", "layer"])
    lens = rng.randrange(1 << 20)
    if op == "scores":
        keys = rng.choice(["fp8", "bf16", "mxfp4"])
        sessions = rng.choice([1, 1, 2, 5, 11, 16])
        hist = _log_int(rng, 8192, 131072)
        # pairs of the largest listed case of this type, shared by the sessions
        pairs = 3e8 if keys == "bf16" else 1.1e9
        new = min(8192, int(pairs / (sessions * 1.1 * hist)))
        new = _log_int(rng, min(64, new), new)
        c = _case("", op, sessions, (max(1, hist // rng.choice([1, 2, 7])), hist), (max(1, new // 4), new), lens=lens,
                  keys=keys, H=64, d=128)
    elif op == "select":
        sessions = rng.choice([1, 1, 3, 8])
        hist = _log_int(rng, 8192, 160000)
        new = _log_int(rng, 1, max(1, min(8192, int(5.5e8 / (sessions * 1.1 * hist)))))
        shards = rng.choice([0, 0, 2, 4, 8])
        c = _case("", op, sessions, (max(1, hist // rng.choice([1, 3])), hist), (max(1, new // 3), new), lens=lens,
                  page=rng.choice([16, 64, 64, 128]), k=rng.choice([512, 1000, 1024, 2048, 2048]), shards=shards)
    elif op == "attn":
        sessions = rng.choice([1, 1, 4, 7])
        hist = _log_int(rng, 4096, 131072)
        new = _log_int(rng, 128, max(128, 8192 // sessions))
        c = _case("", op, sessions, (max(1, hist // rng.choice([1, 4])), hist), (max(1, new // 3), new), lens=lens,
                  k=rng.choice([512, 1000, 2048, 2048]), kv=rng.choice(["bf16", "fp8"]),
                  heads=rng.choice([16, 32, 64, 128, 128]))
    elif op == "decode":
        sessions = _log_int(rng, 1, 64)
        hist = _log_int(rng, 8192, 163840)
        c = _case("", op, sessions, (max(4096, hist // 4), hist), (1, rng.choice([1, 1, 1, 2, 4])), lens=lens,
                  k=rng.choice([1024, 2048, 2048]), keys=rng.choice(["fp8", "mxfp4"]),
                  kv=rng.choice(["bf16", "fp8"]), heads=rng.choice([16, 128, 128]))
    else:
        keys, H, d = rng.choice([("f32", 4, 64), ("f32", 8, 32), ("bf16", 16, 32), ("mxfp4", 64, 128)])
        if keys == "mxfp4":
            c = _case("", op, 1, (_log_int(rng, 131072, 1048576),) * 2, (_log_int(rng, 32, 2048),) * 2, lens=lens,
                      shift=7, k=512, keys=keys, H=H, d=d, kv=rng.choice(["bf16", "fp8"]), heads=128)
        else:
            hist = _log_int(rng, 1024, 16384)
            new = _log_int(rng, 16, 512)
            c = _case("", op, rng.choice([1, 3]), (hist // 2, hist), (max(1, new // 2), new), lens=lens,
                      k=rng.choice([100, 256, 512]), keys=keys, H=H, d=d, kv="mqa", heads=rng.randint(1, 16))
    del c["name"]
    return c


# ---- lengths ---------------------------------------------------------------

def _lengths(c):
    """(histories, appends) of the sessions, in tokens."""
    rng = random.Random(c["lens"] * 7919 + c["sessions"])
    hist = [min(c["hist_hi"], _log_int(rng, c["hist_lo"], c["hist_hi"])) for _ in range(c["sessions"])]
    new = [rng.randint(c["new_lo"], c["new_hi"]) for _ in range(c["sessions"])]
    return hist, new


def _shape(c):
    """Per session: history ids, ids in all, and the candidates of its rows."""
    e = c["shift"]
    out = []
    for M, N in zip(*_lengths(c)):
        out.append((M >> e, (M + N) >> e, [(M + i + 1) >> e for i in range(N)]))
    return out


# ---- inputs ----------------------------------------------------------------

def _hot(c, mh, rng):
    """Ids of the hot spans of a history of mh ids: 5% of it in eight spans,
    one inside each eighth."""
    span, seg = int(0.05 * mh / 8), mh // 8
    ids = []
    for j in range(8):
        s = j * seg + rng.randint(0, max(0, seg - span))
        ids.append(np.arange(s, s + span, dtype=np.int64))
    return np.concatenate(ids)


def _fp8_rows(x):
    flat = x.reshape(x.shape[0], -1)
    scale = flat.abs().amax(dim=1).clamp_min(1e-12) / FP8_MAX
    q = (flat / scale[:, None]).to(torch.float8_e4m3fn).view(torch.uint8).reshape(x.shape)
    return q, scale.float()


def _mxfp4_rows(x):
    n, d = x.shape
    blk = x.reshape(n, d // 32, 32)
    amax = blk.abs().amax(dim=2).clamp_min(1e-30)
    e = torch.ceil(torch.log2(amax / 6.0))
    v = blk / torch.exp2(e)[:, :, None]
    mid = torch.tensor([0.25, 0.75, 1.25, 1.75, 2.5, 3.5, 5.0], device=x.device)
    code = torch.bucketize(v.abs().contiguous(), mid).to(torch.uint8) | ((v < 0).to(torch.uint8) << 3)
    code = code.reshape(n, d)
    return (code[:, 0::2] | (code[:, 1::2] << 4)).contiguous(), (e + 127).to(torch.uint8)


def _indexer(c, s, g, hot):
    """Queries, head weights and keys as a model hands them over."""
    dev, H, d, keys = s["dev"], c["H"], c["d"], c["keys"]
    tq = s["batch"].total_q
    q = torch.randn((tq, H, d), generator=g, device=dev)
    k = torch.randn((s["batch"].total_ctx, d), generator=g, device=dev)
    for b, ids in enumerate(hot):
        k[torch.from_numpy(ids).to(dev) + int(s["batch"].ctx_start_host[b])] *= 3.0
    s["w"] = torch.rand((tq, H), generator=g, device=dev) / 8
    s["sq"] = s["sk"] = s["bs"] = None
    if keys in ("fp8", "mxfp4"):
        s["q"], s["sq"] = _fp8_rows(q)
    else:
        s["q"] = q.to(torch.bfloat16) if keys == "bf16" else q
    if keys == "fp8":
        s["kI"], s["sk"] = _fp8_rows(k)
    elif keys == "mxfp4":
        s["kI"], s["bs"] = _mxfp4_rows(k)
    else:
        s["kI"] = k.to(torch.bfloat16) if keys == "bf16" else k
    s["scores"] = torch.empty(s["batch"].total_scores, dtype=torch.float32, device=dev)


def _selection(c, s, g, hot):
    """[total_q, k] ascending ids shaped like real selections: 60% from the
    hot spans, the rest spread over the row's other candidates; every
    candidate, then -1, where a row has at most k."""
    dev, k = s["dev"], c["k"]
    rows = []
    for (mh, ctx, cand), ids in zip(_shape(c), hot):
        n = torch.tensor(cand, device=dev, dtype=torch.int64)[:, None]
        u = torch.rand((len(cand), k), generator=g, device=dev, dtype=torch.float64)
        j = torch.arange(k, device=dev)[None, :]
        kh = min(int(0.6 * k), len(ids))
        kc = k - kh
        if mh - len(ids) > 2 * kc:
            hid = torch.from_numpy(ids).to(dev)
            mask = torch.ones(ctx, dtype=torch.bool, device=dev)
            mask[hid] = False
            cold = torch.nonzero(mask)[:, 0]
            lo, hi = j[:, :kh] * len(ids) // kh, (j[:, :kh] + 1) * len(ids) // kh
            a = hid[lo + (u[:, :kh] * (hi - lo)).long()]
            cc = n - len(ids)
            lo, hi = j[:, :kc] * cc // kc, (j[:, :kc] + 1) * cc // kc
            b = cold[lo + (u[:, kh:] * (hi - lo)).long()]
            r = torch.sort(torch.cat([a, b], dim=1), dim=1)[0]
        else:
            lo, hi = j * n // k, (j + 1) * n // k
            r = lo + (u * (hi - lo)).long()
            r = torch.where(n <= k, torch.where(j < n, j.expand_as(r), torch.full_like(r, -1)), r)
        rows.append(r.to(torch.int32))
    return torch.cat(rows)


def _pages(c, s, g):
    """A permuted page table and the buffers that page demand fills."""
    dev, ps = s["dev"], c["page"]
    per = [-(-ctx // ps) for _, ctx, _ in _shape(c)]
    P = sum(per)
    perm = torch.randperm(P, generator=g, device=dev).to(torch.int32)
    pt = torch.zeros((len(per), max(1, max(per))), dtype=torch.int32, device=dev)
    at = 0
    for b, n in enumerate(per):
        pt[b, :n] = perm[at:at + n]
        at += n
    s["pt"], s["P"] = pt, P
    z = lambda n: torch.zeros(n, dtype=torch.int32, device=dev)  # noqa: E731
    nw = (P + 31) // 32
    s["pd"] = (z(nw), z(P), z(2 * P), z(2))
    s["diff"] = (z(nw), z(2 * P), z(5))


def _page_bits(s, g, p):
    """A bitmap of pages, each set with probability p."""
    nw = (s["P"] + 31) // 32
    bits = (torch.rand((nw, 32), generator=g, device=s["dev"]) < p).to(torch.int64)
    bits.reshape(-1)[s["P"]:] = 0
    words = (bits << torch.arange(32, device=s["dev"])).sum(dim=1)
    return torch.where(words >= 1 << 31, words - (1 << 32), words).to(torch.int32)


def _attention(c, s, g):
    """The KV pool and the queries.  MLA: 576-element rows, bf16 or fp8 with
    an inline scale; mqa: separate 128-element K and V rows."""
    dev, rows, kv = s["dev"], s["P"] * c["page"], c["kv"]
    tq, Hq = s["batch"].total_q, c["heads"]
    if kv == "mqa":
        s["kpool"] = torch.randn((rows, 128), generator=g, device=dev).to(torch.bfloat16)
        s["vpool"] = torch.randn((rows, 128), generator=g, device=dev).to(torch.bfloat16)
        dqk, dv, s["scale"], odt = 128, 128, 128 ** -0.5, torch.float32
    else:
        width = 576 if kv == "bf16" else KV8_ROW
        pool = torch.zeros((rows, width), dtype=torch.bfloat16 if kv == "bf16" else torch.uint8, device=dev)
        for at in range(0, rows, 1 << 20):
            x = torch.randn((min(1 << 20, rows - at), 576), generator=g, device=dev) / 24.0
            if kv == "bf16":
                pool[at:at + len(x)] = x.to(torch.bfloat16)
            else:
                q8, sc = _fp8_rows(x)
                pool[at:at + len(x), :576] = q8
                pool[at:at + len(x), 576:580] = sc[:, None].contiguous().view(torch.uint8)
        s["kpool"] = s["vpool"] = pool
        dqk, dv, s["scale"], odt = 576, 512, 1.0 / 24.0, torch.bfloat16
    s["qa"] = torch.empty((tq, Hq, dqk), dtype=torch.bfloat16, device=dev)
    for at in range(0, tq, 1024):
        s["qa"][at:at + 1024] = torch.randn((min(1024, tq - at), Hq, dqk), generator=g, device=dev)
    s["out"] = torch.empty((tq, Hq, dv), dtype=odt, device=dev)
    s["lse"] = torch.empty((tq, Hq), dtype=torch.float32, device=dev)


def prepare(case, seed):
    c, dev = case, torch.device("cuda:0")
    g = torch.Generator(device=dev)
    g.manual_seed(seed * 1000003 + 17)
    hist, new = _lengths(c)
    shape = _shape(c)
    rng = random.Random(seed)
    hot = [_hot(c, mh, rng) for mh, _, _ in shape]
    s = {"case": c, "dev": dev, "batch": janus.Batch(hist, new, device=dev, entry_shift=c["shift"])}
    op, tq = c["op"], s["batch"].total_q
    if op in ("scores", "layer", "decode"):
        _indexer(c if op != "decode" else dict(c, H=64, d=128), s, g, hot)
    if op != "scores":
        _pages(c, s, g)
        s["sel"] = torch.empty((tq, c["k"]), dtype=torch.int32, device=dev)
    if op == "select":
        # scores as the indexer leaves them: positive, the hot spans about
        # three times the others, -inf past each token's own position
        parts = []
        for (mh, ctx, cand), ids in zip(shape, hot):
            x = (torch.randn((len(cand), ctx), generator=g, device=dev) * 4.0 + 18.0).abs_()
            x[:, torch.from_numpy(ids).to(dev)] *= 3.0
            n = torch.tensor(cand, device=dev)
            x.masked_fill_(torch.arange(ctx, device=dev)[None, :] >= n[:, None], -math.inf)
            parts.append(x.reshape(-1))
        s["scores"] = torch.cat(parts) if len(parts) > 1 else parts[0]
        s["pred"] = _page_bits(s, g, 0.1)
    if op == "decode":
        s["resident"] = _page_bits(s, g, 0.9)
        s["ws"] = torch.empty(max(1, tq * 16 * c["heads"] * 514 * 4), dtype=torch.uint8, device=dev)
    if op == "attn":
        s["sel"] = _selection(c, s, g, hot)
    if op in ("attn", "decode", "layer"):
        _attention(c, s, g)
    return s


# ---- one pass --------------------------------------------------------------

def _run_scores(c, s):
    if c["keys"] == "mxfp4":
        return janus.index_scores_mxfp4(s["batch"], s["q"], s["kI"], s["bs"], s["w"], q_scale=s["sq"],
                                        scores=s["scores"])
    return janus.index_scores(s["batch"], s["q"], s["kI"], s["w"], q_scale=s["sq"], k_scale=s["sk"],
                              scores=s["scores"])


def _run_demand(c, s):
    return janus.page_demand(s["batch"], s["sel"], s["pt"], c["page"], s["P"], MAX_RUN, out=s["pd"])


def _run_attn(c, s):
    b, ps = s["batch"], c["page"]
    odt = "f32" if c["kv"] == "mqa" else "bf16"
    if c["kv"] == "fp8":
        return janus.sparse_attn_fp8kv(b, s["qa"], s["kpool"], s["pt"], ps, s["sel"], s["scale"],
                                       num_splits=0 if c["op"] == "decode" else 1, out_dtype=odt, out=s["out"],
                                       lse=s["lse"], workspace=s.get("ws"))
    if c["op"] == "decode":
        return janus.sparse_attn_split(b, s["qa"], s["kpool"], s["vpool"], s["pt"], ps, s["sel"], s["scale"],
                                       num_splits=0, dv=512, out_dtype=odt, out=s["out"], lse=s["lse"],
                                       workspace=s["ws"])
    return janus.sparse_attn(b, s["qa"], s["kpool"], s["vpool"], s["pt"], ps, s["sel"], s["scale"],
                             dv=128 if c["kv"] == "mqa" else 512, out_dtype=odt, out=s["out"], lse=s["lse"])


def run(state):
    c, s = state["case"], state
    if c["op"] == "scores":
        return {"scores": _run_scores(c, s)}
    if c["op"] == "attn":
        out, lse = _run_attn(c, s)
        return {"out": out, "lse": lse}
    if c["op"] == "select":
        if c["shards"]:
            janus.topk_sharded(s["batch"], s["scores"], c["k"], c["shards"], c["page"], out=s["sel"])
        else:
            janus.topk(s["batch"], s["scores"], c["k"], out=s["sel"])
        bm, lst, runs, cnt = _run_demand(c, s)
        miss, mruns, mcnt = janus.predict_diff(bm, s["pred"], s["P"], MAX_RUN, out=s["diff"])
        return {"sel": s["sel"], "pages": bm, "list": lst, "runs": runs, "counts": cnt, "miss": miss,
                "miss_runs": mruns, "miss_counts": mcnt}
    _run_scores(c, s)
    janus.topk(s["batch"], s["scores"], c["k"], out=s["sel"])
    bm, lst, runs, cnt = _run_demand(c, s)
    if c["op"] == "decode":
        # the ids, lists and counts in between feed the storage reads; one
        # swap of two equal scores moves all that follow it, so that the page
        # sets stand for them here
        miss = janus.predict_diff(bm, s["resident"], s["P"], MAX_RUN, out=s["diff"])[0]
        out, lse = _run_attn(c, s)
        return {"scores": s["scores"], "pages": bm, "miss": miss, "out": out, "lse": lse}
    out, lse = _run_attn(c, s)
    return {"scores": s["scores"], "sel": s["sel"], "pages": bm, "out": out, "lse": lse}


# ---- what a pass cannot do without ----------------------------------------

def work(case):
    c, shape = case, _shape(case)
    op, k = c["op"], c["k"]
    tq = sum(len(x[2]) for x in shape)
    ctx = sum(x[1] for x in shape)
    cells = sum(len(x[2]) * x[1] for x in shape)
    pairs = sum(sum(x[2]) for x in shape)
    picked = sum(sum(min(k, n) for n in x[2]) for x in shape)
    nbytes = flops = 0
    if op in ("scores", "decode", "layer"):
        H, d = c.get("H", 64), c.get("d", 128)
        el = {"fp8": 1, "mxfp4": 1, "bf16": 2, "f32": 4}[c["keys"]]
        key = {"fp8": d + 4, "mxfp4": d // 2 + d // 32, "bf16": 2 * d, "f32": 4 * d}[c["keys"]]
        nbytes += tq * H * (d * el + 4) + ctx * key + 4 * cells
        flops += 2 * H * d * pairs
    if op == "select":
        nbytes += 4 * pairs
    if op in ("select", "decode", "layer"):
        nbytes += 4 * tq * k + sum(-(-x[1] // c["page"]) for x in shape) // 8
    if op in ("attn", "decode", "layer"):
        mqa = c["kv"] == "mqa"
        dqk, dv = (128, 128) if mqa else (576, 512)
        row = {"mqa": 512, "bf16": 1152, "fp8": 580}[c["kv"]]
        nbytes += tq * c["heads"] * (2 * dqk + (4 if mqa else 2) * dv + 4) + 4 * tq * k
        nbytes += min(picked, ctx) * row
        flops += 2 * picked * c["heads"] * (dqk + dv)
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # measured against 64 bits and taken about four times: fp8 and MXFP4
    # scores round each head's term to bf16 twice; bf16 and fp32 scores sum in
    # fp32; attention rounds the probabilities (and mostly the output) to bf16
    if case["op"] == "select":
        return "exact"
    if case["op"] == "scores":
        return {"rel": {"fp8": 2.5e-3, "mxfp4": 2.5e-3, "bf16": 1e-5}[case["keys"]]}
    # differ: pages or ids that a swap of two scores one rounding apart moves
    return {"rel": 1e-2, "differ": 0.01}


# ---- the same in 64 bits ---------------------------------------------------

def _wide(x, keys):
    if keys == "fp8":
        return x.view(torch.float8_e4m3fn).to(torch.float64)
    return x.to(torch.float64)


def _exact_scores(c, s):
    H, d, dev = c.get("H", 64), c.get("d", 128), s["dev"]
    q = s["q"]
    if c["keys"] == "mxfp4":
        lut = torch.tensor(E2M1 + tuple(-v for v in E2M1), dtype=torch.float64, device=dev)
        n = s["kI"].shape[0]
        code = torch.stack([s["kI"] & 15, s["kI"] >> 4], dim=2).reshape(n, d)
        k = lut[code.long()].reshape(n, d // 32, 32) * torch.exp2(s["bs"].double() - 127)[:, :, None]
        k = k.reshape(n, d)
    else:
        k = _wide(s["kI"], c["keys"])
        if s["sk"] is not None:
            k = k * s["sk"].double()[:, None]
    out = torch.empty(s["batch"].total_scores, dtype=torch.float64, device=dev)
    at = row0 = key0 = 0
    for mh, ctx, cand in _shape(c):
        kb = k[key0:key0 + ctx].t().contiguous()
        n = torch.tensor(cand, device=dev)
        step = max(1, min(32, int(1.5e8 / (H * max(ctx, 1)))))
        for r in range(0, len(cand), step):
            m = min(step, len(cand) - r)
            qq = _wide(q[row0 + r:row0 + r + m], "fp8" if c["keys"] in ("fp8", "mxfp4") else "")
            p = torch.mm(qq.reshape(m * H, d), kb).clamp_(min=0).reshape(m, H, ctx)
            w = s["w"][row0 + r:row0 + r + m].double()
            if s["sq"] is not None:
                w = w * s["sq"][row0 + r:row0 + r + m].double()[:, None]
            v = torch.zeros((m, ctx), dtype=torch.float64, device=dev)
            for h in range(H):
                v.addcmul_(p[:, h], w[:, h, None])
            v.masked_fill_(torch.arange(ctx, device=dev)[None, :] >= n[r:r + m, None], -math.inf)
            out[at:at + m * ctx] = v.reshape(-1)
            at += m * ctx
        row0 += len(cand)
        key0 += ctx
    return out


def _exact_topk(c, s, scores):
    """Selections of the 64-bit scores, ascending and padded with -1."""
    k, at, rows = c["k"], 0, []
    for mh, ctx, cand in _shape(c):
        x = scores[at:at + len(cand) * ctx].reshape(len(cand), ctx)
        at += len(cand) * ctx
        ids = torch.topk(x, min(k, ctx), dim=1)[1]
        n = torch.tensor(cand, device=s["dev"])[:, None]
        ids = torch.where(torch.arange(ids.shape[1], device=s["dev"])[None, :] < n, ids, torch.full_like(ids, ctx))
        ids = torch.sort(ids, dim=1)[0]
        full = torch.full((len(cand), k), -1, dtype=torch.int64, device=s["dev"])
        full[:, :ids.shape[1]] = torch.where(ids < ctx, ids, torch.full_like(ids, -1))
        rows.append(full)
    return torch.cat(rows)


def _exact_attn(c, s, sel):
    dev, ps, kv = s["dev"], c["page"], c["kv"]
    dv = 128 if kv == "mqa" else 512
    tq, Hq = s["qa"].shape[:2]
    out = torch.empty((tq, Hq, dv), dtype=torch.float64, device=dev)
    lse = torch.empty((tq, Hq), dtype=torch.float64, device=dev)
    row0 = 0
    for b, (mh, ctx, cand) in enumerate(_shape(c)):
        for r in range(0, len(cand), 32):
            lo, hi = row0 + r, row0 + min(r + 32, len(cand))
            ids = sel[lo:hi].long()
            ok = ids >= 0
            ids = ids.clamp_min(0)
            slot = s["pt"][b].long()[ids // ps] * ps + ids % ps
            rows = s["kpool"][slot]
            if kv == "fp8":
                sc = rows[..., 576:580].contiguous().view(torch.float32).double()
                K = rows[..., :576].contiguous().view(torch.float8_e4m3fn).double() * sc
            else:
                K = rows.double()
            V = s["vpool"][slot].double() if kv == "mqa" else K[..., :dv]
            x = torch.bmm(s["qa"][lo:hi].double(), K.transpose(1, 2).contiguous()) * s["scale"]
            x.masked_fill_(~ok[:, None, :], -math.inf)
            lse[lo:hi] = torch.logsumexp(x, dim=2)
            p = torch.nan_to_num(torch.exp(x - lse[lo:hi, :, None]), nan=0.0)
            out[lo:hi] = torch.bmm(p, V.contiguous())
        row0 += len(cand)
    return out, lse


def exact(case, seed):
    c = case
    if c["op"] == "select":
        return None  # whole numbers throughout
    s = prepare(case, seed)
    if c["op"] == "attn":
        out, lse = _exact_attn(c, s, s["sel"])
        return {"out": out, "lse": lse}
    scores = _exact_scores(c, s)
    if c["op"] == "scores":
        return {"scores": scores}
    if c["keys"] == "f32":  # fp32 scores select as 64-bit ones do
        out, lse = _exact_attn(c, s, _exact_topk(c, s, scores))
        return {"scores": scores, "sel": None, "pages": None, "out": out, "lse": lse}
    if c["op"] == "decode":
        return {"scores": scores, "pages": None, "miss": None, "out": None, "lse": None}
    return {"scores": scores, "sel": None, "pages": None, "out": None, "lse": None}
