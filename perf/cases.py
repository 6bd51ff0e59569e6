"""Timed cases of the library: what its users have it do, through the binding's entry points.

Serving: a decode step (one index pass, one top-k, L attention layers) from one
short sequence to a batch of long ones, contiguous and paged; the same path
through its three separate calls, as a model whose layers follow one another
makes them; prefill of fresh prompts and of a chunk behind a long context; the
projections of new tokens with their cache write; dense attention of a decode
batch.  Training of the indexer: the dense causal forward of one layer, the
distillation target, and the loss with its gradients.

A case is a dict of plain values; ``kind`` names the path and the sizes follow
the library's own conventions (batch, n_q query rows per sequence, cached tokens
per sequence between len_lo and len_hi, heads, top_k, page_size, ...)."""
import math
import random

import torch

from paper_2606_06467_amd import binding as B

DEV = "cuda"
BF16, F32, F64, I32 = torch.bfloat16, torch.float32, torch.float64, torch.int32
D, IDX = 128, 256  # head dimension, index width


def _case(kind, batch, len_lo, len_hi, **kw):
    c = dict(kind=kind, batch=batch, n_q=1, len_lo=len_lo, len_hi=len_hi, top_k=2048, layers=1,
             q_heads=32, kv_heads=8, page_size=0, causal=False, planted=0, d_model=0,
             with_lse=False)
    c.update(kw)
    return c


def listed():
    return [
        # decoding one short conversation: launches and latency are all there is
        dict(_case("step", 1, 4096, 4096, top_k=512, layers=4), name="step_4k"),
        # a small batch of long contexts in contiguous caches, keys aligned with the query planted
        dict(_case("step", 4, 131072, 131072, layers=16, planted=64), name="step_128k"),
        # a serving batch: ragged lengths, 64-token pages in random physical order
        dict(_case("step", 32, 16384, 65536, layers=24, page_size=64), name="step_paged"),
        # a decode step through the separate index, top-k and attention calls, as a model whose
        # next layer's query needs the layer before issues them
        dict(_case("calls", 8, 20001, 32768, layers=8), name="calls_32k"),
        # fresh prompts of different lengths, padded on the left to one block of rows
        dict(_case("step", 2, 2900, 4096, n_q=4096, causal=True, layers=4, page_size=64),
             name="prefill_prompts"),
        # one chunk of a long prompt behind a 120K context
        dict(_case("step", 1, 131072, 131072, n_q=8192, causal=True, layers=16),
             name="prefill_128k"),
        # index query, index key, K and V of a decode batch's new tokens, into paged caches
        dict(_case("project", 32, 1500, 2048, page_size=64, d_model=2560), name="project_decode"),
        # the same for a prompt chunk
        dict(_case("project", 1, 16384, 16384, n_q=8192, d_model=2560), name="project_prefill"),
        # dense attention of a decode batch (what sparse attention is compared with)
        dict(_case("dense", 8, 32768, 32768), name="dense_decode"),
        # the dense causal forward of one cross-decoder layer in training, with the
        # log-sum-exps that the distillation target takes (20 query / 4 KV heads)
        dict(_case("dense", 1, 8192, 8192, n_q=8192, causal=True, q_heads=20, kv_heads=4,
                   with_lse=True), name="dense_train"),
        # the distillation target of every layer's attention, its own statistics pass included
        dict(_case("target", 1, 16384, 16384, n_q=16384, causal=True, layers=16),
             name="kd_target"),
        # the distillation loss and its gradients over a whole training sequence
        dict(_case("loss", 1, 32768, 32768, n_q=32768, causal=True), name="kd_loss"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same kinds and ranges."""
    qh, kvh = rng.choice([(32, 8), (32, 8), (20, 4), (64, 8), (8, 8)])
    heads = dict(q_heads=qh, kv_heads=kvh)
    page = rng.choice([0, 64])
    k = rng.choice([512, 1024, 2048, rng.randint(100, 2048)])
    what = rng.choice(["decode", "decode", "calls", "prompts", "chunk", "project_decode",
                       "project_prefill", "dense_decode", "dense_train", "target", "loss"])
    if what in ("decode", "calls"):
        batch = _log(rng, 1, 32)
        hi = _log(rng, 3000, min(131072, 2000000 // batch))
        lo = rng.randint(max(1, hi // 4), hi)
        return _case("step" if what == "decode" else "calls", batch, lo, hi, top_k=k,
                     layers=rng.randint(2, 16), page_size=page,
                     planted=rng.choice([0, 64]) if page == 0 else 0, **heads)
    if what == "prompts":
        batch = rng.randint(1, 4)
        t = _log(rng, 200, 16384 // batch)
        return _case("step", batch, rng.randint(max(1, t // 2), t), t, n_q=t, causal=True,
                     top_k=k, layers=rng.randint(1, 4), page_size=page, **heads)
    if what == "chunk":
        t = _log(rng, 256, 4096)
        n = _log(rng, 2 * t, 131072)
        return _case("step", 1, n, n, n_q=t, causal=True, top_k=k, layers=rng.randint(1, 4),
                     page_size=page, **heads)
    if what == "project_decode":
        return _case("project", rng.randint(1, 64), 1000, 2048, page_size=page,
                     d_model=512 * rng.randint(2, 8), **heads)
    if what == "project_prefill":
        t = _log(rng, 100, 8192)
        return _case("project", 1, 16384, 16384, n_q=t, page_size=page,
                     d_model=512 * rng.randint(2, 8), **heads)
    if what == "dense_decode":
        batch = _log(rng, 1, 32)
        hi = _log(rng, 2000, min(131072, 500000 // batch))
        return _case("dense", batch, rng.randint(max(1, hi // 4), hi), hi, page_size=page,
                     with_lse=rng.random() < 0.5, **heads)
    if what == "dense_train":
        batch = rng.randint(1, 3)
        t = _log(rng, 500, 8192 // batch)
        return _case("dense", batch, rng.randint(max(1, t // 2), t), t, n_q=t, causal=True,
                     page_size=page, with_lse=True, **heads)
    if what == "target":
        batch = rng.randint(1, 2)
        t = _log(rng, 500, 8192 // batch)
        return _case("target", batch, rng.randint(max(1, t // 2), t), t, n_q=t, causal=True,
                     page_size=page, layers=rng.randint(2, 16), with_lse=rng.random() < 0.5,
                     **heads)
    batch = rng.randint(1, 3)
    t = _log(rng, 700, 20000 // batch)
    return _case("loss", batch, rng.randint(max(1, t // 2), t), t, n_q=t, causal=True,
                 page_size=page)


def _lens(c):
    """Cached tokens of each sequence: the longest first, the rest between the two bounds."""
    r = random.Random(c["batch"] * 1000003 + c["len_lo"])
    return [c["len_hi"]] + [r.randint(c["len_lo"], c["len_hi"]) for _ in range(c["batch"] - 1)]


def _max_len(c):
    p = c["page_size"]
    return -(-c["len_hi"] // p) * p if p else c["len_hi"]


def _valid(c):
    """Valid keys of every row (b, t), as lists: causal rows are the last n_q of their sequence."""
    t = c["n_q"]
    return [[max(0, n - t + i + 1) if c["causal"] else n for i in range(t)] for n in _lens(c)]


def _shape(c):
    m = _max_len(c)
    p = c["page_size"]
    return B.make_shape(c["batch"], c["n_q"], m, c["top_k"], q_heads=c["q_heads"],
                        kv_heads=c["kv_heads"], page_size=p, max_pages=m // p if p else 0,
                        causal=c["causal"])


def _rand(gen, shape, scale=1.0):
    """N(0, scale^2) in bfloat16, made in blocks."""
    out = torch.empty(shape, dtype=BF16, device=DEV)
    flat = out.view(-1)
    for i in range(0, flat.numel(), 1 << 27):
        n = min(1 << 27, flat.numel() - i)
        flat[i:i + n] = torch.randn(n, generator=gen, device=DEV).mul_(scale)
    return out


def _rows_shape(c):
    p = c["page_size"]
    return (sum(-(-n // p) for n in _lens(c)), p) if p else (c["batch"], _max_len(c))


def _page_table(c, seed):
    p = c["page_size"]
    if not p:
        return None
    need = [-(-n // p) for n in _lens(c)]
    perm = torch.randperm(sum(need), generator=torch.Generator().manual_seed(seed)).to(I32)
    pt = torch.full((c["batch"], _max_len(c) // p), -1, dtype=I32)
    at = 0
    for b, n in enumerate(need):
        pt[b, :n] = perm[at:at + n]
        at += n
    return pt.to(DEV)


def prepare(c, seed):
    """Inputs, output buffers and workspace of one case."""
    gen = torch.Generator(device=DEV).manual_seed(seed)
    kind, bt, t = c["kind"], c["batch"], c["n_q"]
    lens, rows = _lens(c), _rows_shape(c)
    hq, hkv, nl = c["q_heads"], c["kv_heads"], c["layers"]
    s = dict(case=c, shape=_shape(c), page_table=_page_table(c, seed))
    s["seq_lens"] = torch.tensor(lens, dtype=I32, device=DEV)
    s["q_pos"] = None
    if c["causal"]:  # rows before a shorter sequence's first token see nothing
        s["q_pos"] = torch.tensor([[n - t + i for i in range(t)] for n in lens], dtype=I32,
                                  device=DEV)
    if kind in ("step", "calls", "loss"):
        s["q_idx"] = _rand(gen, (bt, t, 4, 64), 1 / 8)
        s["k_idx"] = _rand(gen, rows + (4, 64), 1 / 8)
        if c["planted"]:  # some tokens' index keys aligned with the query, three deviations up
            for b, n in enumerate(lens):
                q = s["q_idx"][b, 0].float()
                at = torch.randperm(n, generator=gen, device=DEV)[:c["planted"]]
                s["k_idx"][b, at] = (s["k_idx"][b, at].float() + 3 / 8 * q / q.norm()).to(BF16)
    if kind in ("step", "calls", "dense", "target"):
        s["k_cache"] = _rand(gen, rows + (hkv, D))
        s["q"] = _rand(gen, (nl, bt, t, hq, D))
    if kind in ("step", "calls", "dense"):
        s["v_cache"] = _rand(gen, rows + (hkv, D))
        s["out"] = torch.zeros((nl, bt, t, hq, D), dtype=BF16, device=DEV)
        s["lse"] = torch.zeros((nl, bt, t, hq), device=DEV)
    if kind in ("step", "calls"):
        s["idx"] = torch.zeros((bt, t, c["top_k"]), dtype=I32, device=DEV)
        s["n_sel"] = torch.zeros((bt, t), dtype=I32, device=DEV)
    if kind == "step":
        s["ws"] = B.workspace(s["shape"], B.CLSA_OP_DECODE, nl, DEV)
    elif kind == "calls":
        s["scores"] = torch.zeros((bt, t, _max_len(c)), device=DEV)
        s["ws_topk"] = B.workspace(s["shape"], B.CLSA_OP_TOPK, 0, DEV)
        s["ws_attn"] = B.workspace(s["shape"], B.CLSA_OP_ATTN, 0, DEV)
    elif kind == "dense":
        s["ws"] = B.workspace(s["shape"], B.CLSA_OP_DENSE, 0, DEV)
    elif kind == "target":
        s["ws"] = B.workspace(s["shape"], B.CLSA_OP_KD_TARGET, nl, DEV)
        s["abar"] = torch.zeros((bt, t, _max_len(c)), device=DEV)
        s["fwd_lse"] = None
        if c["with_lse"]:  # as the dense forward of every layer returns them
            s["fwd_lse"] = torch.empty((nl, bt, t, hq), device=DEV)
            ws = B.workspace(s["shape"], B.CLSA_OP_DENSE, 0, DEV)
            out = torch.empty((bt, t, hq, D), dtype=BF16, device=DEV)
            for l in range(nl):
                B.clsa_dense_attn(s["shape"], s["q"][l], s["k_cache"], s["k_cache"],
                                  s["page_table"], s["seq_lens"], s["q_pos"], out,
                                  s["fwd_lse"][l], ws)
    elif kind == "loss":
        s["ws"] = B.workspace(s["shape"], B.CLSA_OP_KD_LOSS, 0, DEV)
        s["abar"] = torch.zeros((bt, t, _max_len(c)), device=DEV)
        keys = torch.arange(_max_len(c), device=DEV)
        for b in range(bt):  # a peaked distribution over the row's keys
            for i in range(0, t, 2048):
                lim = s["q_pos"][b, i:i + 2048, None] + 1
                z = torch.randn((lim.shape[0], keys.numel()), generator=gen, device=DEV)
                z.masked_fill_(keys >= lim, -math.inf)
                s["abar"][b, i:i + 2048] = torch.softmax(z, -1).nan_to_num_(0.0)
        s["loss"] = torch.zeros(1, device=DEV)
        s["dq"] = torch.zeros((bt, t, IDX), device=DEV)
        s["dk"] = torch.zeros(rows + (IDX,), device=DEV)
    elif kind == "project":
        nf = 512 + 2 * hkv * D
        s["h"] = _rand(gen, (bt, t, c["d_model"]))
        s["w"] = _rand(gen, (nf, c["d_model"]), c["d_model"] ** -0.5)
        s["pos"] = torch.tensor([[n - t + i for i in range(t)] for n in lens], dtype=I32,
                                device=DEV)
        s["q_idx"] = torch.zeros((bt, t, 4, 64), dtype=BF16, device=DEV)
        s["k_idx"] = torch.zeros(rows + (4, 64), dtype=BF16, device=DEV)
        s["k_cache"] = torch.zeros(rows + (hkv, D), dtype=BF16, device=DEV)
        s["v_cache"] = torch.zeros(rows + (hkv, D), dtype=BF16, device=DEV)
    return s


def run(s):
    """One pass through the library's entry points."""
    c, sh, pt, sl, qp = s["case"], s["shape"], s["page_table"], s["seq_lens"], s["q_pos"]
    kind = c["kind"]
    if kind == "step":
        B.clsa_decode_step(sh, s["q_idx"], s["k_idx"], s["k_cache"], s["v_cache"], pt, sl, qp,
                           s["q"], s["out"], s["lse"], s["idx"], s["n_sel"], s["ws"])
        return {"out": s["out"], "lse": s["lse"], "idx": s["idx"], "n_sel": s["n_sel"]}
    if kind == "calls":
        B.clsa_index_scores(sh, s["q_idx"], s["k_idx"], pt, sl, qp, s["scores"])
        B.clsa_topk(sh, s["scores"], sl, qp, s["idx"], s["n_sel"], s["ws_topk"])
        for l in range(c["layers"]):
            B.clsa_sparse_attn(sh, s["q"][l], s["k_cache"], s["v_cache"], pt, s["idx"],
                               s["n_sel"], s["out"][l], s["lse"][l], s["ws_attn"])
        return {"out": s["out"], "lse": s["lse"], "idx": s["idx"], "n_sel": s["n_sel"],
                "scores": s["scores"]}
    if kind == "dense":
        lse = s["lse"][0] if c["with_lse"] else None
        B.clsa_dense_attn(sh, s["q"][0], s["k_cache"], s["v_cache"], pt, sl, qp, s["out"][0], lse,
                          s["ws"])
        return {"out": s["out"], "lse": lse}
    if kind == "target":
        B.clsa_kd_target(sh, c["layers"], s["q"], s["k_cache"], pt, sl, qp, s["abar"], s["ws"],
                         lse_layers=s["fwd_lse"])
        return {"abar": s["abar"]}
    if kind == "loss":
        B.clsa_kd_loss(sh, s["abar"], s["q_idx"], s["k_idx"], pt, sl, qp, s["loss"], s["dq"],
                       s["dk"], s["ws"])
        return {"loss": s["loss"], "dq": s["dq"], "dk": s["dk"]}
    B.clsa_project_append(sh, c["d_model"], s["h"], s["w"], s["pos"], pt, s["q_idx"], s["k_idx"],
                          s["k_cache"], s["v_cache"])
    return {"q_idx": s["q_idx"], "k_idx": s["k_idx"], "k_cache": s["k_cache"],
            "v_cache": s["v_cache"]}


def work(c):
    """Bytes (each input read once, each output written once) and operations of one pass."""
    kind, rows, hq, hkv, nl = c["kind"], c["batch"] * c["n_q"], c["q_heads"], c["kv_heads"], \
        c["layers"]
    valid = [n for b in _valid(c) for n in b]
    pairs, tokens = float(sum(valid)), float(sum(_lens(c)))
    qo = rows * hq * (2 * 2 * D + 4)            # a layer's queries, outputs, log-sum-exps
    if kind in ("step", "calls"):
        sel = float(sum(min(c["top_k"], n) for n in valid))
        kv = min(tokens, sel) * hkv * 2 * 2 * D  # selected K and V rows, at most all of them
        by = tokens * 2 * IDX + rows * 2 * IDX + kv + nl * qo + rows * c["top_k"] * 4
        by += pairs * 4 if kind == "calls" else 0
        return {"bytes": by, "flops": pairs * 2 * IDX + nl * sel * hq * 4 * D}
    if kind == "dense":
        return {"bytes": tokens * hkv * 4 * D + qo, "flops": pairs * hq * 4 * D}
    if kind == "target":
        return {"bytes": tokens * hkv * 2 * D + nl * rows * hq * 2 * D + pairs * 4,
                "flops": pairs * nl * hq * 2 * D}
    if kind == "loss":
        return {"bytes": pairs * 4 + (tokens + rows) * IDX * (2 + 4), "flops": pairs * 6 * IDX}
    nf = 512 + 2 * hkv * D
    return {"bytes": 2.0 * (rows + nf) * c["d_model"] + 2.0 * rows * nf,
            "flops": 2.0 * rows * nf * c["d_model"]}


def tolerance(c):
    """bf16 results of fp32 sums; a tie of two scores within rounding may fall either way."""
    kind = c["kind"]
    if kind in ("step", "calls"):
        return {"rel": 1e-2, "max": 0.1, "differ": 0.01}
    if kind == "dense":
        return {"rel": 1e-2, "max": 0.1}
    if kind == "target":
        return {"rel": 1e-5, "max": 1e-4}
    if kind == "loss":
        return {"rel": 2e-5, "max": 2e-3}
    return {"rel": 2e-3, "max": 0.02}


def _tokens(s, c, cache, b, n):
    """Rows 0 .. n-1 of sequence b of a cache."""
    if c["page_size"]:
        return cache[s["page_table"][b, :-(-n // c["page_size"])].long()].flatten(0, 1)[:n]
    return cache[b, :n]


def _exact_attn(c, q, k, v, keep):
    """q [T, Hq, D], k and v [N, Hkv, D], keep [T, N]: out and natural-log log-sum-exp."""
    t, g = q.shape[0], c["q_heads"] // c["kv_heads"]
    out = torch.zeros((t, c["q_heads"], D), dtype=F64, device=DEV)
    lse = torch.full((t, c["q_heads"]), -math.inf, dtype=F64, device=DEV)
    some = keep.any(-1)
    for h in range(c["q_heads"]):
        z = (q[:, h].double() @ k[:, h // g].double().T.contiguous()) * (1 / math.sqrt(D))
        z.masked_fill_(~keep, -math.inf)
        lse[:, h] = torch.logsumexp(z, -1)
        p = torch.exp(z - lse[:, h].masked_fill(~some, 0.0)[:, None])
        out[:, h] = p @ v[:, h // g].double()
    return out, lse


def exact(c, seed):
    """What run() returns, in 64 bits; None where that takes too long."""
    kind, bt, t, nl = c["kind"], c["batch"], c["n_q"], c["layers"]
    valid = _valid(c)
    pairs = sum(sum(v) for v in valid)
    if kind in ("step", "calls") and t > 1 and nl * t * sum(_lens(c)) > 4.2e8 / (c["q_heads"] / 32):
        return None
    if kind == "target" and pairs * nl * c["q_heads"] > 7.5e10:
        return None
    s = prepare(c, seed)
    lens = _lens(c)
    if kind in ("step", "calls", "dense"):
        out = torch.zeros((nl, bt, t, c["q_heads"], D), dtype=F64, device=DEV)
        lse = torch.zeros((nl, bt, t, c["q_heads"]), dtype=F64, device=DEV)
        idx = torch.full((bt, t, c["top_k"]), -1, dtype=I32, device=DEV)
        n_sel = torch.zeros((bt, t), dtype=I32, device=DEV)
        scores = torch.zeros((bt, t, _max_len(c)), dtype=F64, device=DEV) if kind == "calls" \
            else None
        for b, n in enumerate(lens):
            lim = torch.tensor(valid[b], device=DEV)
            keep = torch.arange(n, device=DEV) < lim[:, None]
            k, v = _tokens(s, c, s["k_cache"], b, n), _tokens(s, c, s["v_cache"], b, n)
            if kind != "dense":
                ki = _tokens(s, c, s["k_idx"], b, n).flatten(1).double()
                sc = s["q_idx"][b].flatten(1).double() @ ki.T.contiguous()
                if scores is not None:
                    scores[b, :, :n] = sc.masked_fill(~keep, 0.0)
                # the selection is decided on the scores rounded to 32 bits, ties to the lowest
                order = torch.sort(sc.float().masked_fill(~keep, -math.inf), dim=-1,
                                   descending=True, stable=True).indices
                m = min(n, c["top_k"])
                n_sel[b] = lim.clamp(max=c["top_k"]).to(I32)
                took = torch.where(torch.arange(m, device=DEV) < n_sel[b, :, None],
                                   order[:, :m], n)
                took = took.sort(-1).values
                idx[b, :, :m] = torch.where(took < n, took, -1).to(I32)
                keep = torch.zeros((t, n + 1), dtype=torch.bool, device=DEV).scatter_(1, took, True)
                keep = keep[:, :n]
                if t == 1:
                    at = took[0, :int(n_sel[b, 0])]
                    k, v, keep = k[at], v[at], keep[:, at]
            for l in range(nl):
                out[l, b], lse[l, b] = _exact_attn(c, s["q"][l, b], k, v, keep)
        if kind == "dense":
            return {"out": out, "lse": lse[0] if c["with_lse"] else None}
        r = {"out": out, "lse": lse, "idx": idx, "n_sel": n_sel}
        return dict(r, scores=scores) if kind == "calls" else r
    if kind == "target":
        abar = torch.zeros((bt, t, _max_len(c)), dtype=F64, device=DEV)
        g = c["q_heads"] // c["kv_heads"]
        for b, n in enumerate(lens):
            k = _tokens(s, c, s["k_cache"], b, n).double()
            for i in range(0, t, 4096):
                lim = torch.tensor(valid[b][i:i + 4096], device=DEV)
                m = int(lim.max())
                drop = torch.arange(m, device=DEV) >= lim[:, None]
                for l in range(nl):
                    for h in range(c["q_heads"]):
                        z = s["q"][l, b, i:i + 4096, h].double() @ k[:m, h // g].T.contiguous()
                        z.mul_(1 / math.sqrt(D)).masked_fill_(drop, -math.inf)
                        abar[b, i:i + 4096, :m] += torch.softmax(z, -1).nan_to_num_(0.0)
        return {"abar": abar.div_(nl * c["q_heads"])}
    if kind == "loss":
        rows = sum(sum(x > 0 for x in v) for v in valid)
        loss = torch.zeros(1, dtype=F64, device=DEV)
        dq = torch.zeros((bt, t, IDX), dtype=F64, device=DEV)
        dk = torch.zeros(s["dk"].shape, dtype=F64, device=DEV)
        for b, n in enumerate(lens):
            ki = _tokens(s, c, s["k_idx"], b, n).flatten(1).double()
            qi = s["q_idx"][b].flatten(1).double()
            acc = torch.zeros((n, IDX), dtype=F64, device=DEV)
            for i in range(0, t, 4096):
                lim = torch.tensor(valid[b][i:i + 4096], device=DEV)
                drop = torch.arange(n, device=DEV) >= lim[:, None]
                z = (qi[i:i + 4096] @ ki.T.contiguous()).masked_fill_(drop, -math.inf)
                logq = torch.log_softmax(z, -1)
                p = s["abar"][b, i:i + 4096, :n].double()
                kl = torch.where(p > 0, p * (p.log() - logq), 0.0)
                loss += kl.masked_fill_(drop, 0.0).sum()
                di = (logq.exp() - p).masked_fill_(drop, 0.0).nan_to_num_(0.0) / rows
                dq[b, i:i + 4096] = di @ ki
                acc += di.T.contiguous() @ qi[i:i + 4096]
            if c["page_size"]:
                j = torch.arange(n, device=DEV)
                page = s["page_table"][b, j // c["page_size"]].long()
                dk[page, j % c["page_size"]] = acc
            else:
                dk[b, :n] = acc
        return {"loss": loss / rows, "dq": dq, "dk": dk}
    y = s["h"].double() @ s["w"].double().T.contiguous()
    r = {"q_idx": y[..., :IDX].reshape(bt, t, 4, 64)}
    at = {"k_idx": (IDX, 2 * IDX), "k_cache": (512, 512 + c["kv_heads"] * D),
          "v_cache": (512 + c["kv_heads"] * D, 512 + 2 * c["kv_heads"] * D)}
    for name, (lo, hi) in at.items():
        r[name] = s[name].double()
        for b, n in enumerate(lens):
            j = torch.arange(n - t, n, device=DEV)
            new = y[b, :, lo:hi].reshape((t,) + s[name].shape[2:])
            if c["page_size"]:
                r[name][s["page_table"][b, j // c["page_size"]].long(), j % c["page_size"]] = new
            else:
                r[name][b, j] = new
    return r
