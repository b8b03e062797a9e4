"""The work a serving engine has this library do, as measurable cases: paged attention with fused rotary embedding in
decode and in question prefill, and the commit of new K/V into pages, through the package's public calls.

A case is one layer's call (the engine makes the same call for every layer). Requests are laid out by the library's
aligner from a seeded mix of private prompt text and reusable chunks with Zipfian popularity; the values of q, K and V
are drawn on the GPU from the seed alone. `structure` seeds the request mix, so that a case always has the same lengths.
"""
import math

import numpy as np
import torch

import paper_2512_16822_amd as M

PROMPT, CHUNK = M.SEG_PROMPT, M.SEG_CHUNK
TORCH_DT = {"f32": torch.float32, "bf16": torch.bfloat16, "f8e4m3": torch.float8_e4m3fn}
ELEM = {"f32": 4, "bf16": 2, "f8e4m3": 1}
E4M3_MAX = 448.0


def _case(name, kind, **kw):
    c = dict(kind=kind, dtype="bf16", B=1, Hq=32, Hkv=8, D=128, P=16, theta=5e5, prefix=0, chunks_lo=1, chunks_hi=1,
             chunk_tokens=512, pool=32, question=0, n_q=0, shared=True, masked=False, interleaved=False, structure=1)
    if name:
        c["name"] = name
    c.update(kw)
    return c


def listed():
    return [
        # the smallest call there is: one request, two chunks, fp32 (a bring-up or verification run); latency counts
        _case("decode_tiny_f32", "decode", dtype="f32", Hq=8, Hkv=8, D=64, theta=1e4, prefix=32, chunks_lo=2, chunks_hi=2,
              chunk_tokens=128, pool=2),
        # a lightly loaded server: four chats on a handful of documents, odd question length
        _case("decode_small_bf16", "decode", B=4, prefix=64, chunks_lo=3, chunks_hi=3, pool=4, question=30),
        # the ordinary decode batch of an 8B-class model: 64 requests of about 4.3 K tokens that share chunk pages
        _case("decode_shared_bf16", "decode", B=64, prefix=64, chunks_lo=8, chunks_hi=8, question=128),
        # the same batch where the engine builds a plan per decode step and reads a shared page once for several requests
        _case("decode_batched_bf16", "batched", B=64, prefix=64, chunks_lo=8, chunks_hi=8, question=128),
        # long contexts without sharing (every page belongs to one request; the engine says so with the hint)
        _case("decode_long_bf16", "decode", B=8, chunks_lo=64, chunks_hi=64, chunk_tokens=1024, pool=256, shared=False),
        # a large batch of mixed lengths on fp8 pages, 28 query heads on 4 KV heads
        _case("decode_mixed_fp8", "decode", dtype="f8e4m3", B=128, Hq=28, Hkv=4, P=32, theta=1e6, chunks_lo=4, chunks_hi=64,
              pool=128),
        # chunks of 500 tokens do not fill their pages: the engine that drops pad slots passes masks and positions
        _case("decode_padmask_bf16", "decode", B=64, prefix=60, chunks_lo=8, chunks_hi=8, chunk_tokens=500, question=121,
              masked=True),
        # time to first token: 256 question tokens per request over 16 K tokens of cached chunks
        _case("prefill_question_bf16", "prefill", B=16, prefix=48, chunks_lo=16, chunks_hi=16, chunk_tokens=1024, pool=64,
              question=256, n_q=256),
        # the same step of a server whose pages are fp8 (the requests that decode_mixed_fp8 later decodes)
        _case("prefill_question_fp8", "prefill", dtype="f8e4m3", B=8, Hq=28, Hkv=4, P=32, theta=1e6, chunks_lo=4,
              chunks_hi=24, pool=64, question=128, n_q=128),
        # question prefill of the engine that drops pad slots, ragged chunk and question lengths
        _case("prefill_padmask_bf16", "prefill", B=4, prefix=60, chunks_lo=8, chunks_hi=8, chunk_tokens=500, question=121,
              n_q=121, masked=True),
        # after the model has computed a batch's new chunks, first blocks and questions: their K/V go into fp8 pages
        _case("commit_new_fp8", "commit", dtype="f8e4m3", B=16, Hq=28, Hkv=4, P=32, theta=1e6, chunks_lo=16, chunks_hi=16,
              pool=128, question=128),
        # one layer of a decode step as the engine's loop runs it: the new token's K/V committed, then attention without
        # a workspace of the caller's
        _case("decode_step_bf16", "step", B=16, prefix=37, chunks_lo=2, chunks_hi=12, chunk_tokens=256, pool=16, question=75),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["decode", "decode", "batched", "masked_decode", "prefill", "prefill", "masked_prefill", "commit", "step"])
    masked = kind.startswith("masked")
    kind = kind[len("masked_"):] if masked else kind
    dtype = rng.choice(["bf16", "bf16", "f8e4m3"] if kind == "batched" else ["bf16", "bf16", "f8e4m3", "f32"])
    Hq, Hkv = rng.choice([(32, 8), (28, 4), (16, 2), (12, 12), (48, 8)])
    # the usual page size of each format and head size 128 most of the time, the other ones now and then
    P, D = (32 if dtype == "f8e4m3" else 16), 128
    if kind != "batched" and rng.random() < 0.25:
        P = 48 - P
    if kind != "batched" and rng.random() < 0.25:
        D = 64
    interleaved = kind in ("decode", "prefill") and rng.random() < 0.2
    chunk = _log(rng, 64, 1024)
    if not masked and rng.random() < 0.5:
        chunk = -(-chunk // P) * P
    hi = max(1, min(_log(rng, 1, 64), 24000 // chunk))
    lo = rng.randint(1, hi)
    question = _log(rng, 1, 300)
    n_q = 0
    B = _log(rng, 1, 64)
    if kind == "prefill":
        n_q = question
        B = _log(rng, 1, 8)
        # at most 2e7 (query token, slot) pairs (fp32: 4e6), so that a draw stays below the largest listed case
        room = (4e6 if dtype == "f32" else 2e7) / B / n_q - n_q - 64
        hi = max(1, min(hi, int(room / (chunk + P)))) if room > 0 else 1
        lo = min(lo, hi)
    elif kind == "decode" and dtype == "f32":
        B = min(B, 16)
    return _case(None, kind, dtype=dtype, B=B, Hq=Hq, Hkv=Hkv, D=D, P=P, theta=rng.choice([1e4, 5e5, 1e6]),
                 prefix=rng.choice([0, 33, 64]), chunks_lo=lo, chunks_hi=hi, chunk_tokens=chunk, pool=_log(rng, 2, 128),
                 question=question, n_q=n_q, shared=kind == "batched" or rng.random() < 0.7, masked=masked,
                 interleaved=interleaved, structure=rng.randint(2, 1 << 30))


# ------------------------------------------------------------------------------------------------ request layout
def _segments(c):
    """Segment lists of the batch: [prefix] chunks [question]; without sharing the chunks are private text."""
    rs = np.random.Generator(np.random.PCG64(c["structure"]))
    w = np.arange(1, c["pool"] + 1, dtype=np.float64) ** -1.1
    cdf = np.cumsum(w / w.sum())
    requests = []
    for _ in range(c["B"]):
        n = int(rs.integers(c["chunks_lo"], c["chunks_hi"] + 1))
        keys = np.minimum(np.searchsorted(cdf, rs.random(n), side="right"), c["pool"] - 1)
        segs = [(PROMPT, c["prefix"], 0)] if c["prefix"] else []
        segs += [(CHUNK, c["chunk_tokens"], 1 + int(k)) if c["shared"] else (PROMPT, c["chunk_tokens"], 0) for k in keys]
        if c["question"]:
            segs.append((PROMPT, c["question"], 0))
        requests.append(segs)
    return requests


def _layout(c):
    """Block tables, lengths and query positions of the batch, as the engine gets them from the aligner."""
    decode = c["kind"] != "prefill"
    requests = _segments(c)
    pool = M.Pool(1 << 20, c["P"])
    al = [pool.align_request(s, 1 if decode and c["kind"] != "commit" else 0) for s in requests]
    nb = [a["info"]["n_blocks"] for a in al]
    width = max(nb)
    bt, bp = np.zeros((c["B"], width), np.int32), np.zeros((c["B"], width), np.int32)
    bm = np.zeros((c["B"], width), np.uint32)
    for b, a in enumerate(al):
        bt[b, :nb[b]], bp[b, :nb[b]], bm[b, :nb[b]] = a["block_table"], a["block_pos"], a["block_valid"]
    kv = np.array([a["info"]["kv_len"] for a in al], np.int32)
    n_q = [c["n_q"] if c["kind"] == "prefill" else 1] * c["B"]
    q_pos = []
    for b, a in enumerate(al):
        last = int(kv[b]) - 1 - (a["info"]["n_pad_slots"] if c["masked"] else 0)
        q_pos += [last - n_q[b] + 1 + i for i in range(n_q[b])]
    used = np.unique(np.concatenate([bt[b, :nb[b]] for b in range(c["B"])]))
    return dict(requests=requests, bt=bt, bp=bp, bm=bm, kv=kv, nb=nb, n_q=n_q, q_pos=np.array(q_pos, np.int32),
                cu=np.concatenate([[0], np.cumsum(n_q)]).astype(np.int32), pages=int(bt.max()) + 1, used=int(used.size))


def _runs(c, lay):
    """What a prefill commits: a chunk that no earlier request of the batch brought wholly, the first block of every
    other one, and all private text. (request, first slot, tokens) each."""
    P, runs, seen = c["P"], [], set()
    for b, segs in enumerate(lay["requests"]):
        slot = 0
        for i, (kind, n, key) in enumerate(segs):
            blocks = -(-n // P)
            if kind == PROMPT:
                runs.append((b, slot, n))
            else:
                pad = blocks * P - n
                runs.append((b, slot + pad, n if key not in seen else min(n, P - pad)))
                seen.add(key)
            slot += blocks * P
    return runs


# ------------------------------------------------------------------------------------------------ inputs
def _pages(c, n, gen, dev):
    """K and V pages of N(0, 1) values in the storage layouts of the C header; fp8 with a scale per page."""
    X, H, D, P = 16 // ELEM[c["dtype"]], c["Hkv"], c["D"], c["P"]

    def make(shape):
        if c["dtype"] != "f8e4m3":
            return torch.randn(shape, generator=gen, device=dev, dtype=TORCH_DT[c["dtype"]]), None
        x = torch.randn(shape, generator=gen, device=dev)
        scale = x.abs().flatten(1).amax(1) / E4M3_MAX
        x.div_(scale.view(-1, *[1] * (len(shape) - 1))).clamp_(-E4M3_MAX, E4M3_MAX)
        return x.to(torch.float8_e4m3fn), scale

    k, ks = make((n, H, D // X, P, X))
    v, vs = make((n, H, D, P))
    return k, v, ks, vs


def _inputs(case, seed):
    """Everything the calls read, on the GPU."""
    c, dev = case, torch.device("cuda:0")
    lay = _layout(c)
    gen = torch.Generator(device=dev).manual_seed(int(seed))
    s = dict(c=c, lay=lay)
    s["k"], s["v"], s["ks"], s["vs"] = _pages(c, lay["pages"], gen, dev)
    src = torch.float32 if c["dtype"] == "f32" else torch.bfloat16
    i32 = lambda a: torch.from_numpy(np.ascontiguousarray(a).view(np.int32)).to(dev)
    s["bt"], s["kv"], s["q_pos"], s["cu"] = i32(lay["bt"]), i32(lay["kv"]), i32(lay["q_pos"]), i32(lay["cu"])
    if c["masked"]:
        s["bp"], s["bm"] = i32(lay["bp"]), i32(lay["bm"])
    if c["kind"] in ("commit", "step"):
        runs = _runs(c, lay) if c["kind"] == "commit" else [(b, int(lay["kv"][b]) - 1, 1) for b in range(c["B"])]
        s["runs"] = runs
        n = sum(r[2] for r in runs)
        s["k_new"] = torch.randn((n, c["Hkv"], c["D"]), generator=gen, device=dev, dtype=src)
        s["v_new"] = torch.randn((n, c["Hkv"], c["D"]), generator=gen, device=dev, dtype=src)
        s["run_req"], s["run_slot"] = i32(np.array([r[0] for r in runs], np.int32)), i32(np.array([r[1] for r in runs], np.int32))
        s["run_cu"] = i32(np.concatenate([[0], np.cumsum([r[2] for r in runs])]).astype(np.int32))
    if c["kind"] != "commit":
        s["q"] = torch.randn((len(lay["q_pos"]), c["Hq"], c["D"]), generator=gen, device=dev, dtype=src)
    return s


def prepare(case, seed):
    c, s = case, _inputs(case, seed)
    lay = s["lay"]
    if c["kind"] in ("commit", "step"):
        s["commit"] = M.make_commit_params(s["k_new"], s["v_new"], s["k"], s["v"], s["bt"], s["run_req"], s["run_slot"],
                                           s["run_cu"], k_scales=s["ks"], v_scales=s["vs"])
    if c["kind"] != "commit":
        s["out"] = torch.empty_like(s["q"])
        flags = (M.FLAG_ROPE_INTERLEAVED if c["interleaved"] else 0) | (0 if c["shared"] else M.FLAG_KV_READ_ONCE)
        make = lambda ws: M.make_params(
            s["q"], s["out"], s["k"], s["v"], s["bt"], s["kv"], s["q_pos"], rope_theta=c["theta"],
            cu_q_lens=s["cu"] if c["kind"] == "prefill" else None, k_scales=s["ks"], v_scales=s["vs"],
            block_positions=s.get("bp"), block_valid_mask=s.get("bm"), flags=flags, max_kv_len=int(lay["kv"].max()),
            max_q_len=max(lay["n_q"]), workspace=ws)
        if c["kind"] == "step":
            s["params"] = make(None)
        else:
            p = make(None)
            if c["kind"] == "batched":
                plan, s["info"] = M.decode_plan_build(lay["bt"], lay["kv"], c["P"], c["Hq"], c["Hkv"], p.kv_dtype)
                s["plan"] = torch.from_numpy(plan).to(s["q"].device)
                n = M.attn_decode_batched_workspace_size(p, s["info"])
            else:
                n = M.attn_workspace_size(p, c["kind"] == "prefill")
            s["ws"] = torch.empty(max(n, 256), dtype=torch.uint8, device=s["q"].device)
            s["params"] = make(s["ws"])
    return s


def _bits(t):
    return t.view({1: torch.uint8, 2: torch.int16, 4: torch.int32}[t.element_size()])


def run(state):
    kind = state["c"]["kind"]
    if kind == "commit":
        M.kv_commit(state["commit"])
        return {"k_pages": _bits(state["k"]), "v_pages": _bits(state["v"])}
    if kind == "step":
        M.kv_commit(state["commit"])
        M.attn_decode_noalloc(state["params"])
        return {"out": state["out"], "k_pages": _bits(state["k"]), "v_pages": _bits(state["v"])}
    if kind == "batched":
        M.attn_decode_batched(state["params"], state["plan"], state["info"])
    elif kind == "prefill":
        M.attn_prefill(state["params"])
    else:
        M.attn_decode(state["params"])
    return {"out": state["out"]}


# ------------------------------------------------------------------------------------------------ cost and error
def work(case):
    """Every distinct page read once, q and out once, the tables once; 4 D operations per visible (query head, slot)."""
    c, lay = case, _layout(case)
    e = 4 if c["dtype"] == "f32" else 2
    page = 2 * c["Hkv"] * c["D"] * c["P"] * ELEM[c["dtype"]]
    token = 2 * c["Hkv"] * c["D"]
    if c["kind"] == "commit":
        n = sum(r[2] for r in _runs(c, lay))
        return {"bytes": n * token * (e + ELEM[c["dtype"]]), "flops": 0}
    rows = len(lay["q_pos"]) * c["Hq"] * c["D"]
    tables = 4 * sum(lay["nb"]) * (3 if c["masked"] else 1)
    pairs = sum(int(lay["kv"][b]) * n - n * (n - 1) // 2 for b, n in enumerate(lay["n_q"]))
    extra = c["B"] * token * (e + ELEM[c["dtype"]]) if c["kind"] == "step" else 0
    scales = 8 * lay["used"] if c["dtype"] == "f8e4m3" else 0
    return {"bytes": lay["used"] * page + 2 * rows * e + tables + scales + extra, "flops": 4 * c["D"] * c["Hq"] * pairs}


def tolerance(case):
    if case["kind"] == "commit":
        return "exact"
    # about four times the largest error against 64 bits measured over listed and drawn cases: 1.9e-5 with fp32 pages
    # (rotary phases at positions of some ten thousand), 3.5e-3 with 16-bit operands and results
    return {"rel": 8e-5 if case["dtype"] == "f32" else 0.014}


def _rotate(x, pos, theta, interleaved):
    """x [n, heads, D] in 64 bits at positions pos [n]."""
    D = x.shape[-1]
    f = theta ** (-2.0 * torch.arange(D // 2, device=x.device, dtype=torch.float64) / D)
    a = pos.to(torch.float64)[:, None] * f
    cos, sin = a.cos()[:, None, :], a.sin()[:, None, :]
    if interleaved:
        x0, x1 = x[..., 0::2], x[..., 1::2]
        return torch.stack([x0 * cos - x1 * sin, x1 * cos + x0 * sin], -1).flatten(-2)
    x0, x1 = x[..., : D // 2], x[..., D // 2:]
    return torch.cat([x0 * cos - x1 * sin, x1 * cos + x0 * sin], -1)


def _commit_plain(s):
    """The decode step's commit with plain indexing (one token per request)."""
    c, X = s["c"], 16 // ELEM[s["c"]["dtype"]]
    for i, (b, slot, _) in enumerate(s["runs"]):
        page, sl = int(s["lay"]["bt"][b, slot // c["P"]]), slot % c["P"]
        for new, scale, pages in ((s["k_new"][i], s["ks"], s["k"]), (s["v_new"][i], s["vs"], s["v"])):
            x = new
            if c["dtype"] == "f8e4m3":
                x = (x.float() / scale[page]).clamp(-E4M3_MAX, E4M3_MAX).to(torch.float8_e4m3fn)
            if pages is s["k"]:
                _bits(pages)[page, :, :, sl, :] = _bits(x.reshape(c["Hkv"], c["D"] // X, X))
            else:
                _bits(pages)[page, :, :, sl] = _bits(x)


def exact(case, seed):
    c = case
    if c["kind"] == "commit":
        return None
    s = _inputs(c, seed)
    if c["kind"] == "step":
        _commit_plain(s)
    lay, dev = s["lay"], s["k"].device
    P, D, H, G = c["P"], c["D"], c["Hkv"], c["Hq"] // c["Hkv"]
    out = torch.zeros((len(lay["q_pos"]), c["Hq"], D), dtype=torch.float64, device=dev)
    for b in range(c["B"]):
        L, q0, q1 = int(lay["kv"][b]), int(lay["cu"][b]), int(lay["cu"][b + 1])
        idx = torch.from_numpy(lay["bt"][b, : -(-L // P)].astype(np.int64)).to(dev)
        wide = lambda pages, scale: pages[idx].to(torch.float64) * (1 if scale is None else scale[idx].double().view(-1, *[1] * (pages.dim() - 1)))
        k = wide(s["k"], s["ks"]).permute(0, 3, 1, 2, 4).reshape(-1, H, D)[:L]
        v = wide(s["v"], s["vs"]).permute(0, 3, 1, 2).reshape(-1, H, D)[:L]
        n = torch.arange(L, device=dev)
        pos, keep = n, torch.ones(L, dtype=torch.bool, device=dev)
        if c["masked"]:
            pos = s["bp"][b][n // P] + n % P
            keep = ((s["bm"][b][n // P] >> (n % P)) & 1).bool()
        q_pos = s["q_pos"][q0:q1]
        q = _rotate(s["q"][q0:q1].double(), q_pos, c["theta"], c["interleaved"]).view(q1 - q0, H, G, D)
        k = _rotate(k, pos, c["theta"], c["interleaved"])
        q = q.permute(1, 0, 2, 3).reshape(H, -1, D).contiguous()
        score = torch.matmul(q, k.permute(1, 2, 0).contiguous()) / math.sqrt(D)
        if c["kind"] == "prefill":
            keep = keep & (pos[None, :] <= q_pos[:, None]).repeat_interleave(G, 0)
        score.masked_fill_(~keep, -math.inf)
        o = torch.matmul(score.softmax(-1), v.permute(1, 0, 2).contiguous())
        out[q0:q1] = o.view(H, q1 - q0, G, D).permute(1, 0, 2, 3).reshape(q1 - q0, c["Hq"], D)
        del score
    if c["kind"] == "step":
        return {"out": out, "k_pages": None, "v_pages": None}
    return {"out": out}
