"""The work this library does for its users, as measurable cases.

A case names one call of the public binding (or the calls of one decode step, with the host tier) on
synthetic inputs of a stated shape.  The listed cases are the calls a serving program makes: decode steps from a short prompt to
a batch of million-token ones, the paper's serving variant (E4M3 rows in pages, dynamic RoPE), a step that
re-uses cached masks, chunked prefill with and without RoPE, the single stages of the path where a stage is what can be compared
value by value, and a decode step whose K/V live in host memory.  `draw` gives other sizes of the same calls.

Shapes follow the repository's own workloads: 128 dims per head, 32 query heads on 8 KV heads (other group sizes are drawn), sink 128 and
window 1024, keys and queries ~ N(0,1) with 16 planted needles per KV head in decode.
"""
import math

import torch

import paper_2502_08910_amd as ih

D = 128
FP8_SCALE = 1.0 / 64          # of the E4M3 tensors: N(0,1) values fill the format's range


def case_of(name, op, **kw):
    c = dict(op=op, B=1, Hq=32, Hkv=8, T=0, ragged=False, Tq=1, b_q=1, n_sink=128, n_stream=1024, stages="", kv="bf16",
             page=0, rope="none", pooling="kv_head", bank_blocks=0)
    c.update(kw)
    if name:
        c["name"] = name
    return c


DECODE3 = "64:512,16:512,4:512"
DECODE4 = "256:256,64:256,16:512,4:1024"
PREFILL2 = "64:256,16:256"


def listed():
    return [
        # a chat-length context, one sequence: the smallest step, a chain of short kernels
        case_of("decode-8k", "decode", T=8192, stages="64:64,16:64,4:128"),
        # one long document
        case_of("decode-128k", "decode", T=131072, stages=DECODE3),
        # a batch of very long contexts: the repository's headline benchmark
        case_of("decode-1m-b8", "decode", B=8, T=1048576, stages=DECODE4),
        # the paper's serving configuration (8-bit K/V in 16-token pages, relative-style RoPE), sequences of unequal length
        case_of("decode-serving-250k-b4", "decode", B=4, T=250007, ragged=True, stages=DECODE4, kv="fp8", page=16, rope="relative"),
        # most steps of a real generation: the coarse stages' lists are cached, only the last stage and the attention run
        case_of("decode-masked-100k-b16", "masked", B=16, T=100003, ragged=True, stages=DECODE3),
        # one prompt chunk on a long prefix: the repository's prefill benchmark
        case_of("prefill-4k-on-256k", "prefill", T=262144 + 4096, Tq=4096, b_q=64, stages=PREFILL2),
        # the same step with the dynamic RoPE of most layers
        case_of("prefill-rope-2k-on-128k", "prefill", T=131072 + 2048, Tq=2048, b_q=64, stages=PREFILL2, rope="relative"),
        # a short chunk for two users, small blocks, 8-bit pages, ragged
        case_of("prefill-fp8-paged-512-b2", "prefill", B=2, T=33001, ragged=True, Tq=512, b_q=32, stages="32:128,8:256", kv="fp8", page=64),
        # first pruning stage of a prefill chunk in the first layers, whose RoPE is chunk-indexed (a chunk's index is its
        # position, so the stage, not the whole layer, is what two correct programs agree on)
        case_of("prune-prefill-chunk-rope", "prune", T=131072 + 4096, Tq=4096, b_q=64, stages="64:256", rope="chunk"),
        # attention of a prefill chunk over a longer key list, streaming-style RoPE, 8-bit rows
        case_of("attn-prefill-rope-fp8", "attn_prefill", T=100000 + 2048, Tq=2048, b_q=64, stages="16:512", kv="fp8", rope="streaming"),
        # arg-top-K alone, a first stage of a prefill chunk
        case_of("select-prefill", "select", T=262144 + 4096, Tq=4096, b_q=64, stages="64:256"),
        # a decode step whose K/V live in pinned host memory behind the hot-block banks, with the LRU update after it
        case_of("decode-offload-128k", "offload", T=131072, stages="256:128,64:128,16:256,4:512", bank_blocks=4096),
    ]


def draw(rng):
    """One more case: a kind, then sizes spread over its range (logarithmically where it is wide)."""
    def log(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    heads = rng.choice(["32/8", "32/8", "64/8", "16/8", "8/8", "16/4"])
    Hq, Hkv = (int(x) for x in heads.split("/"))
    base = dict(Hq=Hq, Hkv=Hkv, n_sink=rng.choice([64, 128, 256, 100]), n_stream=rng.choice([512, 1024, 1000, 2048]))
    kind = rng.choice(["decode", "decode", "decode", "masked", "prefill", "prefill", "prune", "attn_prefill", "attn_decode", "select", "offload"])
    kv, page = rng.choice([("bf16", 0), ("bf16", 0), ("bf16", 16), ("fp8", 0), ("fp8", 64)])
    if kind in ("decode", "masked"):
        T = log(4096, 1 << 20) | 1
        B = max(1, min(log(1, 32), (4 << 20) // T))
        l = rng.choice([64, 128, 256])
        keep = rng.choice([64, 96, 128, 256])
        st = f"{l}:{keep},16:{2 * keep},4:{rng.choice([2, 4]) * keep}"
        if kind == "masked":
            kv, page = "bf16", 0
        rope = rng.choice(["none", "none", "relative"]) if kind == "decode" else "none"
        return case_of("", kind, B=B, T=T, ragged=B > 1, stages=st, kv=kv, page=page, rope=rope,
                       pooling=rng.choice(["kv_head", "kv_head", "all_heads"]) if kind == "decode" else "kv_head", **base)
    if kind == "attn_decode":
        B = log(1, 32)
        T = log(8192, 262144) | 1
        while B * T > 1 << 21:
            B = max(1, B // 2)
        return case_of("", kind, B=B, T=T, ragged=B > 1, stages=f"{rng.choice([4, 8, 16])}:{log(48, 512)}", kv=kv, page=0 if kv == "fp8" else page, **base)
    if kind == "offload":
        T = log(16384, 131072) | 1
        return case_of("", kind, T=T, stages="256:64,64:64,16:128,4:256", bank_blocks=log(512, 8192), **base)
    # prefill: blocks of queries
    b_q = rng.choice([64, 64, 32, 16])
    Tq = b_q * log(2, 2048 // b_q)
    T = Tq + (log(4096, 131072) | 1)
    if kind == "select":
        return case_of("", kind, T=T, Tq=Tq, b_q=b_q, stages=f"{rng.choice([32, 64])}:{log(32, 512)}", **base)
    if kind == "prune":
        return case_of("", kind, T=T, Tq=Tq, b_q=b_q, stages=f"{rng.choice([16, 32, 64])}:256", rope=rng.choice(["chunk", "chunk", "relative", "none"]), **base)
    if kind == "attn_prefill":
        return case_of("", kind, T=T, Tq=Tq, b_q=b_q, stages=f"{rng.choice([8, 16, 32])}:{log(16, 256)}", kv=kv, page=0 if kv == "fp8" else page,
                       rope=rng.choice(["none", "none", "streaming"]), **base)
    return case_of("", kind, T=T, Tq=Tq, b_q=b_q, stages=f"{rng.choice([32, 64])}:{log(64, 256)},{rng.choice([8, 16])}:{log(64, 256)}", kv=kv, page=page,
                   rope=rng.choice(["none", "none", "relative"]), **base)


# ---- inputs ------------------------------------------------------------------
def _plan(case):
    st = [tuple(int(x) for x in s.split(":")) for s in case["stages"].split(",")]
    return [s[0] for s in st], [s[1] for s in st]


def _seq_lens(case, gen):
    B, T = case["B"], case["T"]
    lens = torch.full((B,), T, dtype=torch.int64, device="cuda")
    if case["ragged"]:
        cut = torch.randint(0, max(1, T // 4), (B,), generator=gen, device="cuda")
        cut[0] = 0
        lens -= cut
    return lens.to(torch.int32)


def _rows(shape, kv, gen):
    """bf16 N(0,1) values, or their E4M3 bytes."""
    x = torch.randn(shape, dtype=torch.bfloat16, device="cuda", generator=gen)
    if kv == "bf16":
        return x
    return torch.cat([(p.float() / FP8_SCALE).clamp_(-448, 448).to(torch.float8_e4m3fn).view(torch.uint8) for p in x.split(max(1, shape[0] // 8))])


def _rope_table(n_pos):
    j = torch.arange(D // 2, dtype=torch.float64, device="cuda")
    ang = torch.arange(n_pos, dtype=torch.float64, device="cuda").view(-1, 1) * 10000.0 ** (-2.0 * j / D).view(1, -1)
    return ang.cos().float().contiguous(), ang.sin().float().contiguous()


def _inputs(case, seed):
    """The tensors of a case, all from the seed."""
    gen = torch.Generator(device="cuda").manual_seed(seed * 7919 + 11)
    B, Hq, Hkv, T, Tq = (case[k] for k in ("B", "Hq", "Hkv", "T", "Tq"))
    chunks, keeps = _plan(case)
    x = {"seq_lens": _seq_lens(case, gen), "q": torch.randn((B, Hq, Tq, D), dtype=torch.bfloat16, device="cuda", generator=gen)}
    if case["op"] == "select":
        n_mid = (T - case["n_stream"] - case["n_sink"] + chunks[0] - 1) // chunks[0]
        P = B * Hkv * (Tq // case["b_q"])
        # scores as a pruning stage leaves them: maxima over the heads and queries of a block, -inf behind the last chunk
        sc = 28.0 + 3.0 * torch.randn((P, n_mid), device="cuda", generator=gen)
        m = torch.arange(P, device="cuda") % (Tq // case["b_q"])
        hi = (x["seq_lens"][0] - Tq) + (m + 1) * case["b_q"] - case["n_stream"]
        empty = case["n_sink"] + torch.arange(n_mid, device="cuda").view(1, -1) * chunks[0] >= hi.view(-1, 1)
        x["scores"] = sc.masked_fill_(empty, -math.inf)
        return x
    if case["page"]:
        n = -(-T // case["page"])
        shape = (B * n, Hkv, case["page"], D)
        x["k"], x["v"] = _rows(shape, case["kv"], gen), _rows(shape, case["kv"], gen)
        x["table"] = torch.randperm(B * n, device="cuda", generator=gen).to(torch.int32).view(B, n).contiguous()
    else:
        shape = (B, Hkv, T, D)
        x["k"], x["v"] = _rows(shape, case["kv"], gen), _rows(shape, case["kv"], gen)
        if case["kv"] == "bf16" and Tq == 1:         # needles: keys that resemble a query head
            n, G = 16, Hq // Hkv
            pos = torch.randint(case["n_sink"], max(case["n_sink"] + 1, T - T // 4 - case["n_stream"]), (B, Hkv, n), device="cuda", generator=gen)
            qh = x["q"][:, :, 0].float().view(B, Hkv, G, D)
            qh = qh / qh.norm(dim=-1, keepdim=True)
            rows = 4 * qh[:, :, torch.arange(n, device="cuda") % G] + 0.1 * torch.randn((B, Hkv, n, D), device="cuda", generator=gen)
            x["k"].scatter_(2, pos.unsqueeze(-1).expand(-1, -1, -1, D), rows.bfloat16())
    if case["op"] in ("attn_decode", "attn_prefill"):
        # kept blocks: per problem distinct blocks of its middle range, ascending
        P, Mq = B * Hkv * (Tq // case["b_q"]), Tq // case["b_q"]
        p = torch.arange(P, device="cuda")
        b, m = p // (Hkv * Mq), p % Mq
        hi = (x["seq_lens"].long()[b] - Tq) + (m + 1) * case["b_q"] - case["n_stream"]
        n_blk = ((hi - case["n_sink"]) // chunks[0]).clamp_(min=0)
        pick = torch.rand((P, int(n_blk.max())), device="cuda", generator=gen)
        pick.masked_fill_(torch.arange(pick.shape[1], device="cuda").view(1, -1) >= n_blk.view(-1, 1), 2.0)
        val, idx = pick.topk(min(keeps[0], pick.shape[1]), dim=1, largest=False)
        start = torch.where(val < 1.5, case["n_sink"] + idx * chunks[0], torch.full_like(idx, 1 << 30)).sort(dim=1).values
        start = torch.where(start < (1 << 30), start, torch.full_like(start, -1))
        x["blocks"] = start.to(torch.int32).contiguous()
    if case["op"] == "masked":                       # the previous step's query, whose lists are cached
        x["q_before"] = torch.randn((B, Hq, 1, D), dtype=torch.bfloat16, device="cuda", generator=gen)
    if case["rope"] != "none":
        l0 = chunks[0]
        x["cos"], x["sin"] = _rope_table(max(case["n_stream"] + 2, case["n_sink"] + chunks[-1] * keeps[-1] + case["n_stream"], -(-T // l0) + case["n_stream"]) + 64)
    return x


_STYLE = {"relative": (ih.binding.ROPE_RELATIVE, ih.binding.ROPE_STREAMING), "chunk": (ih.binding.ROPE_CHUNK_INDEXED, ih.binding.ROPE_NONE),
          "streaming": (ih.binding.ROPE_NONE, ih.binding.ROPE_STREAMING)}


def prepare(case, seed):
    chunks, keeps = _plan(case)
    x = _inputs(case, seed)
    s = {"case": case, "chunks": chunks, "keeps": keeps, "q": x["q"], "k": x.get("k"), "v": x.get("v"), "scores": x.get("scores"), "blocks": x.get("blocks")}
    shape_k = torch.empty((case["B"], case["Hkv"], case["T"], 0), dtype=torch.bfloat16)
    s["layer"] = L = ih.Layer(x["q"], shape_k, x["seq_lens"], case["b_q"], case["n_sink"], case["n_stream"])
    s["rope"] = ih.binding.Rope(x["cos"], x["sin"], *_STYLE[case["rope"]]) if case["rope"] != "none" else None
    s["paged"] = ih.binding.PagedKV(x["k"], x["v"], x["table"]) if case["page"] else None
    s["scales"] = (FP8_SCALE, FP8_SCALE) if case["kv"] == "fp8" else None
    s["pooling"] = ih.binding.POOL_ALL_HEADS if case["pooling"] == "all_heads" else None
    B, Hq, Tq = case["B"], case["Hq"], case["Tq"]
    s["out"] = torch.empty((B, Hq, Tq, D), dtype=torch.bfloat16, device="cuda")
    s["lse"] = torch.empty((B, Hq, Tq), dtype=torch.float32, device="cuda")
    op = case["op"]
    if op in ("decode", "masked", "offload"):
        s["ws"] = L.workspace(ih.binding.OP_DECODE_LAYER, chunks, keeps)
    elif op == "prefill":
        s["ws"] = L.workspace(ih.binding.OP_PREFILL_LAYER, chunks, keeps)
    elif op in ("attn_decode", "attn_prefill"):
        s["ws"] = L.workspace(ih.binding.OP_ATTN_DECODE if op == "attn_decode" else ih.binding.OP_ATTN_PREFILL, [chunks[0]], [x["blocks"].shape[1]])
    if op == "masked":
        s["starts"] = L.mask_state(keeps)
        L.decode_layer_masked(x["q_before"], s["k"], s["v"], chunks, keeps, 0, s["starts"], ws=s["ws"], out=s["out"])
    if op == "offload":
        hk, hv = (torch.empty(t.shape, dtype=t.dtype, pin_memory=True) for t in (x["k"], x["v"]))
        hk.copy_(x["k"]), hv.copy_(x["v"])
        s["cache"] = ih.HostKVCache(hk, hv, 64, case["bank_blocks"], max(64, case["bank_blocks"] // 2))
        s["k"] = s["v"] = None
    return s


def run(s):
    case, L, chunks, keeps = s["case"], s["layer"], s["chunks"], s["keeps"]
    op = case["op"]
    if op == "decode":
        L.decode_layer(s["q"], s["k"], s["v"], chunks, keeps, ws=s["ws"], out=s["out"], lse=s["lse"], rope=s["rope"], pooling=s["pooling"],
                       kv_scales=s["scales"], paged=s["paged"])
        return {"out": s["out"], "lse": s["lse"]}
    if op == "masked":
        L.decode_layer_masked(s["q"], s["k"], s["v"], chunks, keeps, len(chunks) - 1, s["starts"], ws=s["ws"], out=s["out"], lse=s["lse"])
        return {"out": s["out"], "lse": s["lse"], "starts": s["starts"]}
    if op == "offload":
        L.decode_layer(s["q"], None, None, chunks, keeps, ws=s["ws"], out=s["out"], lse=s["lse"], cache=s["cache"])
        s["cache"].update()
        return {"out": s["out"], "lse": s["lse"]}
    if op == "prefill":
        L.prefill_layer(s["q"], s["k"], s["v"], chunks, keeps, ws=s["ws"], out=s["out"], lse=s["lse"], rope=s["rope"], kv_scales=s["scales"], paged=s["paged"])
        return {"out": s["out"], "lse": s["lse"]}
    if op == "prune":
        scores, _ = L.prune_stage(s["q"], s["k"], chunks[0], rope=s["rope"])
        return {"scores": scores}
    if op == "select":
        return {"starts": L.select_blocks(s["scores"], chunks[0], keeps[0])}
    fn = L.sparse_attn_decode if op == "attn_decode" else L.sparse_attn_prefill
    out, lse = fn(s["q"], s["k"], s["v"], s["blocks"], chunks[0], want_lse=True, ws=s["ws"], rope=s["rope"], kv_scales=s["scales"], paged=s["paged"])
    return {"out": out, "lse": lse}


# ---- what a pass cannot do without ----------------------------------------------
def _search_rows(l, G, shared=1):
    """Distinct rows the halving searches of `shared` x G heads read in a chunk of l keys (expected, each level's midpoint uniform)."""
    rows = 1.0
    for i in range(1, int(math.log2(l)) + 1):
        n = 2.0 ** (i - 1)
        rows += n * (1.0 - (1.0 - 1.0 / n) ** (G * shared)) if n > 1 else 1.0
    return rows


def work(case):
    chunks, keeps = _plan(case)
    B, Hq, Hkv, T, Tq, b_q = (case[k] for k in ("B", "Hq", "Hkv", "T", "Tq", "b_q"))
    G, Mq = Hq // Hkv, Tq // b_q
    mean_T = T * (1 - (B - 1) / B / 8) if case["ragged"] else T
    row = D * (1 if case["kv"] == "fp8" else 2)
    mid = max(0.0, mean_T - case["n_sink"] - case["n_stream"])
    n1 = math.ceil(mid / chunks[0])
    first = len(chunks) - 1 if case["op"] == "masked" else 0
    nbytes, flops = 2.0 * B * Hq * Tq * D, 0.0
    if case["op"] == "select":
        P = B * Hkv * Mq
        return {"bytes": 4.0 * P * (n1 + min(n1, keeps[0])), "flops": float(P * n1)}
    slots = [n1]
    for i in range(1, len(chunks)):
        slots.append(min(keeps[i - 1], slots[-1]) * (chunks[i - 1] // chunks[i]))
    if case["op"] in ("decode", "masked", "offload", "prefill", "prune"):
        for i in range(first, len(chunks)):
            # a prefill chunk's blocks share the rows of the first stage; later stages' lists differ from block to block
            shared = Mq if i == 0 else 1
            nbytes += B * Hkv * slots[i] * row * (min(_search_rows(chunks[i], G, shared), chunks[i]) * (1 if i == 0 else min(Mq, max(1.0, mid / (slots[i] * chunks[i])))))
            flops += 2.0 * D * B * Hq * Tq * slots[i] * (1 + math.log2(chunks[i]))
        if case["op"] == "prune":
            return {"bytes": nbytes + 4.0 * B * Hkv * Mq * n1, "flops": flops}
    kept = min(keeps[-1], slots[-1] if case["op"] in ("decode", "masked", "offload", "prefill") else n1) * chunks[-1]
    att = case["n_sink"] + case["n_stream"] + kept
    nbytes += B * Hkv * 2 * row * min(mean_T, case["n_sink"] + case["n_stream"] + Tq + kept * min(Mq, max(1.0, mid / max(1, kept)))) + B * Hq * Tq * (2.0 * D + 4)
    flops += 4.0 * D * B * Hq * Tq * att
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    if case["op"] == "select":
        return "exact"
    if case["op"] == "prune":
        # fp32 sums; a search that turns the other way at a near tie ends at another key's score (5e-4 against 64 bits)
        return {"rel": 2e-3, "max": 0.9}
    if case["op"] in ("attn_decode", "attn_prefill"):
        return {"rel": 1e-2, "max": 0.1}             # bf16 results, probabilities and (RoPE) rotated operands: 2e-3 to 3.4e-3
    # A near tie in a selection swaps one block of a problem and its whole output moves a little.  With RoPE on the matrix
    # cores the scores that decide are 2^-17 instead of 2^-24 off: 2.3e-2 against 64 bits, 2e-3 without.
    if case["op"] == "prefill" and case["rope"] != "none":
        return {"rel": 3e-2, "max": 0.99}
    return {"rel": 8e-3, "max": 0.9, "differ": 0.01}


# ---- the same in 64 bits, by plain torch -------------------------------------------
def _rot(x, pos, cos, sin):
    """Rows x [..., D] (float64) turned to positions pos [...] (Su et al., pairs (2j, 2j+1))."""
    c, s = cos[pos].double(), sin[pos].double()
    e, o = x[..., 0::2], x[..., 1::2]
    return torch.stack((e * c - o * s, e * s + o * c), dim=-1).flatten(-2)


class _Ref:
    def __init__(self, case, x):
        self.c, self.x = case, x
        self.G, self.Mq = case["Hq"] // case["Hkv"], case["Tq"] // case["b_q"]
        self.rope = case["rope"]

    def rows(self, name, b, g, pos):
        c, x = self.c, self.x[name]
        if c["page"]:
            r = x[self.x["table"][b].long()[pos // c["page"]], g, pos % c["page"]]
        else:
            r = x[b, g][pos]
        return r.double() if c["kv"] == "bf16" else r.view(torch.float8_e4m3fn).double() * FP8_SCALE

    def bounds(self, b, m):
        E = int(self.x["seq_lens"][b]) - self.c["Tq"] + (m + 1) * self.c["b_q"]
        return E, E - self.c["n_stream"]

    def queries(self, q, b, g, m):
        return q[b, g * self.G:(g + 1) * self.G, m * self.c["b_q"]:(m + 1) * self.c["b_q"]].double()       # [G, b_q, D]

    def stage(self, q, b, g, m, start, l):
        """Chunk scores [S] of the chunks at start [S] (position order, all non-empty)."""
        E, hi = self.bounds(b, m)
        S, G = start.numel(), self.G
        qh = self.queries(q, b, g, m)
        cos, sin = self.x.get("cos"), self.x.get("sin")
        idx = torch.arange(S, device="cuda")
        if self.rope == "relative":
            at = torch.full((1,), self.c["n_stream"] + 1, device="cuda")
            qL, qR = _rot(qh, at, cos, sin), _rot(qh, at - 1, cos, sin)
        elif self.rope == "chunk":
            pos = torch.minimum(E - self.c["b_q"] + torch.arange(self.c["b_q"], device="cuda"), torch.tensor(S - 1 + self.c["n_stream"], device="cuda"))
            qL = qR = _rot(qh, pos.view(1, -1), cos, sin)
        else:
            qL = qR = qh

        def scores(pos, which):                      # pos [G, S]
            out = []
            for h in range(G):
                k = self.rows("k", b, g, pos[h])
                if self.rope == "chunk":
                    k = _rot(k, idx, cos, sin)
                out.append([(k @ w[h].t().contiguous()).amax(dim=1) for w in which])
            return [torch.stack([o[i] for o in out]) for i in range(len(which))]

        st = start.view(1, -1).expand(G, -1)
        length = (hi - st).clamp(max=l)
        off = torch.zeros_like(st)
        two = self.rope == "relative"
        first = scores(st, [qL, qR] if two else [qL])
        left, value = first[0], first[-1]            # the left key as a left branch; what the chunk score takes
        half = l // 2
        while half >= 1:
            ok = off + half < length
            got = scores(torch.where(ok, st + off + half, st), [qL, qR] if two else [qL])
            take = ok & (got[-1] > left)
            off = torch.where(take, off + half, off)
            left, value = torch.where(take, got[0], left), torch.where(take, got[-1], value)
            half //= 2
        return value.amax(dim=0)

    def first_slots(self, b, m, l):
        _, hi = self.bounds(b, m)
        return torch.arange(self.c["n_sink"], max(hi, self.c["n_sink"]), l, device="cuda")

    def prune(self, q, b, gs, m, chunks, keeps, start=None, first=0):
        """Kept starts per KV head of gs after stages first.., from the chunks at `start` (a list per head)."""
        _, hi = self.bounds(b, m)
        kept = start
        for i in range(first, len(chunks)):
            if kept is None:
                slots = [self.first_slots(b, m, chunks[0]) for _ in gs]
            else:
                slots = [(k.view(-1, 1) + torch.arange(0, chunks[i - 1], chunks[i], device="cuda").view(1, -1)).flatten() for k in kept]
                slots = [s[s < hi] for s in slots]
            sc = [self.stage(q, b, g, m, s, chunks[i]) if s.numel() else s.double() for g, s in zip(gs, slots)]
            if self.c["pooling"] == "all_heads":
                sc = [torch.stack(sc).amax(dim=0)] * len(sc)
            kept = []
            for v, s in zip(sc, slots):
                order = torch.sort(v, descending=True, stable=True).indices[:keeps[i]]
                kept.append(s[order.sort().values])
        return kept

    def attend(self, q, b, g, m, start, block, out, lse):
        c = self.c
        E, hi = self.bounds(b, m)
        w0 = max(hi, c["n_sink"])
        mid = (start.view(-1, 1) + torch.arange(block, device="cuda").view(1, -1)).flatten()
        mid = mid[mid < hi]
        pos = torch.cat([torch.arange(min(c["n_sink"], E), device="cuda"), mid, torch.arange(w0, max(E, w0), device="cuda")])
        k, v = self.rows("k", b, g, pos), self.rows("v", b, g, pos)
        qh = self.queries(q, b, g, m)
        qpos = E - c["b_q"] + torch.arange(c["b_q"], device="cuda")
        seen = pos.view(1, -1) <= qpos.view(-1, 1)
        if self.rope in ("relative", "streaming"):
            k = _rot(k, torch.arange(pos.numel(), device="cuda"), self.x["cos"], self.x["sin"])
            qh = _rot(qh, (seen.sum(dim=1) - 1).view(1, -1), self.x["cos"], self.x["sin"])
        kt = k.t().contiguous()
        for h in range(self.G):
            s = (qh[h] @ kt / math.sqrt(D)).masked_fill_(~seen, -math.inf)
            r = torch.logsumexp(s, dim=1)
            rows = slice(m * c["b_q"], (m + 1) * c["b_q"])
            out[b, g * self.G + h, rows] = (s - r.view(-1, 1)).exp_() @ v
            lse[b, g * self.G + h, rows] = r


def exact(case, seed):
    if case["op"] == "select":
        return None                                  # whole numbers
    if case["rope"] == "chunk" and case["op"] != "prune":
        return None
    chunks, keeps = _plan(case)
    x = _inputs(case, seed)
    ref = _Ref(case, x)
    B, Hkv, Tq = case["B"], case["Hkv"], case["Tq"]
    if case["op"] == "prune":
        n1 = -(-(case["T"] - case["n_stream"] - case["n_sink"]) // chunks[0])
        scores = torch.full((B * Hkv * ref.Mq, max(0, n1)), -math.inf, dtype=torch.float64, device="cuda")
        for b in range(B):
            for g in range(Hkv):
                for m in range(ref.Mq):
                    s = ref.first_slots(b, m, chunks[0])
                    if s.numel():
                        scores[(b * Hkv + g) * ref.Mq + m, :s.numel()] = ref.stage(x["q"], b, g, m, s, chunks[0])
        return {"scores": scores}
    out = torch.zeros((B, case["Hq"], Tq, D), dtype=torch.float64, device="cuda")
    lse = torch.zeros((B, case["Hq"], Tq), dtype=torch.float64, device="cuda")
    for b in range(B):
        for m in range(ref.Mq):
            gs = list(range(Hkv))
            if "blocks" in x:
                kept = [x["blocks"][(b * Hkv + g) * ref.Mq + m].long() for g in gs]
                kept = [k[k >= 0] for k in kept]
            elif case["op"] == "masked":
                kept = ref.prune(x["q_before"], b, gs, m, chunks[:-1], keeps[:-1])
                kept = ref.prune(x["q"], b, gs, m, chunks, keeps, start=kept, first=len(chunks) - 1)
            else:
                kept = ref.prune(x["q"], b, gs, m, chunks, keeps)
            for g, k in zip(gs, kept):
                ref.attend(x["q"], b, g, m, k, chunks[-1], out, lse)
    got = {"out": out, "lse": lse}
    if case["op"] == "masked":
        got["starts"] = None
    return got
