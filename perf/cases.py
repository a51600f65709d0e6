"""The work a program has this library do, as measurable cases: one Thinker /
Talker / mixture-of-experts decoder layer over one scheduler step, through the
public entry points (layer_prefill, layer_decode, layer_decode_noalloc).

A case names a layer of the model zoo (LAYERS), its storage type and options,
and the step's ragged batch as text: space-separated groups COUNTxQ@CTX, COUNT
sequences of Q new tokens after CTX cached ones; Q and CTX may be ranges
LO..HI, spread evenly over the logarithm within the group.
"""
import math

import torch

from paper_2606_29629_amd import _lib as tri

BLOCK = 64  # rows per block of a paged cache

# The layer shapes of the workloads: the 7B-class Thinker, the 128-expert
# mixture of experts, the Talker.
LAYERS = {
    "dense": dict(hidden=3584, hq=28, hkv=4, d=128, ffn=18944, experts=0, top_k=0),
    "moe": dict(hidden=2048, hq=32, hkv=4, d=128, ffn=768, experts=128, top_k=8),
    "talker": dict(hidden=896, hq=14, hkv=2, d=64, ffn=4864, experts=0, top_k=0),
}
# frequencies per section (temporal, height, width) of the multimodal rotary positions
MROPE = {64: (8, 12, 12), 128: (16, 24, 24)}
ROPE_BASE, EPS = 1e6, 1e-6


def _case(name, layer, step, batch, **options):
    case = dict(layer=layer, step=step, batch=batch, f32=False, bias=False, qk_norm=False,
                mrope=False, paged=False, noalloc=False)
    case.update(options)
    if name:
        case["name"] = name
    return case


def listed():
    return [
        # one speech stream: the Talker's step per codec token, all latency;
        # a serving loop that allocates nothing
        _case("talker_decode_1", "talker", "decode", "1x1@300", bias=True, noalloc=True),
        # one user: a token of a long multimodal chat, the weights are the work
        _case("dense_decode_1", "dense", "decode", "1x1@5000", bias=True, mrope=True),
        # a served batch: paged cache, lengths of all sizes
        _case("dense_decode_23", "dense", "decode", "23x1@100..8000", bias=True, mrope=True,
              paged=True),
        # the benchmark's decode: 64 sequences at 4096 cached tokens
        _case("dense_decode_64", "dense", "decode", "64x1@4096"),
        # a few users on the mixture of experts: about a third of the experts touched
        _case("moe_decode_7", "moe", "decode", "7x1@60..4000", qk_norm=True),
        # the benchmark's mixture-of-experts decode
        _case("moe_decode_128", "moe", "decode", "128x1@2048"),
        # short ragged Talker prompts
        _case("talker_prefill", "talker", "prefill", "5x190..700@0", bias=True),
        # ragged prompts, one of them continuing a cached prefix (a chat's next turn)
        _case("dense_prefill_ragged", "dense", "prefill", "1x37@0 1x411@900 1x613@0", bias=True,
              mrope=True, paged=True),
        # chunked prefill beside decodes: 512 tokens at 6144 and 32 single tokens
        _case("mixed", "dense", "prefill", "1x512@6144 32x1@1024..8192"),
        # the mixture-of-experts prefill of the benchmark, with its q/k norm
        _case("moe_prefill", "moe", "prefill", "4x1024@0", qk_norm=True),
        # the benchmark's prefill: 8 prompts of 2048 tokens
        _case("dense_prefill", "dense", "prefill", "8x2048@0"),
        # fp32 storage: a small ragged step of the mode that checks parity
        _case("talker_f32", "talker", "prefill", "1x65@0 1x200@130 1x1@77", f32=True),
    ]


def draw(rng):
    def log(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    def flip():
        return rng.random() < 0.5

    kind = rng.choice(["decode", "decode", "decode", "prefill", "prefill", "prefill", "mixed",
                       "f32"])
    layer = rng.choice(["dense", "moe", "talker"])
    options = dict(bias=flip(), mrope=flip(), qk_norm=flip(), paged=flip())
    if kind == "decode":
        n = log(1, 128)
        ctx = log(40, 8000 if n <= 32 else 260000 // n)
        spread = n > 1 and n <= 28
        batch = "%dx1@%s" % (n, "%d..%d" % (max(1, ctx // 20), ctx) if spread else ctx)
        return _case(None, layer, "decode", batch, noalloc=n <= 16 and flip(), **options)
    if kind == "prefill":
        total = log(40, 12000 if layer == "dense" else 4096)
        n = max(rng.randint(1, 5), -(-total // 4096))
        q = max(2, total // n)
        batch = "%dx%s@%d" % (n, "%d..%d" % (max(1, q // 3), q) if n > 1 else q,
                              rng.choice([0, log(20, 2000)]))
        return _case(None, layer, "prefill", batch, **options)
    if kind == "mixed":
        batch = "1x%d@%d %dx1@%d..%d" % (log(30, 1000), log(60, 6000), rng.randint(1, 24),
                                         log(30, 500), log(600, 8000))
        return _case(None, layer, "prefill", batch, **options)
    options["f32"] = True
    return _case(None, "talker", "prefill", "%dx%d@%d" % (rng.randint(1, 4), log(2, 300),
                                                          rng.choice([0, log(10, 300)])), **options)


# ---------------------------------------------------------------- the batch --

def _spread(text, n):
    """n values of "V" or "LO..HI" (evenly over the logarithm, largest in the middle)."""
    if ".." not in text:
        return [int(text)] * n
    lo, hi = (int(v) for v in text.split(".."))
    up = [int(round(lo * (hi / lo) ** (i / max(1, n - 1)))) for i in range(n)]
    return up[0::2] + up[1::2][::-1]


def _seqs(case):
    """[(new tokens, cached tokens)] of the step's sequences."""
    out = []
    for group in case["batch"].split():
        n, rest = group.split("x")
        q, ctx = rest.split("@")
        out += list(zip(_spread(q, int(n)), _spread(ctx, int(n))))
    return out


def _max_seq(seqs):
    return -(-max(q + c for q, c in seqs) // BLOCK) * BLOCK


def _positions(case, seqs):
    """Rotary positions: [T], or three planes [3, T] with mrope: a prompt is a
    third text, then one square image, then text; single tokens are text."""
    planes = []
    for q, c in seqs:
        ids = torch.arange(c, c + q).repeat(3, 1)
        if case["mrope"] and q >= 12:
            t0, side = q // 3, int(math.sqrt(q // 3))
            img = torch.arange(side * side)
            ids[:, t0:t0 + side * side] = c + t0
            ids[1, t0:t0 + side * side] += img // side
            ids[2, t0:t0 + side * side] += img % side
            rest = q - t0 - side * side
            ids[:, t0 + side * side:] = c + t0 + side + torch.arange(rest)
        planes.append(ids)
    pos = torch.cat(planes, 1)
    return pos if case["mrope"] else pos[0]


# --------------------------------------------------------------- the inputs --

def _inputs(case, seed):
    """Weights, cache and activations, from the seed alone."""
    L = LAYERS[case["layer"]]
    H, hq, hkv, D, F = L["hidden"], L["hq"], L["hkv"], L["d"], L["ffn"]
    seqs = _seqs(case)
    dt = torch.float32 if case["f32"] else torch.bfloat16
    g = torch.Generator(device="cuda").manual_seed(int(seed) * 7919 + 13)

    def normal(*shape, std=1.0, mean=0.0):
        return torch.empty(shape, dtype=dt, device="cuda").normal_(mean, std, generator=g)

    experts = (L["experts"],) if L["experts"] else ()
    w = {"attn_norm": normal(H, std=0.1, mean=1.0), "w_qkv": normal((hq + 2 * hkv) * D, H, std=0.02),
         "w_o": normal(H, hq * D, std=0.02), "mlp_norm": normal(H, std=0.1, mean=1.0),
         "w_gate_up": normal(*experts, 2 * F, H, std=0.02),
         "w_down": normal(*experts, H, F, std=0.02)}
    if L["experts"]:
        w["w_router"] = normal(L["experts"], H, std=0.02)
    if case["bias"]:
        w["b_qkv"] = normal((hq + 2 * hkv) * D, std=0.2)
    if case["qk_norm"]:
        w["q_norm"], w["k_norm"] = normal(D, std=0.1, mean=1.0), normal(D, std=0.1, mean=1.0)
    max_seq, n = _max_seq(seqs), len(seqs)
    slots = [(i * 5 + 2) % n if n % 5 else (i + 2) % n for i in range(n)]  # a fixed permutation
    if case["paged"]:
        per = max_seq // BLOCK
        shape = (n * per + 3, hkv, BLOCK, D)
        order = torch.randperm(n * per + 3, generator=torch.Generator().manual_seed(int(seed)))
        table = order[:n * per].reshape(n, per).to(torch.int32).cuda()
    else:
        shape, table = (n, hkv, max_seq, D), None
    k, v = normal(*shape), normal(*shape)
    x = normal(sum(q for q, _ in seqs), H)
    return dict(w=w, k=k, v=v, table=table, x=x, slots=slots, seqs=seqs, max_seq=max_seq,
                pos=_positions(case, seqs))


class _Config:
    """The layer's configuration, by the names the library reads."""

    def __init__(self, case):
        L = LAYERS[case["layer"]]
        self.hidden, self.n_q_heads, self.n_kv_heads = L["hidden"], L["hq"], L["hkv"]
        self.head_dim, self.rms_eps, self.rope_base = L["d"], EPS, ROPE_BASE
        self.n_experts, self.top_k = L["experts"], L["top_k"]
        self.ffn_dim, self.expert_ffn_dim = (0, L["ffn"]) if L["experts"] else (L["ffn"], 0)
        self.qkv_bias, self.qk_norm = case["bias"], case["qk_norm"]
        self.mrope_section = MROPE[L["d"]] if case["mrope"] else None


def _row_pieces(case, i):
    """Per sequence, the (panel, first row, rows) of its new cache rows; one
    entry (None, row, 1) when every sequence writes one row at the same place
    of its slot; None when there would be too many to hand back one by one."""
    seqs = i["seqs"]
    if not case["paged"] and len(set(seqs)) == 1:
        return [(None, seqs[0][1], seqs[0][0])]
    pieces = []
    table = i["table"].cpu() if case["paged"] else None
    for slot, (q, c) in zip(i["slots"], seqs):
        row = c
        while row < c + q:
            if case["paged"]:
                j = row // BLOCK
                rows = min(BLOCK * (j + 1), c + q) - row
                pieces.append((int(table[slot, j]), row - BLOCK * j, rows))
            else:
                rows = q
                pieces.append((slot, row, rows))
            row += rows
    return pieces if len(pieces) <= 30 else None


def _rows(cache, pieces):
    """Views of the cache rows that the step writes (the whole cache without pieces)."""
    if pieces is None:
        return cache
    return [cache[:, :, r:r + n] if p is None else cache[p, :, r:r + n] for p, r, n in pieces]


def prepare(case, seed):
    i = _inputs(case, seed)
    seqs = i["seqs"]
    cfg = tri.make_config(_Config(case), f32=case["f32"])
    pos = i["pos"].numpy() if case["mrope"] else None
    batch = tri.DeviceBatch(i["slots"], [c for _, c in seqs], [q for q, _ in seqs], pos=pos)
    cache = i["k"], i["v"]
    if case["paged"]:
        cache = tri.PagedCache(*cache, i["table"], i["max_seq"])
    state = dict(cfg=cfg, w=i["w"], cache=cache, batch=batch, x=i["x"],
                 out=torch.empty_like(i["x"]), decode=case["step"] == "decode",
                 noalloc=case["noalloc"])
    if not case["noalloc"]:
        state["ws"] = torch.empty(tri.workspace_size(cfg, batch), dtype=torch.uint8,
                                  device="cuda")
    pieces = _row_pieces(case, i)
    state["rows"] = {"k": _rows(i["k"], pieces), "v": _rows(i["v"], pieces)}
    return state


def run(state):
    args = state["cfg"], state["w"], state["cache"], state["batch"], state["x"]
    if state["noalloc"]:
        out = tri.layer_decode_noalloc(*args, out=state["out"])
    elif state["decode"]:
        out, _ = tri.layer_decode(*args, out=state["out"], workspace=state["ws"])
    else:
        out, _ = tri.layer_prefill(*args, out=state["out"], workspace=state["ws"])
    return {"out": out, "new_rows": state["rows"]}


def work(case):
    """One pass: every weight (of the experts expected to be touched), the
    cached rows, the activations once; two flops per multiply-add."""
    L, seqs = LAYERS[case["layer"]], _seqs(case)
    H, hq, hkv, D, F = L["hidden"], L["hq"], L["hkv"], L["d"], L["ffn"]
    E, k, es = L["experts"], L["top_k"], 4 if case["f32"] else 2
    T = sum(q for q, _ in seqs)
    proj = (hq + 2 * hkv) * D * H + H * hq * D
    touched = E * (1 - (1 - k / E) ** T) if E else 1
    weights = proj + touched * 3 * F * H + E * H + 2 * H
    rows = sum(q + c for q, c in seqs)
    nbytes = es * (weights + 2 * T * H + 2 * rows * hkv * D)
    pairs = sum(q * c + q * (q + 1) // 2 for q, c in seqs)
    flops = 2 * T * (proj + (k if E else 1) * 3 * F * H + E * H) + 4 * D * hq * pairs
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # Storage in bf16 rounds at eight places between the input and the output
    # (2^-9 each, 2.3e-3 in the norm): measured against exact(), new cache rows
    # are 2.4e-3 off and outputs 2.5e-3 to 5.4e-3, single values up to 0.03 of
    # the rms.  In fp32 storage the products are of hi + lo bf16 pairs (2^-16
    # each): measured 2e-6 to 5e-6.
    if case["f32"]:
        return {"rel": 2e-5, "max": 2e-4}
    return {"rel": 1e-2, "max": 0.1}


# ------------------------------------------------------ the same in 64 bits --

def _norm(x, g):
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + EPS) * g


def exact(case, seed):
    """The layer of these inputs in plain float64, nothing rounded in between."""
    L, i = LAYERS[case["layer"]], _inputs(case, seed)
    hq, hkv, D, F = L["hq"], L["hkv"], L["d"], L["ffn"]
    w, seqs = i["w"], i["seqs"]
    x = i["x"].double()
    T = x.shape[0]

    def product(a, m):
        """a m^T, a few thousand rows of the weight at a time."""
        return torch.cat([a @ part.double().t() for part in m.split(4096)], -1)

    qkv = product(_norm(x, w["attn_norm"].double()), w["w_qkv"])
    if case["bias"]:
        qkv += w["b_qkv"].double()
    q, k, v = qkv.reshape(T, hq + 2 * hkv, D).split([hq, hkv, hkv], 1)
    if case["qk_norm"]:
        q, k = _norm(q, w["q_norm"].double()), _norm(k, w["k_norm"].double())
    freq = ROPE_BASE ** (-2.0 * torch.arange(D // 2, dtype=torch.float64) / D)
    pos = i["pos"].double()
    if case["mrope"]:
        plane = torch.repeat_interleave(torch.arange(3), torch.tensor(MROPE[D]))
        angle = pos[plane].t() * freq
    else:
        angle = pos[:, None] * freq
    cos, sin = (f(angle).cuda()[:, None] for f in (torch.cos, torch.sin))

    def rotate(a):
        lo, hi = a[..., :D // 2], a[..., D // 2:]
        return torch.cat([lo * cos - hi * sin, hi * cos + lo * sin], -1)

    q, k = rotate(q), rotate(k)

    def cached(cache, slot, rows):
        if i["table"] is None:
            return cache[slot, :, :rows].double()
        blocks = i["table"][slot, :-(-rows // BLOCK)].long()
        return cache[blocks].transpose(0, 1).reshape(hkv, -1, D)[:, :rows].double()

    attn, t0, new = torch.empty_like(q), 0, {"k": [], "v": []}
    for slot, (n, c) in zip(i["slots"], seqs):
        own = {"k": k[t0:t0 + n].transpose(0, 1), "v": v[t0:t0 + n].transpose(0, 1)}
        keys = torch.cat([cached(i["k"], slot, c), own["k"]], 1)
        vals = torch.cat([cached(i["v"], slot, c), own["v"]], 1)
        seen = torch.arange(c + n, device="cuda") <= c + torch.arange(n, device="cuda")[:, None]
        for h in range(hkv):
            group = slice(h * hq // hkv, (h + 1) * hq // hkv)
            s = q[t0:t0 + n, group].transpose(0, 1) @ keys[h].t() / math.sqrt(D)
            p = torch.softmax(s.masked_fill(~seen, -math.inf), -1)
            attn[t0:t0 + n, group] = (p @ vals[h]).transpose(0, 1)
        for name in own:
            new[name].append(own[name])
        t0 += n
    x1 = x + product(attn.reshape(T, hq * D), w["w_o"])
    h2 = _norm(x1, w["mlp_norm"].double())

    def ffn(a, gate_up, down):
        gu = product(a, gate_up)
        return product(torch.nn.functional.silu(gu[:, :F]) * gu[:, F:], down)

    if not L["experts"]:
        out = x1 + ffn(h2, w["w_gate_up"], w["w_down"])
    else:
        top = torch.topk(h2 @ w["w_router"].double().t(), L["top_k"], -1)
        weight = torch.softmax(top.values, -1)
        out = x1.clone()
        for e in range(L["experts"]):
            t, j = torch.nonzero(top.indices == e, as_tuple=True)
            if t.numel():
                y = ffn(h2[t], w["w_gate_up"][e], w["w_down"][e])
                out.index_add_(0, t, y * weight[t, j][:, None])

    pieces = _row_pieces(case, i)
    if pieces is None:
        rows = {"k": None, "v": None}
    elif pieces[0][0] is None:
        at = torch.tensor(i["slots"], device="cuda").argsort()
        rows = {name: [torch.stack(new[name])[at]] for name in new}
    else:
        flat = {name: [] for name in new}
        sizes = iter(pieces)
        for s, (n, _) in enumerate(seqs):
            done = 0
            while done < n:
                size = next(sizes)[2]
                for name in new:
                    flat[name].append(new[name][s][:, done:done + size])
                done += size
        rows = flat
    return {"out": out, "new_rows": rows}
