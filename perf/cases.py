"""The work whose speed counts: what a user of this library has it do, through
the Python binding's entry points, over the sizes it is used at.

Kinds of case
  step            one fused decode step (spot_decode_step / _q): score every
                  pooled key block, select, attend; decode direction.  The
                  caller keeps outputs and workspace, as a serving loop does.
  tokens          one decode step on a per-token selector cache (scorer,
                  selection, sparse attention), 16- or 64-token blocks.
  front           a decode step's selector front end (project, append, re-pool).
  front_prompt    the same for a whole prompt: project every token's query,
                  key and weights, append the keys, pool all blocks.
  prefill_attn    block-sparse causal attention of a prompt; the block lists
                  come from the selector (prefill direction).
  prefill_select  a prompt's block lists from the pooled selector cache:
                  query-block x key-block scores, then the selection.
  prefill_tokens  the same from a per-token selector cache.

Inputs follow the generators of the package's synthetic workloads (Zipf block
relevance, unit-normal K and V), made here on the GPU from the seed alone.
"""
import math

import torch

from paper_2606_22874_amd import spot

DEV = "cuda"
BLK = 64
D = 128                                  # attention head dim
ZIPF, T0, NOISE = 1.1, 16.0, 0.06        # relevance profile of the blocks
ROPE_BASE = 1.0e6


# ------------------------------------------------------------------ cases
def listed():
    return [
        # The smallest call: one sequence of 4K tokens, one layer's decode step.
        dict(name="step_4k_b1", kind="step", batch=1, l_cap=4096, h_q=32, h_kv=8, h_s=8, d_s=64,
             kfmt="bf16", qfmt="bf16", top_p=0.9, k_max=16, full=True),
        # Ordinary serving: eight ragged sequences of up to 32K tokens.
        dict(name="step_32k_b8", kind="step", batch=8, l_cap=32768, h_q=32, h_kv=8, h_s=8, d_s=64,
             kfmt="bf16", qfmt="bf16", top_p=0.9, k_max=64, full=False),
        # The headline workload: four sequences of 128K tokens.
        dict(name="step_128k_b4", kind="step", batch=4, l_cap=131072, h_q=32, h_kv=8, h_s=8,
             d_s=64, kfmt="bf16", qfmt="bf16", top_p=0.95, k_max=128, full=True),
        # 64 query heads, 4-bit selector queries and cache, a larger ragged
        # batch, an odd number of blocks.
        dict(name="step_16k_b16_fp4", kind="step", batch=16, l_cap=16448, h_q=64, h_kv=8, h_s=4,
             d_s=128, kfmt="mxfp4", qfmt="mxfp4", top_p=0.9, k_max=96, full=False),
        # The paper's own selector geometry: per-token keys, 16-token blocks.
        dict(name="tokens16_128k_b4", kind="tokens", batch=4, l_cap=131072, h_q=32, h_kv=8, h_s=4,
             d_s=128, kfmt="bf16", blk=16, top_p=0.95, k_max=512, full=True),
        # Its 4-bit cache over 64-token blocks, ragged lengths.
        dict(name="tokens64_48k_b6_int4", kind="tokens", batch=6, l_cap=49152, h_q=32, h_kv=8,
             h_s=4, d_s=128, kfmt="int4", blk=64, top_p=0.9, k_max=128, full=False),
        # The selector front end of a decode step: one new token a sequence.
        dict(name="front_b4", kind="front", batch=4, l_cap=8192, d_model=4096, h_s=4, d_s=128,
             rope=64),
        # The front end of one prompt of 8100 tokens (ragged last block).
        dict(name="front_prompt_8100", kind="front_prompt", batch=1, tokens=8100, d_model=4096,
             h_s=4, d_s=128, rope=64),
        # The largest: prefill attention of a 32K-token prompt, 64 query heads.
        dict(name="prefill_attn_32k", kind="prefill_attn", batch=1, l_cap=32768, h_q=64, h_kv=8,
             top_p=0.9, k_max=64),
        # Two shorter prompts at once, an odd number of blocks, 32 heads.
        dict(name="prefill_attn_5056_b2", kind="prefill_attn", batch=2, l_cap=5056, h_q=32,
             h_kv=8, top_p=0.9, k_max=32),
        # Block lists of a 20K prompt from an 8-bit pooled cache, odd blocks.
        dict(name="prefill_select_20k_int8", kind="prefill_select", batch=1, l_cap=20288, h_s=8,
             d_s=64, kfmt="int8", top_p=0.9, k_max=64),
        # Block lists of a 16K prompt from the per-token cache.
        dict(name="prefill_tokens_16k", kind="prefill_tokens", batch=1, l_cap=16384, h_s=4,
             d_s=128, kfmt="bf16", blk=64, top_p=0.9, k_max=64),
    ]


def _log(rng, lo, hi):
    return lo * (hi / lo) ** rng.random()


def _blocks(rng, lo, hi):
    """Tokens: a whole number of blocks, spread over the logarithm."""
    return BLK * max(1, int(round(_log(rng, lo, hi) / BLK)))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "tokens", "tokens", "front", "front_prompt",
                       "prefill_attn", "prefill_attn", "prefill_select", "prefill_tokens"])
    heads = rng.choice([(32, 8), (32, 8), (64, 8), (40, 8), (16, 8), (32, 4)])
    h_s, d_s = rng.choice([(8, 64), (4, 128)])
    fmt = rng.choice(["bf16", "bf16", "int4", "mxfp4", "int8", "mxfp8"])
    top_p = rng.choice([0.7, 0.9, 0.95])
    if kind == "step":
        l_cap = _blocks(rng, 1024, 131072)
        batch = max(1, int(_log(rng, 1, min(32, 524288 / l_cap))))
        return dict(kind=kind, batch=batch, l_cap=l_cap, h_q=heads[0], h_kv=heads[1], h_s=h_s,
                    d_s=d_s, kfmt=fmt, qfmt=rng.choice(["bf16", fmt]), top_p=rng.choice([top_p, 1.0]),
                    k_max=int(_log(rng, 8, 256)), full=rng.random() < 0.3)
    if kind == "tokens":
        l_cap = _blocks(rng, 4096, 131072)
        batch = max(1, int(_log(rng, 1, min(16, 524288 / l_cap))))
        blk = rng.choice([16, 64])
        return dict(kind=kind, batch=batch, l_cap=l_cap, h_q=heads[0], h_kv=heads[1], h_s=h_s,
                    d_s=d_s, kfmt=fmt, blk=blk, top_p=top_p,
                    k_max=int(_log(rng, 16, 128)) * (64 // blk), full=rng.random() < 0.3)
    if kind == "front":
        return dict(kind=kind, batch=int(_log(rng, 1, 64.9)), l_cap=_blocks(rng, 1024, 16384),
                    d_model=rng.choice([2560, 4096, 5120]), h_s=h_s, d_s=d_s,
                    rope=rng.choice([64, 32]))
    if kind == "front_prompt":
        tokens = int(_log(rng, 64, 8192))
        return dict(kind=kind, batch=max(1, int(_log(rng, 1, min(4, 8192 / tokens)))),
                    tokens=tokens, d_model=rng.choice([2560, 4096, 5120]), h_s=h_s, d_s=d_s,
                    rope=rng.choice([64, 32]))
    if kind == "prefill_attn":
        l_cap = _blocks(rng, 512, 24576)
        return dict(kind=kind, batch=max(1, int(_log(rng, 1, min(8, 24576 / l_cap)))),
                    l_cap=l_cap, h_q=rng.choice([16, 32, 64]), h_kv=8, top_p=top_p,
                    k_max=int(_log(rng, 8, 64)))
    if kind == "prefill_select":
        l_cap = _blocks(rng, 512, 32768)
        return dict(kind=kind, batch=max(1, int(_log(rng, 1, min(4, 32768 / l_cap)))),
                    l_cap=l_cap, h_s=h_s, d_s=d_s, kfmt=fmt, top_p=top_p,
                    k_max=int(_log(rng, 8, 96)))
    blk = rng.choice([16, 64])
    l_cap = _blocks(rng, 512, 16384)
    return dict(kind=kind, batch=max(1, int(_log(rng, 1, min(4, 16384 / l_cap)))), l_cap=l_cap,
                h_s=h_s, d_s=d_s, kfmt=fmt, blk=blk, top_p=top_p,
                k_max=int(_log(rng, 8, 64)) * (64 // blk))


def _rule(c):
    """(n_sink, n_recent) in the case's selector blocks: 64 + 128 tokens."""
    s = 64 // c.get("blk", BLK)
    return s, 2 * s


# ------------------------------------------------------------------ inputs
def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _normal(g, shape, dtype=torch.bfloat16):
    """N(0, 1), drawn a chunk at a time in FP32."""
    x = torch.empty(shape, dtype=dtype, device=DEV)
    flat = x.view(-1)
    for at in range(0, flat.numel(), 1 << 26):
        part = flat[at:at + (1 << 26)]
        part.copy_(torch.randn(part.numel(), generator=g, device=DEV))
    return x


def _seq_lens(g, c):
    if c["full"]:
        return torch.full((c["batch"],), c["l_cap"], dtype=torch.int32, device=DEV)
    n = torch.rand(c["batch"], generator=g, device=DEV)
    n = (c["l_cap"] * (0.5 + 0.5 * n)).to(torch.int32)
    n[0] = c["l_cap"] - min(5, c["l_cap"] - 1)
    return n


E2M1_MID = [0.25, 0.75, 1.25, 1.75, 2.5, 3.5, 5.0]
E2M1 = [0.0, 0.5, 1.0, 1.5, 2.0, 3.0, 4.0, 6.0]


def _quantize(x, fmt):
    """x [..., h, d] (BF16) as group-32 codes and scales of the cache formats."""
    if fmt == "bf16":
        return x.contiguous(), None
    grp = x.float().reshape(*x.shape[:-1], x.shape[-1] // 32, 32)
    amax = grp.abs().amax(-1)
    if fmt in ("int4", "int8"):
        top = 7.0 if fmt == "int4" else 127.0
        scale = (amax / top).to(torch.float16)
        code = torch.round(grp / scale.float().clamp_min(1e-30)[..., None]).clamp(-top, top)
        code = code.to(torch.int8).reshape(x.shape)
        if fmt == "int8":
            return code.contiguous(), scale.contiguous()
        nib = (code.to(torch.int16) & 0xF).to(torch.uint8)
        return (nib[..., 0::2] | (nib[..., 1::2] << 4)).contiguous(), scale.contiguous()
    emax = 2 if fmt == "mxfp4" else 8
    e = (torch.floor(torch.log2(amax.clamp_min(1e-30))) - emax).clamp(-127, 127)
    y = grp / torch.exp2(e)[..., None]
    scale = (e + 127).to(torch.uint8).contiguous()
    if fmt == "mxfp8":
        code = y.clamp(-448, 448).to(torch.float8_e4m3fn).view(torch.uint8)
        return code.reshape(x.shape).contiguous(), scale
    mag = torch.bucketize(y.abs(), torch.tensor(E2M1_MID, device=DEV)).to(torch.uint8)
    nib = (mag | ((y < 0) & (mag > 0)).to(torch.uint8) << 3).reshape(x.shape)
    return (nib[..., 0::2] | (nib[..., 1::2] << 4)).contiguous(), scale


def _dequantize(code, scale, fmt, d):
    """The values of _quantize's codes, FP64 [..., h, d]."""
    if fmt == "bf16":
        return code.double()
    if fmt in ("int4", "mxfp4"):
        nib = torch.stack((code & 0xF, code >> 4), -1).reshape(*code.shape[:-1], d).long()
        if fmt == "int4":
            v = torch.where(nib > 7, nib - 16, nib).double()
        else:
            v = torch.tensor(E2M1 + [-t for t in E2M1], dtype=torch.float64, device=DEV)[nib]
    elif fmt == "int8":
        v = code.double()
    else:
        v = code.view(torch.float8_e4m3fn).float().double()
    s = scale.double() if fmt in ("int4", "int8") else torch.exp2(scale.double() - 127)
    return (v.reshape(*v.shape[:-1], d // 32, 32) * s[..., None]).reshape(v.shape)


def _unit(x):
    return x / x.norm(dim=-1, keepdim=True)


def _profile(g, n, nblk, n_sink, n_recent):
    """Target scores of one sequence's nblk blocks, n of them present: a Zipf
    law over the residual ones, NaN for reserved and absent blocks."""
    t = torch.full((nblk,), float("nan"), device=DEV)
    lo, hi = min(n_sink, n), max(min(n_sink, n), n - n_recent)
    rank = torch.randperm(max(hi - lo, 0), generator=g, device=DEV) + 1
    t[lo:hi] = T0 - ZIPF * torch.log(rank.float())
    return t


def _decode_selector(g, c, lens):
    """q_sel, w and the cache (pooled, or one key a token) of a decode step."""
    b, h, d = c["batch"], c["h_s"], c["d_s"]
    tokens = c["kind"] == "tokens"
    blk = c.get("blk", BLK)
    n_sink, n_recent = _rule(c)
    q = torch.randn((b, h, d), generator=g, device=DEV)
    q = (q / math.sqrt(d) if tokens else q).bfloat16()
    w = torch.rand((b, h), generator=g, device=DEV)
    nblk = c["l_cap"] // blk
    n = c["l_cap"] if tokens else nblk
    parts = []
    for i in range(b):
        qf = q[i].float()
        qn = qf.norm(dim=-1, keepdim=True)
        t = _profile(g, (int(lens[i]) + blk - 1) // blk, nblk, n_sink, n_recent)
        at = torch.nonzero(~t.isnan()).flatten()
        k = _normal(g, (n, h, d))
        if not tokens:
            k.div_(math.sqrt(d))
        where = at
        if tokens:    # one leading token in each residual block
            room = torch.clamp(int(lens[i]) - at * blk, max=blk)
            where = at * blk + (torch.rand(at.numel(), generator=g, device=DEV) * room).long()
        z = k[where].float()
        qh = qf / qn
        z = z - (z * qh).sum(-1, keepdim=True) * qh
        along = t[at][:, None] / w[i].sum() + NOISE * torch.randn((at.numel(), h), generator=g,
                                                                  device=DEV)
        k[where] = (z + (along[..., None] / qn) * qh).bfloat16()
        parts.append(_quantize(k, c["kfmt"]))
    code = torch.stack([p[0] for p in parts])
    scale = None if parts[0][1] is None else torch.stack([p[1] for p in parts])
    return q, w, code, scale


def _prompt_selector(g, c):
    """Query-block rows and the cache of a prompt's selector: every head looks
    along one direction, key blocks follow one Zipf ranking."""
    b, h, d = c["batch"], c["h_s"], c["d_s"]
    nb = c["l_cap"] // BLK
    tokens = c["kind"] == "prefill_tokens"
    blk = c.get("blk", BLK)
    u = _unit(torch.randn((h, d), generator=g, device=DEV))

    def off(x):
        return x - (x * u).sum(-1, keepdim=True) * u

    size = 1.0 if tokens else 8.0
    q = off(torch.randn((b, nb, h, d), generator=g, device=DEV) * (0.25 / 8.0 * size)) + size * u
    w = torch.rand((b, nb, h), generator=g, device=DEV)
    n = c["l_cap"] // blk
    parts = []
    for _ in range(b):
        rank = torch.randperm(n, generator=g, device=DEV) + 1
        t = (T0 - ZIPF * torch.log(rank.float())) / (h / 2) / size
        if tokens:
            k = _normal(g, (c["l_cap"], h, d))
            at = torch.arange(n, device=DEV) * blk + \
                torch.randint(0, blk, (n,), generator=g, device=DEV)
            k[at] = (off(k[at].float()) + t[:, None, None] * u).bfloat16()
        else:
            k = (off(torch.randn((n, h, d), generator=g, device=DEV) / math.sqrt(d)) +
                 t[:, None, None] * u).bfloat16()
        parts.append(_quantize(k, c["kfmt"]))
    code = torch.stack([p[0] for p in parts])
    scale = None if parts[0][1] is None else torch.stack([p[1] for p in parts])
    return q.reshape(-1, h, d).bfloat16(), w.reshape(-1, h), code, scale


def _block_lists(g, c):
    """The selection of every query block of a prompt, by the rule of the
    method, from synthetic block scores: idx [rows, k_max] ascending, count."""
    nb, k_max = c["l_cap"] // BLK, c["k_max"]
    rows, ids = [], torch.arange(nb, device=DEV)
    qb = ids[:, None]
    reserved = (ids[None] < 1) | (ids[None] > qb - 2)
    seen = ids[None] <= qb
    for _ in range(c["batch"]):
        rank = torch.randperm(nb, generator=g, device=DEV) + 1
        s = (T0 - ZIPF * torch.log(rank.float()))[None] + \
            0.3 * torch.randn((nb, nb), generator=g, device=DEV)
        s = torch.where(seen & ~reserved, s, torch.full_like(s, -math.inf))
        top, order = s.sort(dim=1, descending=True)
        p = torch.softmax(top.double(), 1).nan_to_num(0.0)
        before = p.cumsum(1) - p
        n_res = (seen & reserved).sum(1, keepdim=True)
        keep = (before < c["top_p"]) & (ids[None] < k_max - n_res) & (top > -math.inf)
        chosen = torch.zeros((nb, nb), dtype=torch.bool, device=DEV).scatter_(1, order, keep)
        chosen |= seen & reserved
        key = torch.where(chosen, ids[None].expand(nb, nb), torch.full_like(s, nb).long())
        key = key.sort(dim=1).values[:, :k_max]
        if key.shape[1] < k_max:
            key = torch.nn.functional.pad(key, (0, k_max - key.shape[1]), value=nb)
        rows.append(torch.where(key < nb, key, torch.full_like(key, -1)))
    idx = torch.cat(rows).to(torch.int32).contiguous()
    return idx, (idx >= 0).sum(1).to(torch.int32)


def _front_inputs(g, c, rows):
    dm, n = c["d_model"], c["h_s"] * c["d_s"]
    sd = 1.0 / math.sqrt(dm)
    h = _normal(g, (rows, dm))
    wq, wk = _normal(g, (n, dm)).mul_(sd), _normal(g, (n, dm)).mul_(sd)
    ww = _normal(g, (c["h_s"], dm)).mul_(sd)
    return dict(h=h, w_q=wq, w_k=wk, w_w=ww)


def prepare(case, seed):
    c = case
    kind = c["kind"]
    g = _gen(seed)
    s = {"case": c}
    if kind in ("step", "tokens"):
        b, hq, hkv, cap = c["batch"], c["h_q"], c["h_kv"], c["l_cap"]
        s["seq_len"] = lens = _seq_lens(g, c)
        blk = c.get("blk", BLK)
        s["n_valid"] = ((lens + blk - 1) // blk).to(torch.int32)
        q_sel, s["w"], s["k_sel"], s["k_scale"] = _decode_selector(g, c, lens)
        s["q_sel"], s["q_scale"] = _quantize(q_sel, c.get("qfmt", "bf16"))
        s["q"] = _normal(g, (b, hq, D))
        s["k"], s["v"] = _normal(g, (b, hkv, cap, D)), _normal(g, (b, hkv, cap, D))
        f32, i32 = dict(dtype=torch.float32, device=DEV), dict(dtype=torch.int32, device=DEV)
        s["scores"] = torch.empty((b, cap // blk), **f32)
        s["idx"], s["count"] = torch.empty((b, c["k_max"]), **i32), torch.empty(b, **i32)
        s["mass"] = torch.empty(b, **f32)
        s["out"] = torch.empty((b, hq, D), dtype=torch.bfloat16, device=DEV)
        s["lse"] = torch.empty((b, hq), **f32)
        make = spot.step_workspace if kind == "step" else spot.decode_workspace
        s["ws"] = make(b, hq, hkv, D, c["k_max"], DEV)
    elif kind == "front":
        b, n, cap = c["batch"], c["h_s"] * c["d_s"], c["l_cap"]
        s.update(_front_inputs(g, c, b))
        pos = (cap * torch.rand(b, generator=g, device=DEV)).to(torch.int32).clamp_(0, cap - 1)
        s["pos"], s["seq_len"] = pos, pos + 1
        s["cache"] = _normal(g, (b, cap, n))
        s["pool"] = _normal(g, (b, cap // BLK, n))
        s["q_out"] = torch.empty((b, n), dtype=torch.bfloat16, device=DEV)
        s["w_out"] = torch.empty((b, c["h_s"]), dtype=torch.float32, device=DEV)
    elif kind == "front_prompt":
        b, t, n = c["batch"], c["tokens"], c["h_s"] * c["d_s"]
        cap = (t + BLK - 1) // BLK * BLK
        s.update(_front_inputs(g, c, b * t))
        s["pos"] = torch.arange(t, dtype=torch.int32, device=DEV).repeat(b)
        s["seq_len"] = torch.full((b,), t, dtype=torch.int32, device=DEV)
        s["cache"] = torch.zeros((b, cap, n), dtype=torch.bfloat16, device=DEV)
        s["pool"] = torch.zeros((b, cap // BLK, n), dtype=torch.bfloat16, device=DEV)
        s["q_out"] = torch.empty((b * t, n), dtype=torch.bfloat16, device=DEV)
        s["w_out"] = torch.empty((b * t, c["h_s"]), dtype=torch.float32, device=DEV)
    elif kind == "prefill_attn":
        b, cap = c["batch"], c["l_cap"]
        s["idx"], s["count"] = _block_lists(g, c)
        s["q"] = _normal(g, (b, c["h_q"], cap, D))
        s["k"], s["v"] = (_normal(g, (b, c["h_kv"], cap, D)) for _ in range(2))
    else:
        nb = c["l_cap"] // BLK
        s["q_sel"], s["w"], s["k_sel"], s["k_scale"] = _prompt_selector(g, c)
        last = torch.arange(1, nb + 1, dtype=torch.int32, device=DEV).repeat(c["batch"])
        s["n_valid"] = last * (BLK // c.get("blk", BLK))
        s["seq_len"] = last * BLK
    return s


# ------------------------------------------------------------------ one pass
class _Rule:
    def __init__(self, c):
        self.top_p, self.k_max, self.k_min = c["top_p"], c["k_max"], 0
        self.n_sink, self.n_recent = _rule(c)
        if self.k_max < self.n_sink + self.n_recent:
            raise ValueError("k_max below the reserved blocks")


def run(s):
    c = s["case"]
    kind = c["kind"]
    if kind == "step":
        b, n_sink, n_recent = c["batch"], *_rule(c)
        spot.spot_decode_step(
            s["q_sel"], s["w"], s["k_sel"], s["k_scale"], c["kfmt"], c["h_s"], c["d_s"],
            s["n_valid"], c["top_p"], c["k_max"], 0, n_sink, n_recent, s["q"], s["k"], s["v"],
            s["seq_len"], b, c["h_q"], c["h_kv"], D, c["l_cap"], 1.0 / math.sqrt(D), s["scores"],
            s["idx"], s["count"], s["mass"], s["out"], s["lse"], s["ws"],
            q_scale=s["q_scale"], qfmt=c["qfmt"])
        return {k: s[k] for k in ("scores", "idx", "count", "mass", "out", "lse")}
    if kind == "tokens":
        spot.selector_score_tokens(s["q_sel"], s["w"], s["k_sel"], s["k_scale"], c["kfmt"],
                                   seq_len=s["seq_len"], l_cap=c["l_cap"], out=s["scores"],
                                   blk=c["blk"])
        spot.select_blocks(s["scores"], _Rule(c), s["n_valid"], s["idx"], s["count"], s["mass"])
        spot.sparse_decode(s["q"], s["k"], s["v"], s["seq_len"], s["idx"], s["count"],
                           out=s["out"], lse=s["lse"], ws=s["ws"], blk=c["blk"])
        return {k: s[k] for k in ("scores", "idx", "count", "mass", "out", "lse")}
    if kind == "front":
        spot.spot_selector_project_pooled(
            s["h"], s["w_q"], s["w_k"], s["w_w"], s["pos"], s["seq_len"], c["batch"],
            c["d_model"], c["h_s"], c["d_s"], c["rope"], ROPE_BASE, s["q_out"], s["w_out"],
            s["cache"], s["pool"], c["l_cap"])
        return {k: s[k] for k in ("q_out", "w_out", "cache", "pool")}
    if kind == "front_prompt":
        b, t = c["batch"], c["tokens"]
        cap = s["cache"].shape[1]
        spot.spot_selector_project(
            s["h"], s["w_q"], s["w_k"], s["w_w"], s["pos"], b * t, c["d_model"], c["h_s"],
            c["d_s"], c["rope"], ROPE_BASE, s["q_out"], s["w_out"], s["cache"], t, cap)
        spot.spot_selector_pool(s["cache"], s["pool"], b, cap, c["h_s"], c["d_s"], s["seq_len"])
        return {k: s[k] for k in ("q_out", "w_out", "cache", "pool")}
    if kind == "prefill_attn":
        out, lse = spot.sparse_prefill(s["q"], s["k"], s["v"], s["idx"], s["count"])
        return {"out": out, "lse": lse}
    nb = c["l_cap"] // BLK
    if kind == "prefill_select":
        scores = spot.selector_score(s["q_sel"], s["w"], s["k_sel"], s["k_scale"], c["kfmt"],
                                     rows_per_seq=nb, n_valid=s["n_valid"], nblk=nb)
    else:
        scores = spot.selector_score_tokens(s["q_sel"], s["w"], s["k_sel"], s["k_scale"],
                                            c["kfmt"], rows_per_seq=nb, seq_len=s["seq_len"],
                                            l_cap=c["l_cap"], blk=c["blk"])
    idx, count, mass = spot.select_blocks(scores, _Rule(c), s["n_valid"])
    return {"scores": scores, "idx": idx, "count": count, "mass": mass}


# ------------------------------------------------------------------ its cost
KEY_BYTES = {"bf16": 1024, "int4": 288, "mxfp4": 272, "int8": 544, "mxfp8": 528}


def _selected(c, n):
    """Blocks the rule keeps of n present ones whose relevance is Zipf."""
    n_sink, n_recent = _rule(c)
    res = max(0, n - n_sink - n_recent)
    room = min(res, c["k_max"] - (n_sink + n_recent))
    total = sum(r ** -ZIPF for r in range(1, res + 1))
    mass, kept = 0.0, 0
    while kept < room and (kept == 0 or mass < c["top_p"] * total):
        kept += 1
        mass += kept ** -ZIPF
    return min(n, n_sink + n_recent) + kept


def work(case):
    c = case
    kind = c["kind"]
    hs = c.get("h_s", 0) * c.get("d_s", 0)
    if kind in ("step", "tokens"):
        blk = c.get("blk", BLK)
        fill = 1.0 if c["full"] else 0.75
        b, n = c["batch"], max(1, int(c["l_cap"] * fill) // blk)
        sel = _selected(c, n) * blk
        keys = n * (blk if kind == "tokens" else 1)
        size = b * (keys * KEY_BYTES[c["kfmt"]] + sel * c["h_kv"] * D * 4 + c["h_q"] * D * 4 +
                    4 * n + 4 * c["k_max"])
        return {"bytes": size, "flops": b * (2.0 * keys * hs + 4.0 * sel * c["h_q"] * D)}
    if kind in ("front", "front_prompt"):
        rows = c["batch"] * c.get("tokens", 1)
        outs = 2 * hs + c["h_s"]
        pooled = rows * BLK * hs * 2 if kind == "front" else rows * hs * 2 // BLK
        return {"bytes": 2 * (outs + rows) * c["d_model"] + rows * (4 * hs + 4 * c["h_s"]) + pooled,
                "flops": 2.0 * rows * outs * c["d_model"]}
    nb = c["l_cap"] // BLK
    if kind == "prefill_attn":
        tiles = sum(_selected(c, qb + 1) for qb in range(nb))
        return {"bytes": c["batch"] * c["l_cap"] * D * 4 * (c["h_q"] + c["h_kv"]),
                "flops": 4.0 * c["batch"] * c["h_q"] * BLK * BLK * D * (tiles - nb / 2)}
    blk = c.get("blk", BLK)
    keys = c["l_cap"] if kind == "prefill_tokens" else nb
    cols = c["l_cap"] // blk
    return {"bytes": c["batch"] * (keys * KEY_BYTES[c["kfmt"]] + nb * hs * 2 + 4 * nb * cols +
                                   4 * nb * c["k_max"]),
            "flops": c["batch"] * nb * keys * hs * 1.0}    # the causal half


def tolerance(case):
    kind = case["kind"]
    # Selections compare as whole numbers; a near-tie or a nucleus cut within
    # FP32 rounding of p may move a block or two of a prompt's many rows, and
    # with it that row's mass.
    if kind in ("prefill_select", "prefill_tokens"):
        return {"rel": 1e-4, "max": 1e-2, "differ": 0.01}
    # BF16 outputs: each side rounds to 2^-9 relative.
    return {"rel": 1e-2, "max": 0.1, "differ": 0.0}


# ------------------------------------------------------------------ in 64 bits
def _exact_scores(q, w, k, n_see, blk=1):
    """sum_h w ReLU(q . k) of rows [r, h, d] against keys [n, h, d] (a
    function giving a run of them), the maximum over blk keys; FP64, -inf
    past each row's n_see keys."""
    n, get = k
    step = max(blk, min(n, (1 << 25) // max(1, q.shape[0] * blk) * blk))
    outs = []
    qd, wd = q.double().permute(1, 0, 2).contiguous(), w.double()
    for at in range(0, n, step):
        kd = get(at, min(at + step, n)).permute(1, 2, 0).contiguous()
        s = torch.zeros((q.shape[0], kd.shape[2]), dtype=torch.float64, device=DEV)
        for h in range(qd.shape[0]):
            s += wd[:, h, None] * torch.relu(qd[h] @ kd[h])
        ids = torch.arange(at, at + kd.shape[2], device=DEV)
        s = torch.where(ids[None] < n_see[:, None], s, torch.full_like(s, -math.inf))
        outs.append(s.reshape(s.shape[0], -1, blk).amax(-1))
    return torch.cat(outs, 1)


def _exact_keys(s, i, c):
    code, scale = s["k_sel"][i], None if s["k_scale"] is None else s["k_scale"][i]
    return code.shape[0], lambda a, b: _dequantize(
        code[a:b], None if scale is None else scale[a:b], c["kfmt"], c["d_s"])


def _exact_select(scores, nv, c):
    """One row: the chosen ids in ascending order and the nucleus mass."""
    n_sink, n_recent = _rule(c)
    ids = torch.arange(nv, device=DEV)
    res = (ids >= n_sink) & (ids < nv - n_recent)
    n_res = int((~res).sum())
    cand = ids[res]
    if cand.numel() == 0:
        return ids, 0.0
    order = torch.argsort(scores[cand], descending=True, stable=True)
    p = torch.softmax(scores[cand][order], 0)
    cum = p.cumsum(0)
    n = cand.numel() if c["top_p"] >= 1 else int((cum - p < c["top_p"]).sum())
    n = min(n, c["k_max"] - n_res)
    take = cand[order[:n]]
    chosen = torch.cat((ids[~res], take)).sort().values
    return chosen, float(p[:n].sum())


def _exact_attend(q, k, v):
    """q [g, d], k and v [t, d] in FP64: (out, lse)."""
    s = q @ k.T / math.sqrt(D)
    return torch.softmax(s, -1) @ v, torch.logsumexp(s, -1)


def _rope(x, pos, rope):
    half = rope // 2
    f = ROPE_BASE ** (-2.0 * torch.arange(half, dtype=torch.float64, device=DEV) / rope)
    a = pos.double()[:, None, None] * f
    x0, x1 = x[..., :half], x[..., half:rope]
    return torch.cat((x0 * a.cos() - x1 * a.sin(), x1 * a.cos() + x0 * a.sin(), x[..., rope:]), -1)


def exact(case, seed):
    c, s = case, prepare(case, seed)
    kind = c["kind"]
    if kind in ("step", "tokens"):
        blk, scores, mass, outs, lses = c.get("blk", BLK), [], [], [], []
        q_sel = _dequantize(s["q_sel"], s["q_scale"], c.get("qfmt", "bf16"), c["d_s"])
        grp = c["h_q"] // c["h_kv"]
        for i in range(c["batch"]):
            n, nv = int(s["seq_len"][i]), int(s["n_valid"][i])
            see = torch.tensor([n if kind == "tokens" else nv], device=DEV)
            sc = _exact_scores(q_sel[i:i + 1], s["w"][i:i + 1], _exact_keys(s, i, c), see,
                               blk if kind == "tokens" else 1)[0]
            ids, m = _exact_select(sc, nv, c)
            t = (ids[:, None] * blk + torch.arange(blk, device=DEV)).flatten()
            t = t[t < n]
            for g in range(c["h_kv"]):
                o, e = _exact_attend(s["q"][i, g * grp:(g + 1) * grp].double(),
                                     s["k"][i, g, t].double(), s["v"][i, g, t].double())
                outs.append(o)
                lses.append(e)
            scores.append(sc)
            mass.append(m)
        return {"scores": torch.stack(scores), "idx": None, "count": None,
                "mass": torch.tensor(mass, dtype=torch.float64),
                "out": torch.cat(outs).reshape(c["batch"], c["h_q"], D),
                "lse": torch.cat(lses).reshape(c["batch"], c["h_q"])}
    if kind in ("front", "front_prompt"):
        hs, ds, b = c["h_s"], c["d_s"], c["batch"]
        hd = s["h"].double()
        q = _rope((hd @ s["w_q"].double().T).reshape(-1, hs, ds), s["pos"], c["rope"])
        k = _rope((hd @ s["w_k"].double().T).reshape(-1, hs, ds), s["pos"], c["rope"])
        cache, pool = s["cache"].double(), s["pool"].double()
        seq = torch.arange(b, device=DEV).repeat_interleave(c.get("tokens", 1))
        cache[seq, s["pos"].long()] = k.reshape(-1, hs * ds)
        if kind == "front":
            for i in range(b):
                p = int(s["pos"][i])
                pool[i, p // BLK] = cache[i, p // BLK * BLK:p + 1].mean(0)
        else:
            t = c["tokens"]
            cnt = (t - torch.arange(pool.shape[1], device=DEV) * BLK).clamp(max=BLK).double()
            pool = cache.reshape(b, -1, BLK, hs * ds).sum(2) / cnt[:, None]
        return {"q_out": q.reshape(-1, hs * ds), "w_out": hd @ s["w_w"].double().T,
                "cache": cache, "pool": pool}
    nb = c["l_cap"] // BLK
    if kind == "prefill_attn":
        b, hq, hkv = c["batch"], c["h_q"], c["h_kv"]
        out = torch.empty((b, hq, c["l_cap"], D), dtype=torch.float64, device=DEV)
        lse = torch.empty((b, hq, c["l_cap"]), dtype=torch.float64, device=DEV)
        idx = s["idx"].cpu()
        for i in range(b):
            kd, vd = s["k"][i].double(), s["v"][i].double()
            for qb in range(nb):
                ids = idx[i * nb + qb]
                ids = ids[ids >= 0].long()
                t = (ids[:, None] * BLK + torch.arange(BLK)).flatten().to(DEV)
                pos = torch.arange(qb * BLK, qb * BLK + BLK, device=DEV)
                q = s["q"][i, :, qb * BLK:qb * BLK + BLK].double()
                q = q.reshape(hkv, -1, D)
                sc = torch.bmm(q, kd[:, t].transpose(1, 2).contiguous()) / math.sqrt(D)
                sc = sc.reshape(hq, BLK, -1).masked_fill(t[None, None] > pos[None, :, None],
                                                         -math.inf)
                e = torch.logsumexp(sc, -1)
                p = torch.exp(sc - e[..., None]).reshape(hkv, -1, t.numel())
                out[i, :, qb * BLK:qb * BLK + BLK] = torch.bmm(p, vd[:, t]).reshape(hq, BLK, D)
                lse[i, :, qb * BLK:qb * BLK + BLK] = e
        return {"out": out, "lse": lse}
    scores, mass = [], []
    tokens = kind == "prefill_tokens"
    for i in range(c["batch"]):
        r = slice(i * nb, (i + 1) * nb)
        see = s["seq_len"][r] if tokens else s["n_valid"][r]
        sc = _exact_scores(s["q_sel"][r], s["w"][r], _exact_keys(s, i, c), see,
                           c["blk"] if tokens else 1)
        scores.append(sc)
        mass += [_exact_select(sc[j], int(s["n_valid"][i * nb + j]), c)[1] for j in range(nb)]
    return {"scores": torch.cat(scores), "idx": None, "count": None,
            "mass": torch.tensor(mass, dtype=torch.float64)}
