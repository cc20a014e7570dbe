"""Parity of the selector front end (projections with rotary embedding and
the cache append; block pooling) with the FP64 oracle (needs an MI355X).

Tolerances: a projected value g (FP32 products of BF16, rounded to BF16)
against the oracle o: |g - o| <= 2^-8 |o| + 1e-5 S, with S the sum of
|W_ji h_i| over the terms that make it up (the FP32 summation bound for
4096-term dots, with margin); the weights w_out (FP32) to 1e-5 S.  Pooled
keys: within one BF16 step (2^-8 relative) of the FP64 block mean, and
bitwise equal to the documented FP32 summation order.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2606_22874_amd import spot, synth
from paper_2606_22874_amd.synth import bf16_bits, bf16_value

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

DEV = "cuda:0"


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


def bf(a):
    return spot.to_device_bf16(a, DEV)


def host_bf16(t):
    return t.view(torch.int16).cpu().numpy().view(np.uint16)


def abs_sums(h, w):
    """S[r, j] = sum_i |W[j, i] h[r, i]|."""
    return np.abs(bf16_value(h).astype(np.float64)) @ np.abs(bf16_value(w).astype(np.float64)).T


def rot_sums(S, Hs, ds, rope_dim):
    """Bound terms after the rotation: a rotated value mixes its pair."""
    S = S.reshape(S.shape[0], Hs, ds).copy()
    half = rope_dim // 2
    both = S[..., :half] + S[..., half:rope_dim]
    S[..., :half] = both
    S[..., half:rope_dim] = both
    return S


def run_project(rows, d_model, Hs, ds, rope_dim, base, pos, rows_per_seq, l_cap, seed=1):
    h, wq, wk, ww = synth.selector_frontend(seed, rows, d_model, Hs, ds)
    n_seq = rows // rows_per_seq
    q_out = torch.empty((rows, Hs, ds), dtype=torch.bfloat16, device=DEV)
    w_out = torch.empty((rows, Hs), dtype=torch.float32, device=DEV)
    cache = torch.zeros((n_seq, l_cap, Hs, ds), dtype=torch.bfloat16, device=DEV)
    spot.spot_selector_project(bf(h), bf(wq), bf(wk), bf(ww), dev(np.asarray(pos, np.int32)),
                               rows, d_model, Hs, ds, rope_dim, base, q_out, w_out, cache,
                               rows_per_seq, l_cap)
    torch.cuda.synchronize()
    q_o, k_o, w_o = oracle.selector_project(h, wq, wk, ww, np.asarray(pos, np.int32), Hs, ds,
                                            rope_dim=rope_dim, rope_base=base)
    return (h, wq, wk, ww), (q_out, w_out, cache), (q_o, k_o, w_o)


def check_bf16(g_bits, o, S):
    g = bf16_value(g_bits).astype(np.float64)
    err = np.abs(g - o)
    bound = 2.0 ** -8 * np.abs(o) + 1e-5 * S
    assert np.all(err <= bound), f"max excess {np.max(err - bound)}"


CASES = [
    # rows, d_model, Hs, ds, rope_dim, base, rows_per_seq, l_cap
    (4, 4096, 4, 128, 64, 1.0e6, 1, 131072),     # decode, Qwen3-8B hidden size
    (4, 4096, 8, 64, 32, 1.0e6, 1, 8192),
    (3, 5120, 4, 128, 64, 1.0e6, 1, 4096),       # Qwen3-32B hidden size: two chunk passes
    (20, 2560, 4, 128, 64, 1.0e4, 20, 64),       # prefill rows, two row passes
    (6, 1000, 8, 64, 64, 500.0, 3, 128),         # d_model not a multiple of 512, all dims rotated
    (2, 512, 4, 128, 0, 1.0e6, 1, 64),           # no rotary dims
    (7, 264, 4, 128, 64, 2.0 ** -10, 1, 4096),   # a base below 1 (an FP32 number): angles to 4e6
]


@pytest.mark.parametrize("rows,d_model,Hs,ds,rope_dim,base,rps,l_cap", CASES)
def test_project_parity(rows, d_model, Hs, ds, rope_dim, base, rps, l_cap):
    print(f"[frontend] project rows={rows} d_model={d_model} {Hs}x{ds} rope {rope_dim}",
          flush=True)
    rng = np.random.default_rng(rows * d_model)
    if rps == 1:
        pos = rng.integers(0, l_cap, rows)
        pos[0] = l_cap - 1
    else:
        pos = np.tile(np.arange(rps), rows // rps)
    (h, wq, wk, ww), (q_out, w_out, cache), (q_o, k_o, w_o) = run_project(
        rows, d_model, Hs, ds, rope_dim, base, pos, rps, l_cap)
    Sq = rot_sums(abs_sums(h, wq), Hs, ds, rope_dim)
    Sk = rot_sums(abs_sums(h, wk), Hs, ds, rope_dim)
    check_bf16(host_bf16(q_out), q_o, Sq)
    cache_h = host_bf16(cache)
    k_g = np.stack([cache_h[r // rps, pos[r]] for r in range(rows)])
    check_bf16(k_g, k_o, Sk)
    Sw = abs_sums(h, ww)
    assert np.all(np.abs(w_out.cpu().numpy() - w_o) <= 1e-5 * Sw)
    # nothing else of the cache was written
    mask = np.ones(cache_h.shape[:2], bool)
    for r in range(rows):
        mask[r // rps, pos[r]] = False
    assert np.all(cache_h[mask] == 0)


# Rows at the edges of the kernel choice (row kernel, skinny tiles of 16 and
# 32 tokens, 64 x 64, 128 x 64 and 256 x 128 tiles) and of their token tiles;
# d_model below one step, ragged, and with more steps than buffers; every
# rotary split (none, part, a partial group of 4, all).
MANY_ROWS = [
    # rows, d_model, Hs, ds, rope_dim, rows_per_seq, l_cap
    (33, 4096, 4, 128, 64, 1, 8192),
    (112, 1000, 8, 64, 32, 112, 128),
    (113, 72, 8, 64, 64, 113, 128),
    (225, 8, 4, 128, 0, 225, 256),
    (320, 264, 4, 128, 128, 160, 192),
    (2048, 328, 8, 64, 50, 1024, 1024),
    (2049, 512, 4, 128, 64, 2049, 2112),
    (4097, 136, 8, 64, 6, 4097, 4160),
    (4352, 456, 4, 128, 64, 4352, 4352),
    (48, 8200, 4, 128, 64, 48, 64),      # large d_model: the row kernel up to 48 rows
    (49, 8200, 8, 64, 32, 49, 64),
]


@pytest.mark.parametrize("rows,d_model,Hs,ds,rope_dim,rps,l_cap", MANY_ROWS)
def test_project_many_rows_parity(rows, d_model, Hs, ds, rope_dim, rps, l_cap):
    """The same bounds as test_project_parity; rows of one sequence in a
    shuffled order, one position past the cache (no key stored)."""
    print(f"[frontend] project rows={rows} d_model={d_model} {Hs}x{ds} rope {rope_dim}",
          flush=True)
    rng = np.random.default_rng(rows)
    pos = np.concatenate([rng.permutation(l_cap)[:rps] for _ in range(rows // rps)])
    pos[rows // 2] = l_cap
    (h, wq, wk, ww), (q_out, w_out, cache), (q_o, k_o, w_o) = run_project(
        rows, d_model, Hs, ds, rope_dim, 1.0e6, pos, rps, l_cap)
    check_bf16(host_bf16(q_out), q_o, rot_sums(abs_sums(h, wq), Hs, ds, rope_dim))
    cache_h = host_bf16(cache)
    kept = np.flatnonzero(pos < l_cap)
    k_g = np.stack([cache_h[r // rps, pos[r]] for r in kept])
    check_bf16(k_g, k_o[kept], rot_sums(abs_sums(h, wk), Hs, ds, rope_dim)[kept])
    assert np.all(np.abs(w_out.cpu().numpy() - w_o) <= 1e-5 * abs_sums(h, ww))
    mask = np.ones(cache_h.shape[:2], bool)
    mask[kept // rps, pos[kept]] = False
    assert np.all(cache_h[mask] == 0)


@pytest.mark.parametrize("rows", [40, 300])
def test_project_many_rows_infinities(rows):
    """Infinities, NaN and sums that overflow give what the row kernel gives
    for the same rows 20 at a time (an infinite sum stays one: compensated sums
    must not turn it into NaN), and every other row is untouched by them."""
    d_model, Hs, ds, l_cap = 520, 4, 128, 320
    h, wq, wk, ww = synth.selector_frontend(5, rows, d_model, Hs, ds)
    ww = ww & 0x7FFF                                    # positive weights
    inf, nan, big = 0x7F80, 0x7FC0, bf16_bits(np.float32(3.0e38)).item()
    h[1, 7] = inf
    h[2, :64] = big                                     # sums overflow in FP32
    h[3, [9, 300]] = inf
    h[4, 519] = inf ^ 0x8000
    h[5, [2, 400]] = [inf, inf ^ 0x8000]                # inf - inf: NaN either way
    h[rows - 1, 100] = nan
    W = [bf(x) for x in (wq, wk, ww)]

    def run(part, at):
        n = len(part)
        q_out = torch.empty((n, Hs * ds), dtype=torch.bfloat16, device=DEV)
        w_out = torch.empty((n, Hs), dtype=torch.float32, device=DEV)
        cache = torch.zeros((l_cap, Hs * ds), dtype=torch.bfloat16, device=DEV)
        pos = dev(np.arange(at, at + n, dtype=np.int32))
        spot.spot_selector_project(bf(part), *W, pos, n, d_model, Hs, ds, 64, 1.0e6, q_out, w_out,
                                   cache, n, l_cap)
        torch.cuda.synchronize()
        return w_out, q_out, cache[at:at + n]

    got = run(h, 0)
    ref = [run(h[at:at + 20], at) for at in range(0, rows, 20)]
    for i, (g, name) in enumerate(zip(got, ("w", "q", "k"))):
        g = g.float().cpu().numpy()
        r = np.concatenate([x[i].float().cpu().numpy() for x in ref])
        if i:                    # q and k of the overflowing row depend on the order of the sum
            g, r = np.delete(g, 2, 0), np.delete(r, 2, 0)
        assert np.array_equal(np.isnan(g), np.isnan(r)), name
        assert np.array_equal(np.isinf(g), np.isinf(r)), name
        assert np.array_equal(np.sign(g[np.isinf(g)]), np.sign(r[np.isinf(r)])), name
    w = got[0].cpu().numpy()
    assert np.all(w[1:4] == np.inf) and np.all(w[4] == -np.inf) and np.all(np.isnan(w[5]))
    assert np.all(np.isfinite(np.delete(w, [1, 2, 3, 4, 5, rows - 1], 0)))


@pytest.mark.parametrize("rows", [5, 70])
def test_rotation_stays_bounded(rows):
    """Angles past 2^53 (a rope_base far below 1) carry no phase, but sine and
    cosine stay within [-1, 1]: a rotated pair is at most as long as twice the pair."""
    d_model, Hs, ds, l_cap = 256, 4, 128, 1 << 20
    h, wq, wk, ww = synth.selector_frontend(9, rows, d_model, Hs, ds)
    W = [bf(x) for x in (wq, wk, ww)]
    pos = dev((l_cap - 1 - 1000 * np.arange(rows)).astype(np.int32))
    got = []
    for rope in (64, 0):
        q_out = torch.empty((rows, Hs, ds), dtype=torch.bfloat16, device=DEV)
        w_out = torch.empty((rows, Hs), dtype=torch.float32, device=DEV)
        cache = torch.empty(Hs * ds, dtype=torch.bfloat16, device=DEV)
        spot.spot_selector_project(bf(h), *W, pos, rows, d_model, Hs, ds, rope, 1.0e-30, q_out,
                                   w_out, cache, rows, 0)            # (no key is stored)
        torch.cuda.synchronize()
        got.append(q_out.float().cpu().numpy())
    rot, plain = got
    assert np.all(np.isfinite(rot))
    pair = np.hypot(plain[..., :32], plain[..., 32:64])
    assert np.all(np.hypot(rot[..., :32], rot[..., 32:64]) <= 2.0 * pair + 1e-6)
    assert np.array_equal(rot[..., 64:], plain[..., 64:])


def test_project_skips_keys_outside_the_cache():
    rows, l_cap = 4, 128
    pos = np.array([5, -1, 128, 127], np.int32)
    (h, wq, wk, ww), (q_out, w_out, cache), (q_o, k_o, w_o) = run_project(
        rows, 1024, 4, 128, 64, 1.0e6, pos, 1, l_cap)
    cache_h = host_bf16(cache)
    assert np.all(cache_h[1] == 0) and np.all(cache_h[2] == 0)
    assert np.any(cache_h[0, 5] != 0) and np.any(cache_h[3, 127] != 0)
    # the queries are still produced at the given (even out-of-range) positions
    check_bf16(host_bf16(q_out), q_o, rot_sums(abs_sums(h, wq), 4, 128, 64))


def fp32_quarter_mean(k_tok, b, lo, hi):
    """The documented FP32 order: each 16-token quarter of the block summed
    as a pairwise tree ((t0 + t1) + (t2 + t3), then groups of 4 and 8; absent
    tokens -0.0), the quarters added in order, one division."""
    zero = np.full(k_tok.shape[2:], -0.0, np.float32)
    parts = []
    for q in range(4):
        vals = [bf16_value(k_tok[b, t]).astype(np.float32) if t < hi else zero
                for t in range(lo + 16 * q, lo + 16 * q + 16)]
        while len(vals) > 1:
            vals = [vals[2 * i] + vals[2 * i + 1] for i in range(len(vals) // 2)]
        parts.append(vals[0])
    tot = ((parts[0] + parts[1]) + parts[2]) + parts[3]
    return bf16_bits(tot / np.float32(hi - lo))


@pytest.mark.parametrize("n_seq,L,Hs,ds", [(3, 1024, 4, 128), (2, 4096, 8, 64)])
def test_pool_parity(n_seq, L, Hs, ds):
    rng = np.random.default_rng(L + n_seq)
    k_tok = bf16_bits(rng.standard_normal((n_seq, L, Hs, ds), dtype=np.float32))
    seq_len = np.array([L, L - 100, 1][:n_seq], np.int32)
    pooled = torch.zeros((n_seq, L // 64, Hs, ds), dtype=torch.bfloat16, device=DEV)
    spot.spot_selector_pool(bf(k_tok), pooled, n_seq, L, Hs, ds, dev(seq_len))
    torch.cuda.synchronize()
    g = host_bf16(pooled)
    o = oracle.selector_pool(k_tok, seq_len)
    gv = bf16_value(g).astype(np.float64)
    nv = (seq_len + 63) // 64
    for b in range(n_seq):
        assert np.all(np.abs(gv[b, :nv[b]] - o[b, :nv[b]]) <= 2.0 ** -8 * np.abs(o[b, :nv[b]]))
        assert np.all(g[b, nv[b]:] == 0)                      # blocks without tokens untouched
        for j in (0, nv[b] - 1):
            lo, hi = j * 64, min(j * 64 + 64, int(seq_len[b]))
            np.testing.assert_array_equal(g[b, j], fp32_quarter_mean(k_tok, b, lo, hi))


def test_decode_front_end_step():
    """One decode step's front end: project the new token (append its key),
    re-pool only its block, then score; against the oracle run on the same
    cache contents."""
    B, L, Hs, ds, d_model = 4, 8192, 8, 64, 4096
    rng = np.random.default_rng(99)
    k_tok = bf16_bits(rng.standard_normal((B, L, Hs, ds), dtype=np.float32))
    seq_len = np.array([8192, 5000, 65, 64], np.int32)
    pos = seq_len - 1
    h, wq, wk, ww = synth.selector_frontend(7, B, d_model, Hs, ds)
    cache = bf(k_tok)
    pooled = torch.zeros((B, L // 64, Hs, ds), dtype=torch.bfloat16, device=DEV)
    spot.spot_selector_pool(cache, pooled, B, L, Hs, ds, dev(seq_len))      # the prefill pooling
    q_out = torch.empty((B, Hs, ds), dtype=torch.bfloat16, device=DEV)
    w_out = torch.empty((B, Hs), dtype=torch.float32, device=DEV)
    spot.spot_selector_project(bf(h), bf(wq), bf(wk), bf(ww), dev(pos), B, d_model, Hs, ds, 32,
                               1.0e6, q_out, w_out, cache, 1, L)
    spot.spot_selector_pool(cache, pooled, B, L, Hs, ds, dev(seq_len), dev(pos // 64), 1)
    nv = (seq_len + 63) // 64
    scores = spot.selector_score(q_out, w_out, pooled, n_valid=dev(nv), nblk=L // 64)
    torch.cuda.synchronize()
    cache_h = host_bf16(cache)
    # the appended keys are the GPU's; everything downstream is checked on them
    q_o, k_o, w_o = oracle.selector_project(h, wq, wk, ww, pos, Hs, ds, rope_dim=32,
                                            rope_base=1.0e6)
    check_bf16(np.stack([cache_h[b, pos[b]] for b in range(B)]), k_o,
               rot_sums(abs_sums(h, wk), Hs, ds, 32))
    pooled_o = oracle.selector_pool(cache_h, seq_len)
    pv = bf16_value(host_bf16(pooled)).astype(np.float64)
    for b in range(B):
        assert np.all(np.abs(pv[b, :nv[b]] - pooled_o[b, :nv[b]]) <=
                      2.0 ** -8 * np.abs(pooled_o[b, :nv[b]]))
    s_o = oracle.selector_score(host_bf16(q_out), w_out.cpu().numpy(), host_bf16(pooled),
                                n_valid=nv)
    s_g = scores.cpu().numpy()
    fin = np.isfinite(s_o)
    assert np.array_equal(np.isfinite(s_g), fin)
    assert np.all(np.abs(s_g[fin] - s_o[fin]) <= 1e-4 * np.abs(s_o[fin]) + 1e-6)


@pytest.mark.parametrize("B,L,Hs,ds,rope_dim,with_len", [
    (4, 8192, 8, 64, 32, True),       # decode, Qwen3-8B hidden size
    (4, 32768, 4, 128, 64, False),    # seq_len = pos + 1
    (9, 4096, 4, 128, 0, True),       # more rows than one pass (RP = 16 path)
])
def test_fused_front_end_equals_project_then_pool(B, L, Hs, ds, rope_dim, with_len):
    """spot_selector_project_pooled gives exactly what spot_selector_project
    followed by spot_selector_pool of the new token's block gives: queries,
    weights, the cache and the whole pooled cache, bit for bit.  Positions
    cover the first token of a block, the last, the middle, position 0, a
    seq_len past pos (later tokens of the block count) and a position
    outside the cache (nothing stored or pooled)."""
    d_model = 4096
    rng = np.random.default_rng([B, L, Hs])
    k_tok = bf16_bits(rng.standard_normal((B, L, Hs, ds), dtype=np.float32))
    pos = np.array([L - 1, 64, 127, 0, 5000 % L, 200, 63, L, 1000][:B], np.int32)
    seq_len = np.minimum(pos + 1 + np.array([0, 0, 0, 0, 7, 0, 0, 0, 30][:B]), L).astype(np.int32)
    h, wq, wk, ww = synth.selector_frontend(11, B, d_model, Hs, ds)
    args = (bf(h), bf(wq), bf(wk), bf(ww))
    pool0 = torch.zeros((B, L // 64, Hs, ds), dtype=torch.bfloat16, device=DEV)
    spot.spot_selector_pool(bf(k_tok), pool0, B, L, Hs, ds, dev(np.minimum(pos, L)))
    outs = []
    for fused in (False, True):
        q_out = torch.empty((B, Hs, ds), dtype=torch.bfloat16, device=DEV)
        w_out = torch.empty((B, Hs), dtype=torch.float32, device=DEV)
        cache, pooled = bf(k_tok), pool0.clone()
        sl = dev(seq_len) if with_len else None
        if fused:
            spot.spot_selector_project_pooled(*args, dev(pos), sl, B, d_model, Hs, ds, rope_dim,
                                              1.0e6, q_out, w_out, cache, pooled, L)
        else:
            spot.spot_selector_project(*args, dev(pos), B, d_model, Hs, ds, rope_dim, 1.0e6,
                                       q_out, w_out, cache, 1, L)
            spot.spot_selector_pool(cache, pooled, B, L, Hs, ds,
                                    sl if with_len else dev(pos + 1), dev(pos // 64), 1)
        outs.append((q_out, w_out, cache, pooled))
    torch.cuda.synchronize()
    for name, a, b in zip(("q_out", "w_out", "k_cache", "k_pool"), *outs):
        if a.dtype == torch.bfloat16:
            a, b = a.view(torch.int16), b.view(torch.int16)
        assert torch.equal(a, b), name
    assert not torch.equal(outs[1][3].view(torch.int16), pool0.view(torch.int16))


@pytest.mark.parametrize("B,with_len", [(33, True), (41, False)])
def test_pooled_front_end_of_many_sequences(B, with_len):
    """More sequences than the one-launch kernel takes (projection on the
    matrix cores, then one pooling launch): still bit for bit what
    spot_selector_project and spot_selector_pool of each block give."""
    L, Hs, ds, d_model = 256, 4, 128, 1024
    rng = np.random.default_rng(B)
    k_tok = bf16_bits(rng.standard_normal((B, L, Hs, ds), dtype=np.float32))
    pos = rng.integers(0, L, B).astype(np.int32)
    pos[:4] = [0, 63, 64, L]                                   # L: outside the cache
    seq_len = np.minimum(pos + 1 + np.arange(B) % 3 * 9, L).astype(np.int32)
    seq_len[3] = 0
    h, wq, wk, ww = synth.selector_frontend(13, B, d_model, Hs, ds)
    args = (bf(h), bf(wq), bf(wk), bf(ww), dev(pos))
    outs = []
    for fused in (False, True):
        q_out = torch.empty((B, Hs, ds), dtype=torch.bfloat16, device=DEV)
        w_out = torch.empty((B, Hs), dtype=torch.float32, device=DEV)
        cache = bf(k_tok)
        pooled = torch.zeros((B, L // 64, Hs, ds), dtype=torch.bfloat16, device=DEV)
        sl = dev(seq_len) if with_len else None
        if fused:
            spot.spot_selector_project_pooled(*args, sl, B, d_model, Hs, ds, 64, 1.0e6, q_out,
                                              w_out, cache, pooled, L)
        else:
            spot.spot_selector_project(*args, B, d_model, Hs, ds, 64, 1.0e6, q_out, w_out, cache,
                                       1, L)
            # (the sequence whose position is outside pools nothing)
            spot.spot_selector_pool(cache, pooled, B, L, Hs, ds,
                                    sl if with_len else dev(np.where(pos < L, pos + 1, 0)),
                                    dev(pos // 64), 1)
        outs.append((q_out, w_out, cache, pooled))
    torch.cuda.synchronize()
    for name, a, b in zip(("q_out", "w_out", "k_cache", "k_pool"), *outs):
        if a.dtype == torch.bfloat16:
            a, b = a.view(torch.int16), b.view(torch.int16)
        assert torch.equal(a, b), name


@pytest.mark.parametrize("offset", [2, 8])
def test_pooled_front_end_of_a_misaligned_cache(offset):
    """The C entry asks for no alignment of k_cache (elements are BF16): a cache
    that starts off a 16-byte boundary gives what an aligned one does, with more
    sequences than the one-launch kernel takes as well."""
    L, Hs, ds, d_model, n = 128, 4, 128, 512, 512
    lib = spot.load()
    for B in (20, 37):
        rng = np.random.default_rng(B)
        k_tok = bf16_bits(rng.standard_normal((B, L, Hs, ds), dtype=np.float32))
        h, wq, wk, ww = (bf(x) for x in synth.selector_frontend(17, B, d_model, Hs, ds))
        pos = dev(rng.integers(0, L, B).astype(np.int32))
        outs = []
        for off in (0, offset):
            room = torch.zeros(B * L * n + 8, dtype=torch.bfloat16, device=DEV)
            cache = room[off // 2:off // 2 + B * L * n]
            assert cache.data_ptr() % 16 == off
            cache.copy_(bf(k_tok).reshape(-1))
            q_out = torch.zeros((B, n), dtype=torch.bfloat16, device=DEV)
            w_out = torch.zeros((B, Hs), device=DEV)
            pooled = torch.zeros((B, L // 64, n), dtype=torch.bfloat16, device=DEV)
            torch.cuda.synchronize()
            st = lib.spot_selector_project_pooled(
                h.data_ptr(), wq.data_ptr(), wk.data_ptr(), ww.data_ptr(), pos.data_ptr(), None,
                B, d_model, Hs, ds, 64, 1.0e6, q_out.data_ptr(), w_out.data_ptr(),
                cache.data_ptr(), pooled.data_ptr(), L, torch.cuda.current_stream().cuda_stream)
            assert st == spot.SPOT_OK
            torch.cuda.synchronize()
            outs.append((q_out, w_out, cache.clone(), pooled))
        for a, b in zip(*outs):
            assert torch.equal(a.view(torch.uint8), b.view(torch.uint8))


def test_front_end_in_a_graph_matches_eager():
    """Projection and pooling captured in a HIP graph: every replay (with
    eager work and synchronisations between replays) gives the eager result."""
    B, L, Hs, ds, d_model = 4, 4096, 4, 128, 4096
    h, wq, wk, ww = synth.selector_frontend(5, B, d_model, Hs, ds)
    hd, wqd, wkd, wwd = bf(h), bf(wq), bf(wk), bf(ww)
    seq_len = np.array([4096, 3000, 64, 1], np.int32)
    pos, first, sl = dev(seq_len - 1), dev((seq_len - 1) // 64), dev(seq_len)
    outs = []
    for _ in range(2):
        outs.append((torch.empty((B, Hs, ds), dtype=torch.bfloat16, device=DEV),
                     torch.empty((B, Hs), dtype=torch.float32, device=DEV),
                     torch.zeros((B, L, Hs, ds), dtype=torch.bfloat16, device=DEV),
                     torch.zeros((B, L // 64, Hs, ds), dtype=torch.bfloat16, device=DEV)))

    def run(o, st):
        spot.spot_selector_project(hd, wqd, wkd, wwd, pos, B, d_model, Hs, ds, 64, 1.0e6, o[0],
                                   o[1], o[2], 1, L, st)
        spot.spot_selector_pool(o[2], o[3], B, L, Hs, ds, sl, first, 1, st)

    run(outs[0], torch.cuda.current_stream())
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        run(outs[1], torch.cuda.current_stream())
    for rep in range(3):
        for t in outs[1]:
            t.zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        for a, b in zip(outs[0], outs[1]):
            assert torch.equal(a.view(torch.int16) if a.dtype == torch.bfloat16 else a,
                               b.view(torch.int16) if b.dtype == torch.bfloat16 else b), rep
