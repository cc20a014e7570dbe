"""Parity of the matrix-core scorer of many query rows per sequence (a prompt)
with the FP64 oracle (needs an MI355X): pooled keys, and per-token keys with
blocks of 16 and 64 tokens, in every key and query format.

Sizes lie at the edges of its tiles (64 rows and 32 keys per workgroup step,
runs of several steps) and past the number of (row, key) pairs that sends a call
there (some quantized ones short of it: the row kernels); what each row sees is random: nothing, everything, past the end,
and limits inside a tile.  Tolerance as for the row kernels:
|gpu - oracle| <= 1e-4 |oracle| + 1e-6, the same -inf entries.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2606_22874_amd import spot, synth
from paper_2606_22874_amd.synth import bf16_bits

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

DEV = "cuda:0"
FORMATS = ("bf16", "int4", "mxfp4", "int8", "mxfp8")


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


def bf(a):
    return spot.to_device_bf16(a, DEV)


def assert_scores_close(g, o):
    fin = np.isfinite(o)
    assert np.array_equal(np.isfinite(g), fin)
    assert np.all(g[~fin] == -np.inf)
    err = np.abs(g[fin] - o[fin])
    bound = 1e-4 * np.abs(o[fin]) + 1e-6
    assert np.all(err <= bound), f"max excess {np.max(err - bound)}"


def coded(x, fmt):
    """(host codes, host scales, device codes, device scales) of BF16 bits x."""
    if fmt == "bf16":
        return x, None, bf(x), None
    c, s = synth.QUANTIZERS[fmt](x)
    s = s.view(np.uint16) if fmt in ("int4", "int8") else s
    return c, s, dev(c), dev(s.view(np.int16) if fmt in ("int4", "int8") else s)


def inputs(n_seq, rows, n_keys, Hs, ds):
    rng = np.random.default_rng([n_seq, rows, n_keys, Hs])
    q = bf16_bits(rng.standard_normal((n_seq * rows, Hs, ds), dtype=np.float32))
    w = rng.uniform(0, 1, (n_seq * rows, Hs)).astype(np.float32)
    k = bf16_bits(rng.standard_normal((n_seq, n_keys, Hs, ds), dtype=np.float32))
    see = rng.integers(-3, n_keys + 40, n_seq * rows).astype(np.int32)
    see[:3] = [0, n_keys, 1]
    see[-rows // 2:] = np.minimum(see[-rows // 2:], n_keys // 3)   # some tiles see little
    return q, w, k, see


@pytest.mark.parametrize("n_seq,rows,n_keys,Hs,ds", [
    (1, 64, 1025, 4, 128), (2, 65, 512, 8, 64), (1, 130, 799, 8, 64), (3, 129, 129, 4, 128),
    (1, 1030, 63, 4, 128), (40, 17, 97, 8, 64), (3, 161, 161, 4, 128), (310, 9, 130, 8, 64)])
@pytest.mark.parametrize("fmt", FORMATS)
def test_pooled_keys(n_seq, rows, n_keys, Hs, ds, fmt):
    print(f"[many] pooled {n_seq} x {rows} rows, {n_keys} keys, {Hs}x{ds} {fmt}", flush=True)
    q, w, k, see = inputs(n_seq, rows, n_keys, Hs, ds)
    kc, ks, kd, ksd = coded(k, fmt)
    for lim in (see, None):
        s_o = oracle.selector_score(q, w, kc, ks, fmt, rows_per_seq=rows, n_valid=lim,
                                    nblk=n_keys, h_s=Hs, d_s=ds)
        s_g = spot.selector_score(bf(q), dev(w), kd, ksd, fmt, rows_per_seq=rows,
                                  n_valid=None if lim is None else dev(lim), nblk=n_keys)
        assert_scores_close(s_g.cpu().numpy(), s_o)


@pytest.mark.parametrize("qfmt", FORMATS[1:])
@pytest.mark.parametrize("kfmt", FORMATS)
def test_pooled_keys_quantized_queries(qfmt, kfmt):
    print(f"[many] pooled q={qfmt} k={kfmt}", flush=True)
    for n_seq, rows, n_keys, Hs, ds in ((1, 67, 799, 8, 64), (2, 66, 385, 4, 128),
                                        (1, 131, 1001, 8, 64), (2, 130, 513, 4, 128)):
        q, w, k, see = inputs(n_seq, rows, n_keys, Hs, ds)
        qc, qs, qd, qsd = coded(q, qfmt)
        kc, ks, kd, ksd = coded(k, kfmt)
        s_o = oracle.selector_score_qk(qc, qs, qfmt, w, kc, ks, kfmt, n_seq * rows, n_keys, Hs,
                                       ds, rows_per_seq=rows, n_valid=see)
        out = torch.full((n_seq * rows, n_keys), 7.0, device=DEV)
        spot.spot_selector_score_q(qd, qsd, qfmt, dev(w), kd, ksd, kfmt, n_seq, rows, n_keys, Hs,
                                   ds, dev(see), out)
        assert_scores_close(out.cpu().numpy(), s_o)


def test_pooled_keys_extreme_scales():
    """Key and query scales whose product is no FP32 number (2^117 and 2^-126
    against 2048 and 2^-14), and sums that are none under the key's scale alone
    (32 x 127 x 448 x 2^108, times 2^-10): every score is one, and exact."""
    rows, n_keys, Hs, ds = 128, 1024, 4, 128
    print("[many] pooled extreme scales", flush=True)
    # (query code, scale, key code, scale, elements of a group that are not zero)
    for qv, kv, nz in ((((1, 2048.0), (1, 2.0 ** -14)), ((0x01, 117, 2.0 ** -9), (0x78, -126, 256.0)),
                        1),
                       (((127, 2.0 ** -10), (-127, 2.0 ** -10)), ((0x7E, 108, 448.0),
                                                                (0x7E, 107, 448.0)), 32)):
        q = np.zeros((rows, Hs, 4, 32), np.int8)
        qs = np.zeros((rows, Hs, 4), np.float16)
        kc = np.zeros((1, n_keys, Hs, 4, 32), np.uint8)
        ks = np.zeros((1, n_keys, Hs, 4), np.uint8)
        for i in (0, 1):                       # even and odd rows and keys
            q[i::2, ..., :nz] = qv[i][0]
            qs[i::2] = qv[i][1]
            kc[:, i::2, ..., :nz] = kv[i][0]
            ks[:, i::2] = 127 + kv[i][1]
        w = np.ones((rows, Hs), np.float32)
        got = []
        for n in (rows, 4):                    # all rows, or four a call (the row kernel)
            for at in range(0, rows, n):
                out = torch.zeros((n, n_keys), device=DEV)
                spot.spot_selector_score_q(dev(q[at:at + n]), dev(qs[at:at + n].view(np.int16)),
                                           "int8", dev(w[at:at + n]), dev(kc), dev(ks), "mxfp8", 1,
                                           n, n_keys, Hs, ds, None, out)
                got.append(out.cpu().numpy())
        qval = np.array([v[0] * v[1] for v in qv])[np.arange(rows) % 2]
        kval = np.array([v[2] * 2.0 ** v[1] for v in kv])[np.arange(n_keys) % 2]
        want = np.maximum(16.0 * nz * qval[:, None] * kval, 0.0)
        for g in (got[0], np.concatenate(got[1:])):
            assert np.array_equal(g.astype(np.float64), want)


@pytest.mark.parametrize("n_seq,rows,L,Hs,ds", [
    (1, 96, 1024, 4, 128), (2, 65, 832, 8, 64), (3, 8, 4160, 4, 128), (1, 513, 448, 8, 64)])
@pytest.mark.parametrize("fmt", FORMATS)
def test_token_keys(n_seq, rows, L, Hs, ds, fmt):
    """Both block sizes; the 64-token values are the largest of their four
    16-token values, bit for bit."""
    print(f"[many] tokens {n_seq} x {rows} rows, {L} tokens, {Hs}x{ds} {fmt}", flush=True)
    q, w, k, see = inputs(n_seq, rows, L, Hs, ds)
    kc, ks, kd, ksd = coded(k, fmt)
    for lim in (see, None):
        got = {}
        for blk in (16, 64):
            s_o = oracle.selector_score_tokens(q, w, kc, ks, fmt, rows_per_seq=rows, seq_len=lim,
                                               l_cap=L, blk=blk, h_s=Hs, d_s=ds)
            s_g = spot.selector_score_tokens(bf(q), dev(w), kd, ksd, fmt, rows_per_seq=rows,
                                             seq_len=None if lim is None else dev(lim), l_cap=L,
                                             blk=blk)
            got[blk] = s_g.cpu().numpy()
            assert_scores_close(got[blk], s_o)
        assert np.array_equal(got[16].reshape(len(q), -1, 4).max(2), got[64])


@pytest.mark.parametrize("blk", [16, 64])
@pytest.mark.parametrize("fmt", FORMATS)
def test_token_keys_special_values(fmt, blk):
    """NaN and infinities in w and in BF16 keys: the same blocks are NaN, +inf
    and -inf as from the row kernels, which take the same rows two at a time."""
    rows, L, Hs, ds = 70, 2048, 4, 128
    print(f"[many] special values {fmt} blocks of {blk}", flush=True)
    q, w, k, _ = inputs(1, rows, L, Hs, ds)
    w[3, 1] = np.nan
    w[20:40, 2] = np.nan
    w[40:50, 0] = np.inf
    w[50:60, 3] = -np.inf
    if fmt == "bf16":
        k[0, 640:704, 1, 5] = 0x7FC0            # NaN keys: their head counts nothing
        k[0, 700:900, 2, 9] = 0x7F80            # infinite ones
    see = (L - 29 * np.arange(rows)).astype(np.int32)   # every rest of a block
    see[[20, 21, 22, 23]] = [33, 32, 16, 1]
    see[[40, 50]] = [0, 17]
    _, _, kd, ksd = coded(k, fmt)

    def run(at, n):
        return spot.selector_score_tokens(bf(q[at:at + n]), dev(w[at:at + n]), kd, ksd, fmt,
                                          rows_per_seq=n, seq_len=dev(see[at:at + n]), l_cap=L,
                                          blk=blk).cpu().numpy()

    many = run(0, rows)
    few = np.concatenate([run(at, 2) for at in range(0, rows, 2)])
    assert np.any(np.isnan(few)) or fmt in ("int4", "mxfp4")
    assert np.any(few == np.inf) and np.any(few == -np.inf)
    assert np.array_equal(np.isnan(many), np.isnan(few))
    assert np.array_equal(np.isinf(many) * np.sign(many), np.isinf(few) * np.sign(few),
                          equal_nan=True)
    fin = np.isfinite(few)
    assert np.all(np.abs(many[fin] - few[fin]) <= 1e-4 * np.abs(few[fin]) + 1e-6)


@pytest.mark.parametrize("fmt,offset,tokens", [("int4", 4, False), ("mxfp4", 8, False),
                                               ("int8", 8, False), ("mxfp8", 8, False),
                                               ("int8", 8, True), ("mxfp8", 8, True)])
def test_misaligned_codes(fmt, offset, tokens):
    """The C entries take code caches aligned to what the row kernels read (4
    bytes of 4-bit codes, 8 of 8-bit ones) in a call of any size."""
    rows, n, Hs, ds = 128, 1024, 4, 128
    print(f"[many] {fmt} codes {offset} bytes off, tokens {tokens}", flush=True)
    q, w, k, see = inputs(1, rows, n, Hs, ds)
    kc, ks, kd, ksd = coded(k, fmt)
    room = torch.zeros(kd.numel() + 16, dtype=torch.uint8, device=DEV)
    codes = room[offset:offset + kd.numel()]
    codes.copy_(kd.reshape(-1).view(torch.uint8))
    qd, wd, sd = bf(q), dev(w), dev(see)
    out = torch.zeros((rows, n // 64 if tokens else n), device=DEV)
    torch.cuda.synchronize()
    lib, stream = spot.load(), torch.cuda.current_stream().cuda_stream
    f = lib.spot_selector_score_tokens if tokens else lib.spot_selector_score
    st = f(qd.data_ptr(), wd.data_ptr(), codes.data_ptr(), ksd.data_ptr(), spot.KFMT[fmt], 1, rows,
           n, Hs, ds, sd.data_ptr(), out.data_ptr(), stream)
    assert st == spot.SPOT_OK
    torch.cuda.synchronize()
    if tokens:
        o = oracle.selector_score_tokens(q, w, kc, ks, fmt, rows_per_seq=rows, seq_len=see, l_cap=n,
                                         blk=64, h_s=Hs, d_s=ds)
    else:
        o = oracle.selector_score(q, w, kc, ks, fmt, rows_per_seq=rows, n_valid=see, nblk=n,
                                  h_s=Hs, d_s=ds)
    assert_scores_close(out.cpu().numpy(), o)


@pytest.mark.parametrize("fmt", FORMATS)
def test_pooled_keys_special_values(fmt):
    """NaN, infinities and the smallest numbers in w and in BF16 keys and queries:
    the same scores are NaN, +inf and -inf as from the row kernel, which takes the
    same rows four at a time."""
    rows, n, Hs, ds = 132, 1030, 8, 64
    print(f"[many] pooled special values {fmt}", flush=True)
    q, w, k, see = inputs(1, rows, n, Hs, ds)
    w[3, 1] = np.nan
    w[20:40, 2] = np.nan
    w[40:50, 0] = np.inf
    w[50:60, 7] = -np.inf
    w[60:70] *= 1e-38
    w[70:80] *= -1
    q[90, 5, 3], q[91, 6, 60], q[92, 0, 0] = 0x7FC0, 0x7F80, 0x0001
    if fmt == "bf16":
        k[0, 100:140, 1, 5] = 0x7FC0
        k[0, 300:310, 2, 9] = 0xFF80
        k[0, 700:720] = 0x0001
    _, _, kd, ksd = coded(k, fmt)

    def run(at, m):
        return spot.selector_score(bf(q[at:at + m]), dev(w[at:at + m]), kd, ksd, fmt,
                                   rows_per_seq=m, n_valid=dev(see[at:at + m]),
                                   nblk=n).cpu().numpy()

    many = run(0, rows)
    few = np.concatenate([run(at, 4) for at in range(0, rows, 4)])
    assert np.any(np.isnan(few)) and np.any(few == np.inf)
    assert np.array_equal(np.isnan(many), np.isnan(few))
    assert np.array_equal(np.isinf(many) * np.sign(many), np.isinf(few) * np.sign(few),
                          equal_nan=True)
    fin = np.isfinite(few)
    assert np.all(np.abs(many[fin] - few[fin]) <= 1e-4 * np.abs(few[fin]) + 1e-6)
