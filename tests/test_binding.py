"""The native marshalling of spot.py's calls (csrc/binding.cpp) against the
Python checks it stands in for: what it takes gives the same outputs, bit for
bit, and whatever it does not take is left to the Python path (it answers
None), so that the same calls raise the same errors either way.
"""
import math
import shutil

import numpy as np
import pytest
import torch

from paper_2606_22874_amd import build, spot

DEV = "cuda:0"
ENTRIES = ("selector_score", "selector_score_q", "selector_score_tokens_blk", "selector_project",
           "selector_project_pooled", "selector_pool", "select_blocks", "sparse_decode_blk",
           "dense_decode", "sparse_prefill", "decode_step", "decode_step_static")


def test_native_leaves_the_rest_to_python():
    """No arguments, too many, wrong kinds: None from every entry."""
    if not build.os.path.exists(build.SO):
        build.build()
    spot.load()
    cpu = torch.zeros(64, dtype=torch.int32)
    for name in ENTRIES:
        f = getattr(spot._native, name)
        for args in ((), (None,) * 40, (cpu,) * 20, (1,) * 20, ("bf16",) * 20, (2 ** 70,) * 20):
            assert f(*args) is None, (name, args)


def test_without_the_native_module(monkeypatch, capsys, tmp_path):
    """No marshalling module and no way to build one: the library still loads, and
    every call takes the Python path."""
    if not build.os.path.exists(build.SO):
        build.build()

    def no_compiler():
        raise RuntimeError("g++ failed for binding.cpp")

    monkeypatch.setattr(build, "BINDING", str(tmp_path / "_binding.so"))
    monkeypatch.setattr(build, "build_binding", no_compiler)
    monkeypatch.setattr(spot, "_lib", None)
    monkeypatch.setattr(spot, "_native", None)
    lib = spot.load()
    assert lib is spot._lib and spot._native is None
    assert "marshalled in Python" in capsys.readouterr().err
    with pytest.raises(ValueError, match="scores must be a device tensor"):
        x = torch.zeros(4)
        spot.spot_select_blocks(x, 1, 4, None, 0.9, 4, 0, 1, 1, x, x)


def test_module_of_another_torch_is_rebuilt(monkeypatch, tmp_path):
    """The torch it was built against is read from the file before it is imported."""
    if not build.os.path.exists(build.SO):
        build.build()
    if not build.binding_fits():
        build.build_binding()
    assert build.binding_fits()
    other = tmp_path / "_binding.so"
    shutil.copy(build.BINDING, other)
    tag = f"spot binding for torch {torch.__version__}".encode()
    data = other.read_bytes()
    assert tag in data
    other.write_bytes(data.replace(tag, tag[:-1] + b"?"))
    built = []
    monkeypatch.setattr(build, "BINDING", str(other))
    monkeypatch.setattr(build, "build_binding", lambda: built.append(1))
    monkeypatch.setattr(spot, "_lib", None)
    monkeypatch.setattr(spot, "_native", None)
    spot.load()
    assert built == [1]


def bf(*shape):
    return torch.randn(shape, device=DEV).bfloat16()


def f32(*shape):
    return torch.rand(shape, device=DEV)


def i32(*vals):
    return torch.tensor(vals, dtype=torch.int32, device=DEV)


def calls():
    """(function, positional arguments, outputs' positions, keywords) of every call: B = 2, 256
    tokens, 4 query heads over 1 KV head."""
    B, L, Hq, Hkv, K = 2, 256, 4, 1, 3
    nb, sm = L // 64, 1.0 / math.sqrt(128)
    lens, nv = i32(256, 130), i32(4, 3)
    k_pool, k_tok = bf(B, nb, 8, 64), bf(B, L, 4, 128)
    q_sel, w8, w4 = bf(B, 8, 64), f32(B, 8), f32(B, 4)
    codes = torch.randint(0, 256, (B, nb, 4, 64), dtype=torch.uint8, device=DEV)
    scale = torch.randint(120, 130, (B, nb, 4, 4), dtype=torch.uint8, device=DEV)
    q, k, v = bf(B, Hq, 128), bf(B, Hkv, L, 128), bf(B, Hkv, L, 128)
    idx, cnt = i32(0, 1, 3, 0, 2, -1).reshape(2, 3), i32(3, 2)

    def outs():
        return (torch.zeros((B, nb), device=DEV),
                torch.zeros((B, K), dtype=torch.int32, device=DEV),
                torch.zeros(B, dtype=torch.int32, device=DEV), torch.zeros(B, device=DEV),
                torch.zeros((B, Hq, 128), dtype=torch.bfloat16, device=DEV),
                torch.zeros((B, Hq), device=DEV))

    def ws():
        return spot.decode_workspace(B, Hq, Hkv, 128, nb, DEV)

    def wss():
        return spot.step_workspace(B, Hq, Hkv, 128, K, DEV)

    rule = (0.9, K, 0, 1, 1)
    o = outs
    step = [B, Hq, Hkv, 128, L, sm]
    h, wq, wk, ww = bf(B, 512), bf(512, 512), bf(512, 512), bf(4, 512)
    pq, pk, pv = bf(1, 4, L, 128), bf(1, 1, L, 128), bf(1, 1, L, 128)
    pidx, pcnt = i32(0, 1, 2, 3).reshape(4, 1), i32(1, 1, 1, 1)

    def front():
        return [torch.zeros((B, 512), dtype=torch.bfloat16, device=DEV),
                torch.zeros((B, 4), device=DEV), k_tok.clone()]

    return [
        (spot.spot_selector_score, [q_sel, w8, k_pool, None, "bf16", B, 1, nb, 8, 64, nv, o()[0]],
         [11], {}),
        (spot.spot_selector_score_q, [codes[:, 0].contiguous(), scale[:, 0].contiguous(), "mxfp4",
                                      w4, codes, scale, 2, B, 1, nb, 4, 128, None, o()[0]],
         [13], {}),
        (spot.spot_selector_score_tokens, [bf(B, 4, 128), w4, k_tok, None, 0, B, 1, L, 4, 128,
                                           lens, o()[0]], [11], {}),
        (spot.spot_selector_score_tokens_blk, [bf(B, 4, 128), w4, k_tok, None, "bf16", B, 1, L, 16,
                                               4, 128, lens, torch.zeros((B, 16), device=DEV)],
         [12], {}),
        (spot.spot_selector_project, [h, wq, wk, ww, i32(3, 9), B, 512, 4, 128, 64, 1e6, *front(),
                                      1, L], [11, 12, 13], {}),
        (spot.spot_selector_project_pooled, [h, wq, wk, ww, i32(3, 9), None, B, 512, 4, 128, 64,
                                             1000000, *front(), bf(B, nb, 512), L],
         [12, 13, 14, 15], {}),
        (spot.spot_selector_pool, [k_tok, bf(B, nb, 512), B, L, 4, 128, lens], [1], {}),
        (spot.spot_select_blocks, [f32(B, nb), B, nb, nv, *rule, *o()[1:4]], [9, 10, 11], {}),
        (spot.spot_sparse_decode, [q, k, v, lens, idx, cnt, K, *step, *o()[4:], ws()],
         [13, 14], {}),
        (spot.spot_sparse_decode_blk, [q, k, v, lens, idx, cnt, K, 16, *step, o()[4], None, ws()],
         [14], {}),
        (spot.spot_dense_decode, [q, k, v, lens, *step, *o()[4:], ws()], [10, 11], {}),
        (spot.spot_sparse_prefill, [pq, pk, pv, L, pidx, pcnt, 1, 1, 4, 1, 128, sm,
                                    torch.zeros_like(pq), None], [12], {}),
        (spot.spot_decode_step, [q_sel, w8, k_pool, None, "bf16", 8, 64, nv, *rule, q, k, v, lens,
                                 *step, *o(), wss()], [23, 24, 25, 26, 27, 28], {}),
        (spot.spot_decode_step, [codes[:, 0].contiguous(), w4, codes, scale, "mxfp4", 4, 128, None,
                                 *rule, q, k, v, lens, *step, *o(), wss()],
         [23, 24, 25, 26, 27, 28], dict(q_scale=scale[:, 0].contiguous(), qfmt="mxfp4")),
        (spot.spot_decode_step_static, [q_sel, w8, k_pool, None, 0, 8, 64, nv, *rule, q, k, v,
                                        lens, *step, *o()], [23, 24, 25, 26, 27, 28], {}),
    ]


class Answers:
    """The native module, noting what each entry answered."""

    def __init__(self, module):
        self.module, self.seen = module, []

    def __getattr__(self, name):
        f = getattr(self.module, name)

        def call(*args):
            st = f(*args)
            self.seen.append((name, st))
            return st
        return call


def both(f, args, kw, monkeypatch):
    """What the call does with the native module and without: outputs or the
    error; and what the native entry answered."""
    seen, native = [], Answers(spot._native)
    for module in (native, None):
        with monkeypatch.context() as m:
            m.setattr(spot, "_native", module)
            a = [x.clone() if isinstance(x, torch.Tensor) and x.is_contiguous() and
                 x.data_ptr() % 16 == 0 else x for x in args]
            try:
                f(*a, **kw)
                torch.cuda.synchronize()
                seen.append(a)
            except Exception as e:       # compared below
                seen.append((type(e), str(e)))
    assert len(native.seen) == 1         # every call asks it once
    return (*seen, native.seen[0][1])


def same(nat, py, outs, at):
    """Equal errors, or equal outputs bit for bit."""
    if isinstance(nat, tuple) or isinstance(py, tuple):
        assert nat == py, (*at, nat, py)
        return
    for j in outs:
        if py[j] is not None:
            assert torch.equal(nat[j].view(torch.uint8), py[j].view(torch.uint8)), (*at, j)


@pytest.mark.gpu
@pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")
def test_native_equals_python(monkeypatch):
    """Every call, on the current stream and on a given one, is taken by the native
    entry (a raw stream handle is not) and gives the same outputs, bit for bit.
    Then every tensor argument in turn made unacceptable or optional (other type, one
    element short, not contiguous, misaligned, on the host, None) or larger, and
    every positive size changed (negative, zero, one off, past 32 bits, another
    kind of number): the same outputs or the same error."""
    torch.manual_seed(3)
    spot.load()
    side = torch.cuda.Stream()
    for f, args, outs, kw in calls():
        print(f"[binding] {f.__name__}", flush=True)
        for stream in (None, side, side.cuda_stream):
            torch.cuda.synchronize()
            nat, py, st = both(f, args, dict(kw, stream=stream), monkeypatch)
            assert isinstance(nat, list) and isinstance(py, list), (f, nat, py)
            same(nat, py, outs, (f.__name__, stream))
            assert st == (None if isinstance(stream, int) else spot.SPOT_OK), (f.__name__, stream)
        for j, x in enumerate(args):
            if isinstance(x, torch.Tensor) and x.numel() > 1:
                flat = x.reshape(-1)
                bad = [x.double(), flat[:-1], torch.stack((flat, flat), 1)[:, 0],
                       torch.cat((flat, flat))[1:1 + flat.numel()], x.cpu(), None,
                       torch.cat((flat, flat))]
                if x.dtype == torch.uint8 and j == len(args) - 1:
                    bad = [flat[:16], x.cpu(), None]          # a workspace: any type
            elif isinstance(x, int) and x > 0:
                bad = [-1, 0, x - 1, x + 1, 2 ** 31, x + 2 ** 32, float(x), np.int64(x), True]
            else:
                continue
            for b in bad:
                at = (f.__name__, j, tuple(b.shape) if isinstance(b, torch.Tensor) else b)
                nat, py, st = both(f, args[:j] + [b] + args[j + 1:], kw, monkeypatch)
                same(nat, py, outs, at)
                if isinstance(b, torch.Tensor) and b.is_cuda and b.dtype == x.dtype and \
                        b.numel() == 2 * x.numel():
                    assert st == spot.SPOT_OK, at             # slack is no reason to decline
