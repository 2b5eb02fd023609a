"""Prefill projections over digit operands (24-bit fixed point under one scale per token, three INT8
passes): tile and split remainders of the three tile shapes, ragged K, and rows at the edges of the
number range.

Tolerance: a digit operand is within 2^-23 of its token's largest activation (half a step of a
power-of-two grid of at least 2^22 steps), so a product over K columns is within 2^-23 sqrt(K) times
(largest / rms) of its 2-norm, under 1e-5 for K <= 8192 and a largest value of 8 rms. What exceeds
that is the rounding of k and v to BF16: a value near a tie moves by one step (2^-8 of it), for a
share of the entries of about the relative error before it over 2^-8. 2e-4 of the 2-norm covers one
entry in a thousand moving. (Hi/lo BF16 operands on the same cases: up to 1e-4.)"""
import numpy as np
import pytest
import torch

import synth
from tests.gpu_case import PrefillCase

pytestmark = pytest.mark.gpu
REL = 2e-4


def _rel(got, want):
    return float(np.linalg.norm(got - want) / np.linalg.norm(want))


def _case(sh, T, pos0=0, seed=5, p_f=0.6):
    return PrefillCase(sh, synth.raw_mask(sh, seed, p_f=p_f), T, pos0)


@pytest.mark.parametrize("T", [1, 31, 32, 33, 64, 65, 128, 129, 300])
def test_token_remainders(T):
    """Token counts around the 32-, 64- and 128-token tiles; width 528 and a per-channel mask leave
    K and N without any alignment beyond 16, and every projection splits K where T is small."""
    print(f"case digits T={T}", flush=True)
    sh = synth.tiny_shape(d=528, hq=6, hkv=3, dh=64, f=2000)
    case = _case(sh, T, pos0=7)
    assert _rel(case.run(), case.oracle()) < REL


@pytest.mark.parametrize("d,hq,hkv,dh,f,T", [(16, 1, 1, 64, 16, 5),        # one chunk, mostly padding
                                             (128, 2, 1, 128, 144, 40),
                                             (1040, 8, 8, 128, 8208, 70),   # long ragged down rows
                                             (4096, 32, 8, 128, 4096, 520)])   # 128 x 256 tiles
def test_widths(d, hq, hkv, dh, f, T):
    print(f"case digits d={d} hq={hq} hkv={hkv} dh={dh} f={f} T={T}", flush=True)
    case = _case(synth.tiny_shape(d=d, hq=hq, hkv=hkv, dh=dh, f=f), T)
    assert _rel(case.run(), case.oracle()) < REL


@pytest.mark.parametrize("shared,d,f,T", [(False, 4096, 8192, 600), (True, 4096, 8192, 600), (True, 8192, 2048, 1200)])
def test_cut_launch(shared, d, f, T):
    """Token counts at which a projection is cut in two launches (whole rounds of 128 x 256 tiles, then
    smaller ones): gate/up with about 7950 channels at 600 tokens, and the column-mapped down
    projection of 8192 rows at 1200 tokens, whose chunk list stays behind the first launch's first
    token."""
    print(f"case digits cut shared={shared} d={d} f={f} T={T}", flush=True)
    sh = synth.tiny_shape(d=d, hq=4, hkv=2, dh=64, f=f)
    case = PrefillCase(sh, synth.raw_mask(sh, 3, p_f=0.97, block=16), T, 0, shared=shared)
    assert _rel(case.run(), case.oracle()) < REL


@pytest.mark.parametrize("shared", [False, True])
@pytest.mark.parametrize("d,f,T", [(384, 640, 20),        # three chunks for four groups
                                   (640, 12800, 20),      # 32 x 64 tiles, one row tile of tokens
                                   (1152, 12800, 33),     # nine chunks; a second, nearly empty token tile
                                   (1152, 13056, 120)])   # 64 x 128 tiles, nine chunks over two groups
def test_chunk_groups(shared, d, f, T):
    """Tiles whose chunks are dealt to groups of waves (short prompts, and up to one workgroup per CU):
    chunk counts that are no multiple of the groups, and fewer chunks than groups."""
    print(f"case digits groups shared={shared} d={d} f={f} T={T}", flush=True)
    sh = synth.tiny_shape(d=d, hq=4, hkv=2, dh=64, f=f)
    case = PrefillCase(sh, synth.raw_mask(sh, 4, p_f=0.6, block=16), T, 3, shared=shared)
    assert _rel(case.run(), case.oracle()) < REL


def test_number_range():
    """Rows of zeros, of tiny and of large values, and rows with one value far above the rest: each
    token has its own scale, so a token's result does not depend on its neighbours, and its error
    stays relative to its own result."""
    print("case digits number range", flush=True)
    sh = synth.tiny_shape(d=512, hq=8, hkv=2, dh=64, f=1536)
    case = _case(sh, 8)
    x = case.x.copy()
    x[1] = 0.0
    x[2] *= 1e-20
    x[3] *= 1e12
    x[4, 7] = 3e3
    x[5, :] = 0.0
    x[5, 9] = -2.5
    case.x, case.xd = x, torch.from_numpy(x).cuda()
    got, want = case.run(), case.oracle()
    for t in (0, 2, 3, 4, 5, 6, 7):
        assert _rel(got[t], want[t]) < REL, t
    assert np.abs(got[1] - want[1]).max() <= REL * max(1.0, np.abs(want[1]).max())


def test_non_finite_rows():
    """A non-finite token gives a non-finite row and leaves the other tokens' bits alone (a layer
    without heads, so that no token reads another's key)."""
    print("case digits non-finite", flush=True)
    sh = synth.tiny_shape(d=512, hq=8, hkv=2, dh=64, f=1536)
    q, kv, f = synth.all_kept_mask(sh)
    q[:] = 0
    case = PrefillCase(sh, (q, kv, f), 8, 0)
    got = case.run()
    assert _rel(got, case.oracle()) < REL
    for bad in (np.inf, np.nan):
        case.xd = torch.from_numpy(case.x).cuda()
        case.xd[6, 3] = float(bad)
        out = case.run()
        assert np.array_equal(np.delete(out, 6, 0), np.delete(got, 6, 0))
        assert not np.isfinite(out[6]).any()


@pytest.mark.parametrize("dh,T", [(64, 5), (64, 70), (128, 40), (128, 200)])
def test_groupwise_store(dh, T):
    """The groupwise store with channel blocks of 16 and single dropped heads: with head_dim 64 a
    store chunk of 128 columns holds a kept and a dropped head, the down projection's chunks hold
    anything from one to eight blocks, and some chunks none."""
    print(f"case digits groupwise dh={dh} T={T}", flush=True)
    sh = synth.tiny_shape(d=512, hq=8, hkv=4, dh=dh, f=2048)
    q, kv, f = synth.raw_mask(sh, 21, p_q=0.6, p_f=0.4, block=16)
    f[:, 256:512] = 0
    f[:, 1024:1040] = 1
    case = PrefillCase(sh, (q, kv, f), T, 9, shared=True)
    assert _rel(case.run(), case.oracle()) < REL


@pytest.mark.parametrize("what", ["no_heads", "no_ffn", "wide"])
def test_groupwise_store_edges(what):
    """Empty modules, and the 128 x 256 tile shape with K splits."""
    print(f"case digits groupwise {what}", flush=True)
    wide = what == "wide"
    sh = synth.tiny_shape(d=4096 if wide else 256, hq=8, hkv=2, dh=128 if wide else 64, f=8192 if wide else 512)
    q, kv, f = synth.raw_mask(sh, 22, p_f=0.7, block=16)
    if what == "no_heads":
        q[:] = 0
    elif what == "no_ffn":
        f[:] = 0
    case = PrefillCase(sh, (q, kv, f), 520 if wide else 33, 0, shared=True)
    assert _rel(case.run(), case.oracle()) < REL


def _outlier_case(shared, d, f, T, ratio, where, some):
    """A layer without heads (no rounding of k and v between the input and the result) whose outputs do
    not use the columns with the outliers. where "x": column 3 of the tokens in `some` is `ratio` times the
    rms of the others, and no gate or up row reads it; "h": channel 5's up row is `ratio` times the
    others', and the down projection does not read it. The scales make the layer's own contribution
    larger than the residual, which float32 adds to it."""
    sh = synth.tiny_shape(d=d, hq=2, hkv=1, dh=64, f=f)
    layer = synth.layer_weights(sh, 0, quant="group" if shared else "row")

    def scale(name, factor, rows=slice(None)):
        w, s = layer[name]
        s = s.copy()
        s[rows] = synth.to_bf16_bits(synth.bf16_bits_to_f32(s[rows]) * np.float32(factor)) if shared else s[rows] * np.float32(factor)
        layer[name] = (w, s)

    def drop(name, column):
        w = layer[name][0].copy()
        w[:, column] = 0
        layer[name] = (w, layer[name][1])

    scale("wd", 64.0)
    if where == "x":
        # the RMS of a row with the outlier is ratio / sqrt(d)
        up = 2.0 ** max(0, round(np.log2(ratio / np.sqrt(d))))
        for n in ("wg", "wu"):
            scale(n, up)
            drop(n, 3)
    else:
        scale("wu", 2.0 ** round(np.log2(ratio)), slice(5, 6))
        drop("wd", 5)
    q, kv, ff = synth.all_kept_mask(sh)
    q[:] = 0
    case = PrefillCase(sh, (q, kv, ff), T, 0, store=[layer], shared=shared)
    if where == "x":
        x = case.x.copy()
        x[some, 3] = ratio * np.sign(x[some, 3] + 0.5)
        case.x, case.xd = x, torch.from_numpy(x).cuda()
    return case


OUTLIER_CASES = [   # store, widths, tokens, launches: every tile shape of both projections
    (False, 512, 512, 5, dict(gateup=(2, 1, 0, 0), down=(2, 2, 0, 0))),
    (False, 1024, 512, 5, dict(gateup=(3, 1, 0, 0))),
    (False, 512, 12288, 33, dict(gateup=(1, 1, 0, 0))),
    (False, 4096, 2048, 33, dict(down=(1, 8, 0, 0))),
    (False, 1024, 1024, 700, dict(gateup=(4, 1, 0, 0))),
    (False, 512, 6144, 330, dict(gateup=(0, 1, 0, 0))),
    (False, 4096, 528, 1040, dict(down=(0, 1, 0, 0))),
    (False, 1024, 4096, 1040, dict(gateup=(0, 1, 1024, 3))),
    (True, 512, 512, 520, dict(down=(3, 1, 0, 0))),
    (True, 512, 12288, 5, dict(gateup=(2, 1, 0, 0), down=(3, 8, 0, 0))),
    (True, 512, 8192, 33, dict(gateup=(1, 1, 0, 0))),
    (True, 1024, 8192, 130, dict(down=(4, 8, 0, 0))),
    (True, 512, 16384, 200, dict(gateup=(0, 1, 0, 0))),
    (True, 8192, 512, 1000, dict(down=(0, 1, 0, 0))),
    (True, 8192, 2048, 1060, dict(down=(0, 1, 1024, 3)))]


@pytest.mark.parametrize("shared,d,f,T,launches", OUTLIER_CASES)
def test_outlier_rows(shared, d, f, T, launches):
    """Rows with one value far above the others: what does not use that value is as exact as with hi/lo
    BF16 operands. Such an operand is off by rms 2.4e-6 (2^-16 sqrt(0.308 / 12)) of its rms; the layer's
    result takes that from gate, up and down, 2.4e-6 sqrt(3) with silu's slope up to 1.1, so 5e-6; four
    times that is allowed (with digits alone: 7e-5 to 2e-3 at these ratios)."""
    every = np.arange(T)
    for where, ratio, some in (("x", 1000.0, every[every % 5 == 2]),       # digit and pair rows in a tile
                               ("x", 3e5, every),                          # pair rows only
                               ("h", 60.0, every),                         # about half of the rows
                               ("h", 1e4, every)):
        print(f"case outliers shared={shared} d={d} f={f} T={T} {where} {ratio}", flush=True)
        case = _outlier_case(shared, d, f, T, ratio, where, some)
        for kind, want in launches.items():
            assert case.launch(kind) == want
        # (the outlier's own column holds it in float32 beside the layer's result)
        got, want = (np.delete(y - case.x, 3, axis=1) for y in (case.run(), case.oracle()))
        rel = np.linalg.norm(got - want, axis=1) / np.linalg.norm(want, axis=1)
        print(f"  relative error: largest {rel.max():.2e}, median {np.median(rel):.2e}", flush=True)
        assert rel.max() < 2e-5, (where, ratio, int(rel.argmax()))
