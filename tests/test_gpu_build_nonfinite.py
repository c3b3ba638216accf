"""GPU: a span side with a NaN or an infinite token keeps no component: its stored factors are
zeros throughout (its block then adds nothing to a step), and every other span's block has the
bytes that it has without that token.  Sketch-spanned and longer spans, with and without
iterations, in the kernels of one and of four waves per span side."""

import numpy as np
import pytest

import oracle
from synth import make_prefill
from tests.gpu_common import banner
from tests.test_gpu_build import S, _build  # noqa: F401

pytestmark = pytest.mark.gpu
LENGTHS = [15, 16, 33, 3, 130, 40, 41, 257]


@pytest.mark.parametrize("dtype,d,rank,sketch,power,heads", [
    ("bf16", 128, 32, 40, 1, 2), ("bf16", 128, 32, 40, 1, 36), ("bf16", 64, 16, 24, 0, 36), ("f32", 128, 32, 40, 1, 36),
    ("f32", 64, 12, 18, 2, 2), ("bf16", 64, 40, 40, 2, 36)])
def test_non_finite_tokens_keep_nothing(S, dtype, d, rank, sketch, power, heads):  # noqa: F811
    banner(f"non-finite tokens {dtype} d{d} r{rank} l{sketch} p{power} heads {heads}")
    n = sum(LENGTHS) + len(LENGTHS)
    p = make_prefill(1, heads, d, [n], dtype=dtype, true_rank=min(rank, 20), noise=0.05, sketch=sketch, seed=83)
    p.surprisal[:] = 1.0
    end = np.cumsum([L + 1 for L in LENGTHS]) - 1
    p.surprisal[0, end] = 9.0
    c = dict(rank=rank, sketch=sketch, min_span=2, window=0, power=power, Hkv=heads, d=d)
    clean, _, lay = _build(S, p, c)
    odd = {"nan": np.nan, "inf": np.inf, "-inf": -np.inf}
    odd = {k: (oracle.narrow(np.float32(v), dtype) if dtype == "bf16" else np.float32(v)) for k, v in odd.items()}
    hit = {}
    for i, side, what in ((1, "K", "nan"), (4, "V", "inf"), (4, "K", "nan"), (7, "K", "-inf"), (3, "V", "nan")):
        rows = p.keys if side == "K" else p.values
        for g in (0, heads - 1):
            rows[0, g, int(end[i]) - LENGTHS[i] // 2, 5 + i] = odd[what]
            hit[i, g, side] = what
    got, _, lay2 = _build(S, p, c)
    assert np.array_equal(lay["block_off"], lay2["block_off"])
    spans = dict(oracle.segment(p.surprisal[0], n, 1.0, 2, 0)[1])
    for i, L in enumerate(LENGTHS):
        s0 = int(end[i]) - L
        assert spans[s0] == L
        at = sorted(spans).index(s0)
        for g in range(heads):
            w = int(lay["block_rank"][0, g, at])
            a, b = (oracle.read_span_block(t["factors"], int(lay["block_off"][0, g, at]), L, w & 0xFFFF, d, dtype, w >> 16)
                    for t in (clean, got))
            for side in ("K", "V"):
                for name in ("U" + side, "s" + side, "Vt" + side):
                    if (i, g, side) in hit:
                        assert np.all(b[name] == 0), (i, g, name, hit[i, g, side])
                    else:
                        assert np.array_equal(a[name], b[name]), (i, g, name)
