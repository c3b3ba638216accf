"""GPU: infinite stored values in a bfloat16 step, entry by entry.

A value of plus or minus infinity under a positive weight makes its output infinite with that sign, and
touches no other output: an anchor's or a summary's value its own column, a token's U_V entry or
a sigma_V every column with the sign of Vt_V there, a Vt_V entry its column with the sign of the
weighted sum above it.  A key factor that drives a token's (or a whole span's) score to minus
infinity takes that token (span) out of the softmax, as a huge finite one does.  Untouched outputs
follow the CPU oracle on the same case with the entry finite."""

import numpy as np
import pytest

import oracle
from synth import custom_spec, make_case
from synth.cases import from_storage
from tests.gpu_common import assert_out_close, banner, case_arrays, dims_for, oracle_result, out_to_f64

pytestmark = pytest.mark.gpu
INF, NINF = 0x7F80, 0xFF80
SHAPES = [(1, 64, 8, 3), (2, 128, 16, 5), (4, 128, 32, 2), (8, 64, 64, 4)]      # group, d, rank, top-k


def make(g, d, r, k):
    case = make_case(custom_spec(batch=2, n_q_heads=2 * g, n_kv_heads=2, head_dim=d, rank=r, top_k=k, context=2400,
                                 n_prefix_anchors=40, window=30, span_min=20, span_max=70, dtype="bf16", seed=200 + g))
    for name in ("anchor_v", "sum_v", "factors"):
        setattr(case, name, getattr(case, name).copy())
    return case


def parts(case, b, g, span):
    """Writable views of one block: UK, sK, VtK, UV, sV, VtV (bfloat16 words)."""
    L, r, d = int(case.span_len[b, span]), case.spec.rank, case.spec.head_dim
    x = case.factors.view(np.uint8).reshape(-1)[int(case.block_off[b, g, span]):].view(np.uint16)
    out, at = {}, 0
    for side in ("K", "V"):
        for name, shape in (("U", (L, r)), ("s", (r,)), ("Vt", (r, d))):
            n = int(np.prod(shape))
            out[name + side] = x[at:at + n].reshape(shape)
            at += n
    return out


def run(case):
    import torch
    from paper_2606_31145_amd import sekv as S
    dev = torch.device("cuda:0")
    dc = S.DeviceCache.from_arrays(case_arrays(case), case.dtype, dev)
    dims = dims_for(S, case, out_dtype="f32")
    ws = S.Workspace(dims, dev)
    sel, out = S.decode_step(dims, dc, ws)
    torch.cuda.synchronize()
    assert ws.status() == 0
    return sel.cpu().numpy(), out_to_f64(out)


@pytest.mark.parametrize("g,d,r,k", SHAPES)
@pytest.mark.parametrize("what", ["anchor_v", "sum_v", "UV", "sV", "VtV"])
def test_infinite_values(what, g, d, r, k):
    banner(f"infinite {what} g{g} d{d} r{r} k{k}")
    case = make(g, d, r, k)
    sel = oracle_result(case)["sel"]
    b, h, col, comp = 1, 1, d // 2 + 3, r - 2
    if what == "anchor_v":
        at = case.anchor_v[b, h, 17:18, col]
    elif what == "sum_v":
        free = next(s for s in range(int(case.n_spans[b])) if s not in sel[b, h])
        at = case.sum_v[b, h, free:free + 1, col]
    else:
        blk = parts(case, b, h, int(sel[b, h, k - 1]))
        blk["UV"][:, comp] &= 0x7FFF                        # so that the weighted sum above is positive
        blk["sV"][comp] = 0x3F80
        at = {"UV": blk["UV"][5:6, comp], "sV": blk["sV"][comp:comp + 1], "VtV": blk["VtV"][comp, col:col + 1]}[what]
        row = from_storage(blk["VtV"][comp].copy(), "bf16")
    at[0] &= 0x7FFF
    ref = oracle_result(case)["out"].copy()
    heads = slice(h * g, (h + 1) * g)
    if what in ("UV", "sV"):
        assert np.all(row != 0)
        ref[b, heads] = np.where(row > 0, np.inf, -np.inf)
        at[0] = INF
    else:
        ref[b, heads, col] = -np.inf
        at[0] = NINF
    got_sel, got = run(case)
    assert np.array_equal(got_sel, sel)
    odd = ~np.isfinite(ref)
    assert np.array_equal(got[odd], ref[odd]), (got[odd][:4], ref[odd][:4])
    assert_out_close(np.where(odd, 0.0, got), np.where(odd, 0.0, ref), "f32")


@pytest.mark.parametrize("what", ["UK", "VtK"])
@pytest.mark.parametrize("d,r,k", [(64, 8, 3), (128, 32, 5), (64, 64, 2)])
def test_scores_of_minus_infinity_drop_out(what, d, r, k):
    banner(f"infinite {what} d{d} r{r} k{k}")
    case = make(1, d, r, k)
    sel = oracle_result(case)["sel"]
    b, h, comp, col = 1, 1, r - 3, 7
    blk = parts(case, b, h, int(sel[b, h, k - 1]))
    q = from_storage(case.q, "bf16")[b, h]
    blk["sK"][comp] = 0x3F80
    if what == "UK":
        blk["UK"][5, comp] = 0x0000
        minus = float(q @ from_storage(blk["VtK"][comp].copy(), "bf16")) > 0        # the entry's sign
        at = blk["UK"][5:6, comp]
    else:
        blk["UK"][:, comp] |= 0x3000
        blk["UK"][:, comp] &= 0x7FFF                        # every token's factor positive
        minus = float(q[col]) > 0
        at = blk["VtK"][comp, col:col + 1]
    at[0] = oracle.narrow(np.float32(-1e30 if minus else 1e30), "bf16")
    _, ref = run(case)
    assert np.all(np.isfinite(ref))
    want = oracle_result(case)["out"]
    assert_out_close(ref, want, "f32")
    at[0] = NINF if minus else INF
    got_sel, got = run(case)
    assert np.array_equal(got_sel, sel)
    assert_out_close(got, want, "f32")
