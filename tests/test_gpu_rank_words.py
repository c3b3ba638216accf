"""GPU: the ranking by key high words (32 of 64 bits) hands ties to the whole keys.

Spans whose float64 selection keys share the high word but not the low one, placed inside one
routing chunk, across chunks and across the k-th place; with up to 128 candidates, up to 512
(one thread per candidate) and more (the single merger).  Selections of the fused step and of
the selection call are compared with the oracle's order bit for bit."""

import numpy as np
import pytest

from synth import custom_spec, make_case
from synth.cases import from_storage
from tests.gpu_common import banner, case_arrays, dims_for, oracle_result

pytestmark = pytest.mark.gpu


def near_ties(dtype, k, spans, group=2, heads=2, d=64):
    """Equal lengths and, on every third span, one key row up to a component of 2^-24 steps."""
    import oracle
    case = make_case(custom_spec(batch=1, n_q_heads=group * heads, n_kv_heads=heads, head_dim=d, rank=8, top_k=k,
                                 context=8 + 8 * spans, span_min=8, span_max=8, dtype=dtype, seed=7 + k + spans))
    case.sum_k = case.sum_k.copy()
    m = int(case.n_spans[0])
    rng = np.random.default_rng(k + spans)
    for g in range(heads):
        q = from_storage(case.q, dtype).reshape(heads, group, d)[g]
        best = int(np.argmax((from_storage(case.sum_k, dtype)[0, g, :m] @ q.T).max(1)))
        row = case.sum_k[0, g, best].copy()
        ids = rng.permutation(np.union1d(np.arange(0, m, 3), [best]))
        for n, t in enumerate(ids):
            case.sum_k[0, g, t] = row
            tiny = np.float32((n % 97 + 1) * 2.0 ** -24).view(np.uint32)
            case.sum_k[0, g, t, 0] = tiny.view(np.float32) if dtype == "f32" else np.uint16(tiny >> 16)
    lg = oracle.routing_logits(from_storage(case.q, dtype), from_storage(case.sum_k, dtype), case.span_logsize,
                               case.n_spans, case.spec.softmax_scale)
    words = np.sort(oracle.group_keys(lg, heads)[0, 0, :m])[::-1][: k + 1].view(np.uint64)
    hi = words >> np.uint64(32)
    assert np.any((hi[1:] == hi[:-1]) & (words[1:] != words[:-1]))
    return case


@pytest.mark.parametrize("dtype,k,spans", [("bf16", 3, 40), ("f32", 16, 128), ("bf16", 16, 900), ("f32", 8, 1000),
                                           ("bf16", 64, 129), ("bf16", 40, 1300), ("f32", 64, 1300), ("bf16", 1, 257)])
def test_equal_high_words(dtype, k, spans):
    import torch
    from paper_2606_31145_amd import sekv as S
    banner(f"equal high words {dtype} k{k} spans {spans}")
    case = near_ties(dtype, k, spans)
    ref = oracle_result(case)["sel"]
    dev = torch.device("cuda:0")
    dc = S.DeviceCache.from_arrays(case_arrays(case), case.dtype, dev)
    dims = dims_for(S, case)
    ws = S.Workspace(dims, dev)
    sel, _ = S.decode_step(dims, dc, ws)
    assert np.array_equal(sel.cpu().numpy(), ref)
    sel, _ = S.route_topk(dims, dc, ws)
    assert np.array_equal(sel.cpu().numpy(), ref)
    assert ws.status() == 0
