"""GPU: the bfloat16 share item at the edges of its matrix tiles (16 tokens of a span, 16 and
32 full-resolution or summary rows, 16 and 32 components), against the CPU oracle.

Rows past a sequence's own counts hold NaN, which must not reach the output.  Tolerance of
the fp32 output: a score is a sum of at most 12 roundings of 2^-24 at |score| < 16 (base 2),
so a weight is off by at most 12 * 16 * 2^-24 = 1.2e-5 relative, a value sum by as much of its
own size; assert_out_close asks for 2e-5 of the output's largest value.
"""

import numpy as np
import pytest

from synth import custom_spec, make_case
from tests.gpu_common import assert_out_close, banner, case_arrays, dims_for, oracle_result, out_to_f64

pytestmark = pytest.mark.gpu

# group, d, rank, top-k, batch, kv heads, prefix anchors, window, span lengths, rank mode
CASES = [
    (1, 64, 8, 1, 1, 1, 1, 0, (1, 3), "fixed"),
    (2, 128, 16, 3, 2, 2, 15, 1, (15, 17), "fixed"),
    (4, 128, 32, 5, 3, 2, 33, 0, (31, 33), "adaptive"),
    (8, 64, 64, 9, 5, 1, 129, 128, (63, 65), "adaptive"),
    (4, 64, 8, 64, 5, 8, 32, 31, (8, 9), "fixed"),          # several spans a slot, whole waves
    (1, 128, 64, 2, 1, 1, 64, 65, (250, 530), "adaptive"),  # one span in four parts
    (8, 128, 16, 6, 40, 4, 16, 1, (16, 16), "fixed"),       # two and more spans a slot
    (2, 64, 32, 33, 1, 16, 500, 300, (127, 129), "adaptive"),
]


@pytest.mark.parametrize("g,d,r,k,batch,heads,prefix,window,span,ranks", CASES)
def test_share_tiles(g, d, r, k, batch, heads, prefix, window, span, ranks):
    import torch
    from paper_2606_31145_amd import sekv as S
    banner(f"share tiles g{g} d{d} r{r} k{k}")
    case = make_case(custom_spec(batch=batch, n_q_heads=g * heads, n_kv_heads=heads, head_dim=d, rank=r, top_k=k,
                                 context=prefix + window + max(40 * span[1], 700), n_prefix_anchors=prefix,
                                 window=window, span_min=span[0], span_max=span[1], dtype="bf16", rank_mode=ranks,
                                 seed=100 + g + d + r))
    case.n_anchors, case.n_spans = case.n_anchors.copy(), case.n_spans.copy()
    if batch > 1:
        case.n_anchors[1] = case.n_anchors[1] * 2 // 3
        case.n_spans[1] = max(1, int(case.n_spans[1]) - 7)
        case.n_anchors[batch - 1] = 0
    for rows, n in ((("anchor_k", "anchor_v"), case.n_anchors), (("sum_k", "sum_v"), case.n_spans)):
        for name in rows:
            t = getattr(case, name).copy()
            for b in range(batch):
                t[b, :, int(n[b]):] = 0     # what the oracle's arithmetic may touch
            setattr(case, name, t)
    ref = oracle_result(case)
    for name, n in (("anchor_k", case.n_anchors), ("anchor_v", case.n_anchors), ("sum_v", case.n_spans)):
        t = getattr(case, name)
        for b in range(batch):
            t[b, :, int(n[b]):] = 0x7FC0
    dc = S.DeviceCache.from_arrays(case_arrays(case), case.dtype, torch.device("cuda:0"))
    dims = dims_for(S, case, out_dtype="f32")
    ws = S.Workspace(dims, torch.device("cuda:0"))
    for _ in range(2):
        sel, out = S.decode_step(dims, dc, ws)
        torch.cuda.synchronize()
        assert ws.status() == 0
        assert np.array_equal(sel.cpu().numpy(), ref["sel"])
        assert_out_close(out_to_f64(out), ref["out"], "f32")
