"""GPU: the wait for the single merger's selection (more than 512 candidates of a pair).

Every workgroup of a pair polls one ready word and all its waves must leave the wait in the
same round, or its later barriers pair up wrongly.  Many pairs with many slots each poll here
while a pair's last routing chunk sorts its candidates, launch after launch; every launch gives
the oracle's selection and the first launch's bits."""

import numpy as np
import pytest

from synth import custom_spec, make_case
from tests.gpu_common import assert_out_close, banner, case_arrays, dims_for, oracle_result, out_to_f64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,d,group,heads,batch", [("bf16", 64, 2, 4, 3), ("f32", 64, 1, 2, 2)])
def test_waits_for_the_merger_end_together(dtype, d, group, heads, batch):
    import torch
    from paper_2606_31145_amd import sekv as S
    banner(f"merger wait {dtype} pairs {heads * batch}")
    case = make_case(custom_spec(batch=batch, n_q_heads=group * heads, n_kv_heads=heads, head_dim=d, rank=8, top_k=64,
                                 context=8 * 1200, span_min=8, span_max=8, dtype=dtype, seed=31))
    assert -(-int(case.max_spans) // 128) * 64 > 512
    dev = torch.device("cuda:0")
    dc = S.DeviceCache.from_arrays(case_arrays(case), case.dtype, dev)
    dims = dims_for(S, case)
    ws = S.Workspace(dims, dev)
    ref = oracle_result(case)
    first = None
    for _ in range(24):
        sel, out = S.decode_step(dims, dc, ws)
        torch.cuda.synchronize()
        assert ws.status() == 0
        assert np.array_equal(sel.cpu().numpy(), ref["sel"])
        if first is None:
            first = out
            assert_out_close(out_to_f64(out), ref["out"], case.dtype)
        assert torch.equal(out, first)
