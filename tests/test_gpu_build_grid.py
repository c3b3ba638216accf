"""GPU: a build whose anchor blocks and spans together pass the 2^32 threads of one launch, though
neither does alone: the tables are wide (max_anchors, max_spans), the sequences short."""

import numpy as np
import pytest

from tests.gpu_common import banner

pytestmark = pytest.mark.gpu


def test_gather_past_one_launch():
    import torch
    from paper_2606_31145_amd import sekv as S
    B, H, d, N, A, M = 64, 64, 64, 120, 64 * 100, 4000
    blocks = A // 64
    assert B * H * M * 256 < 2 ** 32 and B * H * blocks * 256 < 2 ** 32 <= B * H * (M + blocks) * 256
    banner(f"gather grid {B * H} pairs, {blocks} anchor blocks + {M} spans")
    gen = torch.Generator(device="cuda").manual_seed(9)
    k, v = (torch.randn((B, H, N, d), generator=gen, device="cuda").to(torch.bfloat16) for _ in range(2))
    h = torch.ones((B, N), device="cuda")
    h[:, [20, 60, 61, 90]] = 9.0
    n = torch.full((B,), N, dtype=torch.int32, device="cuda")
    omega = torch.randn((d, 16), generator=gen, device="cuda")
    small = S.make_dims(batch=1, n_q_heads=1, n_kv_heads=1, head_dim=64, rank=8, top_k=1, max_anchors=1, max_spans=1,
                        max_span_len=1, dtype="f32", softmax_scale=1.0)
    ws = S.Workspace(small)
    bd = S.make_build_dims(batch=B, n_kv_heads=H, head_dim=d, max_tokens=N, rank=8, sketch=16, min_span=10, window=0,
                           dtype="bf16")
    seg = S.segment(bd, h, n)
    ns, span_len = seg["n_spans"].cpu().numpy(), seg["span_len"].cpu().numpy()
    off, _, nbytes = S.build_layout(bd, M, ns, span_len)
    cache = S.build_cache(bd, k, v, h, n, seg, omega, A, M, torch.from_numpy(off).cuda(), nbytes, ws)
    torch.cuda.synchronize()
    assert ws.status() == 0
    na = int(seg["n_anchors"][0])
    idx = seg["anchor_idx"][0, :na].long()
    spans = [(int(s), int(e)) for s, e in zip(seg["span_start"][0, :ns[0]], seg["span_len"][0, :ns[0]])]
    assert na == 4 and spans == [(0, 20), (21, 39), (62, 28), (91, 29)] and np.all(ns == 4)
    assert torch.equal(cache["anchor_k"][:, :, :na], k[:, :, idx]) and torch.equal(cache["anchor_v"][:, :, :na], v[:, :, idx])
    for i, (s, L) in enumerate(spans):
        ref = k[:, :, s:s + L].double().mean(dim=2)
        # a float32 mean of at most 40 values below 6 (40 x 2^-24 x 6), then bfloat16 (2^-8)
        assert torch.all((cache["sum_k"][:, :, i].double() - ref).abs() <= 2.0 ** -8 * ref.abs() * 1.01 + 2e-5)
