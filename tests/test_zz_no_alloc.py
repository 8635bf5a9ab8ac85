"""GPU test of the no-allocation forward (vc_jointattn_fwd_noalloc), through the C ABI.

Its output is compared with the workspace-taking forward's (vc_jointattn_fwd, the same
kernels, with its queried workspace) bit for bit, and with the fp64 oracle to the parity bar, on two calls in a row,
the second with a smaller input: the ragged-text workload first (4 x 9,856 tokens, 216 MB
of the 256 MiB scratch array), then a small ragged, key-masked problem at head_dim 64.
A problem larger than the array is refused before anything runs.
"""
import numpy as np
import pytest

import oracle.ref_attention as ora
import workloads as W
from parity_util import assert_close, bf16_values, log, lse_bound, to_gpu_bf16

pytestmark = pytest.mark.gpu


def _call_both(w, x, key_mask=None):
    import torch
    import paper_2501_08453_amd as vc
    q, k, v = (to_gpu_bf16(x[n]) for n in ("q", "k", "v"))
    tl = None if x["text_len"] is None else torch.from_numpy(x["text_len"]).to("cuda")
    km = None if key_mask is None else torch.from_numpy(key_mask).to("cuda")
    desc = vc.desc_for(w)
    B, N, H, D = w.shape
    assert vc.vc_jointattn_fwd_workspace_bytes(desc) <= vc.NOALLOC_SCRATCH_BYTES
    o_n = torch.full_like(q, float("nan"))
    l_n = torch.full((B, H, N), float("nan"), dtype=torch.float32, device="cuda")
    vc.vc_jointattn_fwd_noalloc(desc, q, k, v, tl, km, o_n, l_n)
    o_w, l_w = vc.fwd(q, k, v, desc, tl, km)
    torch.cuda.synchronize()
    assert torch.equal(o_n, o_w), "no-allocation forward differs from vc_jointattn_fwd (O)"
    assert torch.equal(l_n, l_w), "no-allocation forward differs from vc_jointattn_fwd (LSE)"
    return q, k, v, o_n, l_n


def test_noalloc_forward_two_calls_then_refusal():
    import torch
    import paper_2501_08453_amd as vc
    # call 1: the ragged-text workload; oracle on sampled rows of two (sample, head) pairs
    w1 = W.WORKLOADS[4]
    x1 = W.make_inputs(w1, with_do=False)
    log("no-alloc forward, call 1:", w1.shape, "text_len", x1["text_len"].tolist())
    q, k, v, o, lse = _call_both(w1, x1)
    B, N, H, D = w1.shape
    valid = ora.key_validity(B, N, w1.text_slot, x1["text_len"])
    rng = np.random.Generator(np.random.PCG64(5))
    rows = np.unique(np.r_[0, w1.text_slot - 1, w1.text_slot, N - 1, rng.integers(0, N, 40)])
    rows_t = torch.from_numpy(rows).to("cuda")
    for b, h in ((0, 0), (3, 15)):
        qh, kh, vh = (bf16_values(t[b:b + 1, :, h:h + 1]) for t in (q, k, v))
        o_r, l_r = ora.forward_rows(qh, kh, vh, valid[b], ora.default_scale(D), 0, 0, rows)
        assert_close("O", bf16_values(o[b, :, h].index_select(0, rows_t)), o_r)
        assert_close("LSE", lse[b, h].index_select(0, rows_t).double().cpu().numpy(), l_r)
    del q, k, v, o, lse
    # call 2: smaller, head_dim 64, ragged text and a key mask; oracle on every element
    w2 = W.custom(2, 2, 64, 16, 2, 8, 9, ragged_text=True)
    x2 = W.make_inputs(w2, seed=31, with_do=False)
    km = W.random_key_mask(w2, seed=32, keep=0.85)
    log("no-alloc forward, call 2:", w2.shape)
    q, k, v, o, lse = _call_both(w2, x2, km)
    B, N, H, D = w2.shape
    valid = ora.key_validity(B, N, w2.text_slot, x2["text_len"], km)
    o_r, l_r = ora.attention_forward(bf16_values(q), bf16_values(k), bf16_values(v), valid)
    assert_close("O", bf16_values(o), o_r)
    assert_close("LSE", lse.double().cpu().numpy(), l_r)
    # a problem beyond the array: refused with VC_ERR_SCRATCH, nothing launched
    big = vc.make_desc(1, 24, 128, 256, 16, 45, 80)
    with pytest.raises(vc.JointAttnError) as e:
        vc.vc_jointattn_fwd_noalloc(big, q, k, v, None, None, o, lse)
    assert e.value.status == -10


@pytest.mark.parametrize("shape", [(1, 2, 64, 77, 3, 30, 61), (1, 13, 128, 16, 6, 30, 31), (1, 3, 128, 0, 1, 200, 200)],
                         ids=lambda s: "x".join(map(str, s)))
def test_noalloc_forward_where_the_last_round_is_split(shape):
    """Split last rounds (44 items; 30 of 286; 215 of 471): bitwise the workspace-taking forward's
    results with a workspace of the queried size or more; with the least accepted one, whose
    fewer split workgroups round other sums, within two roundings of the LSE and 2^-7 of O's
    2-norm (each side's probabilities are bf16, relative 2^-9 on average)."""
    import torch
    import paper_2501_08453_amd as vc
    w = W.custom(*shape)
    B, N, H, D = w.shape
    gen = torch.Generator(device="cuda").manual_seed(N)
    q, k, v = (torch.randn((B, N, H, D), generator=gen, device="cuda").to(torch.bfloat16) for _ in range(3))
    desc = vc.desc_for(w)
    o_n, l_n = torch.empty_like(q), torch.empty((B, H, N), device="cuda")
    vc.vc_jointattn_fwd_noalloc(desc, q, k, v, None, None, o_n, l_n)
    need = vc.vc_jointattn_fwd_workspace_bytes(desc)
    for size in (need, 2 * need + 12345):
        o, lse = vc.fwd(q, k, v, desc, ws=torch.empty(size, dtype=torch.uint8, device="cuda"))
        assert torch.equal(o, o_n) and torch.equal(lse, l_n)
    up = lambda x: (x + 255) & ~255  # noqa: E731
    least = up(B * H * ((N + 63) // 64) * D * 72 * 2) + up(min(256, (N + 255) // 256 * H * B) * 256 * (D + 2) * 4)
    o, lse = vc.fwd(q, k, v, desc, ws=torch.empty(least, dtype=torch.uint8, device="cuda"))
    assert float((lse - l_n).abs().max()) <= 2 * lse_bound(N)
    assert float((o.float() - o_n.float()).norm() / o_n.float().norm()) <= 2.0 ** -7
