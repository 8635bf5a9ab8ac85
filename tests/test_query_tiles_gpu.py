"""GPU parity of the key-stationary backward at the edges of its query walk, against the fp64
oracle: tiles of 32 queries (one row short, exact, one row over), the row statistics copied
for 256 queries at a time, key blocks of 256, and dQ turns that do not divide the tile
count. A wrong edge shifts or drops whole rows, far outside the bf16 bounds of
parity_util (mean-rel 5e-3, max-abs 2e-2 or one bf16 spacing)."""
import numpy as np
import pytest

import oracle.ref_attention as ora
import workloads as W
from parity_util import assert_close, bf16_values, run_gpu, to_gpu_bf16

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("det", [False, True], ids=["fused", "deterministic"])
@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("tokens", [31, 32, 33, 64, 95, 255, 256, 257, 289, 513])
def test_tile_edges(tokens, head_dim, det):
    import paper_2501_08453_amd as vc
    w = W.custom(2, 2, head_dim, 0, 1, 1, tokens)
    x = W.make_inputs(w, seed=tokens + head_dim)
    g = {n: to_gpu_bf16(x[n]) for n in ("q", "k", "v", "do")}
    out = run_gpu(vc.desc_for(w, deterministic=det), g["q"], g["k"], g["v"], g["do"])
    q, k, v, do = (bf16_values(g[n]) for n in ("q", "k", "v", "do"))
    valid = np.ones((2, tokens), dtype=bool)
    c = ora.default_scale(head_dim)
    o, lse = ora.attention_forward(q, k, v, valid, c)
    dq, dk, dv = ora.attention_backward(q, k, v, do, valid, c, lse=lse)
    for name, a, r in (("O", out["o"], o), ("LSE", out["lse"], lse), ("dQ", out["dq"], dq), ("dK", out["dk"], dk),
                       ("dV", out["dv"], dv)):
        assert_close(name, a, r)


@pytest.mark.parametrize("head_dim", [64, 128])
def test_infinite_value_in_the_last_row(head_dim):
    """The value row of key N-1 stands in for the rows past N of the last tile of 64; those
    have probability 0, which must not turn an infinite value into a NaN: O is infinite in
    that dim for every query, and finite and equal to the oracle's elsewhere."""
    import torch
    import paper_2501_08453_amd as vc
    w = W.custom(1, 2, head_dim, 0, 1, 1, 131)
    x = W.make_inputs(w, seed=3)
    g = {n: to_gpu_bf16(x[n]) for n in ("q", "k", "v")}
    g["v"][0, 130, 1, 5] = float("inf")
    o, _ = vc.fwd(g["q"], g["k"], g["v"], vc.desc_for(w))
    assert bool(torch.isinf(o[0, :, 1, 5]).all())
    o = bf16_values(o)
    v = bf16_values(g["v"])
    v[0, 130, 1, 5] = 0.0
    ref, _ = ora.attention_forward(bf16_values(g["q"]), bf16_values(g["k"]), v, np.ones((1, 131), dtype=bool),
                                   ora.default_scale(head_dim))
    keep = np.ones_like(ref, dtype=bool)
    keep[0, :, 1, 5] = False
    assert_close("O", o[keep], ref[keep])


@pytest.mark.parametrize("tokens", [131, 289])
@pytest.mark.parametrize("head_dim", [64, 128])
def test_infinite_output_gradient_in_the_last_row(head_dim, tokens):
    """Separate dK/dV pass: the dO row of query N-1 stands in for the rows past N of the last tile of 32; those have
    probability 0, which must not turn an infinite gradient into a NaN: dV is infinite in that
    dim for every key (each has a positive probability), and the oracle's in every other."""
    import torch
    import paper_2501_08453_amd as vc
    w = W.custom(1, 2, head_dim, 0, 1, 1, tokens)
    x = W.make_inputs(w, seed=3)
    g = {n: to_gpu_bf16(x[n]) for n in ("q", "k", "v", "do")}
    do = bf16_values(g["do"])
    do[0, -1, 1, 5] = 0.0
    g["do"][0, -1, 1, 5] = float("inf")
    desc = vc.desc_for(w, deterministic=True)
    o, lse = vc.fwd(g["q"], g["k"], g["v"], desc)
    _, _, dv = vc.bwd(g["q"], g["k"], g["v"], o, lse, g["do"], desc)
    assert bool(torch.isposinf(dv[0, :, 1, 5]).all())
    q, k, v = (bf16_values(g[n]) for n in ("q", "k", "v"))
    _, _, ref = ora.attention_backward(q, k, v, do, np.ones((1, tokens), dtype=bool), ora.default_scale(head_dim))
    keep = np.ones_like(ref, dtype=bool)
    keep[0, :, 1, 5] = False
    assert_close("dV", bf16_values(dv)[keep], ref[keep])


@pytest.mark.parametrize("det", [False, True], ids=["fused", "deterministic"])
@pytest.mark.parametrize("scale", [1e-30, 1e-37, 1e-39])
def test_tiny_scale(scale, det):
    """The key-stationary pass starts its scores from -LSE / c, which overflows for the smallest
    scales: every probability must still be 1/N (O and dV the oracle's, within the bounds of
    parity_util; so dQ and dK over the scale, where bf16 has its full precision)."""
    import paper_2501_08453_amd as vc
    w = W.custom(1, 2, 128, 0, 1, 1, 131)
    x = W.make_inputs(w, seed=5)
    g = {n: to_gpu_bf16(x[n]) for n in ("q", "k", "v", "do")}
    out = run_gpu(vc.desc_for(w, scale=scale, deterministic=det), g["q"], g["k"], g["v"], g["do"])
    q, k, v, do = (bf16_values(g[n]) for n in ("q", "k", "v", "do"))
    valid = np.ones((1, 131), dtype=bool)
    o, lse = ora.attention_forward(q, k, v, valid, scale)
    dq, dk, dv = ora.attention_backward(q, k, v, do, valid, scale, lse=lse)
    assert_close("O", out["o"], o)
    assert_close("dV", out["dv"], dv)
    if scale == 1e-30:
        assert_close("dQ/c", out["dq"] / scale, dq / scale)
        assert_close("dK/c", out["dk"] / scale, dk / scale)
    assert np.abs(out["dq"]).max() < 1e3 * scale and np.abs(out["dk"]).max() < 1e3 * scale


@pytest.mark.parametrize("det", [False, True], ids=["fused", "deterministic"])
@pytest.mark.parametrize("branch", ["joint", "spatial"])
@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("scale", [1e-20, 1e-30, 1e-37, 1e-39, 1e20, 1e37])
def test_extreme_scales_with_matching_scores(scale, head_dim, branch, det):
    """Extreme scales are used with scores of the inverse size: q and k such that the logits c q.k are of
    order 0.5 (scores up to about 2e38 of the 3.4e38 that fp32 holds; for 1e-39 a tenth of
    that). Results are those of ordinary sizes: dQ and dK are compared in units of c |k|
    and c |q|, within the bounds of parity_util."""
    import torch
    import oracle.ref_branches as orb
    import paper_2501_08453_amd as vc
    T, F = (16, 2) if branch == "spatial" else (0, 1)
    w = W.custom(1, 2, head_dim, T, F, 1, 99)
    x = W.make_inputs(w, seed=7)
    size = np.sqrt(min(0.5 / scale, 5e37) / np.sqrt(head_dim))  # of a q or k element
    g = {n: to_gpu_bf16(x[n] * (np.float32(size) if n in "qk" else np.float32(1))) for n in ("q", "k", "v", "do")}
    q, k, v, do = (bf16_values(g[n]) for n in ("q", "k", "v", "do"))
    desc = vc.desc_for(w, scale=scale, deterministic=det)
    if branch == "joint":
        out = run_gpu(desc, g["q"], g["k"], g["v"], g["do"])
        valid = np.ones((1, w.tokens), dtype=bool)
        o, lse = ora.attention_forward(q, k, v, valid, scale)
        dq, dk, dv = ora.attention_backward(q, k, v, do, valid, scale, lse=lse)
    else:
        to, tl = vc.spatial_fwd(g["q"], g["k"], g["v"], desc)
        grads = vc.spatial_bwd(g["q"], g["k"], g["v"], to, tl, g["do"], desc)
        torch.cuda.synchronize()
        out = dict(zip(("o", "dq", "dk", "dv"), map(bf16_values, (to, *grads))))
        o, lse = orb.spatial_forward(q, k, v, T, F, scale=scale)
        dq, dk, dv = orb.spatial_backward(q, k, v, do, T, F, scale=scale, lse=lse)
    unit = scale * size
    for n, a, r in (("O", out["o"], o), ("dV", out["dv"], dv), ("dQ", out["dq"] / unit, dq / unit),
                    ("dK", out["dk"] / unit, dk / unit)):
        assert_close(n, a, r)
