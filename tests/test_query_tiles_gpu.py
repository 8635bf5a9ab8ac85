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


@pytest.mark.parametrize("det", [False, True], ids=["fused", "deterministic"])
@pytest.mark.parametrize("scale", [1e-30, 1e-37, 1e-39])
def test_tiny_scale(scale, det):
    """The key-stationary pass starts its scores from -LSE / c, which overflows for the smallest
    scales: every probability must still be 1/N (O and dV the oracle's, within the bounds of
    parity_util; dQ and dK are of the order of the scale)."""
    import paper_2501_08453_amd as vc
    w = W.custom(1, 2, 128, 0, 1, 1, 131)
    x = W.make_inputs(w, seed=5)
    g = {n: to_gpu_bf16(x[n]) for n in ("q", "k", "v", "do")}
    out = run_gpu(vc.desc_for(w, scale=scale, deterministic=det), g["q"], g["k"], g["v"], g["do"])
    q, k, v, do = (bf16_values(g[n]) for n in ("q", "k", "v", "do"))
    valid = np.ones((1, 131), dtype=bool)
    o, lse = ora.attention_forward(q, k, v, valid, scale)
    _, _, dv = ora.attention_backward(q, k, v, do, valid, scale, lse=lse)
    assert_close("O", out["o"], o)
    assert_close("dV", out["dv"], dv)
    assert np.abs(out["dq"]).max() < 1e3 * scale and np.abs(out["dk"]).max() < 1e3 * scale
