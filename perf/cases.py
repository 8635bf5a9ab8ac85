"""Performance cases of the attention library: what a user's program has it do.

The calls are those of the parallel diffusion block: joint text-video attention, the
spatial branch (each frame with the text), the temporal branch (each position across the
frames) and the differentiable sum of the three, forward alone (sampling) and forward with
backward (training), at both head dims, with padded captions, key masks and the
reproducible backward where they are used. Sizes are the repository's workloads plus a
single image and a clip of odd sizes; `draw` spreads further cases over the same ranges.
"""
from __future__ import annotations

import math

import torch

import paper_2501_08453_amd as vc

DEV = "cuda"


def _case(name, op, mode, B, H, D, T, F, gh, gw, ragged=False, mask=False, det=False, api="call", q_scale=1.0):
    return {"name": name, "op": op, "mode": mode, "B": B, "H": H, "D": D, "T": T, "F": F, "gh": gh, "gw": gw,
            "ragged": ragged, "mask": mask, "det": det, "api": api, "q_scale": q_scale}


def listed():
    return [
        # The smallest call: a toy clip, one training step; launches and host work decide.
        _case("joint-tiny-train", "joint", "train", 1, 2, 64, 16, 2, 8, 8),
        # One image (a one-frame clip) through the differentiable call, as image training
        # steps between video steps make it: fewer workgroups than compute units.
        _case("joint-image-train", "joint", "train", 1, 24, 128, 256, 1, 32, 32, api="autograd"),
        # The medium clip at head_dim 64, training.
        _case("joint-medium-train", "joint", "train", 2, 16, 64, 128, 8, 32, 32, q_scale=0.125),
        # A batch of clips whose captions have different lengths, training.
        _case("joint-ragged-train", "joint", "train", 4, 16, 128, 256, 8, 30, 40, ragged=True),
        # The headline: a 720p clip of 57,856 tokens, training.
        _case("joint-long-train", "joint", "train", 1, 24, 128, 256, 16, 45, 80),
        # The longest joint clip (123,136 tokens), forward only: a sampling step.
        _case("joint-max-infer", "joint", "infer", 1, 24, 128, 256, 32, 48, 80),
        # One GPU's 3 heads of the 720p clip under 8-way head sharding, sampled through the
        # call that takes no workspace (serving loops).
        _case("joint-shard-infer", "joint", "infer", 1, 3, 128, 256, 16, 45, 80, api="noalloc"),
        # Odd sizes throughout, ragged captions, a key mask and the reproducible backward:
        # debugging and regression runs of a fine-tune on cropped clips.
        _case("joint-odd-masked-det", "joint", "train", 2, 6, 128, 77, 7, 23, 37, ragged=True, mask=True, det=True),
        # The spatial branch of the 720p clip, training.
        _case("spatial-long-train", "spatial", "train", 1, 24, 128, 256, 16, 45, 80),
        # The temporal branch of the 720p clip (16 frames), training.
        _case("temporal-long-train", "temporal", "train", 1, 24, 128, 256, 16, 45, 80),
        # The temporal branch of the longest clip (144 frames), training.
        _case("temporal-clip144-train", "temporal", "train", 1, 24, 128, 256, 144, 45, 80),
        # The whole parallel block (three branches, summed) through the differentiable call.
        _case("block-medium-train", "block", "train", 2, 16, 64, 128, 8, 32, 32, api="autograd"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges: 64 to about 60,000 tokens, 1 to 24 heads, both head
    dims, with the options in the shares real use has them."""
    while True:
        op = rng.choice(["joint"] * 4 + ["spatial"] * 2 + ["temporal"] * 3 + ["block"])
        mode = "infer" if op != "block" and rng.random() < 0.3 else "train"
        D = rng.choice([64, 128, 128])
        H = rng.choice([2, 3, 6, 8, 12, 16, 24, rng.randint(1, 24)])
        B = rng.choice([1, 1, 2, rng.randint(1, 4)])
        T = rng.choice([0, 16, 77, 128, 256, rng.randint(1, 256)])
        F = _log(rng, 2, 144) if op == "temporal" else _log(rng, 1, 32)
        gh, gw = _log(rng, 6, 48), _log(rng, 6, 80)
        ragged = T > 0 and op != "temporal" and rng.random() < 0.4
        mask = rng.random() < 0.15
        det = mode == "train" and op == "joint" and rng.random() < 0.2
        api = "autograd" if op == "block" or (mode == "train" and rng.random() < 0.4) else "call"
        c = _case("", op, mode, B, H, D, T, F, gh, gw, ragged, mask, det, api)
        del c["name"]
        w = work(c)
        if w["flops"] <= 6e13 and w["bytes"] <= 3e10:
            return c


def _tokens(c):
    return c["T"] + c["F"] * c["gh"] * c["gw"]


def work(c):
    """Algorithmic bytes (inputs read and outputs written once per call) and flops (matrix
    products over every query and key, recomputation not counted) of one pass."""
    B, H, D, T, F, L = c["B"], c["H"], c["D"], c["T"], c["F"], c["gh"] * c["gw"]
    N = _tokens(c)
    rows = B * H * N
    pairs = {"joint": N * N, "spatial": F * L * (L + T), "temporal": L * F * F}
    ops = ["joint", "spatial", "temporal"] if c["op"] == "block" else [c["op"]]
    train = c["mode"] == "train"
    flops = sum((12 if train else 4) * B * H * D * pairs[o] for o in ops)
    per = rows * (8 * D + 4) + (rows * (16 * D + 4) if train else 0)
    nbytes = len(ops) * per
    if c["op"] == "block":  # the sum, and the three branches' gradients added
        nbytes += rows * D * 2
    return {"bytes": float(nbytes), "flops": float(flops)}


def tolerance(c):
    # bf16 outputs and bf16 operands of the products (probabilities and their gradients):
    # 2-norm errors of about 2 to 3e-3 against 64 bits on every output; a single value is off
    # by up to a few of its bf16 spacings.
    return {"rel": 1e-2, "max": 0.15}


def _inputs(c, seed):
    """bf16 q, k, v, dO ([B, N, H, D], standard normal; q scaled where logits are flat), and
    int32 caption lengths and the uint8 key mask where the case has them."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    B, N, H, D = c["B"], _tokens(c), c["H"], c["D"]
    x = {}
    for n in ("q", "k", "v", "do") if c["mode"] == "train" else ("q", "k", "v"):
        t = torch.empty((B, N, H, D), dtype=torch.bfloat16, device=DEV)
        for b in range(B):  # frame-sized float32 pieces, so that drawing needs little memory
            for n0 in range(0, N, 65536):
                p = torch.randn((min(65536, N - n0), H, D), generator=gen, device=DEV)
                t[b, n0:n0 + 65536] = p * c["q_scale"] if n == "q" else p
        x[n] = t
    x["tl"] = x["km"] = None
    if c["ragged"]:
        x["tl"] = torch.randint(min(8, c["T"]), c["T"] + 1, (B,), generator=gen, device=DEV, dtype=torch.int32)
    if c["mask"]:
        x["km"] = (torch.rand((B, N), generator=gen, device=DEV) < 0.9).to(torch.uint8)
    return x


def prepare(c, seed):
    x = _inputs(c, seed)
    desc = vc.make_desc(c["B"], c["H"], c["D"], c["T"], c["F"], c["gh"], c["gw"], deterministic=c["det"])
    s = {"case": c, "desc": desc, **x}
    if c["api"] == "autograd":
        for n in ("q", "k", "v"):
            s[n].requires_grad_(True)
    elif c["api"] == "noalloc":
        s["o"] = torch.empty_like(s["q"])
        s["lse"] = torch.empty((c["B"], c["H"], _tokens(c)), dtype=torch.float32, device=DEV)
    elif c["op"] in ("joint", "spatial"):
        s["fws"] = vc.fwd_workspace(desc, DEV)
        if c["mode"] == "train":
            s["bws"] = vc.workspace(desc, DEV) if c["op"] == "joint" else vc.spatial_workspace(desc, DEV)
    return s


def run(s):
    c, d, q, k, v, tl, km = s["case"], s["desc"], s["q"], s["k"], s["v"], s["tl"], s["km"]
    op, train = c["op"], c["mode"] == "train"
    if c["api"] == "autograd":
        if op == "temporal":
            o = vc.temporal_attention(q, k, v, d, km)
        else:
            f = {"joint": vc.joint_attention, "spatial": vc.spatial_attention, "block": vc.parallel_block_attention}[op]
            o = f(q, k, v, d, tl, km)
        return (o.detach(),) + torch.autograd.grad(o, (q, k, v), s["do"])
    if c["api"] == "noalloc":
        vc.vc_jointattn_fwd_noalloc(d, q, k, v, tl, km, s["o"], s["lse"])
        return s["o"], s["lse"]
    if op == "joint":
        o, lse = vc.fwd(q, k, v, d, tl, km, ws=s["fws"])
        return (o, lse) + (vc.bwd(q, k, v, o, lse, s["do"], d, tl, km, ws=s["bws"]) if train else ())
    if op == "spatial":
        o, lse = vc.spatial_fwd(q, k, v, d, tl, km, ws=s["fws"])
        return (o, lse) + (vc.spatial_bwd(q, k, v, o, lse, s["do"], d, tl, km, ws=s["bws"]) if train else ())
    o, lse = vc.temporal_fwd(q, k, v, d, km)
    return (o, lse) + (vc.temporal_bwd(q, k, v, o, lse, s["do"], d, km) if train else ())


# --- the same results in 64 bits -------------------------------------------------------------

def _softmax64(s):
    """(probabilities, log-sum-exp) of masked scores; rows without a valid key: 0, -inf."""
    m = s.amax(-1, keepdim=True)
    e = torch.exp(s - torch.where(torch.isinf(m), torch.zeros_like(m), m))
    l = e.sum(-1, keepdim=True)
    lse = torch.where(l > 0, torch.log(l) + torch.where(torch.isinf(m), torch.zeros_like(m), m),
                      torch.full_like(l, -math.inf))
    return e / torch.where(l > 0, l, torch.ones_like(l)), lse[..., 0]


def _attend64(q, k, v, do, ok, scale):
    """Attention of queries [n, D] over keys [m, D] with validity ok [m], over blocks of
    query rows: o, lse, dq, dk, dv (the last three None without do)."""
    o, lse = torch.empty_like(q), torch.empty(q.shape[0], dtype=torch.float64, device=q.device)
    dq = dk = dv = None
    if do is not None:
        dq, dk, dv = torch.empty_like(q), torch.zeros_like(k), torch.zeros_like(v)
    kt, vt = k.t().contiguous(), v.t().contiguous()
    step = max(1, (1 << 28) // max(1, k.shape[0]))
    for r in range(0, q.shape[0], step):
        i = slice(r, r + step)
        s = (q[i] @ kt).mul_(scale).masked_fill_(~ok, -math.inf)
        p, lse[i] = _softmax64(s)
        o[i] = p @ v
        if do is not None:
            dv += p.t() @ do[i]
            ds = (do[i] @ vt).sub_((do[i] * o[i]).sum(-1, keepdim=True)).mul_(p)
            dq[i] = (ds @ k).mul_(scale)
            dk += (ds.t() @ q[i]).mul_(scale)
    return o, lse, dq, dk, dv


def _temporal64(q, k, v, do, ok, scale):
    """Attention of every position across the frames: [F, L, D] tensors, ok [F, L]."""
    q, k, v = (t.permute(1, 0, 2).contiguous() for t in (q, k, v))
    s = torch.bmm(q, k.transpose(1, 2).contiguous()).mul_(scale).masked_fill_(~ok.t()[:, None, :], -math.inf)
    p, lse = _softmax64(s)
    o = torch.bmm(p, v)
    dq = dk = dv = None
    back = lambda t: t.permute(1, 0, 2)  # noqa: E731
    if do is not None:
        do = do.permute(1, 0, 2).contiguous()
        dv = back(torch.bmm(p.transpose(1, 2).contiguous(), do))
        ds = p * (torch.bmm(do, v.transpose(1, 2).contiguous()) - (do * o).sum(-1, keepdim=True))
        dq = back(torch.bmm(ds, k).mul_(scale))
        dk = back(torch.bmm(ds.transpose(1, 2).contiguous(), q).mul_(scale))
    return back(o), lse.t(), dq, dk, dv


def _branch64(op, x, c):
    B, N, H, D, T, F, L = c["B"], _tokens(c), c["H"], c["D"], c["T"], c["F"], c["gh"] * c["gw"]
    train = c["mode"] == "train"
    scale = 1.0 / math.sqrt(D)
    new = lambda: torch.zeros((B, N, H, D), dtype=torch.float64, device=DEV)  # noqa: E731
    o, lse = new(), torch.full((B, H, N), -math.inf, dtype=torch.float64, device=DEV)
    dq, dk, dv = (new(), new(), new()) if train else (None, None, None)
    pos = torch.arange(N, device=DEV)
    for b in range(B):
        ok = torch.ones(N, dtype=torch.bool, device=DEV)
        if x["tl"] is not None and op != "temporal":
            ok &= (pos >= T) | (pos < x["tl"][b])
        if x["km"] is not None:
            ok &= x["km"][b] != 0
        for h in range(H):
            q, k, v, do = (x[n][b, :, h].double() if n in x else None for n in ("q", "k", "v", "do"))
            if op == "joint":
                groups = [(slice(0, N), pos)]
            elif op == "spatial":
                groups = [(slice(T + f * L, T + (f + 1) * L), torch.cat([pos[:T], pos[T + f * L:T + (f + 1) * L]]))
                          for f in range(F)]
            else:
                t = [None if a is None else a[T:].reshape(F, L, D) for a in (q, k, v, do)]
                r = _temporal64(*t, ok[T:].reshape(F, L), scale)
                o[b, T:, h] = r[0].reshape(F * L, D)
                lse[b, h, T:] = r[1].reshape(F * L)
                if train:
                    for dst, g in zip((dq, dk, dv), r[2:]):
                        dst[b, T:, h] = g.reshape(F * L, D)
                continue
            for rows, keys in groups:
                r = _attend64(q[rows], k[keys], v[keys], do[rows] if train else None, ok[keys], scale)
                o[b, rows, h], lse[b, h, rows] = r[0], r[1]
                if train:
                    dq[b, rows, h] = r[2]
                    dk[b, :, h].index_add_(0, keys, r[3])
                    dv[b, :, h].index_add_(0, keys, r[4])
    return [o, lse] + ([dq, dk, dv] if train else [])


def exact(c, seed):
    """What run() returns for these inputs, in 64 bits by plain torch."""
    x = _inputs(c, seed)
    with torch.no_grad():
        if c["op"] == "block":
            total = None
            for op in ("joint", "spatial", "temporal"):
                r = _branch64(op, x, c)
                r = [r[0]] + r[2:]
                total = r if total is None else [a + b for a, b in zip(total, r)]
            return tuple(total)
        r = _branch64(c["op"], x, c)
    return tuple([r[0]] + r[2:] if c["api"] == "autograd" else r)
