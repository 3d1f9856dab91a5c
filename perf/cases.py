"""Timed workloads of the framework's public calls: the segmented gated linear
recurrence (scalar and per-key-channel gate), the gated delta rule and the
short convolution, from one short call to the 256K-context layer.

A case is a dict of plain values:
  op      "scalar", "vector" (gate per key channel), "gdn" (gated delta rule) or "conv"
  api     "chain" (consecutive segments, the state carried) or "segment" (one call)
  train   True: forward and backward of one layer; False: the forward alone
  segs    segment lengths in tokens, comma separated
  keep    the forward keeps its superchunk states for the backward
  state   a state (tail) enters the first segment and a gradient the last one
"""
import math

import torch

import paper_2608_06838_amd as sf
from paper_2608_06838_amd import synth

CHUNK = 64  # tokens per block of the closed form below, and of the flop counts
SEGS_256K = "65536,40960,32768,28672,26624,24576,22528,20480"
_IO = {"f32": torch.float32, "bf16": torch.bfloat16}


def _lens(case):
    return [int(x) for x in case["segs"].split(",")]


def listed():
    return [
        # The 256K-context layer of a hidden-5120 model (40 heads of 128) in 8
        # nonuniform segments, states recomputed by the backward: the layer a
        # long-context training run spends its time in.
        dict(name="scalar_ctx256k", op="scalar", api="chain", train=True, B=1, H=40, D=128, segs=SEGS_256K,
             io="bf16", g_mu=3.0, keep=False, state=False),
        # A mid-size layer, 32K tokens in uniform segments with an entering
        # state, the forward's states kept for the backward.
        dict(name="scalar_mid_keep", op="scalar", api="chain", train=True, B=1, H=16, D=128,
             segs=",".join(["4096"] * 8), io="bf16", g_mu=3.0, keep=True, state=True),
        # A batch of sequences in many short segments with stronger decay: the
        # time goes to segment boundaries and to launches.
        dict(name="scalar_short_segs", op="scalar", api="chain", train=True, B=4, H=32, D=128,
             segs=",".join(["512"] * 32), io="bf16", g_mu=1.0, keep=False, state=False),
        # Prefill of one segment of odd length on one tensor-parallel rank (10
        # of 40 heads): forward only.
        dict(name="scalar_prefill_tp", op="scalar", api="segment", train=False, B=1, H=10, D=128, segs="8256",
             io="bf16", g_mu=3.0, keep=False, state=True),
        # A small fp32 layer (numerics work, small models): one 1024-token
        # segment, forward and backward; latency counts.
        dict(name="scalar_f32_small", op="scalar", api="segment", train=True, B=1, H=2, D=64, segs="1024",
             io="f32", g_mu=3.0, keep=False, state=False),
        # The per-key-channel (GLA) gate, two sequences of 64K tokens.
        dict(name="vector_train", op="vector", api="chain", train=True, B=2, H=16, D=128,
             segs=",".join(["4096"] * 16), io="bf16", g_mu=3.0, keep=False, state=False),
        # The per-key-channel gate on few heads of 64 channels, ragged segments.
        dict(name="vector_ragged", op="vector", api="chain", train=True, B=1, H=6, D=64, segs="1984,1088,4160",
             io="bf16", g_mu=3.0, keep=False, state=True),
        # The gated delta rule on the 256K-context layer.
        dict(name="gdn_ctx256k", op="gdn", api="chain", train=True, B=1, H=40, D=128, segs=SEGS_256K,
             io="bf16", g_mu=3.0, keep=False, state=True),
        # The same operator on one tensor-parallel rank (8 heads), 16K tokens
        # in two segments of odd length.
        dict(name="gdn_tp", op="gdn", api="chain", train=True, B=1, H=8, D=128, segs="10112,6272",
             io="bf16", g_mu=3.0, keep=False, state=True),
        # Prefill of a short prompt chunk through the gated delta rule.
        dict(name="gdn_prefill", op="gdn", api="segment", train=False, B=1, H=10, D=128, segs="1088",
             io="bf16", g_mu=3.0, keep=False, state=True),
        # The short convolution in front of the 256K-context layer (q, k and v
        # of 40 heads), its first two segments.
        dict(name="conv_train", op="conv", api="chain", train=True, B=1, C=15360, W=4, segs="65536,40960",
             io="bf16", act="silu", state=True),
        # The convolution of a small fp32 model on a ragged batch.
        dict(name="conv_small", op="conv", api="segment", train=True, B=2, C=1536, W=4, segs="1037",
             io="f32", act="silu", state=True),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _split(rng, L, step):
    """L tokens in 1 to 8 segments at random multiples of step."""
    n = min(rng.choice((1, 1, 2, 3, 4, 8)), L // step)
    cuts = sorted(rng.sample(range(1, L // step), n - 1)) if n > 1 else []
    ends = [c * step for c in cuts] + [L]
    return ",".join(str(b - a) for a, b in zip([0] + ends[:-1], ends))


def draw(rng):
    op = rng.choice(("scalar", "scalar", "vector", "gdn", "gdn", "conv"))
    train = rng.random() < 0.75
    B = rng.choice((1, 1, 1, 2, 3, 4))
    state = rng.random() < 0.5
    if op == "conv":
        C = 8 * int(_log(rng, 32, 1920))
        L = int(_log(rng, 16, min(65536, (1 << 30) // (B * C))))
        segs = _split(rng, L, 1)
        return dict(op=op, api="chain" if "," in segs else "segment", train=train, B=B, C=C,
                    W=rng.choice((2, 3, 4, 4, 4)), segs=segs, io=rng.choice(("bf16", "bf16", "f32")),
                    act=rng.choice(("silu", "silu", "none")), state=state)
    D = rng.choice((64, 128, 128, 128))
    io = "bf16" if op == "gdn" or rng.random() < 0.75 else "f32"
    if op == "vector" and io == "f32":
        D = 64
    H = int(_log(rng, 2, 41))
    L = 64 * int(_log(rng, 1, min(1024, (1 << 15) // (B * H)) + 1))
    segs = _split(rng, L, 64)
    api = "chain" if "," in segs else rng.choice(("chain", "segment"))
    keep = train and api == "chain" and rng.random() < 0.4
    return dict(op=op, api=api, train=train, B=B, H=H, D=D, segs=segs, io=io, g_mu=rng.choice((1.0, 3.0, 3.0)),
                keep=keep, state=state)


def prepare(case, seed):
    dev = torch.device("cuda:0")
    segs = _lens(case)
    L = sum(segs)
    st = dict(case=case, segs=segs)
    if case["op"] == "conv":
        st.update(synth.make_conv_inputs(case["B"], L, case["C"], case["W"], io=case["io"], device=dev, seed=seed,
                                         tails=case["state"]))
        return st
    B, H, D = case["B"], case["H"], case["D"]
    s_std = 0.1 if case["state"] else 0.0
    if case["op"] == "gdn":
        st.update(synth.make_gdn_inputs(B, L, H, D, device=dev, seed=seed, s_in_std=s_std, g_mu=case["g_mu"]))
        gen = torch.Generator(device=dev).manual_seed(seed + 1)
        st["dO"] = torch.randn((B, L, H, D), device=dev, generator=gen).to(torch.bfloat16)
        st["dS_out"] = torch.randn((B, H, D, D), device=dev, generator=gen) * 0.1 if case["state"] else None
        return st
    w = dict(B=B, H=H, D=D, seg_lens=segs, io=case["io"], gate=case["op"], g_mu=case["g_mu"], s_in_std=s_std)
    st.update(synth.make_inputs(w, device=dev, seed=seed, dS_out_std=s_std))
    return st


def _run_conv(st):
    case, segs = st["case"], st["segs"]
    x, w, dy, act = st["x"], st["w"], st["dy"], case["act"]
    if case["api"] == "segment":
        y, tail = sf.conv_fwd(x, w, st["tail_in"], act)
        if not case["train"]:
            return dict(y=y, tail=tail)
        dx, dw, dtail = sf.conv_bwd(x, w, st["tail_in"], dy, st["dtail_out"], act)
        return dict(y=y, tail=tail, dx=dx, dw=dw, dtail=dtail)
    starts = [sum(segs[:i]) for i in range(len(segs))]
    y, tails = torch.empty_like(x), [st["tail_in"]]
    for t, n in zip(starts, segs):
        tail = torch.empty((x.shape[0], w.shape[1] - 1, x.shape[2]), dtype=torch.float32, device=x.device)
        sf.conv_fwd(x[:, t:t + n], w, tails[-1], act, out=(y[:, t:t + n], tail))
        tails.append(tail)
    if not case["train"]:
        return dict(y=y, tail=tails[-1])
    dx, dw, dtail = torch.empty_like(x), None, st["dtail_out"]
    for i in reversed(range(len(segs))):
        xs, dxs = x[:, starts[i]:starts[i] + segs[i]], dx[:, starts[i]:starts[i] + segs[i]]
        ws = torch.empty(sf.conv_bwd_workspace_bytes(xs, w, act), dtype=torch.uint8, device=x.device)
        dwi, dti = torch.empty_like(w), torch.empty_like(tails[i + 1])
        sf.conv_bwd(xs, w, tails[i], dy[:, starts[i]:starts[i] + segs[i]], dtail, act, out=(dxs, dwi, dti, ws))
        dw, dtail = dwi if dw is None else dw.add_(dwi), dti
    return dict(y=y, tail=tails[-1], dx=dx, dw=dw, dtail=dtail)


def run(st):
    case = st["case"]
    if case["op"] == "conv":
        return _run_conv(st)
    q, k, v, g, S_in = st["q"], st["k"], st["v"], st["g"], st["S_in"]
    gdn, keep = case["op"] == "gdn", case["keep"]
    extra = (st["beta"],) if gdn else ()
    if case["api"] == "segment":
        fwd, bwd = (sf.gdn_fwd, sf.gdn_bwd) if gdn else (sf.segment_fwd, sf.segment_bwd)
        o, S = fwd(q, k, v, g, *extra, S_in)
        out = dict(o=o, S=S)
        if case["train"]:
            out["grads"] = bwd(q, k, v, g, *extra, S_in, st["dO"], st["dS_out"])
        return out
    fwd, bwd = (sf.gdn_chain_fwd, sf.gdn_chain_bwd) if gdn else (sf.chain_fwd, sf.chain_bwd)
    o, S, *ck = fwd(q, k, v, g, *extra, st["segs"], S_in, keep_states=keep)
    out = dict(o=o, S=S)
    if case["train"]:
        out["grads"] = bwd(q, k, v, g, *extra, st["segs"], S, st["dO"], st["dS_out"], ckpt=ck[0] if keep else None)
    return out


def work(case):
    segs, B = _lens(case), case["B"]
    L, io = sum(segs), 2 if case["io"] == "bf16" else 4
    if case["op"] == "conv":
        n, W = B * L * case["C"], case["W"]
        tails = 4 * B * (W - 1) * case["C"]
        nbytes = n * io * (5 if case["train"] else 2) + tails * 2 + 4 * case["C"] * W
        return dict(bytes=nbytes, flops=n * (2 * W + 4 + (6 * W + 8 if case["train"] else 0)))
    H, D, C = case["H"], case["D"], CHUNK
    th, states = B * H * L, 4 * B * H * D * D
    gate = {"scalar": 4, "vector": 4 * D, "gdn": 8}[case["op"]]
    nbytes = th * (4 * D * io + gate) + states * (len(segs) + (1 if case["state"] else 0))
    if case["train"]:
        nbytes += th * (7 * D * io + 2 * gate) + states * (len(segs) + (1 if case["state"] else 0) + 1)
    # causal products at their triangular size, per 64-token chunk; a backward
    # starts from the segments' states, so it forms the inner ones again
    if case["op"] == "gdn":
        tri = C * (C + 1) * D
        fl = 6 * C * D * D + 4 * tri + C ** 3 // 3
        if case["train"]:
            fl += 18 * C * D * D + 13 * tri + 2 * (C ** 3 // 3)
    else:
        fl = 2 * C * (C + 1) * D + 4 * C * D * D
        if case["train"]:
            fl += 5 * C * (C + 1) * D + 10 * C * D * D
    return dict(bytes=nbytes, flops=fl * (th // C))


def tolerance(case):
    if case["io"] == "f32":
        # sums in 32 bits (measured rel 1.9e-7 to 4.2e-7 against 64 bits, dg the largest)
        return {"rel": 1e-5, "max": 4e-4}
    # outputs rounded to bf16 (measured rel 1.7e-3 against 64 bits)
    return {"rel": 6e-3, "max": 2e-2}


# --- the same outputs in 64 bits, in plain torch -----------------------------------------

def _rows(x, h0, h1):
    """[B, L, H, ...] heads h0..h1 as [B (h1 - h0), L / C, C, ...] in float64."""
    x = x[:, :, h0:h1].double().transpose(1, 2)
    return x.reshape(-1, x.shape[2] // CHUNK, CHUNK, *x.shape[3:]).contiguous()


def _closed_form(op, q, k, v, g, beta, S0):
    """o and the states before every chunk and after the last one."""
    b = g.cumsum(2)
    end = b[:, :, -1:]
    tril = torch.ones(CHUNK, CHUNK, dtype=torch.bool, device=q.device).tril()
    if op == "vector":
        qd, kd, gam = q * b.exp(), k * (end - b).exp(), end[:, :, 0].exp()[..., None]
        A = (qd @ (k * (-b).exp()).transpose(2, 3)).masked_fill(~tril, 0.0)
    else:
        M = (b[..., :, None] - b[..., None, :]).masked_fill(~tril, float("-inf")).exp()
        qd, kd, gam = q * b.exp()[..., None], k * (end - b).exp()[..., None], end.exp()[..., None]
        gam = gam[:, :, 0]
        A = (q @ k.transpose(2, 3)) * M
    S, Ss = S0, [S0]
    if op == "gdn":
        N = (beta[..., None] * M * (k @ k.transpose(2, 3))).tril(-1)
        eye = torch.eye(CHUNK, dtype=q.dtype, device=q.device)
        T = torch.linalg.solve_triangular(eye + N, eye.expand_as(N), upper=False, unitriangular=True)
        W, U0, us = T @ (k * (beta * b.exp())[..., None]), T @ (v * beta[..., None]), []
        for w, u0, kc, gc in zip(W.unbind(1), U0.unbind(1), kd.transpose(2, 3).unbind(1), gam.unbind(1)):
            u = u0 - w @ S
            S = gc[..., None] * S + kc @ u
            us.append(u)
            Ss.append(S)
        v = torch.stack(us, 1)
    else:
        for d, gc in zip((kd.transpose(2, 3) @ v).unbind(1), gam.unbind(1)):
            S = (gc if op == "vector" else gc[..., None]) * S + d
            Ss.append(S)
    return qd @ torch.stack(Ss[:-1], 1) + A @ v, Ss


def _exact_conv(case, st):
    x, dy, w = st["x"].double(), st["dy"].double(), st["w"].double()
    B, L, C, W = case["B"], x.shape[1], case["C"], case["W"]
    zero = torch.zeros(B, W - 1, C, dtype=x.dtype, device=x.device)
    xe = torch.cat([zero if st["tail_in"] is None else st["tail_in"].double(), x], 1)
    u = sum(xe[:, j:j + L] * w[:, j] for j in range(W))
    s = torch.sigmoid(u) if case["act"] == "silu" else torch.ones_like(u)
    out = dict(y=u * s if case["act"] == "silu" else u, tail=xe[:, L:].clone())
    if not case["train"]:
        return out
    du = dy * (s * (1 + u * (1 - s)) if case["act"] == "silu" else s)
    dxe = torch.zeros_like(xe)
    for j in range(W):
        dxe[:, j:j + L] += du * w[:, j]
    if st["dtail_out"] is not None:
        dxe[:, L:] += st["dtail_out"].double()
    dw = torch.stack([(du * xe[:, j:j + L]).sum((0, 1)) for j in range(W)], 1)
    return dict(out, dx=dxe[:, W - 1:], dw=dw, dtail=dxe[:, :W - 1].clone())


def exact(case, seed):
    st = prepare(case, seed)
    if case["op"] == "conv":
        return _exact_conv(case, st)
    op, segs, B, H, D = case["op"], st["segs"], case["B"], case["H"], case["D"]
    L, dev, train = sum(segs), st["q"].device, case["train"]
    names = ["q", "k", "v", "g"] + (["beta"] if op == "gdn" else [])
    f64 = dict(dtype=torch.float64, device=dev)
    o = torch.empty((B, L, H, D), **f64)
    S = torch.empty((len(segs) + 1, B, H, D, D), **f64)
    grads = [torch.empty(st[n].shape, **f64) for n in names] + [torch.empty((B, H, D, D), **f64)]
    ends = [sum(segs[:i]) // CHUNK for i in range(len(segs) + 1)]
    step = max(1, (1 << 28) // (B * L * D))  # heads at a time, so that the intermediates fit
    for h0 in range(0, H, step):
        h1 = min(H, h0 + step)
        x = {n: _rows(st[n], h0, h1) for n in names}
        n = B * (h1 - h0)
        S0 = torch.zeros((n, D, D), **f64) if st["S_in"] is None else \
            st["S_in"][:, h0:h1].double().reshape(n, D, D)
        args = [t.requires_grad_(train) for t in list(x.values()) + [S0]]
        out, Ss = _closed_form(op, *args[:4], args[4] if op == "gdn" else None, args[-1])

        def back(t):  # [n, L / C, C, ...] -> [B, L, h, ...]
            return t.reshape(B, h1 - h0, L, *t.shape[3:]).transpose(1, 2)

        o[:, :, h0:h1] = back(out.detach())
        for i, e in enumerate(ends):
            S[i, :, h0:h1] = Ss[e].detach().reshape(B, h1 - h0, D, D)
        if train:
            loss = (out * _rows(st["dO"], h0, h1)).sum()
            if st["dS_out"] is not None:
                loss = loss + (Ss[-1] * st["dS_out"][:, h0:h1].double().reshape(n, D, D)).sum()
            *ds, dS = torch.autograd.grad(loss, args)
            for t, d in zip(grads, ds):
                t[:, :, h0:h1] = back(d)
            grads[-1][:, h0:h1] = dS.reshape(B, h1 - h0, D, D)
        del x, args, out, Ss
    res = dict(o=o, S=S[-1] if case["api"] == "segment" else S)
    if train:
        res["grads"] = tuple(grads)
    return res
