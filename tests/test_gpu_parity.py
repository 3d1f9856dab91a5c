"""GPU parity: the HIP path (through the C ABI) against the fp64 oracle.

Sizes span several chunks and superchunks with ragged tails; the workloads of
the paper's evaluation shapes run at full size, with the oracle on all heads
where it finishes in seconds and on sampled (batch, head) pairs otherwise.
"""
import numpy as np
import pytest
import torch

import paper_2608_06838_amd as sf
from paper_2608_06838_amd import synth
from tests._helpers import assert_close, assert_dg_apriori, oracle_run, select, select_state, to64

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def say(*a):
    print(*a, flush=True)


def on_gpu(inp):
    out = {}
    for key, x in inp.items():
        out[key] = x.to(DEV) if isinstance(x, torch.Tensor) else x
    return out


def check_all(io, got, ref, inp, names=("o", "S_out", "dq", "dk", "dv", "dg", "dS_in"), dg_apriori_ts=None):
    """Every output against the oracle.  dg_apriori_ts: for near-memoryless
    gates, whose exact dg is ~1e-13, dg is held to its elementwise fp32 bound
    over superchunks of that many tokens instead of the relative bar."""
    pairs = ref["pairs"]
    for n in names:
        X = got[n]
        X = select_state(X, pairs) if n in ("S_out", "dS_in") else select(X, pairs)
        if n == "dg" and dg_apriori_ts:
            assert_dg_apriori(n, X, ref, to64(select(inp["q"], pairs)), to64(select(inp["k"], pairs)),
                              dg_apriori_ts)
        else:
            assert_close(n, X, ref[n], io)


def seg_case(w, L, ts, seed, dS_std=0.1, s_in_std=None):
    if s_in_std is not None:
        w = dict(w, s_in_std=s_in_std)
    inp = synth.make_inputs(w, device="cpu", seed=seed, dS_out_std=dS_std, L=L)
    g = on_gpu(inp)
    say(f"[seg] {w['name']} L={L} ts={ts} seed={seed}")
    o, S_out = sf.segment_fwd(g["q"], g["k"], g["v"], g["g"], g["S_in"], ts=ts)
    dq, dk, dv, dg, dS_in = sf.segment_bwd(g["q"], g["k"], g["v"], g["g"], g["S_in"], g["dO"], g["dS_out"],
                                           ts=ts)
    torch.cuda.synchronize()
    return inp, dict(o=o, S_out=S_out, dq=dq, dk=dk, dv=dv, dg=dg, dS_in=dS_in)


@pytest.mark.parametrize("ts", [1024, 256, 192])
def test_tiny_fp32_segment(ts):
    """B=1, H=2, d=64, L=1024, fp32 I/O; one superchunk, four, and a ragged split."""
    w = synth.workload("tiny_fp32")
    inp, got = seg_case(w, 1024, ts, seed=1000, dS_std=0.0)
    check_all("f32", got, oracle_run(inp), inp)
    inp, got = seg_case(w, 1024, ts, seed=1001, dS_std=0.1, s_in_std=0.1)
    check_all("f32", got, oracle_run(inp), inp)


@pytest.mark.parametrize("D", [128, 64])
@pytest.mark.parametrize("ts", [4096, 128, 64])
def test_bf16_segment_paths(D, ts):
    """B=2, H=3, L=448 (7 chunks): single superchunk, ragged 128-token
    superchunks (128,128,128,64), and one superchunk per chunk."""
    w = synth.workload("mid_bf16", B=2, H=3, D=D)
    inp, got = seg_case(w, 448, ts, seed=7 + D + ts)
    check_all("bf16", got, oracle_run(inp), inp)


@pytest.mark.parametrize("name,D,io", [("mid_bf16", 64, "bf16"), ("tiny_fp32", 64, "f32"), ("vector_gate", 64, "bf16"),
                                       ("vector_gate", 64, "f32"), ("mid_bf16", 128, "bf16")])
@pytest.mark.parametrize("ts", [64, 128])
def test_more_items_than_cus(name, D, io, ts):
    """B=1, H=88, L=192: 264 or 176 items and, at d = 64, 352 scan workgroups on 256
    CUs.  Launches of more items than CUs, and of a scan workgroup per CU, take other
    kernel forms than the small cases do; the scans' rows are then shared out
    otherwise too."""
    w = synth.workload(name, B=1, H=88, D=D, io=io)
    inp, got = seg_case(w, 192, ts, seed=83 + D + ts, s_in_std=0.1)
    check_all(io, got, oracle_run(inp), inp)


@pytest.mark.parametrize("ts", [1024, 128, 192])
def test_fp32_d128_segment(ts):
    """fp32 I/O at d = 128 (scalar gate; its dk/dv walk runs as two workgroups
    per superchunk): B=1, H=2, L=1024 as one superchunk, eight, and a ragged
    192-token split, with S_in and dS_out; fp32 bar."""
    w = synth.workload("tiny_fp32", D=128)
    inp, got = seg_case(w, 1024, ts, seed=1200 + ts, dS_std=0.1, s_in_std=0.1)
    check_all("f32", got, oracle_run(inp), inp)


@pytest.mark.parametrize("ts", [0, 64, 128])
def test_fp32_d128_chain(ts):
    """fp32 I/O at d = 128 over four nonuniform segments, in one set of launches (ts =
    0, 64) and segment by segment (128): overlap on and off and kept superchunk states
    give bitwise the same outputs; fp32 bar."""
    w = synth.workload("tiny_fp32", B=1, H=3, D=128)
    seg_lens = [192, 64, 320, 128]
    inp = synth.make_inputs(w, device="cpu", seed=1210 + ts, dS_out_std=0.1, L=sum(seg_lens))
    g = on_gpu(inp)
    say(f"[chain] fp32 d=128 ts={ts}")
    assert in_one(g, seg_lens, ts) == (ts != 128)
    a = run_chain(g, seg_lens, ts=ts, overlap=True)
    for kw in (dict(overlap=False), dict(overlap=2), dict(overlap=True, keep=True), dict(overlap=2, keep=True)):
        b = run_chain(g, seg_lens, ts=ts, **kw)
        for key in a:
            assert torch.equal(a[key], b[key]), (key, kw)
    check_chain("f32", inp, a, seg_lens)


def test_fp32_strong_decay_and_memoryless():
    """Very negative gates (a_t -> 0): each token sees only itself."""
    w = synth.workload("tiny_fp32", g_mu=-30.0)
    inp, got = seg_case(w, 256, 128, seed=3)
    check_all("f32", got, oracle_run(inp), inp, dg_apriori_ts=128)


@pytest.mark.parametrize("io", ["f32", "bf16"])
def test_strong_decay_dg(io):
    """a_t ~ e^-3 (x ~ N(-3, 1)): a short memory, yet dg is of the order of its
    per-token terms, so it is held to the plain relative bar."""
    w = synth.workload("tiny_fp32", g_mu=-3.0) if io == "f32" else synth.workload("mid_bf16", B=1, H=2, D=128,
                                                                                    g_mu=-3.0)
    inp, got = seg_case(w, 512, 128, seed=13)
    check_all(io, got, oracle_run(inp), inp)


def test_empty_segment():
    w = synth.workload("mid_bf16", B=1, H=2, D=128)
    inp = on_gpu(synth.make_inputs(w, device="cpu", seed=5, dS_out_std=0.1, L=64))
    q0 = inp["q"][:, :0]
    g0 = inp["g"][:, :0]
    say("[seg] empty segment")
    o, S_out = sf.segment_fwd(q0, q0, q0, g0, inp["S_in"])
    _, _, _, _, dS_in = sf.segment_bwd(q0, q0, q0, g0, inp["S_in"], q0, inp["dS_out"])
    torch.cuda.synchronize()
    assert o.numel() == 0
    assert torch.equal(S_out, inp["S_in"])
    assert torch.equal(dS_in, inp["dS_out"])


def launches(fn, *kernels):
    """(fn(timing), launches per kernel kind of that call)"""
    t = sf.KernelTimer(kernels, capacity=512)
    try:
        out = fn(t)
        return out, {k: n for k, (_, n) in t.read().items()}
    finally:
        t.close()


def in_one(g, seg_lens, ts):
    """Whether the chain goes out as one set of launches over all its segments."""
    _, n = launches(lambda t: sf.chain_fwd(g["q"], g["k"], g["v"], g["g"], seg_lens, g["S_in"], ts=ts, overlap=False,
                                           timing=t), "fwd_out")
    assert n["fwd_out"] in (1, len(seg_lens))
    return n["fwd_out"] == 1


def run_chain(g, seg_lens, ts=0, overlap=True, keep=False):
    """keep: the backward reads the superchunk states the forward kept."""
    ck = None
    if keep:
        o, S_bnd, ck = sf.chain_fwd(g["q"], g["k"], g["v"], g["g"], seg_lens, g["S_in"], ts=ts, overlap=overlap,
                                    keep_states=True)
    else:
        o, S_bnd = sf.chain_fwd(g["q"], g["k"], g["v"], g["g"], seg_lens, g["S_in"], ts=ts, overlap=overlap)
    dq, dk, dv, dg, dS0 = sf.chain_bwd(g["q"], g["k"], g["v"], g["g"], seg_lens, S_bnd, g["dO"], g["dS_out"],
                                       ts=ts, overlap=overlap, ckpt=ck)
    torch.cuda.synchronize()
    return dict(o=o, S_bnd=S_bnd, S_out=S_bnd[-1], dq=dq, dk=dk, dv=dv, dg=dg, dS_in=dS0)


def check_chain(io, inp, got, seg_lens, pairs=None):
    pos = np.cumsum([0] + list(seg_lens)).tolist()
    ref = oracle_run(inp, pairs=pairs, snap_pos=pos)
    check_all(io, got, ref, inp)
    for i in range(1, len(pos) - 1):  # interior boundary states
        X = got["S_bnd"][i]
        X = select_state(X, ref["pairs"])
        assert_close(f"S_bnd{i}", X, ref["snaps"][i], io)


@pytest.mark.parametrize("ts", [0, 64, 128])
def test_chain_nonuniform_small(ts):
    """Four nonuniform segments, chained, in one set of launches (ts = 0, 64) and
    segment by segment (128); every overlap mode (serial, scans on the aux stream,
    preparation and scans there) agrees bitwise."""
    w = synth.workload("mid_bf16", B=1, H=4, D=128)
    seg_lens = [192, 64, 320, 128]
    inp = synth.make_inputs(w, device="cpu", seed=11, dS_out_std=0.1, L=sum(seg_lens))
    g = on_gpu(inp)
    say(f"[chain] small nonuniform ts={ts}")
    assert in_one(g, seg_lens, ts) == (ts != 128)
    a = run_chain(g, seg_lens, ts=ts, overlap=True)
    for mode in (False, 2):
        b = run_chain(g, seg_lens, ts=ts, overlap=mode)
        for key in a:
            assert torch.equal(a[key], b[key]), (key, mode)
    check_chain("bf16", inp, a, seg_lens)


@pytest.mark.parametrize("name,D,io,head_major", [("mid_bf16", 128, "bf16", False), ("mid_bf16", 64, "bf16", True),
                                                  ("tiny_fp32", 64, "f32", False), ("vector_gate", 128, "bf16", True)])
def test_chain_launched_as_one_segment(name, D, io, head_major):
    """32 short segments go out as one set of launches, 33 segment by segment:
    both against a segment call per segment, handing over S_out and dS_in, with
    the superchunks that ts = 64 gives all three.  Only how the scans round between
    segments differs, so the oracle's bars hold; and the 33 agree bitwise in every
    overlap mode (their scans and preparations do run on the aux stream)."""
    w = synth.workload(name, B=2, H=3, D=D, io=io)
    for n in (32, 33):
        seg_lens = [64, 192, 128] * 10 + [64] * (n - 30)
        inp = synth.make_inputs(w, device="cpu", seed=71 + n, dS_out_std=0.1, L=sum(seg_lens))
        g = on_gpu(inp)
        if head_major:
            for key in ("q", "k", "v", "g", "dO"):
                p = (0, 2, 1, 3)[:g[key].dim()]
                g[key] = g[key].permute(*p).contiguous().permute(*p)
        say(f"[chain] {n} segments {name} D={D} {io} against segment calls")
        assert in_one(g, seg_lens, 64) == (n == 32)
        a = run_chain(g, seg_lens, ts=64, overlap=False)
        for mode in (True, 2) if n > 32 else ():
            b = run_chain(g, seg_lens, ts=64, overlap=mode)
            for key in a:
                assert torch.equal(a[key], b[key]), (key, mode)
        pos = np.cumsum([0] + seg_lens).tolist()
        S = a["S_bnd"][0]
        bnd, outs, grads = [S], [], [None] * n
        for i in range(n):
            part = [g[key][:, pos[i]:pos[i + 1]] for key in ("q", "k", "v", "g")]
            o, S = sf.segment_fwd(*part, S, ts=64)
            outs.append(o)
            bnd.append(S)
        dS = g["dS_out"]
        for i in reversed(range(n)):
            part = [g[key][:, pos[i]:pos[i + 1]] for key in ("q", "k", "v", "g")]
            *grads[i], dS = sf.segment_bwd(*part, bnd[i], g["dO"][:, pos[i]:pos[i + 1]], dS, ts=64)
        torch.cuda.synchronize()
        want = dict(o=torch.cat(outs, 1), S_bnd=torch.stack(bnd), dS_in=dS)
        for j, key in enumerate(("dq", "dk", "dv", "dg")):
            want[key] = torch.cat([x[j] for x in grads], 1)
        for key in want:
            X, R = to64(a[key]), to64(want[key])
            if a[key].dtype == torch.bfloat16:  # both rounded: a step apart (2^-7) where they fall either side
                assert np.all(np.abs(X - R) <= 2.0 ** -7 * np.abs(R) + 2e-3 * np.sqrt(np.mean(R * R))), key
            else:
                assert_close(key, X, R, io)


@pytest.mark.parametrize("name,D,io", [("mid_bf16", 128, "bf16"), ("tiny_fp32", 64, "f32"), ("vector_gate", 128, "bf16")])
def test_chain_replay_starts_from_the_given_states(name, D, io):
    """A backward over several segments in one set of launches replays each segment
    from the S_bnd it is given: infinities in the first segment's v leave every
    gradient of the later segments, and the gradient of the initial state (which
    depends on no v), bitwise as they were."""
    w = synth.workload(name, B=1, H=3, D=D, io=io)
    seg_lens = [128, 64, 192, 128]
    inp = synth.make_inputs(w, device="cpu", seed=91 + D, dS_out_std=0.1, L=sum(seg_lens))
    g = on_gpu(inp)
    say(f"[chain] replay from the given states {name} D={D} {io}")
    _, S_bnd = sf.chain_fwd(g["q"], g["k"], g["v"], g["g"], seg_lens, g["S_in"], ts=64, overlap=False)

    def bwd(v):
        out, n = launches(lambda t: sf.chain_bwd(g["q"], g["k"], v, g["g"], seg_lens, S_bnd, g["dO"], g["dS_out"],
                                                 ts=64, overlap=False, timing=t), "scan")
        assert n == {"scan": 1}  # one set of launches
        return out

    bad = g["v"].clone()
    bad[:, 5, :, 3] = float("inf")
    a, b = bwd(g["v"]), bwd(bad)
    assert not torch.isfinite(b[0][:, :seg_lens[0]]).all()
    for x, y in zip(a[:4], b[:4]):
        assert torch.isfinite(x).all()
        assert torch.equal(x[:, seg_lens[0]:], y[:, seg_lens[0]:])
    assert torch.equal(a[4], b[4])


@pytest.mark.parametrize("name,D,io", [("mid_bf16", 128, "bf16"), ("tiny_fp32", 64, "f32"), ("vector_gate", 128, "bf16")])
def test_two_segments_of_one_chunk(name, D, io):
    """Two segments of one chunk each: the forward runs segment by segment and keeps
    nothing, the backward as one set of launches from S_bnd, with the kept states' buffer
    or without it."""
    w = synth.workload(name, B=1, H=3, D=D, io=io)
    seg_lens = [64, 64]
    inp = synth.make_inputs(w, device="cpu", seed=97 + D, dS_out_std=0.1, L=128)
    g = on_gpu(inp)
    say(f"[chain] two segments of one chunk {name} D={D} {io}")
    assert not in_one(g, seg_lens, 0) and sf.chain_ckpt_bytes(g["q"], g["g"], seg_lens, ts=0) == 0
    a = run_chain(g, seg_lens, ts=0, overlap=False)
    _, n = launches(lambda t: sf.chain_bwd(g["q"], g["k"], g["v"], g["g"], seg_lens, a["S_bnd"], g["dO"], g["dS_out"], ts=0,
                                           overlap=False, timing=t), "bwd_dq")
    assert n == {"bwd_dq": 1}
    b = run_chain(g, seg_lens, ts=0, overlap=False, keep=True)
    for key in a:
        assert torch.equal(a[key], b[key]), key
    check_chain(io, inp, a, seg_lens)


KEPT_CASES = [("mid_bf16", 128, "bf16", 0), ("mid_bf16", 128, "bf16", 64), ("mid_bf16", 64, "bf16", 128),
              ("tiny_fp32", 64, "f32", 128), ("vector_gate", 128, "bf16", 128), ("vector_gate", 64, "f32", 64),
              ("mid_bf16", 128, "bf16", 128), ("tiny_fp32", 128, "f32", 128), ("vector_gate", 64, "f32", 128),
              ("vector_gate", 128, "bf16", 64)]


@pytest.mark.parametrize("name,D,io,ts", KEPT_CASES)
def test_kept_states(name, D, io, ts):
    """Backward from the superchunk states the forward kept: bitwise the
    outputs of the backward that replays them (segments of one and of several
    superchunks; in one set of launches, or, for ts = 128, segment by segment in
    every overlap mode), and within the bar of the oracle."""
    w = synth.workload(name, B=1, H=3, D=D, io=io)
    seg_lens = [192, 64, 320, 128]
    inp = synth.make_inputs(w, device="cpu", seed=53 + D + ts, dS_out_std=0.1, L=sum(seg_lens))
    g = on_gpu(inp)
    say(f"[chain] kept states {name} D={D} {io} ts={ts}")
    assert in_one(g, seg_lens, ts) == (ts != 128)
    for overlap in (False, True, 2):
        a = run_chain(g, seg_lens, ts=ts, overlap=overlap)
        b = run_chain(g, seg_lens, ts=ts, overlap=overlap, keep=True)
        for key in a:
            assert torch.equal(a[key], b[key]), (key, overlap)
    check_chain(io, inp, b, seg_lens)


def test_mid_layer_chain():
    """B=1, H=16, d=128, L=32768 in 8 segments of 4096, bf16 I/O, S_in ~ 0.1 N(0,1)."""
    w = synth.workload("mid_bf16")
    say("[chain] mid_bf16 full size")
    inp = synth.make_inputs(w, device=DEV, seed=1001, dS_out_std=0.1)
    got = run_chain(inp, w["seg_lens"])
    check_chain("bf16", inp, got, w["seg_lens"])


def test_scan_stress_sampled():
    """B=4, H=32, L=16384 in 32 segments of 512 with strong decay; oracle on
    six (batch, head) pairs."""
    w = synth.workload("scan_stress")
    say("[chain] scan_stress full size")
    inp = synth.make_inputs(w, device=DEV, seed=1004, dS_out_std=0.1)
    got = run_chain(inp, w["seg_lens"])
    again = run_chain(inp, w["seg_lens"], overlap=False, keep=True)
    for key in got:
        assert torch.equal(got[key], again[key]), key
    check_chain("bf16", inp, got, w["seg_lens"], pairs=[(0, 0), (1, 7), (2, 31), (3, 16), (0, 20), (3, 3)])


def test_ctx256k_sampled():
    """B=1, H=40, d=128, L=262144 in 8 nonuniform segments (the 256K-context
    workload) with a nonzero gradient of the final state.  Full-size run; the
    oracle checks the first, a middle and the last head end to end, interior
    boundary states included; the run is repeated with the backward reading the
    forward's kept superchunk states, and every output must be bitwise
    identical."""
    w = synth.workload("ctx256k_h40")
    say("[chain] ctx256k_h40 full size")
    inp = synth.make_inputs(w, device=DEV, seed=1002, dS_out_std=0.1)
    got = run_chain(inp, w["seg_lens"])
    again = run_chain(inp, w["seg_lens"], keep=True)
    for key in ("o", "S_bnd", "dq", "dk", "dv", "dg", "dS_in"):
        assert torch.equal(got[key], again[key]), key
    say("[chain] ctx256k_h40 oracle on heads 0, 17, 39")
    check_chain("bf16", inp, got, w["seg_lens"], pairs=[(0, 0), (0, 17), (0, 39)])


# ------------------------------------------------------------------ vector gate
@pytest.mark.parametrize("D,io", [(128, "bf16"), (64, "bf16"), (64, "f32")])
@pytest.mark.parametrize("ts", [4096, 128, 64])
def test_vector_gate_segment(D, io, ts):
    """Per-key-channel gate, B=2, H=3, L=448 (7 chunks): one superchunk, ragged
    128-token superchunks, one superchunk per chunk."""
    w = synth.workload("vector_gate", B=2, H=3, D=D, io=io)
    inp, got = seg_case(w, 448, ts, seed=31 + D + ts, s_in_std=0.1)
    check_all(io, got, oracle_run(inp), inp)


@pytest.mark.parametrize("g_mu", [-0.5, -30.0])
def test_vector_gate_decay_regimes(g_mu):
    """Gates strong enough that some chunks (g_mu = -0.5: a mix) or all chunks
    (g_mu = -30: memoryless) decay below 2^-100 in some channel and are walked
    token by token; the rest take the tiled path."""
    w = synth.workload("vector_gate", B=1, H=2, D=128, g_mu=g_mu)
    inp, got = seg_case(w, 512, 128, seed=41, s_in_std=0.1)
    check_all("bf16", got, oracle_run(inp), inp, dg_apriori_ts=128 if g_mu < -10 else None)


@pytest.mark.parametrize("ts", [0, 64, 128])
def test_vector_gate_chain_nonuniform(ts):
    """As test_chain_nonuniform_small, with the per-key-channel gate."""
    w = synth.workload("vector_gate", B=1, H=3, D=128)
    seg_lens = [192, 64, 320, 128]
    inp = synth.make_inputs(w, device="cpu", seed=43, dS_out_std=0.1, L=sum(seg_lens))
    g = on_gpu(inp)
    say(f"[chain] vector gate nonuniform ts={ts}")
    assert in_one(g, seg_lens, ts) == (ts != 128)
    a = run_chain(g, seg_lens, ts=ts, overlap=True)
    for mode in (False, 2):
        b = run_chain(g, seg_lens, ts=ts, overlap=mode)
        for key in a:
            assert torch.equal(a[key], b[key]), (key, mode)
    check_chain("bf16", inp, a, seg_lens)


def test_vector_gate_workload_sampled():
    """B=2, H=16, d=128, L=65536 in 16 segments of 4096 with the per-key-channel
    gate; the oracle checks two (batch, head) pairs end to end."""
    w = synth.workload("vector_gate")
    say("[chain] vector_gate full size")
    inp = synth.make_inputs(w, device=DEV, seed=1003, dS_out_std=0.0)
    got = run_chain(inp, w["seg_lens"])
    check_chain("bf16", inp, got, w["seg_lens"], pairs=[(0, 5), (1, 12)])


@pytest.mark.parametrize("gate", ["scalar", "vector"])
def test_head_major_layout(gate):
    """q, k, v, dO stored head-major ([B, H, L, D] in memory) and g as [B, H, L]
    (vector gate: [B, H, L, D]), passed as [B, L, H, ...] views: the strides go
    through the ABI, the outputs come back in the same layout, every value is
    bitwise that of the packed layout, and the oracle bar holds (chained
    nonuniform segments, several superchunks)."""
    name = "vector_gate" if gate == "vector" else "mid_bf16"
    w = synth.workload(name, B=2, H=3, D=128)
    seg_lens = [192, 64, 320]
    inp = synth.make_inputs(w, device="cpu", seed=61, dS_out_std=0.1, L=sum(seg_lens))
    say(f"[chain] head-major layout, {gate} gate")

    def hm(x):  # the same values in head-major memory
        p = (0, 2, 1, 3) if x.dim() == 4 else (0, 2, 1)
        return x.permute(*p).contiguous().permute(*p).to(DEV)

    g = on_gpu(inp)
    h = dict(g, **{n: hm(inp[n]) for n in ("q", "k", "v", "g", "dO")})
    assert h["q"].stride(2) == sum(seg_lens) * 128 and h["q"].stride(1) == 128
    a = run_chain(g, seg_lens, ts=128)
    b = run_chain(h, seg_lens, ts=128)
    assert b["o"].stride() == h["q"].stride() and b["dg"].stride() == h["g"].stride()
    for key in a:
        assert torch.equal(a[key].contiguous(), b[key].contiguous()), key
    check_chain("bf16", inp, b, seg_lens)


def test_tuned_setting_is_applied(monkeypatch):
    """chain_fwd / chain_bwd with ts and overlap left unset take the profiled
    per-shape setting (paper_2608_06838_amd.tuned): bitwise the outputs of
    passing that setting explicitly, different from the automatic stride's
    rounding, and within the parity bar of the oracle."""
    from paper_2608_06838_amd import tuned
    w = synth.workload("mid_bf16", B=1, H=4, D=128)
    seg_lens = [512, 256, 448]
    key = tuned.key(1, 4, 128, "bf16", "scalar", seg_lens)
    monkeypatch.setitem(tuned.TABLE, key, dict(ts=128, overlap=False))
    inp = synth.make_inputs(w, device="cpu", seed=17, dS_out_std=0.1, L=sum(seg_lens))
    g = on_gpu(inp)
    say("[chain] tuned setting lookup")

    def chain(**kw):
        o, S_bnd = sf.chain_fwd(g["q"], g["k"], g["v"], g["g"], seg_lens, g["S_in"], **kw)
        grads = sf.chain_bwd(g["q"], g["k"], g["v"], g["g"], seg_lens, S_bnd, g["dO"], g["dS_out"], **kw)
        torch.cuda.synchronize()
        return (o, S_bnd) + tuple(grads)

    looked_up, explicit, other = chain(), chain(ts=128, overlap=False), chain(ts=0, overlap=False)
    for x, y in zip(looked_up, explicit):
        assert torch.equal(x, y)
    # a different stride sums in another order: some output differs in its last bits
    assert any(not torch.equal(x, y) for x, y in zip(looked_up, other))
    got = dict(zip(("o", "S_bnd", "dq", "dk", "dv", "dg", "dS_in"), looked_up))
    got["S_out"] = got["S_bnd"][-1]
    check_chain("bf16", inp, got, seg_lens)
