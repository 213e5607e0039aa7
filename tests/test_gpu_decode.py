"""GPU parity of the recurrent (decode) kernel and the chunk -> decode hand-off."""

import numpy as np
import pytest

from oracle import gdr2_recurrent_fwd
from paper_2605_22791_amd.inputs import make_inputs
from tests.helpers import rel_l2
from tests.gpu_common import dev_inputs, host, heads, pick

pytestmark = pytest.mark.gpu

TOL = {"fp32": 1e-5, "bf16": 2e-3}


def _case(msg):
    print(f"\n[gpu case] {msg}", flush=True)


@pytest.mark.parametrize("Dk,Dv,dtype,T", [(128, 128, "fp32", 50), (64, 128, "bf16", 33),
                                           (128, 64, "fp32", 7), (64, 64, "bf16", 1)])
def test_recurrent_multi_token(Dk, Dv, dtype, T):
    import paper_2605_22791_amd as g2
    d = make_inputs(3, T, 2, Dk, Dv, seed=70 + T, dtype=dtype, s0_std=0.05)
    _case(f"recurrent T={T} Dk{Dk} Dv{Dv} {dtype}")
    x = dev_inputs(d)
    S = x["S0"].clone()
    o = g2.gdr2_recurrent_step(x["q"], x["k"], x["v"], x["log_alpha"], x["b"], x["w"], S, scale=d["scale"])
    o_ref, S_ref = gdr2_recurrent_fwd(d["q"], d["k"], d["v"], d["log_alpha"], d["b"], d["w"], d["S0"], d["scale"])
    assert rel_l2(host(o), o_ref) < TOL[dtype]
    assert rel_l2(host(S), S_ref) < TOL[dtype] / 4


def test_decode_config4_full_horizon_sampled():
    """Config 4 over its whole horizon: B=256, H=16, d=128, 1024 consecutive
    one-token calls on one fp32 state kept in HBM (App. C.5), from S = 0.
    Inputs are drawn on the device; four (batch, head) pairs, among them the
    first and the last, are run through the oracle over all 1024 tokens.
    Checked: o of all calls (rel-L2 over the whole output and over every
    window of 64 calls), and the sampled states after every 128 calls, so a
    drift of the fp32 state over the horizon shows where it starts."""
    import torch
    import paper_2605_22791_amd as g2
    from paper_2605_22791_amd.inputs import make_decode_device
    steps, B, H, D = 1024, 256, 16, 128
    _case(f"decode B{B} H{H} d{D}, {steps} consecutive calls")
    x = make_decode_device(steps, B, H, D, seed=4)
    pairs = [(0, 0), (255, 15), (100, 7), (31, 3)]
    names = ("q", "k", "v", "log_alpha", "b", "w")
    S = torch.zeros((B, H, D, D), dtype=torch.float32, device="cuda")
    o = torch.empty((B, 1, H, D), dtype=torch.bfloat16, device="cuda")
    o_s = torch.empty((steps, len(pairs), D), dtype=torch.float32, device="cuda")
    S_s = {}
    bi = torch.tensor([p[0] for p in pairs], device="cuda")
    hi = torch.tensor([p[1] for p in pairs], device="cuda")
    for t in range(steps):
        g2.gdr2_recurrent_step(*[x[n][t] for n in names], S, o=o, scale=x["scale"])
        o_s[t] = o[bi, 0, hi].float()
        if (t + 1) % 128 == 0:
            S_s[t + 1] = S[bi, hi].double().cpu().numpy()
    torch.cuda.synchronize()
    o_got = o_s.double().cpu().numpy()                     # (steps, pairs, D)
    d = {n: np.stack([x[n][:, b_, 0, h_].float().cpu().numpy() for (b_, h_) in pairs])[:, :, None]
         for n in names}                                   # (pairs, steps, 1, D)
    del x
    o_ref = np.empty((steps, len(pairs), D))
    S_ref = {}
    Sr = None
    for lo in range(0, steps, 128):
        sl = {n: np.ascontiguousarray(d[n][:, lo:lo + 128]) for n in names}
        o_r, Sr = gdr2_recurrent_fwd(sl["q"], sl["k"], sl["v"], sl["log_alpha"], sl["b"], sl["w"], Sr, 1.0 / np.sqrt(D))
        o_ref[lo:lo + 128] = np.moveaxis(o_r[:, :, 0], 0, 1)
        S_ref[lo + 128] = Sr[:, 0]
    e_all = rel_l2(o_got, o_ref)
    e_win = max(rel_l2(o_got[t:t + 64], o_ref[t:t + 64]) for t in range(0, steps, 64))
    e_S = {t: rel_l2(S_s[t], S_ref[t]) for t in S_s}
    print(f"rel o {e_all:.3e}, worst 64-call window {e_win:.3e}; S after calls:",
          {t: f"{v:.2e}" for t, v in e_S.items()}, flush=True)
    assert e_all < TOL["bf16"] and e_win < TOL["bf16"]
    # the state stays fp32: its error is that of fp32 arithmetic, far below the bf16 bound
    assert max(e_S.values()) < 1e-4, e_S


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
def test_chunk_then_decode_handoff(dtype):
    """chunk_fwd over a 256-token prompt, then 8 recurrent steps == oracle over 264 tokens."""
    import paper_2605_22791_amd as g2
    d = make_inputs(2, 264, 2, 128, 128, seed=80, dtype=dtype, s0_std=0.05)
    _case(f"chunk->decode hand-off {dtype}")
    x = dev_inputs(d)
    pre = [x[n][:, :256].contiguous() for n in ("q", "k", "v", "log_alpha", "b", "w")]
    o1, S = g2.gdr2_chunk_fwd(*pre, x["S0"], scale=d["scale"])
    outs = [host(o1)]
    for t in range(256, 264):
        step = [x[n][:, t:t + 1].contiguous() for n in ("q", "k", "v", "log_alpha", "b", "w")]
        outs.append(host(g2.gdr2_recurrent_step(*step, S, scale=d["scale"])))
    o_ref, S_ref = gdr2_recurrent_fwd(d["q"], d["k"], d["v"], d["log_alpha"], d["b"], d["w"], d["S0"], d["scale"])
    assert rel_l2(np.concatenate(outs, axis=1), o_ref) < TOL[dtype]
    assert rel_l2(host(S), S_ref) < TOL[dtype]


# the sizes where the recurrent kernels change: one token or several, and 16 columns a wave
# (apart, together) or 32 by the number of (sequence, head) pairs, these up to four tokens by rows
@pytest.mark.parametrize("B,T,H,Dk,Dv,dtype", [
    (1, 1, 1, 64, 64, "fp32"), (3, 1, 2, 128, 64, "bf16"), (2, 1, 3, 64, 128, "bf16"), (2, 1, 1, 128, 128, "fp32"),
    (32, 2, 4, 64, 128, "bf16"), (43, 3, 3, 128, 128, "bf16"), (64, 2, 4, 128, 128, "fp32"),
    (257, 2, 1, 128, 128, "bf16"), (513, 3, 1, 128, 64, "fp32"), (260, 4, 1, 64, 128, "fp32"),
    (260, 5, 1, 64, 128, "bf16"), (520, 4, 1, 64, 64, "bf16")])
@pytest.mark.parametrize("fused", [False, True])
def test_recurrent_routes(B, T, H, Dk, Dv, dtype, fused):
    import torch
    import paper_2605_22791_amd as g2
    from paper_2605_22791_amd.inputs import make_fused
    from oracle import gdr2_fused_fwd
    _case(f"recurrent B{B} T{T} H{H} Dk{Dk} Dv{Dv} {dtype} fused={fused}")
    dev = lambda a, t: torch.from_numpy(np.ascontiguousarray(a)).cuda().to(t)
    io = torch.bfloat16 if dtype == "bf16" else torch.float32
    if fused:
        d = make_fused(B, T, H, Dk, Dv, seed=90 + B, dtype=dtype, s0_std=0.05)
        S = dev(d["S0"], torch.float32)
        o = g2.gdr2_fused_recurrent(*[dev(d[n], io) for n in ("q", "k", "v")], dev(d["f"], torch.float32),
                                    dev(d["a"], torch.float32), dev(d["delta"], torch.float32), dev(d["b"], io),
                                    dev(d["w"], io), S, scale=d["scale"], eps=d["eps"])
        o_ref, S_ref = gdr2_fused_fwd(*[d[n] for n in ("q", "k", "v", "f", "a", "delta", "b", "w")], d["S0"],
                                      scale=d["scale"], eps=d["eps"], dtype=dtype)
    else:
        d = make_inputs(B, T, H, Dk, Dv, seed=90 + B, dtype=dtype, s0_std=0.05)
        x = dev_inputs(d)
        S = x["S0"].clone()
        o = g2.gdr2_recurrent_step(x["q"], x["k"], x["v"], x["log_alpha"], x["b"], x["w"], S, scale=d["scale"])
        o_ref, S_ref = gdr2_recurrent_fwd(d["q"], d["k"], d["v"], d["log_alpha"], d["b"], d["w"], d["S0"], d["scale"])
    assert rel_l2(host(o), o_ref) < TOL[dtype]
    # fp32 state arithmetic; fused bf16 rounds the normalised k, where a value next to a tie can go
    # either way (2^-8 of that value)
    assert rel_l2(host(S), S_ref) < (1e-4 if fused and dtype == "bf16" else 1e-5)


@pytest.mark.parametrize("Dk,Dv,H,Hv,dtype", [(128, 128, 1, 1, "bf16"), (64, 128, 1, 2, "fp32"), (128, 64, 2, 2, "bf16"),
                                              (64, 64, 2, 4, "bf16")])
def test_recurrent_packed_mixed_counts(Dk, Dv, H, Hv, dtype):
    """A packed batch past the line of 1024 32-column waves whose sequences take 0 to 9 tokens: those of
    up to four go by rows, the others by columns, side by side in one launch."""
    import torch
    import paper_2605_22791_amd as g2
    from oracle import gdr2_packed_fwd
    rng = np.random.default_rng(77)
    N = 1024 // (Hv * Dv // 32) + 3
    lengths = rng.choice([0, 1, 1, 2, 3, 4, 5, 9], size=N)
    lengths[:3], lengths[-2:] = (4, 5, 0), (9, 1)
    cu = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    T = int(cu[-1])
    d = make_inputs(1, T, Hv, Dk, Dv, seed=97, dtype=dtype)
    for n in ("q", "k", "log_alpha", "b"):
        d[n] = np.ascontiguousarray(d[n][:, :, :H])
    S0 = (0.1 * rng.standard_normal((N, Hv, Dk, Dv))).astype(np.float32)
    _case(f"recurrent packed {N} sequences, T = {T}, H{H} Hv{Hv} Dk{Dk} Dv{Dv} {dtype}")
    x = dev_inputs(dict(d, S0=S0))
    S = x["S0"].clone()
    o = g2.gdr2_recurrent_varlen(x["q"], x["k"], x["v"], x["log_alpha"], x["b"], x["w"], torch.from_numpy(cu).cuda(), S,
                                 scale=d["scale"])
    rep = {n: np.repeat(d[n].astype(np.float64), Hv // H, axis=2) for n in ("q", "k", "log_alpha", "b")}
    o_ref, S_ref = gdr2_packed_fwd(rep["q"], rep["k"], d["v"], rep["log_alpha"], rep["b"], d["w"], cu, S0, d["scale"])
    assert rel_l2(host(o), o_ref) < TOL[dtype]
    assert rel_l2(host(S), S_ref) < 1e-5
    none = torch.from_numpy(np.flatnonzero(lengths == 0)).cuda()
    assert torch.equal(S[none], x["S0"][none])
