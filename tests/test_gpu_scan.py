"""GPU parity of the bf16 fused chunkwise scan (forward) against the fp64 oracle.

Precision of the bf16 path: Y is stored in bfloat16 (App. D's model-dtype
auxiliaries) and Y S reads the bf16 part of the state; every other product,
the Gram T and A's products into Y and U included, is fp32-accurate (split
hi/lo bf16), and the solve runs in fp32.  The fp32-typed final state S_T must
therefore stay well inside the 2e-3 bound: these tests hold it to 1e-3 (o is
bounded by its own bf16 rounding, ~1.66e-3).
"""

import numpy as np
import pytest

from oracle import gdr2_recurrent_fwd
from paper_2605_22791_amd.inputs import make_inputs
from tests.helpers import rel_l2
from tests.gpu_common import dev_inputs, host

pytestmark = pytest.mark.gpu

TOL_O = 2e-3
TOL_S = 1e-3


def _case(msg):
    print(f"\n[gpu case] {msg}", flush=True)


def _fwd(d, S0=True):
    import paper_2605_22791_amd as g2
    x = dev_inputs(d)
    o, ST = g2.gdr2_chunk_fwd(x["q"], x["k"], x["v"], x["log_alpha"], x["b"], x["w"],
                              x["S0"] if S0 else None, scale=d["scale"])
    return host(o), host(ST)


def _check(d, tol_s=TOL_S):
    o, ST = _fwd(d)
    o_ref, S_ref = gdr2_recurrent_fwd(d["q"], d["k"], d["v"], d["log_alpha"], d["b"], d["w"], d["S0"],
                                      d["scale"])
    ro, rs = rel_l2(o, o_ref), rel_l2(ST, S_ref)
    print(f"rel o {ro:.3e} S_T {rs:.3e}")
    assert np.all(np.isfinite(o)) and np.all(np.isfinite(ST))
    assert ro < TOL_O, ro
    assert rs < tol_s, rs


@pytest.mark.parametrize("Dk,Dv", [(64, 64), (64, 128), (128, 64), (128, 128)])
def test_bf16_head_dims(Dk, Dv):
    # B*H = 6: not a multiple of 8 (plain block order); 5 chunks
    d = make_inputs(2, 320, 3, Dk, Dv, seed=70 + Dk + Dv, dtype="bf16", s0_std=0.05)
    _case(f"bf16 scan B2 H3 T320 Dk{Dk} Dv{Dv}")
    _check(d)


def test_bf16_xcd_grouped_order():
    # B*H = 8: the value slices of one head are placed on one XCD
    d = make_inputs(2, 256, 4, 128, 128, seed=75, dtype="bf16", s0_std=0.05)
    _case("bf16 scan B2 H4 T256 d128 (XCD-grouped slices)")
    _check(d)


def test_bf16_single_chunk_and_no_initial_state():
    d = make_inputs(1, 64, 2, 128, 128, seed=76, dtype="bf16")
    _case("bf16 scan one chunk, S0 = 0")
    _check(d)


def test_bf16_extreme_decay_diagonal_blocks():
    """Decay spikes push a block's internal decay past e^60: the diagonal T / A_qk
    tiles of that block are formed element by element."""
    d = make_inputs(1, 192, 2, 128, 128, seed=77, dtype="bf16", s0_std=0.1)
    la = d["log_alpha"].copy()
    la[0, 20, 0, :8] = -90.0
    la[0, 70, 1, 5:40] = -200.0
    la[0, 75, 1, 30:] = -70.0
    la[0, 140:150, 0, :] = -9.0
    d["log_alpha"] = la
    _case("bf16 scan extreme decay spikes")
    _check(d)


def test_bf16_state_passing():
    import paper_2605_22791_amd as g2
    d = make_inputs(1, 384, 2, 128, 128, seed=78, dtype="bf16", s0_std=0.05)
    _case("bf16 scan state passing 384 = 128 + 256")
    x = dev_inputs(d)
    o_all, S_all = g2.gdr2_chunk_fwd(x["q"], x["k"], x["v"], x["log_alpha"], x["b"], x["w"], x["S0"],
                                     scale=d["scale"])
    sl = lambda t, a, b_: t[:, a:b_].contiguous()
    o1, S1 = g2.gdr2_chunk_fwd(*[sl(x[n], 0, 128) for n in ("q", "k", "v", "log_alpha", "b", "w")], x["S0"],
                               scale=d["scale"])
    o2, S2 = g2.gdr2_chunk_fwd(*[sl(x[n], 128, 384) for n in ("q", "k", "v", "log_alpha", "b", "w")], S1,
                               scale=d["scale"])
    # the split is exact up to fp32 rounding of the hand-over state
    assert rel_l2(np.concatenate([host(o1), host(o2)], axis=1), host(o_all)) < 1e-3
    assert rel_l2(host(S2), host(S_all)) < 1e-5


@pytest.mark.parametrize("Dk,Dv", [(64, 128), (128, 128)])
def test_bf16_workspace_intermediates(Dk, Dv):
    """Fragment-ordered workspace of the intra-chunk kernel against App. A's chunk
    algebra: Q_g, Ktail, A_qk, gamma_C are fp32-accurate (split hi/lo); U = A Z
    comes from fp32-accurate products and the fp32 solve, so it stays near fp32
    rounding (a bf16 operand anywhere in T or A would put it near 1e-3);
    Y is stored in bf16, so its error is its own rounding (~1.7e-3 rel-L2)."""
    import torch
    from oracle.chunkwise import gdr2_chunk_fwd_ref
    from tests.gpu_common import ws_layout_bf16, decode_frag_blocks, decode_u_tiles, CH
    B, T, H = 1, 192, 2
    d = make_inputs(B, T, H, Dk, Dv, seed=79, dtype="bf16", s0_std=0.05)
    lay, total, NC = ws_layout_bf16(B, T, H, Dk, Dv)
    ws = torch.full((total,), 0xFF, dtype=torch.uint8, device="cuda")
    _case(f"bf16 workspace intermediates Dk{Dk} Dv{Dv}")
    import paper_2605_22791_amd as g2
    x = dev_inputs(d)
    g2.gdr2_chunk_fwd(x["q"], x["k"], x["v"], x["log_alpha"], x["b"], x["w"], x["S0"], scale=d["scale"], ws=ws)
    torch.cuda.synchronize()
    raw = ws.cpu().numpy()
    _, _, it = gdr2_chunk_fwd_ref(d["q"], d["k"], d["v"], d["log_alpha"], d["b"], d["w"], d["S0"], d["scale"],
                                  C=CH, keep=True)
    NT = T // CH
    worst = {}
    for ch in range(NC):
        bh, n = divmod(ch, NT)
        bi, hi = divmod(bh, H)

        def region(name):
            off, per = lay[name]
            return raw[off + ch * per: off + (ch + 1) * per]

        got = {
            "Y": decode_frag_blocks(region("Y").view(np.uint16), 4, Dk // 32, False, True),
            "Qg": decode_frag_blocks(region("Qg").view(np.uint16), 4, Dk // 32, True, False),
            "Aqk": decode_frag_blocks(region("Aqk").view(np.uint16), 4, 2, True, True),
            "Kt": decode_frag_blocks(region("KtT").view(np.uint16), Dk // 16, 2, True, False).T,
            "U": decode_u_tiles(region("U").view(np.float32), Dv),
            "GC": region("GC").view(np.float32)[:Dk].astype(np.float64),
        }
        # query rows 0..31 against keys 32..63 of A_qk are causal zeros that the
        # bf16 workspace does not store (its two all-zero fragment blocks)
        got["Aqk"][:32, 32:] = 0.0
        ref = {"Y": it["Y"][bi, hi, n], "Qg": it["Qg"][bi, hi, n], "Aqk": it["Aqk"][bi, hi, n],
               "Kt": it["Ktail"][bi, hi, n], "U": it["U"][bi, hi, n], "GC": it["gC"][bi, hi, n]}
        for k_ in ref:
            worst[k_] = max(worst.get(k_, 0.0), rel_l2(got[k_], ref[k_]))
    print({k_: f"{v_:.2e}" for k_, v_ in worst.items()})
    for k_ in ("Qg", "Aqk", "Kt", "GC"):
        assert worst[k_] < 1e-4, (k_, worst[k_])
    assert worst["U"] < 1e-5, worst["U"]   # about 3e-7
    assert worst["Y"] < 3e-3, worst["Y"]


@pytest.mark.parametrize("T", [1, 64, 130, 200])
@pytest.mark.parametrize("Dk,Dv", [(64, 64), (64, 128), (128, 64), (128, 128)])
def test_narrow_scans_equal_wide(Dk, Dv, T):
    """A few heads alone (32-wide value slices) give the bits that the same heads give inside a
    batch large enough for the 64-wide scans: one to four chunks, whole and partial last ones."""
    import torch
    import paper_2605_22791_amd as g2
    B, H = 9, 16 * 128 // Dv   # 288 wide scans
    d = make_inputs(B, T, H, Dk, Dv, seed=500 + T + Dk, dtype="bf16", decay_shift=-2.0, s0_std=0.05, with_dST=True)
    _case(f"narrow against wide scans, Dk{Dk} Dv{Dv} T{T}")
    x = dev_inputs(d)

    def run(t, save):
        args = [t[n] for n in ("q", "k", "v", "log_alpha", "b", "w")]
        need = g2.gdr2_chunk_workspace_bytes(g2._problem(t["q"], t["v"], d["scale"]), 1)
        ws = torch.full((need,), 0xFF, dtype=torch.uint8, device="cuda")
        o, ST = g2.gdr2_chunk_fwd(*args, t["S0"], scale=d["scale"], ws=ws, save=save)
        g = g2.gdr2_chunk_bwd(*args, t["S0"], t["do"], t["dST"], scale=d["scale"], ws=ws, saved=save)
        return {"o": o, "S_T": ST, **g}

    wide = run(x, True)
    for h0, nh in ((0, 1), (3, 5)):   # one head; five (no multiple of the XCDs)
        sub = {n: (t[2:3, :, h0:h0 + nh] if n not in ("S0", "dST") else t[2:3, h0:h0 + nh]).contiguous()
               for n, t in x.items()}
        for save in (True, False):
            for n, t in run(sub, save).items():
                w = wide[n]
                w = w[2:3, h0:h0 + nh] if n in ("S_T", "dS0") else w[2:3, :, h0:h0 + nh]
                assert torch.equal(t, w), (n, h0, save)


STATES = ("S0", "S_T", "dST", "dS0")
VALUE_SIDE = ("v", "w", "o", "do", "dv", "dw")


def _device_problem(B, T, H, Hv, Dk, Dv, seed, states):
    """A bf16 problem drawn on the device (S0 and dST for `states` sequences)."""
    import torch
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    nrm = lambda *s: torch.randn(s, generator=gen, device="cuda")
    unit = lambda t: (t / t.norm(dim=-1, keepdim=True)).bfloat16()
    return {"q": unit(nrm(B, T, H, Dk)), "k": unit(nrm(B, T, H, Dk)), "v": nrm(B, T, Hv, Dv).bfloat16(),
            "log_alpha": -torch.nn.functional.softplus(nrm(B, T, H, Dk) - 2.0),
            "b": torch.sigmoid(nrm(B, T, H, Dk)).bfloat16(), "w": torch.sigmoid(nrm(B, T, Hv, Dv)).bfloat16(),
            "S0": 0.05 * nrm(states, Hv, Dk, Dv), "do": nrm(B, T, Hv, Dv).bfloat16(), "dST": nrm(states, Hv, Dk, Dv)}


def _fwd_bwd_device(x, save, cu=None):
    import torch
    import paper_2605_22791_amd as g2
    args = [x[n] for n in ("q", "k", "v", "log_alpha", "b", "w")]
    prob = g2._problem(x["q"], x["v"], None)
    need = g2.gdr2_chunk_workspace_bytes(prob, 1) if cu is None else \
        g2.gdr2_varlen_workspace_bytes(prob, cu.numel() - 1, 1)
    ws = torch.full((need,), 0xFF, dtype=torch.uint8, device="cuda")
    if cu is None:
        o, ST = g2.gdr2_chunk_fwd(*args, x["S0"], ws=ws, save=save)
        g = g2.gdr2_chunk_bwd(*args, x["S0"], x["do"], x["dST"], ws=ws, saved=save)
    else:
        o, ST = g2.gdr2_chunk_fwd_varlen(*args, cu, x["S0"], ws=ws, save=save)
        g = g2.gdr2_chunk_bwd_varlen(*args, cu, x["S0"], x["do"], x["dST"], ws=ws, saved=save)
    return {"o": o, "S_T": ST, **g}


# more than 512 wide scans; at most 512, of more than 32 chunks for each of 256 compute units;
# the same with Dk = 64 and grouped value heads
@pytest.mark.parametrize("H,Hv,Dk,Dv,lengths", [
    (16, 16, 128, 128, [70, 0, 130, 64, 5, 300, 1, 200, 128, 0, 65, 63, 90, 33, 250, 77, 140, 12]),
    (8, 16, 64, 128, [1300, 1984, 40, 0, 2500, 64, 1700, 2049, 800, 1900, 1, 2300, 2500]),
    (16, 16, 128, 128, [2048, 1, 2047, 2000, 1999, 2100, 0, 2050, 2048, 2113])])
def test_packed_wide_scans_equal_narrow(H, Hv, Dk, Dv, lengths):
    """The 64-wide scans over a chunk table (empty sequences, partial chunks) give the bits that two of
    the sequences give in a batch of their own, whose few heads take the 32-wide scans."""
    import torch
    T, N, G = sum(lengths), len(lengths), Hv // H
    x = _device_problem(1, T, H, Hv, Dk, Dv, 600 + N, N)
    off = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    slots = T // 64 + N
    per_seq = Hv * Dv // 64
    assert N * per_seq > 512 or slots * per_seq > 32 * 256   # the wide route whatever the lengths are
    _case(f"packed wide scans H{H} Hv{Hv} Dk{Dk} Dv{Dv}, {N} sequences, T = {T}")
    cu = torch.from_numpy(off).cuda()
    for save in (True, False):
        wide = _fwd_bwd_device(x, save, cu)
        for seqs, heads in (((2, 4), slice(0, 1)), ((0, N - 1), slice(H - 3, H))):
            assert len(seqs) * 3 * G * Dv // 64 <= 128
            rows = torch.cat([torch.arange(off[s], off[s + 1]) for s in seqs]).cuda()
            vheads = slice(heads.start * G, heads.stop * G)
            side = lambda n, t: (t[list(seqs)][:, vheads] if n in STATES else
                                 t[:, rows][:, :, vheads if n in VALUE_SIDE else heads]).contiguous()
            few = torch.tensor([0] + list(np.cumsum([lengths[s] for s in seqs])), dtype=torch.int32, device="cuda")
            for n, t in _fwd_bwd_device({n: side(n, t) for n, t in x.items()}, save, few).items():
                assert torch.equal(t, side(n, wide[n])), (n, seqs, save)


@pytest.mark.parametrize("H", [8, 7])
@pytest.mark.parametrize("Dk,Dv", [(128, 128), (64, 64)])
def test_grouped_wide_scans_equal_narrow(H, Dk, Dv):
    """Grouped value heads on the unsegmented 64-wide scans, with a multiple of eight (sequence, key head)
    units (placed by XCD) and without: the bits of one sequence's three key heads alone."""
    import torch
    B, G, T = 9, 2 * 128 // Dv, 150
    Hv = G * H
    assert B * Hv * Dv // 64 > 128 and ((B * H) % 8 == 0) == (H == 8)
    x = _device_problem(B, T, H, Hv, Dk, Dv, 620 + H + Dk, B)
    _case(f"grouped wide scans B{B} H{H} Hv{Hv} Dk{Dk} Dv{Dv}")
    side = lambda n, t: (t[2:3, 3 * G:6 * G] if n in STATES else
                         t[2:3, :, 3 * G:6 * G] if n in VALUE_SIDE else t[2:3, :, 3:6]).contiguous()
    few = {n: side(n, t) for n, t in x.items()}
    for save in (True, False):
        wide = _fwd_bwd_device(x, save)
        for n, t in _fwd_bwd_device(few, save).items():
            assert torch.equal(t, side(n, wide[n])), (n, save)
