"""GPU parity of packed variable-length batches and of partial last chunks (App. C.6).

A packed batch lays its sequences end to end along T; the operator chunks each
sequence on its own, so the state restarts at every boundary and the result
for sequence s is the recurrence (Sec. 3.1) over its tokens alone, from its own
S0.  The oracle is exactly that: the fp64 token recurrence and its adjoint run
per sequence.  Lengths mix empty sequences, single tokens, exact multiples of
the chunk and ragged tails.  Tolerances as elsewhere (rel-L2 2e-3 bf16, 1e-5 fp32).
"""

import numpy as np
import pytest

from oracle import gdr2_packed_bwd, gdr2_packed_fwd, gdr2_recurrent_bwd, gdr2_recurrent_fwd
from paper_2605_22791_amd.inputs import make_inputs, make_packed
from tests.helpers import rel_l2
from tests.gpu_common import dev_inputs, host, ws_layout_bf16

pytestmark = pytest.mark.gpu

TOL = {"fp32": 1e-5, "bf16": 2e-3}
GRADS = ("dq", "dk", "dv", "dlog_alpha", "db", "dw")
REF = {"dlog_alpha": "dg"}


def _case(msg):
    print(f"\n[gpu case] {msg}", flush=True)


def oracle_packed(d, backward=True):
    """The oracle's packed batch (App. C.6): the fp64 recurrence and adjoint per sequence."""
    args = [d[n] for n in ("q", "k", "v", "log_alpha", "b", "w")]
    o, ST = gdr2_packed_fwd(*args, d["cu_seqlens"], d["S0"], d["scale"])
    out = {"o": o, "S_T": ST}
    if backward:
        g = gdr2_packed_bwd(*args, d["cu_seqlens"], d["S0"], d["do"], d.get("dST"), d["scale"])
        out.update({n: g[REF.get(n, n)] for n in GRADS})
        out["dS0"] = g["dS0"]
    return out


def _run_packed(d, save=False):
    import torch
    import paper_2605_22791_amd as g2
    x = dev_inputs(d)
    cu = torch.from_numpy(d["cu_seqlens"]).cuda()
    args = [x[n] for n in ("q", "k", "v", "log_alpha", "b", "w")]
    ws = None
    if save:
        prob = g2._problem(x["q"], x["v"], d["scale"])
        ws = torch.empty(g2.gdr2_varlen_workspace_bytes(prob, len(d["lengths"]), 1), dtype=torch.uint8,
                         device="cuda")
    o, ST = g2.gdr2_chunk_fwd_varlen(*args, cu, x["S0"], scale=d["scale"], ws=ws, save=save)
    g = g2.gdr2_chunk_bwd_varlen(*args, cu, x["S0"], x["do"], x["dST"], scale=d["scale"], ws=ws, saved=save)
    out = {"o": host(o), "S_T": host(ST)}
    out.update({n: host(t) for n, t in g.items()})
    return out


def _compare(got, ref, tol):
    err = {n: rel_l2(got[n], ref[n]) for n in ("o", "S_T", "dS0") + GRADS}
    print({k: f"{v:.2e}" for k, v in err.items()})
    for k, v in err.items():
        assert v < tol, (k, v)


LENGTHS = [100, 64, 1, 0, 257, 130, 63, 65]


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("Dk,Dv", [(128, 128), (64, 128), (128, 64)])
def test_packed_batch_matches_per_sequence_oracle(dtype, Dk, Dv):
    d = make_packed(LENGTHS, 2, Dk, Dv, seed=120 + Dk + Dv, dtype=dtype, decay_shift=-1.0, s0_std=0.05,
                    with_dST=True)
    _case(f"packed {dtype} lengths {LENGTHS} H2 Dk{Dk} Dv{Dv}")
    _compare(_run_packed(d), oracle_packed(d), TOL[dtype])


def test_packed_saved_path_and_many_sequences():
    """40 sequences of 0..300 tokens, H = 4: the stored training path returns
    the same as the recomputing one, and both match the oracle."""
    rng = np.random.default_rng(7)
    lengths = [int(x) for x in rng.integers(0, 301, size=40)]
    d = make_packed(lengths, 4, 128, 128, seed=125, dtype="bf16", decay_shift=-2.0, s0_std=0.05, with_dST=True)
    _case(f"packed bf16, 40 sequences, T = {sum(lengths)}, H4, saved vs recompute")
    got_s = _run_packed(d, save=True)
    got_r = _run_packed(d)
    for n in got_r:
        assert np.array_equal(got_s[n], got_r[n]), n
    _compare(got_r, oracle_packed(d), TOL["bf16"])


def test_packed_equals_separate_calls():
    """Each sequence of a packed batch gives exactly what a fixed-length call on
    its tokens alone gives (same chunking from the sequence start)."""
    import torch
    import paper_2605_22791_amd as g2
    lengths = [130, 64, 7, 200]
    d = make_packed(lengths, 2, 128, 128, seed=126, dtype="bf16", s0_std=0.05, with_dST=True)
    _case(f"packed vs separate fixed-length calls, lengths {lengths}")
    got = _run_packed(d)
    cu = d["cu_seqlens"]
    for s in range(len(lengths)):
        a, b = int(cu[s]), int(cu[s + 1])
        ds = {n: (d[n][:, a:b] if d[n] is not None else None) for n in ("q", "k", "v", "log_alpha", "b", "w", "do")}
        ds.update(S0=d["S0"][s:s + 1], dST=d["dST"][s:s + 1], dtype="bf16", scale=d["scale"])
        x = dev_inputs(ds)
        args = [x[n] for n in ("q", "k", "v", "log_alpha", "b", "w")]
        o, ST = g2.gdr2_chunk_fwd(*args, x["S0"], scale=d["scale"])
        g = g2.gdr2_chunk_bwd(*args, x["S0"], x["do"], x["dST"], scale=d["scale"])
        torch.cuda.synchronize()
        assert np.array_equal(host(o), got["o"][:, a:b]), s
        assert np.array_equal(host(ST)[0], got["S_T"][s]), s
        assert np.array_equal(host(g["dS0"])[0], got["dS0"][s]), s
        for n in GRADS:
            assert np.array_equal(host(g[n]), got[n][:, a:b]), (s, n)


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
def test_fixed_length_partial_last_chunk(dtype):
    """T = 100 and T = 65: the last chunk of every sequence is partial."""
    import paper_2605_22791_amd as g2
    for T in (100, 65):
        d = make_inputs(2, T, 2, 128, 128, seed=127 + T, dtype=dtype, s0_std=0.05, with_dST=True)
        _case(f"fixed-length {dtype} B2 T{T} H2")
        x = dev_inputs(d)
        args = [x[n] for n in ("q", "k", "v", "log_alpha", "b", "w")]
        o, ST = g2.gdr2_chunk_fwd(*args, x["S0"], scale=d["scale"])
        g = g2.gdr2_chunk_bwd(*args, x["S0"], x["do"], x["dST"], scale=d["scale"])
        o_ref, S_ref = gdr2_recurrent_fwd(d["q"], d["k"], d["v"], d["log_alpha"], d["b"], d["w"], d["S0"],
                                          d["scale"])
        ref = gdr2_recurrent_bwd(d["q"], d["k"], d["v"], d["log_alpha"], d["b"], d["w"], d["S0"], d["do"],
                                 d["dST"], d["scale"])
        err = {"o": rel_l2(host(o), o_ref), "S_T": rel_l2(host(ST), S_ref), "dS0": rel_l2(host(g["dS0"]), ref["dS0"])}
        for n in GRADS:
            err[n] = rel_l2(host(g[n]), ref[REF.get(n, n)])
        print({k: f"{v:.2e}" for k, v in err.items()})
        for k, v in err.items():
            assert v < TOL[dtype], (T, k, v)


def test_recurrent_varlen_matches_oracle():
    import torch
    import paper_2605_22791_amd as g2
    lengths = [5, 0, 1, 17]
    d = make_packed(lengths, 3, 64, 128, seed=128, dtype="bf16", s0_std=0.05)
    _case(f"recurrent packed lengths {lengths}")
    x = dev_inputs(d)
    cu = torch.from_numpy(d["cu_seqlens"]).cuda()
    S = x["S0"].clone()
    o = g2.gdr2_recurrent_varlen(*[x[n] for n in ("q", "k", "v", "log_alpha", "b", "w")], cu, S,
                                 scale=d["scale"])
    ref = oracle_packed(d, backward=False)
    e_o, e_s = rel_l2(host(o), ref["o"]), rel_l2(host(S), ref["S_T"])
    print("o", e_o, "S", e_s)
    assert e_o < TOL["bf16"] and e_s < 1e-5


def test_chunk_table_in_workspace():
    """The device chunk table: every sequence cut into ceil(L/64) chunks from its
    own first token, the last one holding the remainder; empty sequences none;
    the scans take the sequences longest first."""
    import torch
    import paper_2605_22791_amd as g2
    lengths = [100, 0, 64, 1, 129]
    d = make_packed(lengths, 2, 64, 64, seed=129, dtype="bf16")
    x = dev_inputs(d)
    cu = torch.from_numpy(d["cu_seqlens"]).cuda()
    prob = g2._problem(x["q"], x["v"], d["scale"])
    T, N = sum(lengths), len(lengths)
    lay, total, _ = ws_layout_bf16(1, T, 2, 64, 64, bwd=False, nseq=N)
    assert total == g2.gdr2_varlen_workspace_bytes(prob, N, 0)
    ws = torch.zeros(total, dtype=torch.uint8, device="cuda")
    _case("varlen chunk table")
    g2.gdr2_chunk_fwd_varlen(*[x[n] for n in ("q", "k", "v", "log_alpha", "b", "w")], cu, None, scale=d["scale"],
                             ws=ws)
    torch.cuda.synchronize()
    raw = ws.cpu().numpy()
    region = lambda n: raw[lay[n][0]: lay[n][0] + lay[n][1]].view(np.int32)
    coff, ct0, clen = region("coff"), region("ct0"), region("clen")
    exp_off, exp_t0, exp_len = [0], [], []
    for s, L in enumerate(lengths):
        for j in range(-(-L // 64)):
            exp_t0.append(int(d["cu_seqlens"][s]) + 64 * j)
            exp_len.append(min(64, L - 64 * j))
        exp_off.append(len(exp_t0))
    assert list(coff) == exp_off
    assert list(ct0[:len(exp_t0)]) == exp_t0 and list(clen[:len(exp_len)]) == exp_len
    # scan order: a permutation of the sequences by non-increasing chunk count
    order = list(region("sorder"))
    counts = [exp_off[s + 1] - exp_off[s] for s in range(N)]
    assert sorted(order) == list(range(N))
    assert all(counts[order[i]] >= counts[order[i + 1]] for i in range(N - 1))


@pytest.mark.parametrize("lengths", [[1], [0, 0, 65], [64] * 1024, [0] * 1023 + [3, 200], [1, 0, 70] * 700],
                         ids=["one", "empty first", "1024", "1025", "2100"])
def test_chunk_table_passes(lengths):
    """The table at the edges of its passes of 1024 sequences, empty sequences among them."""
    import torch
    import paper_2605_22791_amd as g2
    d = make_packed(lengths, 1, 64, 64, seed=130, dtype="bf16")
    x = dev_inputs(d)
    cu = torch.from_numpy(d["cu_seqlens"]).cuda()
    T, N = sum(lengths), len(lengths)
    lay, total, _ = ws_layout_bf16(1, T, 1, 64, 64, bwd=False, nseq=N)
    ws = torch.zeros(total, dtype=torch.uint8, device="cuda")
    _case(f"varlen chunk table, {N} sequences, T = {T}")
    g2.gdr2_chunk_fwd_varlen(*[x[n] for n in ("q", "k", "v", "log_alpha", "b", "w")], cu, None, scale=d["scale"],
                             ws=ws)
    raw = ws.cpu().numpy()
    region = lambda n: raw[lay[n][0]: lay[n][0] + lay[n][1]].view(np.int32)
    L = np.array(lengths)
    n = -(-L // 64)
    off = np.concatenate([[0], np.cumsum(n)])
    first = np.arange(off[-1]) - np.repeat(off[:-1], n)     # chunk number within its sequence
    assert np.array_equal(region("coff")[:N + 1], off)
    assert np.array_equal(region("ct0")[:off[-1]], np.repeat(d["cu_seqlens"][:-1], n) + 64 * first)
    assert np.array_equal(region("clen")[:off[-1]], np.minimum(64, np.repeat(L, n) - 64 * first))
    order = region("sorder")[:N]
    assert np.array_equal(np.sort(order), np.arange(N)) and np.all(np.diff(n[order]) <= 0)


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("entry", [0x7FFFFFFF, -1, -2 ** 31, 1000])
def test_saved_backward_on_a_foreign_workspace(dtype, entry):
    """A saved backward takes its chunk table from the workspace.  One that no forward has filled gives
    undefined gradients, but whatever the table's entries are, nothing outside the tensors is written, and
    the forward that fills it makes the next backward right."""
    import torch
    import paper_2605_22791_amd as g2
    lengths = [70, 0, 130, 64, 5]
    d = make_packed(lengths, 2, 64, 64, seed=131, dtype=dtype, s0_std=0.05, with_dST=True)
    x = dev_inputs(d)
    cu = torch.from_numpy(d["cu_seqlens"]).cuda()
    args = [x[n] for n in ("q", "k", "v", "log_alpha", "b", "w")]
    need = g2.gdr2_varlen_workspace_bytes(g2._problem(x["q"], x["v"], d["scale"]), len(lengths), 1)
    guard = 1 << 16
    room = torch.full((need + 2 * guard,), 0x5A, dtype=torch.uint8, device="cuda")
    ws = room[guard:guard + need]
    shapes = {"dq": x["q"], "dk": x["k"], "dv": x["v"], "dlog_alpha": x["log_alpha"], "db": x["b"], "dw": x["w"],
              "dS0": x["S0"]}
    bufs = {n: torch.full((t.numel() + 2 * guard,), 3.0, dtype=t.dtype, device="cuda") for n, t in shapes.items()}
    grads = {n: bufs[n][guard:guard + t.numel()].view(t.shape) for n, t in shapes.items()}
    _case(f"saved backward on a workspace of {entry}, {dtype}")

    def bwd():
        return g2.gdr2_chunk_bwd_varlen(*args, cu, x["S0"], x["do"], x["dST"], scale=d["scale"], ws=ws, saved=True,
                                        grads=dict(grads))

    ws.view(torch.int32).fill_(entry)
    bwd()
    torch.cuda.synchronize()
    assert bool((room[:guard] == 0x5A).all()) and bool((room[guard + need:] == 0x5A).all())
    for n, t in bufs.items():
        assert bool((t[:guard] == 3.0).all()) and bool((t[-guard:] == 3.0).all()), n
    o, ST = g2.gdr2_chunk_fwd_varlen(*args, cu, x["S0"], scale=d["scale"], ws=ws, save=True)
    got = {n: host(t) for n, t in bwd().items()}
    got.update(o=host(o), S_T=host(ST))
    _compare(got, oracle_packed(d), TOL[dtype])


@pytest.mark.parametrize("H,Dk,Dv,lengths", [
    (16, 128, 128, [700] * 10),                             # alike: wide slices by the table
    (16, 128, 128, [5000, 200, 64, 1, 0, 130, 77, 300]),    # one long sequence: narrow ones
    (16, 64, 64, [1792] * 8 + [0]),                         # at the line: 8 x 28 chunks x 16 scans = 128 x 28
    (16, 64, 64, [1792, 1] + [1792] * 7),                   # a chunk past it
    (24, 64, 128, [400] * 9), (8, 128, 64, [0] * 40 + [22016])])
def test_packed_scan_slices(H, Dk, Dv, lengths):
    """Batches whose scans run in wide or narrow slices by the table's lengths (both kernels are
    launched): the bits of the sequences in batches so small that the host takes the narrow ones."""
    import torch
    import paper_2605_22791_amd as g2
    T, N = sum(lengths), len(lengths)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(140 + N)
    nrm = lambda *s: torch.randn(s, generator=gen, device="cuda")
    unit = lambda t: (t / t.norm(dim=-1, keepdim=True)).bfloat16()
    x = {"q": unit(nrm(1, T, H, Dk)), "k": unit(nrm(1, T, H, Dk)), "v": nrm(1, T, H, Dv).bfloat16(),
         "log_alpha": -torch.nn.functional.softplus(nrm(1, T, H, Dk) - 2.0),
         "b": torch.sigmoid(nrm(1, T, H, Dk)).bfloat16(), "w": torch.sigmoid(nrm(1, T, H, Dv)).bfloat16(),
         "do": nrm(1, T, H, Dv).bfloat16(), "S0": 0.05 * nrm(N, H, Dk, Dv), "dST": nrm(N, H, Dk, Dv)}
    off = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    per_seq = H * Dv // 64
    assert 128 < N * per_seq <= 512 and 12 * 256 < (T // 64 + N) * per_seq <= 32 * 256  # the table's choice
    _case(f"packed scan slices H{H} Dk{Dk} Dv{Dv} lengths {lengths}")

    def run(t, cu, save):
        args = [t[n] for n in ("q", "k", "v", "log_alpha", "b", "w")]
        need = g2.gdr2_varlen_workspace_bytes(g2._problem(t["q"], t["v"], None), cu.numel() - 1, 1)
        ws = torch.full((need,), 0xFF, dtype=torch.uint8, device="cuda")
        o, ST = g2.gdr2_chunk_fwd_varlen(*args, cu, t["S0"], ws=ws, save=save)
        g = g2.gdr2_chunk_bwd_varlen(*args, cu, t["S0"], t["do"], t["dST"], ws=ws, saved=save)
        return {"o": o, "S_T": ST, **g}

    cu = torch.from_numpy(off).cuda()
    few = 128 // per_seq
    for save in (True, False):
        whole = run(x, cu, save)
        for s0 in range(0, N, few):
            s1 = min(N, s0 + few)
            if off[s1] == off[s0]:
                continue
            part = lambda n, t: (t[s0:s1] if n in ("S0", "dST", "S_T", "dS0") else t[:, off[s0]:off[s1]]).contiguous()
            sub = torch.from_numpy(off[s0:s1 + 1] - off[s0]).cuda()
            for n, t in run({n: part(n, t) for n, t in x.items()}, sub, save).items():
                assert torch.equal(t, part(n, whole[n])), (n, s0, save)
