"""The forward over a few tokens: up to eight run as the token recurrence in
one launch, more as chunks.  Both sides of that line and the ends of its range,
over every write key, gate, element type and head size, against the float64
oracle; and a sequence fed in pieces of mixed lengths against the same sequence
at once (states carried through the two forms)."""
import numpy as np
import pytest

import pdn_inputs as pi
from oracle import abi as oabi

from gpu_util import rel_err, run_fwd, to_device, tol

pytestmark = pytest.mark.gpu

CASES = [
    # (io, gate, precond, knorm, dk, dv, T)
    ("bf16", "scalar", "squash", "none", 128, 128, 1),
    ("bf16", "channel", "squash", "none", 128, 64, 2),
    ("bf16", "none", "squash", "m", 64, 128, 3),
    ("bf16", "scalar", "squash", "beta", 128, 128, 5),
    ("bf16", "none", "squash", "beta", 64, 64, 8),
    ("bf16", "channel", "squash", "1pm", 128, 128, 7),
    ("bf16", "scalar", "identity", "none", 64, 128, 8),
    ("bf16", "channel", "external", "none", 128, 128, 8),
    ("bf16", "scalar", "diag_sm", "none", 128, 64, 6),
    ("bf16", "channel", "atq", "none", 64, 64, 4),
    ("bf16", "scalar", "atq", "none", 128, 128, 8),
    ("f32", "scalar", "squash", "none", 128, 128, 8),
    ("f32", "none", "external", "none", 64, 64, 1),
    ("f32", "channel", "diag_sm", "none", 64, 128, 5),
    ("f32", "channel", "squash", "m", 128, 128, 3),
    # just past the line
    ("bf16", "scalar", "squash", "none", 128, 128, 9),
    ("f32", "channel", "squash", "none", 64, 64, 9),
]


@pytest.mark.parametrize("io,gate,precond,knorm,dk,dv,T", CASES)
def test_few_tokens(io, gate, precond, knorm, dk, dv, T):
    gram = precond in ("squash", "diag_sm", "atq")
    spec = pi.small_spec(io=io, gate=gate, dk=dk, dv=dv, B=2, H=3, T=T, s0="normal",
                         a0="lognormal" if gram else "zero", scale=0.7)
    inp = pi.generate(spec, 7000 + T)
    if precond == "external":
        kt = inp["k"] * np.random.default_rng(3).uniform(1 / 1.5, 1.5, inp["k"].shape)
        inp["ktilde"] = pi.round_bf16(kt) if io == "bf16" else kt.astype(np.float32)
    kw = dict(knorm=knorm, ridge=0.5)
    o, S_T, A_T = run_fwd(spec, inp, precond, **kw)
    ref = oabi.forward(inp, gate=gate, precond=precond, x=spec.x, scale=spec.scale, B=2, H=3, **kw)
    e_o = rel_err(np.stack([o[b, :, h] for b in range(2) for h in range(3)]), ref["o"])
    e_s = rel_err(S_T.reshape(6, dk, dv), ref["S_T"])
    msg = f"{io}/{gate}/{precond}/{knorm} {dk}x{dv} T={T}: o={e_o:.2e} S_T={e_s:.2e}"
    print(msg)
    # fp32 arithmetic throughout: only o is rounded to io (bf16 keeps eight
    # significant bits, so half an ulp is at most 2^-8 of the value); past the
    # line the chunk kernels' bars hold
    bar_s = 1e-5 if T <= 8 else tol(io)
    bar_o = (2 ** -8 + 1e-5 if io == "bf16" else 1e-5) if T <= 8 else tol(io)
    assert e_o <= bar_o and e_s <= bar_s, msg
    if gram:
        assert rel_err(A_T.reshape(6, dk), ref["A_T"]) <= 1e-5


@pytest.mark.parametrize("gate", ["scalar", "channel"])
def test_pieces_equal_whole(gate):
    import torch
    import paper_2604_21100_amd as pdn
    spec = pi.small_spec(io="f32", gate=gate, dk=64, dv=128, B=1, H=2, T=90, s0="normal", a0="lognormal")
    d = to_device(pi.generate(spec, 77), "f32")
    names = ("q", "k", "v", "beta", "g", "beta_p", "g_p")

    def run(lo, hi, S0, A0):
        p = {n: d[n][:, lo:hi].clone() for n in names}
        return pdn.pdn_chunk_fwd(p["q"], p["k"], p["v"], p["beta"], g=p["g"], gate=gate, beta_p=p["beta_p"],
                                 g_p=p["g_p"], log_a_scale=d["log_a_scale"], A0=A0, S0=S0)

    whole = run(0, 90, d["S0"], d["A0"])
    S, A, t, parts = d["S0"], d["A0"], 0, []
    for n in (1, 8, 40, 3, 9, 1, 1, 27):
        o, S, A = run(t, t + n, S, A)
        parts.append(o)
        t += n
    assert t == 90
    torch.cuda.synchronize()
    for x, y in ((torch.cat(parts, 1), whole[0]), (S, whole[1]), (A, whole[2])):
        assert rel_err(x.cpu().numpy(), y.cpu().numpy()) <= 1e-5


@pytest.mark.parametrize("precond,gate,dk,dv,H,T,recurrence", [
    # bf16 at chunk 32: past 512 slabs of 32 columns (1024 with a Gram recurrence) the line falls to 4 or 6 tokens
    ("identity", "none", 64, 64, 256, 8, True),
    ("identity", "none", 64, 64, 257, 5, False),
    ("identity", "none", 64, 64, 257, 4, True),
    ("external", "scalar", 128, 128, 129, 7, False),
    ("external", "channel", 128, 128, 129, 6, True),
    ("squash", "scalar", 64, 128, 256, 8, True),
    ("squash", "channel", 64, 128, 257, 7, False),
    ("squash", "none", 64, 128, 257, 6, True),
    ("squash", "none", 128, 128, 300, 8, True),
])
def test_few_tokens_of_many_heads(precond, gate, dk, dv, H, T, recurrence):
    """Which form takes the call (the recurrence is one launch), and that it
    returns what the same heads return in calls of few heads."""
    import ctypes
    import torch
    import paper_2604_21100_amd as pdn
    sq = precond == "squash"
    spec = pi.small_spec(gate=gate, dk=dk, dv=dv, B=1, H=H, T=T, chunk=32, s0="normal",
                         a0="lognormal" if sq else "zero")
    d = to_device(pi.generate(spec, 7300 + H + T), "bf16")
    if precond == "external":
        d["ktilde"] = (d["k"].float() * 1.2).to(torch.bfloat16)
    names = ("g", "beta_p", "g_p", "log_a_scale", "A0", "S0", "ktilde") if sq else ("g", "S0", "ktilde")

    def call(lo, hi, out=None):
        cut = lambda n: None if d.get(n) is None else (  # noqa: E731  (a copy: aligned)
            d[n][lo:hi] if n == "log_a_scale" else d[n][:, lo:hi] if n in ("A0", "S0") else d[n][:, :, lo:hi]).clone(memory_format=torch.contiguous_format)
        main, kw = [cut(n) for n in ("q", "k", "v", "beta")], {n: cut(n) for n in names}
        kw.update(gate=gate, precond=precond, chunk=32, **(out or {}))
        return main, kw

    main, kw = call(0, H)
    whole = pdn.pdn_chunk_fwd(*main, **kw)
    n = 64
    for lo in (0, H - n):
        main, kw = call(lo, lo + n)
        few = pdn.pdn_chunk_fwd(*main, **kw)   # the recurrence: the oracle's check is above
        for x, y in ((whole[0][:, :, lo:lo + n], few[0]), (whole[1][:, lo:lo + n], few[1])):
            e = rel_err(x.float().cpu().numpy(), y.float().cpu().numpy())
            assert e == 0 if recurrence else e <= tol("bf16")
    main, kw = call(0, H, dict(zip(("o", "S_T", "A_T"), whole)))
    prob = pdn.make_problem(1, T, H, dk, dv, gate=gate, precond=precond, chunk=32)
    kw["workspace"] = torch.empty(pdn.pdn_workspace_size(prob), dtype=torch.uint8, device="cuda")
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph):
        pdn.pdn_chunk_fwd(*main, **kw)
    nodes = ctypes.c_size_t(0)
    hip = ctypes.CDLL(pdn.loaded_hip_runtimes()[0])
    assert hip.hipGraphGetNodes(ctypes.c_void_p(graph.raw_cuda_graph()), None, ctypes.byref(nodes)) == 0
    assert (nodes.value == 1) == recurrence, nodes.value
