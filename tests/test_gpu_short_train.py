"""Training over a few tokens: the token recurrence takes the state scan's
place in the training forward and in the backward's recompute, and leaves the
chunk-start states and E rows the backward reads.  At the ends of its range,
on a workspace of NaN bytes: forward outputs equal the inference forward's and
gradients the recomputing backward's bit for bit, gradients meet the oracle;
and the training forward launches as many kernels as with the scan."""
import ctypes

import numpy as np
import pytest

import pdn_inputs as pi

from gpu_util import to_device
from test_gpu_bwd import compare

pytestmark = pytest.mark.gpu

CASES = [
    # (io, gate, precond, dk, dv, T, chunk)
    ("bf16", "scalar", "squash", 128, 128, 1, 64),
    ("bf16", "channel", "squash", 128, 64, 2, 32),
    ("bf16", "none", "identity", 64, 128, 4, 64),
    ("bf16", "scalar", "external", 64, 64, 8, 64),
    ("bf16", "none", "squash", 128, 128, 8, 32),
    ("bf16", "channel", "external", 64, 128, 7, 64),
    ("f32", "scalar", "squash", 64, 64, 1, 32),
    ("f32", "channel", "squash", 64, 64, 8, 64),
    ("f32", "none", "external", 64, 64, 5, 32),
]


def _spec(io, gate, precond, dk, dv, T):
    spec = pi.small_spec(io=io, gate=gate, dk=dk, dv=dv, B=2, H=3, T=T, s0="normal",
                         a0="lognormal" if precond == "squash" else "zero", with_do=True)
    inp = pi.generate(spec, 8100 + T)
    if precond == "external":
        kt = inp["k"] * np.random.default_rng(9).uniform(1 / 1.5, 1.5, inp["k"].shape)
        inp["ktilde"] = pi.round_bf16(kt) if io == "bf16" else kt.astype(np.float32)
    return spec, inp


def _args(spec, inp, precond, chunk):
    d = to_device(inp, spec.io)
    sq = precond == "squash"
    kw = dict(g=d["g"], gate=spec.gate, precond=precond, beta_p=d["beta_p"] if sq else None,
              g_p=d["g_p"] if sq else None, log_a_scale=d["log_a_scale"] if sq else None,
              A0=d["A0"] if sq else None, S0=d["S0"], ktilde=d.get("ktilde") if precond == "external" else None,
              x=spec.x, scale=spec.scale, chunk=chunk)
    return (d["q"], d["k"], d["v"], d["beta"]), d["dO"], kw


def _workspace(spec, precond, chunk):
    import torch
    import paper_2604_21100_amd as pdn
    prob = pdn.make_problem(spec.B, spec.T, spec.H, spec.dk, spec.dv, io=spec.io, gate=spec.gate, precond=precond,
                            x=spec.x, scale=spec.scale, chunk=chunk)
    return torch.full((pdn.pdn_workspace_size(prob, True),), 255, dtype=torch.uint8, device="cuda")


@pytest.mark.parametrize("io,gate,precond,dk,dv,T,chunk", CASES)
def test_short_training(io, gate, precond, dk, dv, T, chunk):
    import torch
    import paper_2604_21100_amd as pdn
    spec, inp = _spec(io, gate, precond, dk, dv, T)
    main, dO, kw = _args(spec, inp, precond, chunk)
    dS_T = (0.1 * np.random.default_rng(T).standard_normal((2, 3, dk, dv))).astype(np.float32)
    dST = torch.from_numpy(dS_T).cuda()
    ws = _workspace(spec, precond, chunk)
    tag = f"short {io}/{gate}/{precond} {dk}x{dv} T={T} C={chunk}"
    for x, y in zip(pdn.pdn_chunk_fwd(*main, workspace=ws, train=True, **kw), pdn.pdn_chunk_fwd(*main, **kw)):
        assert (x is None and y is None) or torch.equal(x, y), tag
    saved = pdn.pdn_chunk_bwd(*main, dO, dS_T=dST, workspace=ws, saved=True, **kw)
    ws2 = _workspace(spec, precond, chunk)
    again = pdn.pdn_chunk_bwd(*main, dO, dS_T=dST, workspace=ws2, **kw)
    for name, x in saved.items():
        assert torch.equal(x, again[name]), f"{tag} {name}"
    compare(spec, inp, precond, dS_T, tag=tag, chunk=chunk)


def _launches(spec, inp, precond):
    """Kernel launches of the training forward: the nodes of its capture."""
    import torch
    import paper_2604_21100_amd as pdn
    main, _, kw = _args(spec, inp, precond, 64)
    ws = _workspace(spec, precond, 64)
    out = dict(zip(("o", "S_T", "A_T"), pdn.pdn_chunk_fwd(*main, workspace=ws, train=True, **kw)))
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph):
        pdn.pdn_chunk_fwd(*main, workspace=ws, train=True, **kw, **out)
    hip = ctypes.CDLL(pdn.loaded_hip_runtimes()[0])
    n = ctypes.c_size_t(0)
    assert hip.hipGraphGetNodes(ctypes.c_void_p(graph.raw_cuda_graph()), None, ctypes.byref(n)) == 0
    return n.value


@pytest.mark.parametrize("io,precond", [("bf16", "squash"), ("f32", "identity")])
def test_short_training_forward_launches(io, precond):
    want = _launches(*_spec(io, "scalar", precond, 64, 64, 9), precond)
    for T in (1, 8):
        assert _launches(*_spec(io, "scalar", precond, 64, 64, T), precond) == want, T
