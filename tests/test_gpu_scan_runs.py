"""The bf16 state scans over every short run length: their waves walk the
chunks differently (the chain by two, the output waves by four with their ends
peeled, the loaders one at a time, two ahead), so a run of n chunks is checked
for n = 1 .. 13 (three trips of the longest unrolled loop and every remainder)
at both chunk lengths, whole and ragged, with head counts that leave the grid's
last group of eight heads part empty, and unsplit.  Forward outputs and states
and every gradient against the float64 oracle's token recurrence, to the bars
of the other GPU tests (bf16 rounding of inputs, stored rows and operands)."""
import numpy as np
import pytest

import pdn_inputs as pi
from oracle import abi as oabi

from gpu_util import rel_err, run_fwd, to_device, tol
from test_gpu_bwd import compare

pytestmark = pytest.mark.gpu

GATES = ("none", "scalar", "channel")
DIMS = ((128, 128), (64, 128), (128, 64), (64, 64))


@pytest.mark.parametrize("ragged", [False, True])
@pytest.mark.parametrize("chunk", [32, 64])
@pytest.mark.parametrize("n", range(1, 14))
def test_scan_runs(n, chunk, ragged):
    import paper_2604_21100_amd as pdn
    k = n + 2 * (chunk // 64) + ragged
    gate, (dk, dv) = GATES[k % 3], DIMS[(k // 2 + n) % 4]
    T = n * chunk - (1 + 2 * n if ragged else 0)
    assert (T + chunk - 1) // chunk == n
    # from ten chunks on few heads would be split
    H = 1 + k % 3 if n < 10 else 43
    assert pdn.pdn_scan_segments(pdn.make_problem(1, T, H, dk, dv, gate=gate, chunk=chunk)) == 1
    heads = [(0, h) for h in (range(H) if n < 10 else (0, 8, H - 1))]
    spec = pi.small_spec(B=1, H=H, T=T, gate=gate, dk=dk, dv=dv, chunk=chunk, s0="normal", a0="lognormal",
                         with_do=True)
    inp = pi.generate(spec, 4000 + 10 * n + chunk + ragged)
    ref = oabi.forward(inp, gate=gate, x=spec.x, scale=spec.scale, heads=heads)
    o, S_T, _ = run_fwd(spec, inp, chunk=chunk)
    e_o = rel_err(np.stack([o[b, :, h] for b, h in heads]), ref["o"])
    e_s = rel_err(np.stack([S_T[b, h] for b, h in heads]), ref["S_T"])
    msg = f"n={n} C={chunk} {gate} {dk}x{dv} T={T}"
    assert max(e_o, e_s) <= tol("bf16"), f"{msg}: o={e_o:.2e} S_T={e_s:.2e}"
    dS_T = (0.1 * np.random.default_rng(n).standard_normal((1, H, dk, dv))).astype(np.float32)
    compare(spec, inp, "squash", dS_T, heads=heads, tag=f"runs {msg}", chunk=chunk)


@pytest.mark.parametrize("gate,precond,knorm,dk,dv,chunk,B,H,T", [
    ("scalar", "squash", "none", 128, 128, 64, 4, 16, 32 * 64 - 63),   # 32 chunks, the last of one token
    ("none", "squash", "none", 64, 128, 32, 8, 8, 33 * 32 - 5),
    ("scalar", "squash", "none", 128, 64, 32, 8, 16, 32 * 32),
    ("none", "squash", "none", 64, 64, 64, 16, 8, 33 * 64 - 1),
    ("none", "squash", "none", 128, 128, 64, 4, 16, 32 * 64),
    ("none", "identity", "none", 128, 128, 32, 4, 16, 32 * 32 + 7),
    ("scalar", "external", "none", 64, 128, 64, 8, 8, 32 * 64 - 9),
    ("scalar", "identity", "none", 64, 64, 32, 16, 8, 33 * 32),
    ("none", "external", "none", 128, 64, 32, 16, 8, 32 * 32 - 1),
    ("scalar", "squash", "m", 128, 128, 32, 8, 8, 32 * 32 - 3),
    ("none", "squash", "1pm", 64, 64, 32, 8, 16, 32 * 32),
    ("scalar", "squash", "beta", 128, 64, 32, 8, 16, 33 * 32 - 30),
    ("scalar", "diag_sm", "none", 64, 128, 32, 8, 8, 32 * 32 - 31),
])
def test_scan_forms_p(gate, precond, knorm, dk, dv, chunk, B, H, T):
    """Problems whose scan forms P itself (its slabs fill the chip and its
    runs have 32 chunks or more), whose chunk preparation reads no queries:
    sampled heads, forward and every gradient against the oracle; and the
    training pair, whose forward leaves that P for the backward, bit for bit
    against the inference forward and the recomputing backward."""
    import torch
    import paper_2604_21100_amd as pdn
    assert B * H * dv // 32 >= 256 and -(-T // chunk) >= 32
    sq, ext = precond == "squash", precond == "external"
    spec = pi.small_spec(B=B, H=H, T=T, gate=gate, dk=dk, dv=dv, chunk=chunk, with_do=True)
    inp = pi.generate(spec, 4500 + dk + chunk)
    if ext:
        kt = inp["k"] * np.random.default_rng(2).uniform(1 / 1.5, 1.5, inp["k"].shape)
        inp["ktilde"] = pi.round_bf16(kt)
    heads = [(0, 0), (B - 1, H - 1)]
    kw = dict(knorm=knorm, ridge=0.5)
    ref = oabi.forward(inp, gate=gate, precond=precond, x=spec.x, scale=spec.scale, heads=heads, **kw)
    o, S_T, _ = run_fwd(spec, inp, precond, chunk=chunk, **kw)
    e_o = rel_err(np.stack([o[b, :, h] for b, h in heads]), ref["o"])
    e_s = rel_err(np.stack([S_T[b, h] for b, h in heads]), ref["S_T"])
    msg = f"forms P C={chunk} {gate}/{precond}/{knorm} {dk}x{dv}"
    assert max(e_o, e_s) <= tol("bf16"), f"{msg}: o={e_o:.2e} S_T={e_s:.2e}"
    if precond == "diag_sm" or knorm != "none":
        return   # forward only
    compare(spec, inp, precond, None, heads=heads, tag=msg, chunk=chunk)
    d = to_device(inp, "bf16")
    main = (d["q"], d["k"], d["v"], d["beta"])
    more = dict(g=d["g"], gate=gate, precond=precond, beta_p=d["beta_p"] if sq else None, g_p=d["g_p"] if sq else None,
                log_a_scale=d["log_a_scale"] if sq else None, A0=d["A0"] if sq else None, S0=d["S0"],
                ktilde=d["ktilde"] if ext else None, x=spec.x, scale=spec.scale, chunk=chunk)
    prob = pdn.make_problem(B, T, H, dk, dv, gate=gate, precond=precond, x=spec.x, scale=spec.scale, chunk=chunk)
    ws = torch.full((pdn.pdn_workspace_size(prob, True),), 255, dtype=torch.uint8, device="cuda")   # (NaN bytes)
    for x, y in zip(pdn.pdn_chunk_fwd(*main, workspace=ws, train=True, **more), pdn.pdn_chunk_fwd(*main, **more)):
        assert (x is None and y is None) or torch.equal(x, y), msg
    saved = pdn.pdn_chunk_bwd(*main, d["dO"], workspace=ws, saved=True, **more)
    again = pdn.pdn_chunk_bwd(*main, d["dO"], **more)
    for name, x in saved.items():
        assert torch.equal(x, again[name]), f"{msg} {name}"
