"""The bf16 state scans over every short run length: their chain, output and
loader waves unroll the chunk loop differently (by two, by three, not at all)
and peel its ends, so a run of n chunks is checked for n = 1 .. 8 at both chunk
lengths, whole and ragged, with head counts that leave the grid's last group
of eight heads part empty.  Forward outputs and states and every gradient
against the float64 oracle's token recurrence, to the bars of the other GPU
tests (bf16 rounding of inputs, stored rows and operands)."""
import numpy as np
import pytest

import pdn_inputs as pi
from oracle import abi as oabi

from gpu_util import rel_err, run_fwd, tol
from test_gpu_bwd import compare

pytestmark = pytest.mark.gpu

GATES = ("none", "scalar", "channel")
DIMS = ((128, 128), (64, 128), (128, 64), (64, 64))


@pytest.mark.parametrize("chunk", [32, 64])
@pytest.mark.parametrize("n", range(1, 9))
def test_scan_runs(n, chunk):
    gate, (dk, dv) = GATES[n % 3], DIMS[(n // 2) % 4]
    T = n * chunk - (0 if n % 2 else 1 + 5 * n)
    spec = pi.small_spec(B=1, H=1 + n % 3, T=T, gate=gate, dk=dk, dv=dv, chunk=chunk, s0="normal", a0="lognormal",
                         with_do=True)
    inp = pi.generate(spec, 4000 + 10 * n + chunk)
    H = spec.H
    ref = oabi.forward(inp, gate=gate, x=spec.x, scale=spec.scale, B=1, H=H)
    o, S_T, _ = run_fwd(spec, inp, chunk=chunk)
    e_o = rel_err(np.stack([o[0, :, h] for h in range(H)]), ref["o"])
    e_s = rel_err(S_T.reshape(H, dk, dv), ref["S_T"])
    assert max(e_o, e_s) <= tol("bf16"), f"n={n} C={chunk} {gate} {dk}x{dv}: o={e_o:.2e} S_T={e_s:.2e}"
    dS_T = (0.1 * np.random.default_rng(n).standard_normal((1, H, dk, dv))).astype(np.float32)
    compare(spec, inp, "squash", dS_T, tag=f"runs n={n} C={chunk} {gate} {dk}x{dv}", chunk=chunk)


@pytest.mark.parametrize("gate,dk,dv,chunk,B,H,T", [
    ("scalar", 128, 128, 64, 4, 16, 32 * 64 - 63),   # 32 chunks, the last of one token
    ("none", 64, 128, 32, 8, 8, 33 * 32 - 5),
    ("scalar", 128, 64, 32, 8, 16, 32 * 32),
    ("none", 64, 64, 64, 16, 8, 33 * 64 - 1),
])
def test_scan_forms_p(gate, dk, dv, chunk, B, H, T):
    """Problems whose scan forms P itself (its slabs fill the chip and its
    runs have 32 chunks or more): sampled heads, forward and every gradient."""
    spec = pi.small_spec(B=B, H=H, T=T, gate=gate, dk=dk, dv=dv, chunk=chunk, with_do=True)
    inp = pi.generate(spec, 4500 + dk + chunk)
    heads = [(0, 0), (B - 1, H - 1)]
    ref = oabi.forward(inp, gate=gate, x=spec.x, scale=spec.scale, heads=heads)
    o, S_T, _ = run_fwd(spec, inp, chunk=chunk)
    e_o = rel_err(np.stack([o[b, :, h] for b, h in heads]), ref["o"])
    e_s = rel_err(np.stack([S_T[b, h] for b, h in heads]), ref["S_T"])
    assert max(e_o, e_s) <= tol("bf16"), f"C={chunk} {gate} {dk}x{dv}: o={e_o:.2e} S_T={e_s:.2e}"
    compare(spec, inp, "squash", None, heads=heads, tag=f"forms P C={chunk} {gate} {dk}x{dv}", chunk=chunk)
