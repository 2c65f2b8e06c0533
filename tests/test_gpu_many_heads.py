"""Calls of very many heads and few tokens: hundreds of thousands of heads in a
sequence (a chunk's rows past its end lie beyond 32-bit byte offsets, while
the valid rows do not), and millions of sequences (a scan's grid passes 2^32
work items).  A head's result does not depend on the others, so the
call must return bit for bit what calls on parts of the heads return."""
import pytest

pytestmark = pytest.mark.gpu


def _inputs(B, T, H, dk, dv, gate, seed):
    """Seeded tensors of a few thousand heads, repeated over B and H."""
    import torch
    gen = torch.Generator(device="cuda").manual_seed(seed)

    def tiled(*tail, f=lambda z: z, dtype=torch.float32):
        n = min(B * H, 3001)
        z = f(torch.randn((n, T) + tail, generator=gen, device="cuda")).to(dtype)
        out = torch.empty((B, T, H) + tail, device="cuda", dtype=dtype)
        for b0 in range(0, B, max(1, 1 << 20)):
            b1 = min(B, b0 + (1 << 20))
            idx = torch.arange(b0 * H, b1 * H, device="cuda") % n
            out[b0:b1] = z[idx].view((b1 - b0, H, T) + tail).transpose(1, 2)
        return out

    unit = lambda z: z / z.norm(dim=-1, keepdim=True)  # noqa: E731
    decay = lambda z: -0.1 * torch.nn.functional.softplus(z)  # noqa: E731
    bf = torch.bfloat16
    d = dict(q=tiled(dk, f=unit, dtype=bf), k=tiled(dk, f=unit, dtype=bf), v=tiled(dv, dtype=bf),
             beta=tiled(f=torch.sigmoid))
    if gate == "scalar":
        d["g"] = tiled(f=decay)
    return d


def test_rows_past_the_end_with_wide_strides():
    """300000 heads of 128: rows 56 .. 63 of the chunk start past 2^32 bytes,
    and wrapped they would fall on the nine valid rows of other heads."""
    import torch
    import paper_2604_21100_amd as pdn
    T, H, parts = 9, 300_000, 4
    d = _inputs(1, T, H, 128, 128, "scalar", 11)
    assert 63 * H * 256 - 2 ** 32 < (T - 1) * H * 256 < 2 ** 32 < 63 * H * 256
    kw = dict(gate="scalar", precond="identity")
    dO = torch.randn(d["v"].shape, generator=torch.Generator(device="cuda").manual_seed(5), device="cuda",
                     dtype=torch.bfloat16)

    def step(x, dO):
        main = (x["q"], x["k"], x["v"], x["beta"])
        o = pdn.pdn_chunk_fwd(*main, g=x["g"], want_state=False, **kw)[0]
        grads = pdn.pdn_chunk_bwd(*main, dO, g=x["g"], want_optional=False, **kw)
        return dict(grads, o=o)

    whole = step(d, dO)
    n = H // parts
    for i in range(parts):
        cut = lambda x: x[:, :, i * n:(i + 1) * n].contiguous()  # noqa: E731
        part = step({k: cut(x) for k, x in d.items()}, cut(dO))
        for name, x in part.items():
            assert torch.equal(cut(whole[name]), x), f"{name}, heads {i * n} .. {(i + 1) * n}"


def test_scan_grid_past_two_to_the_32():
    """3000000 sequences of one 64 x 128 head: the state scan's four slabs a
    head of 384 threads are more work items than one grid dimension takes."""
    import torch
    import paper_2604_21100_amd as pdn
    T, B, parts = 9, 3_000_000, 3
    assert B * 4 * 384 > 2 ** 32
    d = _inputs(B, T, 1, 64, 128, "none", 12)

    def forward(x):
        return pdn.pdn_chunk_fwd(x["q"], x["k"], x["v"], x["beta"], gate="none", precond="identity", chunk=32,
                                 want_state=False)[0]

    whole = forward(d)
    n = B // parts
    for i in range(parts):
        part = forward({k: x[i * n:(i + 1) * n] for k, x in d.items()})
        assert torch.equal(whole[i * n:(i + 1) * n], part), f"sequences {i * n} .. {(i + 1) * n}"
