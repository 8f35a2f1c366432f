"""Feed-forward and decoder blocks with less room than their queries ask for: from the least that is taken on, results are right, nothing
beyond the room is written, and below it the call is refused before its first launch."""
import numpy as np
import pytest
import torch

import paper_2604_26666_amd as fact
import workloads as wl
from oracle import block as blk
from oracle import check
import test_gpu_block as gb

pytestmark = pytest.mark.gpu
WORKSPACE = -6


# T, d_model, d_ff, bytes that are taken, bytes asked for (one fp32 plane for each range of the down projection's K)
@pytest.mark.parametrize("T,d,dff,least,full", [(96, 768, 3072, 2 * 96 * 768 * 4, 6 * 96 * 768 * 4), (610, 5040, 13784, 0, 2 * 610 * 5040 * 4)])
def test_mlp(T, d, dff, least, full):
    assert fact.fact_block_mlp_workspace_bytes(T, d, dff, fact.ACT_GELU_TANH) == full
    g = torch.Generator(device="cuda").manual_seed(8)
    r = lambda std, *s: torch.randn(*s, generator=g, device="cuda").mul_(std).bfloat16()
    X, W1, b1, W2, b2, R = r(1.0, T, d), r(d ** -0.5, dff, d), r(0.1, dff), r(dff ** -0.5, d, dff), r(0.1, d), r(1.0, T, d)
    H = torch.empty(T, dff, dtype=torch.bfloat16, device="cuda")
    outs = {}
    for have in [n for n in (least - 16, least, least + 16, (least + full) // 32 * 16, full - 16, full, None) if n is None or n >= 0]:
        ws = torch.full(((have or 0) + 4096,), 0x5A, dtype=torch.uint8, device="cuda")
        Y = torch.full((T, d), 77.0, dtype=torch.bfloat16, device="cuda")
        H.fill_(77.0)
        rc = fact.fact_block_mlp(T, d, dff, X, W1, None, b1, fact.ACT_GELU_TANH, W2, b2, R, H, Y, None if have is None else ws, have or 0)
        torch.cuda.synchronize()
        assert (ws[have or 0:] == 0x5A).all(), "wrote past the workspace"
        if (have or 0) < least:
            assert rc == WORKSPACE and (Y == 77.0).all() and (H == 77.0).all() and (ws == 0x5A).all(), have
            continue
        assert rc == 0, (have, rc)
        outs[have] = Y
        # Y of the H that was stored: one rounding to bfloat16 (2^-9 of the value), and on either side sums in fp32 of at most d_ff / 32 + 16 steps (2^-24 of the
        # sum of magnitudes each)
        ref = H.float() @ W2.float().t() + b2.float() + R.float()
        size = H.float().abs() @ W2.float().abs().t() + b2.float().abs() + R.float().abs()
        assert ((Y.float() - ref).abs() <= ref.abs() * 2.0 ** -8 + size * (dff // 32 + 16) * 2.0 ** -23).all(), have
    # one plan where there is no room for the ranges, and with none at all
    rest = [outs[n] for n in outs if n != full]
    assert all(torch.equal(rest[0], y) for y in rest)


@pytest.mark.parametrize("ranges", [1, 2, 4, 6])
def test_block(ranges):
    T, d, dff = 96, 768, 3072
    p, t, X = gb.make_block("gpt", 1, T, d, 12, 12, 64, dff)
    b = fact.Block(1, T, d, 12, 12, 64, dff, 0, p["act"], 0, 1e-5, 0.0, **{k: v.cuda() for k, v in t.items()})
    offs = fact.fact_block_scratch_offsets(b)
    assert fact.fact_block_scratch_bytes(b) == offs[6] + 6 * T * d * 4
    have = offs[6] + ranges * T * d * 4
    scratch = torch.full((have + 4096,), 0x5A, dtype=torch.uint8, device="cuda")
    Y = torch.full((T, d), 77.0, dtype=torch.bfloat16, device="cuda")
    rc = fact.fact_block_forward(b, X.cuda(), Y, scratch, have)
    torch.cuda.synchronize()
    assert (scratch[have:] == 0x5A).all(), "wrote past the scratch"
    if ranges < 2:
        assert rc == WORKSPACE and (scratch == 0x5A).all() and (Y == 77.0).all()
        return
    assert rc == 0
    raw, got = scratch.cpu().numpy(), {"Y": gb.host_bits(Y)}
    for name, off, cols in zip(("N1", "QKVR", "A", "X1", "N2", "H"), offs, (d, 3 * d, d, d, d, dff)):
        got[name] = raw[off: off + T * cols * 2].view(np.uint16).reshape(T, cols).copy()
    strict = blk.block_forward(wl.bits(X), p, given={k: got[k] for k in ("N1", "QKVR", "A", "X1", "N2", "H")})
    for name in ("X1", "H", "Y"):
        check.assert_close(got[name], strict[name], what=f"{name}, room for {ranges} ranges")
