"""Decode-step kernel variants at the edges of their 128-row chunks, against the oracle."""
import sys

import numpy as np
import pytest
import torch

import parity
from oracle import vatp_oracle as orc
import paper_2406_12335_amd as vatp

pytestmark = pytest.mark.gpu


# one case per instantiation of the group kernel (up to 2, 4, 8, 16 query heads), full and not, for every row layout
@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("bf16", 64), ("fp32", 128), ("fp32", 64)])
@pytest.mark.parametrize("g", [1, 2, 3, 4, 7, 8, 16])
def test_decode_step_at_chunk_edges(gpu_device, dtype, d, g):
    """Scores and attention outputs; the caches hold NaN in every row the step must not read."""
    n0s, H = [0, 1, 127, 128, 129, 300], 2
    b, cap = len(n0s), max(n0s) + 3
    tdt = torch.float32 if dtype == "fp32" else torch.bfloat16
    gen = torch.Generator().manual_seed(17 * d + g)
    K = (torch.randn(b, H, cap, d, generator=gen) * 1.2).to(tdt)
    V = (torch.randn(b, H, cap, d, generator=gen) * torch.exp(0.5 * torch.randn(b, H, cap, 1, generator=gen))).to(tdt)
    S0 = torch.rand(b, H, cap, generator=gen) + 0.1
    for bb, n0 in enumerate(n0s):
        for t in (K, V, S0):
            t[bb, :, n0:] = float("nan")
    q = (torch.randn(b, H * g, d, generator=gen) * 1.5).to(tdt)
    k, v = ((torch.randn(b, H, d, generator=gen) * 1.5).to(tdt) for _ in range(2))
    print("[case] decode %s d=%d g=%d" % (dtype, d, g), flush=True)
    sys.stdout.flush()
    dev = gpu_device
    ctx = vatp.vatp_create(0)
    try:
        p = vatp.Params(b, H, d, tdt, 0, 0, cap, n0s, None, q_per_kv=g)
        res = []
        for attend in (False, True):
            Kd, Vd, Sd = K.to(dev), V.to(dev), S0.to(dev)
            Nd = torch.zeros(b, H, cap, device=dev)
            out = torch.full((b, H * g, d), 9.0, device=dev)
            call = vatp.CALL_DECODE_ATTEND_STEP if attend else vatp.CALL_DECODE_STEP
            ws = torch.empty(vatp.vatp_workspace_bytes(ctx, p, call), dtype=torch.uint8, device=dev)
            args = (ctx, p, q.to(dev), k.to(dev), v.to(dev), Kd, Vd, Sd, Nd, None, None)
            if attend:
                vatp.vatp_decode_attend_step(*args, out, ws)
            else:
                vatp.vatp_decode_step(*args, ws)
            torch.cuda.synchronize()
            res.append((Kd.cpu(), Vd.cpu(), Sd.cpu(), Nd.cpu(), out.cpu()))
    finally:
        vatp.vatp_destroy(ctx)
    rtol = parity.rtol_for(tdt)
    (_, _, Sa, _, _), (Kb, Vb, Sb, Nb, out) = res
    for bb, n0 in enumerate(n0s):
        n = n0 + 1
        assert torch.equal(Sa[bb, :, :n], Sb[bb, :, :n])
        for h in range(H):
            Kfull = torch.cat([K[bb, h, :n0], k[bb, h][None]], 0).double().numpy()
            Vfull = torch.cat([V[bb, h, :n0], v[bb, h][None]], 0).double().numpy()
            assert torch.equal(Kb[bb, h, n0], k[bb, h]) and torch.equal(Vb[bb, h, n0], v[bb, h])
            parity.assert_scores_close(Nb[bb, h, n0:n].numpy(), orc.l1norm(Vfull[n0:n]), rtol, "norm")
            S_start = np.concatenate([S0[bb, h, :n0].double().numpy(), np.zeros(1)])
            S_want, _ = orc.decode_scores_group(q[bb, h * g:(h + 1) * g].double().numpy(), Kfull, S_start)
            parity.assert_scores_close(Sb[bb, h, :n].numpy(), S_want, rtol, "S (%d,%d)" % (bb, h))
            for r in range(g):
                want, scale = orc.attention_output(q[bb, h * g + r].double().numpy(), Kfull, Vfull)
                err = np.abs(out[bb, h * g + r].double().numpy() - want)
                assert np.all(err <= rtol * scale + 1e-12), "output (%d,%d,%d): max err %.3g" % (bb, h, r, err.max())
