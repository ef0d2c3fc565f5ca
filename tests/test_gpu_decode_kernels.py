"""Decode-step kernel variants at the edges of their 128-row chunks, against the oracle."""
import sys

import numpy as np
import pytest
import torch

import parity
import vatp_synth as vs
from oracle import vatp_oracle as orc
import paper_2406_12335_amd as vatp
from paper_2406_12335_amd.runner import PrunedKVCache
from test_gpu_fused_step import _seed_state

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


# edges of what the second launch of the fused step requests ahead: a workgroup's share of the rows (64-row steps; one
# workgroup for all, shares that wrap round the end, shares beyond the rows held in registers) and of the recent window
@pytest.mark.parametrize("dtype,d,H,g,lens,recent", [
    ("bf16", 128, 2, 1, [63, 64, 65, 1], 8), ("fp32", 64, 2, 1, [128, 127, 5], 0), ("bf16", 128, 1, 1, [1023, 1025], 1000),
    ("bf16", 64, 1, 2, [33500], 64), ("bf16", 64, 32, 16, [1100], 300), ("fp32", 128, 43, 4, [260, 513, 90], 40),
    ("bf16", 128, 65, 8, [2300], 128),
])
def test_fused_second_launch_at_the_edges_of_its_shares(gpu_device, dtype, d, H, g, lens, recent):
    """Bit for bit the state that vatp_decode_attend_step followed by vatp_select_compact leaves."""
    tdt = torch.float32 if dtype == "fp32" else torch.bfloat16
    b, dev, F = len(lens), gpu_device, 0 if recent == 0 else 1
    budgets = [max(n, F + recent) for n in lens]
    print("[case] fused shares %s d=%d H=%d g=%d lens=%s" % (dtype, d, H, g, lens), flush=True)
    gen = torch.Generator().manual_seed(7)
    two, fused = [PrunedKVCache(b, H, d, tdt, F, recent, budgets, dev, cap_cache=max(budgets) + 1, q_per_kv=g) for _ in range(2)]
    try:
        weak = [(bb, h, min(F + 37 * h, lens[bb] - 1)) for bb in range(b) for h in range(0, H, 2)]
        _seed_state([two, fused], lens, gen, d, tdt, dev, weak_rows=weak)
        ws = torch.empty(vatp.vatp_workspace_bytes(two.ctx, two._p_dec, vatp.CALL_DECODE_ATTEND_STEP) + 256, dtype=torch.uint8,
                         device=dev)
        for t in range(4):
            q = torch.randn(b, H * g, d, generator=gen).to(tdt).to(dev)
            k, v = (torch.randn(b, H, d, generator=gen).to(tdt).to(dev) for _ in range(2))
            out_two, out_fused = (torch.full((b, H * g, d), x, device=dev) for x in (0.0, 1.0))
            c = two.cur
            two._p_dec.set_len(two.lens)
            vatp.vatp_decode_attend_step(two.ctx, two._p_dec, q, k, v, two.K[c], two.V[c], two.S[c], two.nrm[c], two.pos[c],
                                         [900 + t] * b, out_two, ws)
            two.lens = [n + 1 for n in two.lens]
            two.prune()
            fused.decode_prune_step(q, k, v, [900 + t] * b, out=out_fused)
            assert torch.equal(out_two, out_fused) and two.lens == fused.lens
            for bb, n in enumerate(two.lens):
                for name in ("K", "V", "S", "nrm", "pos"):
                    x, y = getattr(two, name)[two.cur], getattr(fused, name)[fused.cur]
                    assert torch.equal(x[bb, :, :n], y[bb, :, :n]), (t, bb, name)
                assert torch.equal(two.kept_idx[bb, :, :n], fused.kept_idx[bb, :, :n]), (t, bb)
    finally:
        two.close()
        fused.close()


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("fp32", 64)])
@pytest.mark.parametrize("g", [1, 4])
def test_infinity_in_the_new_value_row_stays_an_infinity(gpu_device, dtype, d, g):
    """The rows of a chunk past the new one have no part in the outputs, whatever the new row holds."""
    tdt, dev, n0 = (torch.float32 if dtype == "fp32" else torch.bfloat16), gpu_device, 130
    print("[case] infinite value %s g=%d" % (dtype, g), flush=True)
    gen = torch.Generator().manual_seed(3)
    K, V = (torch.randn(1, 2, n0 + 1, d, generator=gen).to(tdt).to(dev) for _ in range(2))
    q = torch.randn(1, 2 * g, d, generator=gen).to(tdt).to(dev)
    k, v = (torch.randn(1, 2, d, generator=gen).to(tdt).to(dev) for _ in range(2))
    v[:, :, 3] = float("inf")
    S, N = (torch.zeros(1, 2, n0 + 1, device=dev) for _ in range(2))
    out = torch.zeros(1, 2 * g, d, device=dev)
    ctx = vatp.vatp_create(0)
    try:
        p = vatp.Params(1, 2, d, tdt, 0, 0, n0 + 1, [n0], None, q_per_kv=g)
        ws = torch.empty(vatp.vatp_workspace_bytes(ctx, p, vatp.CALL_DECODE_ATTEND_STEP), dtype=torch.uint8, device=dev)
        vatp.vatp_decode_attend_step(ctx, p, q, k, v, K, V, S, N, None, None, out, ws)
        torch.cuda.synchronize()
    finally:
        vatp.vatp_destroy(ctx)
    want = torch.zeros(d, dtype=torch.bool)
    want[3] = True
    assert torch.equal(torch.isinf(out.cpu()), want.expand(1, 2 * g, d)) and not torch.isnan(out).any()


# the same launch with a history window, whose rows come by way of the ring's columns: shares of more rows than a workgroup
# holds in registers (2048, of more than 8 query heads 512), by one workgroup per head and by sixteen
@pytest.mark.parametrize("dtype,d,b,H,g,L,window", [
    ("bf16", 64, 1, 1, 1, 35000, 5), ("fp32", 128, 1, 64, 8, 2300, 9), ("bf16", 64, 1, 32, 16, 700, 12), ("bf16", 128, 8, 64, 1, 2200, 3),
])
def test_windowed_second_launch_with_large_shares(gpu_device, dtype, d, b, H, g, L, window):
    print("[case] windowed shares %s d=%d b=%d H=%d g=%d L=%d w=%d" % (dtype, d, b, H, g, L, window), flush=True)
    cfg = vs.scaled(vs.CONFIGS["llama7b_layer"], batch=b, n_heads=H, head_dim=d, dtype=dtype, q_per_kv=g, prompt_len=L,
                    decode_steps=window + 4, recent=40)
    inp = vs.make_inputs(cfg, seed=71, device=gpu_device)
    inp.budgets = [L * 97 // 100] * b
    rep = parity.run_trajectory(inp, gpu_device, units=[(0, 0)] if b * H == 1 else [(0, 1), (b - 1, H - 1)], fused=True, window=window)
    print("report %r" % rep, flush=True)
    assert rep.admitted_near_ties <= 1
