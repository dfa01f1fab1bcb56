"""The general path on both sides of the line between its two kinds of kernels (one wavefront a row for few rows or keys a
head, 16-row tiles otherwise), at the sizes next to it, and at as many heads as a call takes.  Bounds as in
test_gpu_general.py."""
import numpy as np
import pytest
import torch

from oracle import nfd_oracle as orc
from paper_2506_01380_amd import binding as nb
from paper_2506_01380_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,B,H,T,D,kvf,qf,rows", [
    ("fp32", 64, 64, 1, 64, 1, 1, True),     # one key
    ("fp32", 64, 64, 2, 129, 2, 2, True),    # rows of two frames
    ("fp32", 16, 64, 16, 32, 1, 1, False),   # one whole tile
    ("fp32", 16, 64, 1, 129, 64, 1, True),   # one by one: 64 keys
    ("fp32", 1, 2, 1, 129, 64, 1, False),    # the same, few heads
    ("fp32", 16, 64, 4, 100, 1, 1, True),
    ("fp32", 16, 64, 4, 100, 16, 1, False),
    ("fp32", 64, 64, 1, 5, 65, 1, True),     # a second pass over the lanes
    ("bf16", 16, 64, 4, 33, 4, 1, True),
    ("bf16", 16, 64, 16, 33, 4, 1, False),
    ("bf16", 24, 24, 3, 62, 2, 2, True),
    ("bf16", 64, 32, 2, 256, 2, 1, True),
])
def test_rows_and_tiles(dtype, B, H, T, D, kvf, qf, rows):
    dt = nb.NFD_FP32 if dtype == "fp32" else nb.NFD_BF16
    assert (nb.nfd_attn_plan(dt, B, H, kvf + 1, T, D, kvf, qf)["block_m"] == 4) == rows
    q, k, v = wl.make_qkv(B, H, D, T, kvf, qf, kvf + 1, dtype, seed=wl.BASE_SEED + 6000 + D)
    g = wl.randn(q.shape, wl.BASE_SEED + 6001, dtype)
    k[:, :, kvf * T:] = np.nan
    v[:, :, kvf * T:] = np.nan
    td = torch.float32 if dtype == "fp32" else torch.bfloat16
    a = nb.Attention(dtype)
    qd, kd, vd, gd = (torch.from_numpy(x).cuda().to(td) for x in (q, k, v, g))
    out, lse = a.forward_lse(qd, kd, vd, T, kv_frames=kvf, q_frames=qf)
    dq, dk, dv = a.backward(qd, kd, vd, out, gd, lse, T, kv_frames=kvf, q_frames=qf)
    torch.cuda.synchronize()
    a.close()
    kz, vz = np.nan_to_num(k), np.nan_to_num(v)
    ref = orc.block_causal_attn(q, kz, vz, T, kv_frames=kvf, q_frames=qf)
    rdq, rdk, rdv, rlse = orc.block_causal_attn_bwd(q, kz, vz, g, T, kv_frames=kvf, q_frames=qf)
    for got, want, tag in ((out, ref, "out"), (dq, rdq, "dq"), (dk, rdk, "dk"), (dv, rdv, "dv")):
        d = got.double().cpu().numpy() - want
        scale = max(np.linalg.norm(want), 0.1 * np.sqrt(want.size))  # one visible key: dq = dk = 0 (see test_gpu_general.py)
        assert np.linalg.norm(d) <= (1e-5 if dtype == "fp32" else 1e-2) * scale, (tag, np.linalg.norm(d) / scale)
    assert np.abs(lse.cpu().numpy() - rlse).max() <= 1e-5


@pytest.mark.parametrize("T", [1, 3])
def test_as_many_heads_as_a_call_takes(T):
    """2^24 heads: a launch holds fewer than 2^32 threads, 256 of them a tile."""
    B = H = 4096
    gen = torch.Generator(device="cuda").manual_seed(T)
    q, k, v, g = (torch.randn((B, H, T, 1), device="cuda", generator=gen) for _ in range(4))
    a = nb.Attention("fp32", workspace_bytes=1 << 28)
    out, lse = a.forward_lse(q, k, v, T)
    dq, dk, dv = a.backward(q, k, v, out, g, lse, T)
    a.close()
    s = (q * k.transpose(2, 3)).double()  # [B, H, T, T], width 1: scale 1
    p = torch.softmax(s, -1)
    assert (out.double() - (p * v.transpose(2, 3)).sum(-1, keepdim=True)).abs().max() <= 1e-5
    assert (lse.double() - torch.logsumexp(s, -1)).abs().max() <= 1e-5
    assert (dv.double() - (p * g).sum(2).unsqueeze(-1)).abs().max() <= 1e-5
    ds = p * (g * v.transpose(2, 3) - (g * out))
    assert (dq.double() - (ds * k.transpose(2, 3)).sum(-1, keepdim=True)).abs().max() <= 1e-4
    assert (dk.double() - (ds * q).sum(2).unsqueeze(-1)).abs().max() <= 1e-4
