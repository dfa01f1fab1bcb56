"""How the general path loads features: vectors at a full padded width, vectors with those past the width left out (multiples
of four), one by one (other widths, tensors off a 16-byte boundary).  The last feature of every row is what a wrong
group would lose or take from the next row.  Bounds as in test_gpu_general.py."""
import numpy as np
import pytest
import torch

from oracle import nfd_oracle as orc
from paper_2506_01380_amd import binding as nb
from paper_2506_01380_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _on_gpu(x, dtype, offset):
    """x as a dense tensor that starts `offset` elements behind an aligned address."""
    buf = torch.full((x.size + 16,), float("nan"), dtype=dtype, device="cuda")
    t = buf[offset:offset + x.size].view(x.shape)
    t.copy_(torch.from_numpy(x))
    return t


@pytest.mark.parametrize("dtype,D,offset", [
    ("fp32", 4, 0), ("fp32", 28, 0), ("fp32", 36, 0), ("fp32", 100, 0), ("fp32", 132, 0), ("fp32", 252, 0),
    ("bf16", 4, 0), ("bf16", 20, 0), ("bf16", 60, 0), ("bf16", 68, 0), ("bf16", 196, 0),
    ("fp32", 64, 0), ("fp32", 64, 1), ("fp32", 36, 2), ("bf16", 32, 4), ("bf16", 96, 1),
])
@pytest.mark.parametrize("B,H,T,kvf,qf", [(1, 2, 21, 4, 3), (4, 24, 93, 8, 8)])  # one column block, two (D <= 64)
def test_loads(dtype, D, offset, B, H, T, kvf, qf):
    q, k, v = wl.make_qkv(B, H, D, T, kvf, qf, kvf, dtype, seed=wl.BASE_SEED + 5000 + D)
    g = wl.randn(q.shape, wl.BASE_SEED + 5001, dtype)
    td = torch.float32 if dtype == "fp32" else torch.bfloat16
    a = nb.Attention(dtype)
    qd, kd, vd, gd = (_on_gpu(x, td, offset) for x in (q, k, v, g))
    out, lse = a.forward_lse(qd, kd, vd, T, kv_frames=kvf, q_frames=qf)
    dq, dk, dv = a.backward(qd, kd, vd, out, gd, lse, T, kv_frames=kvf, q_frames=qf)
    torch.cuda.synchronize()
    a.close()
    ref = orc.block_causal_attn(q, k, v, T, kv_frames=kvf, q_frames=qf)
    rdq, rdk, rdv, rlse = orc.block_causal_attn_bwd(q, k, v, g, T, kv_frames=kvf, q_frames=qf)
    for got, want, tag in ((out, ref, "out"), (dq, rdq, "dq"), (dk, rdk, "dk"), (dv, rdv, "dv")):
        d = got.double().cpu().numpy() - want
        assert np.linalg.norm(d) <= (1e-5 if dtype == "fp32" else 1e-2) * np.linalg.norm(want), tag
        assert np.abs(d[..., -1]).max() <= (1e-4 if dtype == "fp32" else 2e-2) * np.abs(want).max(), tag
    assert np.abs(lse.cpu().numpy() - rlse).max() <= 1e-5
