"""The general path (fp32 matrix instruction; fp32 at any width, bf16 at widths other than 64) at the edges of its
dispatch and tiles: every padded width with and without 16-byte loads, one and two column blocks per workgroup, fewer key
blocks than wavefronts, rows that leave the last block ragged.  fp32 bound: sums of at most 1600 products of unit-variance
values in fp32, relative 2-norm 1600^.5 x 2^-24 = 2.4e-6 per product stage, three stages: 1e-5."""
import numpy as np
import pytest
import torch

from oracle import nfd_oracle as orc
from paper_2506_01380_amd import binding as nb
from paper_2506_01380_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,B,H,T,D,kvf,qf", [
    ("fp32", 1, 1, 1, 64, 1, 1),       # one row, one key
    ("fp32", 1, 2, 15, 32, 2, 1),      # 30 keys: two key blocks for four wavefronts, ragged row block
    ("fp32", 1, 1, 17, 17, 5, 5),      # odd width: single loads, padded to 32
    ("fp32", 1, 2, 33, 60, 3, 2),      # padded to 64
    ("fp32", 1, 3, 16, 128, 4, 4),
    ("fp32", 1, 1, 40, 129, 3, 3),     # padded to 256
    ("fp32", 1, 1, 40, 256, 2, 2),
    ("fp32", 2, 24, 95, 64, 8, 8),     # 48 heads x 24 tiles of 32 rows: two column blocks, ragged by 8 rows
    ("fp32", 2, 24, 95, 33, 8, 8),     # ... with single loads
    ("bf16", 1, 2, 33, 32, 3, 3),
    ("bf16", 1, 2, 33, 62, 3, 3),
    ("bf16", 1, 1, 65, 256, 2, 1),
])
def test_general_path_edges(dtype, B, H, T, D, kvf, qf):
    q, k, v = wl.make_qkv(B, H, D, T, kvf, qf, kvf + 1, dtype, seed=wl.BASE_SEED + 3000 + D + T)
    g = wl.randn(q.shape, wl.BASE_SEED + 3001, dtype)
    k[:, :, kvf * T:] = np.nan  # capacity past the frames present is never read
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
        # With one visible key dq = dk = 0 in exact arithmetic; what is left is the rounding of two equal dot products of
        # 64 terms, at most 2 x 64 x 2^-24 x E|xy| = 5e-6, times the scale 1/8: 1e-6 an element is allowed there.
        scale = max(np.linalg.norm(want), 0.1 * np.sqrt(want.size))
        assert np.linalg.norm(d) <= (1e-5 if dtype == "fp32" else 1e-2) * scale, (tag, np.linalg.norm(d) / scale)
    assert np.abs(lse.cpu().numpy() - rlse).max() <= 1e-5
