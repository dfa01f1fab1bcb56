"""The launch forms of the matrix-core backward, each at sizes where its work items go wrong first: separate kernels (many
short heads), one launch with both kinds of items in the large and in the small size; ragged last row tiles and key
blocks, a cached form with spare capacity, head counts off the XCD count.  Bounds as in test_gpu_bwd.py."""
import numpy as np
import pytest
import torch

from oracle import nfd_oracle as orc
from paper_2506_01380_amd import binding as nb
from paper_2506_01380_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,H,T,kvf,qf,F,form", [
    (24, 32, 40, 6, 6, 6, nb.NFD_BWD_SEPARATE),     # 768 heads of 240 rows
    (24, 33, 23, 9, 9, 9, nb.NFD_BWD_SEPARATE),     # 207 rows: a second key block of 15 keys
    (28, 32, 40, 8, 3, 9, nb.NFD_BWD_SEPARATE),     # cached form, capacity to spare
    (4, 24, 150, 7, 7, 7, nb.NFD_BWD_MERGED),       # 96 heads of 1050 rows
    (3, 25, 151, 7, 6, 8, nb.NFD_BWD_MERGED),       # cached form, head count off the XCD count
    (1, 2, 65, 1, 1, 1, nb.NFD_BWD_MERGED_SMALL),   # one frame, one row past a 64-row step
    (1, 3, 129, 1, 1, 2, nb.NFD_BWD_MERGED_SMALL),  # one row past a 128-row tile
    (2, 5, 43, 6, 2, 7, nb.NFD_BWD_MERGED_SMALL),   # cached form
])
def test_backward_launch_forms(B, H, T, kvf, qf, F, form):
    assert nb.nfd_attn_bwd_form(nb.NFD_BF16, B, H, F, T, 64, kvf, qf) == form
    q, k, v = wl.make_qkv(B, H, 64, T, kvf, qf, F, "bf16", seed=wl.BASE_SEED + 4000 + T)
    g = wl.randn(q.shape, wl.BASE_SEED + 4001)
    k[:, :, kvf * T:] = np.nan
    v[:, :, kvf * T:] = np.nan
    a = nb.Attention("bf16")
    qd, kd, vd, gd = (torch.from_numpy(x).cuda().to(torch.bfloat16) for x in (q, k, v, g))
    out, lse = a.forward_lse(qd, kd, vd, T, kv_frames=kvf, q_frames=qf)
    got = a.backward(qd, kd, vd, out, gd, lse, T, kv_frames=kvf, q_frames=qf)
    again = a.backward(qd, kd, vd, out, gd, lse, T, kv_frames=kvf, q_frames=qf)
    torch.cuda.synchronize()
    a.close()
    ref = orc.block_causal_attn_bwd(q, np.nan_to_num(k), np.nan_to_num(v), g, T, kv_frames=kvf, q_frames=qf)
    for x, y, r, tag in zip(got, again, ref, ("dq", "dk", "dv")):
        assert torch.equal(x, y), tag
        d = x.double().cpu().numpy() - r
        rel = np.linalg.norm(d) / np.linalg.norm(r)
        assert rel <= 1e-2 and np.abs(d).max() <= 2e-2 * np.abs(r).max(), (tag, rel, np.abs(d).max())
