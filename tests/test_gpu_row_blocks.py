"""The forward's kernels by the number of 32-row blocks in a query tile: 48 rows per wavefront at six (first and second row
block of a wavefront in different frames, ragged last rows, key splits and none), the 128-row kernel at four and fewer with
a log-sum-exp, 64 rows per wavefront otherwise.  Plain, with log-sum-exp, and the one-call cached step."""
import numpy as np
import pytest
import torch

from oracle import nfd_oracle as orc
from paper_2506_01380_amd import binding as nb
from paper_2506_01380_amd import workloads as wl
from parity_bounds import BF16_MAX_ABS

pytestmark = pytest.mark.gpu

CASES = [
    # B, H, T, kv_frames, q_frames, F: blocks in the largest tile
    ((1, 64, 192, 1, 1, 1), 6),    # three key tiles: too short for the pipelined loop's second round
    ((1, 64, 161, 6, 1, 7), 6),    # the last block has one row; key splits
    ((2, 256, 48, 5, 4, 5), 6),    # no splits, four frames in a tile: both row blocks straddle frames
    ((1, 64, 90, 4, 2, 4), 6),     # 180 rows: the last wavefront's second block has four rows, in the later frame
    ((1, 32, 576, 3, 1, 3), 6),    # three whole tiles
    ((1, 64, 150, 4, 1, 4), 5),
    ((1, 64, 120, 5, 1, 5), 4),
    ((1, 64, 33, 9, 3, 9), 4),
    ((1, 64, 20, 7, 1, 8), 1),
]


@pytest.mark.parametrize("shape,blocks", CASES)
def test_forward_row_blocks(shape, blocks):
    B, H, T, kvf, qf, F = shape
    D = 64
    plan = nb.nfd_attn_plan(nb.NFD_BF16, B, H, F, T, D, kvf, qf)
    assert plan["block_m"] == 256 and -(-(-(-qf * T // 32)) // plan["n_q_tiles"]) == blocks
    q, k, v = wl.make_qkv(B, H, D, T, kvf, qf, F, "bf16", seed=wl.BASE_SEED + 3000 + T)
    attn = nb.Attention("bf16")
    qd, kd, vd = (torch.from_numpy(x).cuda().to(torch.bfloat16) for x in (q, k, v))
    out = attn.forward(qd, kd, vd, T, kv_frames=kvf, q_frames=qf)
    out_l, lse = attn.forward_lse(qd, kd, vd, T, kv_frames=kvf, q_frames=qf)
    kc, vc = kd.clone(), vd.clone()
    new = slice((kvf - qf) * T, kvf * T)
    kn, vn = kd[:, :, new].contiguous(), vd[:, :, new].contiguous()
    kc[:, :, new] = float("nan")
    vc[:, :, new] = float("nan")
    step = torch.empty_like(qd)
    nb.nfd_kvcache_append_attn_fwd(attn.h, qd, kc, vc, kn, vn, step, B, H, F, T, D, kvf, qf)
    torch.cuda.synchronize()
    assert torch.equal(step, out) and torch.equal(kc, kd) and torch.equal(vc, vd)
    heads = sorted({0, B * H // 2, B * H - 1})  # the oracle on three heads, every row
    flat = lambda x: x.reshape(1, B * H, *x.shape[2:])[:, heads]
    hq, hk, hv = flat(q), flat(k), flat(v)
    ref = orc.block_causal_attn(hq, hk, hv, T, kv_frames=kvf, q_frames=qf)
    for name, o in (("forward", out), ("lse", out_l)):
        got = flat(o.float().cpu().numpy().astype(np.float64))
        assert np.all(np.isfinite(got)) and np.abs(got - ref).max() <= BF16_MAX_ABS, (name, np.abs(got - ref).max())
        assert np.linalg.norm(got - ref) <= 1e-2 * np.linalg.norm(ref), name
    s = np.einsum("bhid,bhjd->bhij", hq.astype(np.float64), hk[:, :, :kvf * T].astype(np.float64)) / 8.0
    seen = np.arange(kvf * T)[None, :] // T <= kvf - qf + np.arange(qf * T)[:, None] // T
    s = np.where(seen, s, -np.inf)
    m = s.max(-1)
    want = m + np.log(np.exp(s - m[..., None]).sum(-1))
    # exact products of bf16 inputs summed in fp32, fp32 exponentials and sums
    assert np.abs(flat(lse.cpu().numpy().astype(np.float64)) - want).max() <= 2e-4
    attn.close()
