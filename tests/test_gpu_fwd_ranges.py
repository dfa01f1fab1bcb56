"""The matrix-core forward over row ranges smaller than the plan's tiles, and the shapes it leaves to whole tiles: 32 rows per
wavefront (every count of wavefronts with rows, chains of one key tile to several turns of the ring, frame bounds inside a unit of 32
keys, ragged last rows and keys, key splits and none), 48 and 64 rows.  Plain, with log-sum-exp, the one-call cached step and
the 8-bit cache."""
import numpy as np
import pytest
import torch

from oracle import fp8_cache as f8
from oracle import nfd_oracle as orc
from paper_2506_01380_amd import binding as nb
from paper_2506_01380_amd import workloads as wl
from parity_bounds import BF16_MAX_ABS, BF16_REL_L2_INTERNAL

CASES = [
    # (B, H, T, kv_frames, q_frames, F), (row ranges per head, key splits), the same over the 8-bit cache
    ((1, 64, 64, 2, 2, 2), (1, 1), (1, 1)),          # four blocks, two key tiles
    ((1, 40, 33, 9, 9, 10), (3, 1), (3, 1)),         # ranges of 4, 3 and 3 blocks, bounds inside every unit
    ((1, 40, 100, 5, 5, 5), (4, 1), (4, 1)),
    ((1, 64, 7, 50, 40, 51), (3, 1), (3, 1)),        # nine blocks, cached form, five bounds a unit
    ((1, 64, 192, 1, 1, 1), (2, 1), (2, 1)),         # three key tiles, no mask
    ((1, 64, 90, 4, 2, 4), (2, 1), (2, 1)),          # the last block has 20 rows
    ((2, 20, 52, 13, 8, 14), (4, 1), (4, 1)),        # eleven key tiles: the ring's round and its remainder
    ((1, 24, 121, 8, 8, 8), (8, 1), (8, 1)),
    ((1, 12, 247, 11, 11, 11), (22, 1), (11, 3)),    # chains of 4 to 43 tiles
    ((1, 36, 1, 200, 200, 200), (2, 2), (2, 2)),     # one token a frame, key splits: rows that see none of a split
    ((1, 16, 336, 33, 1, 34), (3, 10), (3, 16)),     # long splits of the pipelined shape
    ((1, 32, 576, 3, 1, 3), (5, 3), (3, 5)),         # splits of ranges that are no plan tiles
    ((1, 16, 336, 20, 1, 21), (3, 15), (3, 15)),     # short splits
    ((1, 300, 40, 5, 5, 5), (1, 1), (2, 1)),         # whole tiles: seven blocks
    ((1, 512, 192, 3, 3, 3), (3, 1), (3, 1)),        # six: 48 rows per wavefront
    ((1, 500, 48, 5, 4, 5), (1, 1), (1, 1)),         # six, frame bounds in both row blocks of a wavefront
    ((1, 512, 250, 2, 2, 2), (2, 1), (2, 1)),        # eight
    ((1, 64, 161, 6, 1, 7), (1, 4), (1, 4)),         # six, splits
]


@pytest.mark.parametrize("shape,plain,fp8", CASES)
def test_ranges(shape, plain, fp8):
    B, H, T, kvf, qf, F = shape
    args = (nb.NFD_BF16, B, H, F, T, 64, kvf, qf)
    plan = nb.nfd_attn_plan(*args)
    blocks = -(-qf * T // 32)
    assert nb.nfd_attn_fwd_ranges(*args) == plain and nb.nfd_attn_fwd_ranges(*args, fp8kv=True) == fp8
    assert plain[1] == plan["n_splits"]
    for ranges, _ in (plain, fp8):
        assert ranges == plan["n_q_tiles"] or (ranges > plan["n_q_tiles"] and -(-blocks // ranges) <= 4)


@pytest.mark.gpu
@pytest.mark.parametrize("shape", [c[0] for c in CASES])
def test_forward_over_ranges(shape):
    B, H, T, kvf, qf, F = shape
    D, Sk, Sq = 64, kvf * T, qf * T
    gen = torch.Generator(device="cuda").manual_seed(wl.BASE_SEED + 5000 + T)
    q, k, v = (torch.randn((B, H, n * T, D), generator=gen, device="cuda").to(torch.bfloat16) for n in (qf, F, F))
    k[:, :, Sk:] = float("nan")
    v[:, :, Sk:] = float("nan")
    attn = nb.Attention("bf16")
    out = attn.forward(q, k, v, T, kv_frames=kvf, q_frames=qf)
    out_l, lse = attn.forward_lse(q, k, v, T, kv_frames=kvf, q_frames=qf)
    kc, vc, new = k.clone(), v.clone(), slice(Sk - Sq, Sk)
    kc[:, :, new] = vc[:, :, new] = float("nan")
    step = torch.empty_like(q)
    nb.nfd_kvcache_append_attn_fwd(attn.h, q, kc, vc, k[:, :, new].contiguous(), v[:, :, new].contiguous(), step, B, H, F, T, D, kvf, qf)
    nbytes = nb.nfd_fp8_cache_bytes(B, H, F, T, D)
    k8, v8 = (torch.full((nbytes,), 0x7F, dtype=torch.uint8, device="cuda") for _ in range(2))
    sc = torch.full((B, H), 6.0 / 448.0, device="cuda")
    out8 = torch.empty_like(q)
    nb.nfd_kvcache_append_fp8(attn.h, k8, v8, sc, sc, k[:, :, :Sk].contiguous(), v[:, :, :Sk].contiguous(), B, H, F, T, D, 0, kvf)
    nb.nfd_block_causal_attn_fwd_fp8kv(attn.h, q, k8, v8, sc, sc, out8, B, H, F, T, D, kvf, qf)
    torch.cuda.synchronize()
    assert torch.equal(step, out) and torch.equal(kc[:, :, :Sk], k[:, :, :Sk]) and torch.equal(vc[:, :, :Sk], v[:, :, :Sk])
    heads = sorted({0, B * H // 2, B * H - 1})  # the oracle on three heads, every row
    pick = lambda x: x.reshape(1, B * H, *x.shape[2:])[:, heads].float().cpu().numpy()
    hq, hk, hv = pick(q), pick(k[:, :, :Sk]), pick(v[:, :, :Sk])
    scale = np.float32(6.0 / 448.0)
    d8 = lambda x: f8.e4m3_decode(f8.quantize(x, np.full((1, len(heads), 1, 1), scale))) * np.float64(scale)
    ref = orc.block_causal_attn(hq, hk, hv, T, kv_frames=kvf, q_frames=qf)
    ref8 = orc.block_causal_attn(hq, d8(hk), d8(hv), T, kv_frames=kvf, q_frames=qf)
    for name, o, r in (("forward", out, ref), ("lse", out_l, ref), ("8-bit", out8, ref8)):
        got = pick(o).astype(np.float64)
        assert np.all(np.isfinite(got)) and np.abs(got - r).max() <= BF16_MAX_ABS, (name, np.abs(got - r).max())
        assert np.linalg.norm(got - r) <= BF16_REL_L2_INTERNAL * np.linalg.norm(r), (name, np.linalg.norm(got - r) / np.linalg.norm(r))
    s = (hq.astype(np.float64) @ np.swapaxes(hk.astype(np.float64), 2, 3)) / 8.0
    seen = np.arange(Sk)[None, :] // T <= kvf - qf + np.arange(Sq)[:, None] // T
    s = np.where(seen, s, -np.inf)
    m = s.max(-1)
    want = m + np.log(np.exp(s - m[..., None]).sum(-1))
    # exact products of bf16 inputs summed in fp32, fp32 exponentials and sums
    assert np.abs(pick(lse[..., None])[..., 0] - want).max() <= 2e-4
    attn.close()
