"""The general path keeps infinities and NaNs where the mask says: a row must not change, bit for bit, whatever later
frames hold, nor a key's gradients whatever rows that cannot see it hold, also where frames meet inside a block of 16 rows
or keys.  An infinity that is seen comes out as that infinity, also from the last row of a ragged block."""
import pytest
import torch

from paper_2506_01380_amd import binding as nb

pytestmark = pytest.mark.gpu

SHAPES = [
    ("fp32", 1, 2, 20, 64, 3, 3),
    ("fp32", 1, 2, 5, 64, 9, 7),      # four frames in a block
    ("fp32", 1, 3, 1, 32, 40, 40),    # a frame a row
    ("fp32", 4, 24, 95, 64, 8, 8),    # two column blocks per workgroup
    ("fp32", 1, 2, 21, 129, 6, 6),
    ("fp32", 1, 1, 40, 256, 3, 2),
    ("bf16", 1, 2, 33, 62, 3, 3),
    ("bf16", 1, 2, 100, 128, 4, 2),
]


def _inputs(dtype, B, H, T, D, kvf, qf):
    td = torch.float32 if dtype == "fp32" else torch.bfloat16
    gen = torch.Generator(device="cuda").manual_seed(T + D)
    mk = lambda frames: torch.randn((B, H, frames * T, D), device="cuda", generator=gen).to(td)
    return mk(qf), mk(kvf), mk(kvf), mk(qf)


@pytest.mark.parametrize("dtype,B,H,T,D,kvf,qf", SHAPES)
def test_later_frames_do_not_reach_earlier_rows(dtype, B, H, T, D, kvf, qf):
    q, k, v, g = _inputs(dtype, B, H, T, D, kvf, qf)
    a = nb.Attention(dtype)
    out, lse = a.forward_lse(q, k, v, T, kvf, qf)
    dq = a.backward(q, k, v, out, g, lse, T, kvf, qf)[0]
    for bad in (float("nan"), float("inf"), float("-inf")):
        k2, v2 = k.clone(), v.clone()
        k2[:, :, (kvf - 1) * T:] = bad
        v2[:, :, (kvf - 1) * T:] = bad
        out2, lse2 = a.forward_lse(q, k2, v2, T, kvf, qf)
        dq2 = a.backward(q, k2, v2, out, g, lse, T, kvf, qf)[0]
        early = (qf - 1) * T
        assert torch.equal(out2[:, :, :early], out[:, :, :early]), bad
        assert torch.equal(lse2[:, :, :early], lse[:, :, :early]), bad
        assert torch.equal(dq2[:, :, :early], dq[:, :, :early]), bad
        assert not torch.isfinite(out2[:, :, early:]).any(), bad
    a.close()


@pytest.mark.parametrize("dtype,B,H,T,D,kvf,qf", SHAPES)
def test_blind_rows_do_not_reach_a_key(dtype, B, H, T, D, kvf, qf):
    q, k, v, g = _inputs(dtype, B, H, T, D, kvf, qf)
    a = nb.Attention(dtype)
    out, lse = a.forward_lse(q, k, v, T, kvf, qf)
    dq, dk, dv = a.backward(q, k, v, out, g, lse, T, kvf, qf)
    hidden = (kvf - qf + 1) * T  # from this key on, the first query frame sees nothing
    for bad in (float("nan"), float("inf")):
        q2, g2, o2, l2 = q.clone(), g.clone(), out.clone(), lse.clone()
        for x in (q2, g2, o2, l2):
            x[:, :, :T] = bad
        eq, ek, ev = a.backward(q2, k, v, o2, g2, l2, T, kvf, qf)
        assert torch.equal(ek[:, :, hidden:], dk[:, :, hidden:]) and torch.equal(ev[:, :, hidden:], dv[:, :, hidden:]), bad
        assert torch.equal(eq[:, :, T:], dq[:, :, T:]), bad
    a.close()


@pytest.mark.parametrize("dtype,B,H,T,D,kvf,qf", SHAPES)
def test_a_seen_infinity_stays_one(dtype, B, H, T, D, kvf, qf):
    q, k, v, g = _inputs(dtype, B, H, T, D, kvf, qf)
    a = nb.Attention(dtype)
    out, lse = a.forward_lse(q, k, v, T, kvf, qf)
    dv = a.backward(q, k, v, out, g, lse, T, kvf, qf)[2]
    v2 = v.clone()
    v2[:, :, -1, 0] = float("inf")
    out2 = a.forward(q, k, v2, T, kvf, qf)
    assert (out2[:, :, (qf - 1) * T:, 0] == float("inf")).all() and torch.equal(out2[:, :, :(qf - 1) * T], out[:, :, :(qf - 1) * T])
    assert torch.equal(out2[..., 1:], out[..., 1:])
    g2 = g.clone()
    g2[:, :, -1, 0] = float("inf")
    dv2 = a.backward(q, k, v, out, g2, lse, T, kvf, qf)[2]
    assert (dv2[..., 0] == float("inf")).all() and torch.equal(dv2[..., 1:], dv[..., 1:])
    a.close()
