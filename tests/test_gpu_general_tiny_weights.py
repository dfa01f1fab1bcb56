"""The general path keeps weights below 2^-126, fp32's smallest normal number: their products with large values are ordinary
numbers.  Two keys whose scores differ by 130 binary orders; the lesser one's weight has 149 - 130 = 19 bits, and the
score's rounding (130 x 2^-23 binary orders at most, once for the scale and once for the sum) is 2.2e-5 of the weight: 5e-5."""
import pytest
import torch

from paper_2506_01380_amd import binding as nb

pytestmark = pytest.mark.gpu

LN2 = 0.6931471805599453


@pytest.mark.parametrize("D,n_keys", [(64, 2), (64, 130), (33, 20), (256, 40)])
def test_subnormal_weights_count(D, n_keys):
    T, big = 1, 2.0 ** 60
    q = torch.zeros((1, 1, 1, D), device="cuda")
    k = torch.zeros((1, 1, n_keys, D), device="cuda")
    v = torch.zeros_like(k)
    g = torch.zeros_like(q)
    q[..., 0] = 130.0 * LN2 * D ** 0.5
    k[:, :, 0, 0] = 1.0     # weight 1; all others 2^-130
    v[:, :, 1:, 1] = big
    g[..., 2] = big
    a = nb.Attention("fp32")
    out, lse = a.forward_lse(q, k, v, T, kv_frames=n_keys, q_frames=1)
    dv = a.backward(q, k, v, out, g, lse, T, kv_frames=n_keys, q_frames=1)[2]
    g2 = torch.zeros_like(q)
    g2[..., 1] = 1.0
    dk = a.backward(q, k, v, out, g2, lse, T, kv_frames=n_keys, q_frames=1)[1]
    a.close()
    w = 2.0 ** -130
    assert abs(out[0, 0, 0, 1].item() / ((n_keys - 1) * w * big) - 1.0) <= 5e-5
    assert (dv[0, 0, 1:, 2].double() / (w * big) - 1.0).abs().max() <= 5e-5
    want = w * big * D ** -0.5 * q[0, 0, 0, 0].item()  # of the lesser keys: the score's gradient is p (big - delta)
    assert (dk[0, 0, 1:, 0].double() / want - 1.0).abs().max() <= 5e-5
