"""Window moves (nfd_kvcache_shift, nfd_kvcache_shift_fp8) where the one-pass kernels can go wrong: chains of exactly,
one fewer and one more link than are read at a time, chains past the limit of the staged copy (with and without the
workspace for it), feature rows longer than one piece, element widths without 16-byte vectors.  Byte work: exact."""
import numpy as np
import pytest
import torch

from oracle import spec_driver as sd
from paper_2506_01380_amd import binding as nb

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,B,H,T,D,F,kv,drop,ws", [
    ("bf16", 1, 2, 8, 64, 9, 9, 1, 0),       # 8 links: one batch
    ("bf16", 1, 3, 8, 64, 11, 10, 1, 0),     # 9
    ("bf16", 2, 1, 8, 64, 8, 8, 1, 0),       # 7
    ("bf16", 1, 2, 12, 64, 40, 37, 5, 0),    # last link of a chain missing for part of the chains
    ("bf16", 1, 2, 4, 64, 99, 98, 1, 0),     # 97 links: staged copy
    ("bf16", 1, 2, 4, 64, 99, 98, 1, 1024),  # the same, no workspace for it
    ("bf16", 1, 2, 3, 33, 12, 11, 2, 0),     # two-byte units
    ("fp32", 1, 2, 5, 31, 20, 19, 3, 0),     # four-byte units
    ("bf16", 1, 2, 8, 64, 9, 9, 6, 0),       # three kept, six dropped: copied
    ("bf16", 1, 2, 8, 64, 9, 9, 5, 0),       # four kept, five dropped: chains of one link
    ("bf16", 1, 2, 3, 33, 12, 12, 6, 0),     # two-byte units, as many kept as dropped: copied
    ("fp32", 1, 2, 5, 31, 20, 19, 9, 0),     # one more kept: chains
])
def test_shift_bit_exact(dtype, B, H, T, D, F, kv, drop, ws):
    a = nb.Attention(dtype, workspace_bytes=ws)
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator(device="cuda").manual_seed(kv)
    k, v = (torch.randn((B, H, F * T, D), device="cuda", generator=g).to(td) for _ in range(2))
    hk, hv = k.float().cpu().numpy(), v.float().cpu().numpy()
    nb.nfd_kvcache_shift(a.h, k, v, B, H, F, T, D, kv, drop)
    keep = (kv - drop) * T
    for dev, host in ((k, hk), (v, hv)):
        got = dev.float().cpu().numpy()
        np.testing.assert_array_equal(got[:, :, :keep], sd.kvcache_shift(host, T, kv, drop)[:, :, :keep])
        np.testing.assert_array_equal(got[:, :, kv * T:], host[:, :, kv * T:])
    a.close()


@pytest.mark.parametrize("B,H,T,F,kv,drop", [
    (1, 1, 336, 100, 100, 1),  # a feature row of more than one piece of 2048 vectors; 99 links of K: staged
    (1, 2, 100, 24, 23, 3),    # T no multiple of 16: V key by key, 2000 keys, one piece
    (1, 1, 100, 24, 24, 1),    # ... 2300 keys, two pieces
    (2, 3, 48, 9, 9, 6),       # K and V copied
    (2, 3, 48, 9, 9, 5),       # chains, or copied off the boundary
    (2, 3, 37, 9, 8, 6),       # K copied, V key by key
])
@pytest.mark.parametrize("offset", [0, 4])  # 4: caches not 16-byte aligned
def test_shift_fp8_bit_exact(B, H, T, F, kv, drop, offset):
    from test_gpu_fp8 import _host_views, _spad, _v_physical
    a = nb.Attention("bf16")
    S, D, n = _spad(F, T), 64, nb.nfd_fp8_cache_bytes(B, H, F, T, 64)
    rng = np.random.default_rng(T)
    hk = rng.integers(0, 256, size=(B, H, S, D), dtype=np.uint8)
    hv = rng.integers(0, 256, size=(B, H, D, S), dtype=np.uint8)
    bufs = [torch.zeros(n + 16, dtype=torch.uint8, device="cuda")[offset:offset + n] for _ in range(2)]
    for b, x in zip(bufs, (hk, _v_physical(hv))):
        b.copy_(torch.from_numpy(x.reshape(-1)))
    nb.nfd_kvcache_shift_fp8(a.h, bufs[0], bufs[1], B, H, F, T, D, kv, drop)
    gk, gv = _host_views(bufs[0], bufs[1], B, H, F, T)
    keep = (kv - drop) * T
    assert np.array_equal(gk[:, :, :keep], hk[:, :, drop * T: kv * T]) and np.array_equal(gk[:, :, kv * T:], hk[:, :, kv * T:])
    assert np.array_equal(gv[..., :keep], hv[..., drop * T: kv * T]) and np.array_equal(gv[..., kv * T:], hv[..., kv * T:])
    a.close()


def test_shift_fp8_more_threads_than_a_launch():
    """2^18 heads have 2^24 feature rows: at one workgroup a row, 2^32 threads and more."""
    B, H, T, F = 512, 512, 16, 2
    n = nb.nfd_fp8_cache_bytes(B, H, F, T, 64)
    gen = torch.Generator(device="cuda").manual_seed(3)
    k8, v8 = (torch.randint(0, 2 ** 62, (n // 8,), device="cuda", generator=gen, dtype=torch.int64).view(torch.uint8) for _ in range(2))
    want_k, want_v = k8.view(B * H, 64, 64)[:, T:2 * T].clone(), v8.view(B * H * 64, 64)[:, T:2 * T].clone()
    a = nb.Attention("bf16")
    nb.nfd_kvcache_shift_fp8(a.h, k8, v8, B, H, F, T, 64, 2, 1)
    assert torch.equal(k8.view(B * H, 64, 64)[:, :T], want_k) and torch.equal(v8.view(B * H * 64, 64)[:, :T], want_v)
    a.close()


@pytest.mark.parametrize("dtype,T,D,F,kv,drop", [
    ("bf16", 97, 65, 9, 9, 4),   # two-byte units, 12.1 million chains a tensor
    ("bf16", 96, 64, 40, 37, 12),
    ("fp32", 33, 63, 12, 11, 9),  # fewer kept than dropped
])
def test_shift_many_chains(dtype, T, D, F, kv, drop):
    B, H = 8, 60
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    gen = torch.Generator(device="cuda").manual_seed(kv)
    k, v = (torch.randn((B, H, F * T, D), device="cuda", generator=gen).to(td) for _ in range(2))
    k0, v0 = k.clone(), v.clone()
    a = nb.Attention(dtype)
    nb.nfd_kvcache_shift(a.h, k, v, B, H, F, T, D, kv, drop)
    keep = (kv - drop) * T
    for x, x0 in ((k, k0), (v, v0)):
        assert torch.equal(x[:, :, :keep], x0[:, :, drop * T:kv * T]) and torch.equal(x[:, :, kv * T:], x0[:, :, kv * T:])
    a.close()
