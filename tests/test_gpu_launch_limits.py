"""Calls whose blocks number more than one launch dimension takes: a launch has
fewer than 2^32 threads along x, so kernels of 512 and 1024 threads reach the
limit at 2^23 and 2^22 blocks."""
import numpy as np
import pytest

from paper_2608_02032_amd import dart

pytestmark = pytest.mark.gpu


def test_sma_forward_of_a_very_large_batch():
    """65535 x 129 (batch, head) pairs of one token, bf16, S 16: a block each."""
    import torch
    B, H, N, S = 65535, 129, 32, 16
    print("\n[gpu-case] sma of %d pairs" % (B * H), flush=True)
    q, Cm = (torch.ones(B, 1, 1, N, dtype=torch.bfloat16, device="cuda") for _ in range(2))
    e = torch.ones(B, 1, 1, 64, dtype=torch.bfloat16, device="cuda")
    z = torch.ones(B, 1, H, dtype=torch.bfloat16, device="cuda")
    ys = torch.randn(B, 1, H, 64, dtype=torch.bfloat16, device="cuda")
    mem = torch.zeros(1, 1, 1, N, 64, dtype=torch.bfloat16, device="cuda")  # one chunk: never read
    y, lse = dart.sma_fwd(q, e, Cm, mem, z, ys, S)
    torch.cuda.synchronize()
    assert torch.equal(y, ys) and bool(torch.isneginf(lse).all())


def test_dt_softplus_bwd_of_very_many_heads():
    """2^28 heads: the sums over rows take 2^22 blocks of 1024 threads."""
    import torch
    H = 1 << 28
    print("\n[gpu-case] dt softplus bwd of %d heads" % H, flush=True)
    raw = torch.randn(1, H, dtype=torch.bfloat16, device="cuda")
    ddt = torch.randn(1, H, device="cuda")
    bias = torch.zeros(H, device="cuda")
    draw, dbias = dart.dt_softplus_bwd(raw, ddt, bias=bias)
    torch.cuda.synchronize()
    assert torch.equal(draw[0], dbias)  # one row
    for s in (slice(0, 4096), slice(H // 2, H // 2 + 4096), slice(H - 4096, H)):
        ref = ddt[0, s].double() * torch.sigmoid(raw[0, s].double())
        # the hardware exponential and an IEEE division: a few 2^-24 of the value
        assert float(((draw[0, s].double() - ref).abs() / ref.abs().clamp_min(1e-30)).max()) < 2e-6


def test_decode_updates_every_state_once():
    """65535 x 129 (batch, head) pairs with a memory each: the streaming kernel's blocks fill more
    than one row of its grid, whose last row is not full, and the state updates
    run in a kernel of their own (a cache of 17 GB)."""
    import torch
    torch.cuda.empty_cache()
    B, H, N, S, pos = 65535, 129, 16, 16, 20
    print("\n[gpu-case] decode of %d pairs" % (B * H), flush=True)
    bf = dict(dtype=torch.bfloat16, device="cuda")
    x = torch.zeros(B, H, 64, **bf)
    dt = torch.full((B, H), 0.1, device="cuda")
    A = torch.full((H,), -1.0, device="cuda")
    Bm, Cm, q = (torch.ones(B, 1, N, **bf) for _ in range(3))
    e, z = torch.ones(B, 1, 64, **bf), torch.zeros(B, H, **bf)
    hs, ca = (torch.ones(B, H, N, 64, device="cuda") for _ in range(2))
    mem = torch.ones(B, 1, H, N, 64, **bf)
    y = dart.decode_step(pos, x, dt, A, Bm, Cm, q, e, z, hs, ca, mem, S)
    torch.cuda.synchronize()
    a = float(np.exp(np.float64(np.float32(0.1)) * -1.0))
    for t in (hs, ca):
        for v in torch.aminmax(t):
            assert abs(float(v) - a) < 1e-6
    assert abs(float(y.float().max()) - N * a) < 0.05 and abs(float(y.float().min()) - N * a) < 0.05
    del hs, ca, mem
    torch.cuda.empty_cache()
