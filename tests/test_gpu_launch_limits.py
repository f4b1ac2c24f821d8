"""Calls whose blocks number more than one launch dimension takes: a launch has
fewer than 2^32 threads along x, so kernels of 512 and 1024 threads reach the
limit at 2^23 and 2^22 blocks."""
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
