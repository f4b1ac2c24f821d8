"""Backward of the block kernels where their launch forms change: four channels
per thread in the convolution (channel counts and strides that are multiples
of 4, runs of 32 tokens and their remainders, sequences shorter than the
filter), rows tiled over few or many heads in the step sizes, and two to eight
register pieces of 256 channels per row in the gated RMSNorm."""
import numpy as np
import pytest

import oracle
from paper_2608_02032_amd import dart, synth
from tests.helpers import assert_close_slices, f32_dev, to_dev, to_np

pytestmark = pytest.mark.gpu

# sums of n fp32 products in any order: about sqrt(n) 2^-24 of the largest, with
# the hardware exponential and reciprocal (a few ulp per element) on top
TOL = 2e-5


@pytest.mark.parametrize("dtype,B,L,C,pad", [("bf16", 1, 1, 4, 0), ("fp32", 2, 2, 8, 4), ("bf16", 2, 3, 260, 8),
                                             ("fp32", 1, 32, 64, 0), ("bf16", 3, 33, 252, 4), ("bf16", 2, 130, 512, 12)])
@pytest.mark.parametrize("with_state", [False, True])
def test_conv1d_silu_bwd_four_channels_per_thread(dtype, B, L, C, pad, with_state):
    import torch
    print("\n[gpu-case] conv1d bwd v4 %s B=%d L=%d C=%d pad=%d state=%s" % (dtype, B, L, C, pad, with_state), flush=True)
    rng = np.random.default_rng(L + C)
    x = synth.to_storage(rng.standard_normal((B, L, C + pad)).astype(np.float32), dtype)
    w = (rng.standard_normal((C, 4)) * 0.5).astype(np.float32)
    bias = (rng.standard_normal(C) * 0.1).astype(np.float32)
    st0 = rng.standard_normal((B, C, 3)).astype(np.float32) if with_state else None
    dout = rng.standard_normal((B, L, C)).astype(np.float32)
    dbuf = torch.full((B, L, C + pad + 4), 7.0, dtype=torch.float32, device="cuda")
    g = dart.conv1d_silu_bwd(to_dev(x, dtype), f32_dev(w), f32_dev(dout), bias=f32_dev(bias),
                             state_in=f32_dev(st0) if with_state else None, channels=C,
                             din=dbuf[:, :, 4:4 + C], want_state=True)
    torch.cuda.synchronize()
    ref = oracle.conv1d_silu_bwd(x[:, :, :C], w, dout, bias=bias, state=st0)
    assert_close_slices(to_np(g["din"]), ref["din"], TOL, axes_keep=(), what="din")
    assert_close_slices(to_np(g["dweight"]), ref["dw"], TOL, axes_keep=(), what="dweight")
    assert_close_slices(to_np(g["dbias"]), ref["db"], TOL, axes_keep=(), what="dbias")
    assert_close_slices(to_np(g["dstate"]), ref["dstate"], TOL, axes_keep=(), what="dstate")
    b = to_np(dbuf)
    assert np.all(b[:, :, :4] == 7.0) and np.all(b[:, :, 4 + C:] == 7.0)


@pytest.mark.parametrize("rows,H", [(1, 1), (257, 24), (256, 256), (513, 300), (4100, 7)])
def test_dt_softplus_bwd_row_tiles(rows, H):
    import torch
    print("\n[gpu-case] dt softplus bwd rows=%d H=%d" % (rows, H), flush=True)
    rng = np.random.default_rng(rows + H)
    raw = synth.to_storage((rng.standard_normal((rows, H + 3)) * 4).astype(np.float32), "bf16")
    bias = rng.standard_normal(H).astype(np.float32)
    ddt = rng.standard_normal((rows, H)).astype(np.float32)
    draw, dbias = dart.dt_softplus_bwd(to_dev(raw, "bf16"), f32_dev(ddt), bias=f32_dev(bias), nheads=H)
    torch.cuda.synchronize()
    rr, rb = oracle.dt_softplus_bwd(raw[:, :H], ddt, bias=bias)
    assert_close_slices(to_np(draw), rr, TOL, axes_keep=(), what="draw")
    assert_close_slices(to_np(dbias), rb, TOL, axes_keep=(), what="dbias")


@pytest.mark.parametrize("dtype,rows,D,group", [("bf16", 1, 512, 512), ("fp32", 17, 520, 520), ("bf16", 33, 1024, 1024),
                                                ("bf16", 15, 1536, 1536), ("fp32", 31, 1544, 1544), ("bf16", 50, 4096, 2048)])
def test_gated_rmsnorm_bwd_register_pieces(dtype, rows, D, group):
    import torch
    print("\n[gpu-case] gated rmsnorm bwd %s rows=%d D=%d group=%d" % (dtype, rows, D, group), flush=True)
    rng = np.random.default_rng(rows + D)
    y = synth.to_storage(rng.standard_normal((rows, D)).astype(np.float32), dtype)
    z = synth.to_storage(rng.standard_normal((rows, D)).astype(np.float32), dtype)
    w = (1 + 0.1 * rng.standard_normal(D)).astype(np.float32)
    dout = rng.standard_normal((rows, D)).astype(np.float32)
    g = dart.gated_rmsnorm_bwd(to_dev(y, dtype), to_dev(z, dtype), f32_dev(dout), weight=f32_dev(w), group=group)
    torch.cuda.synchronize()
    ref = oracle.gated_rmsnorm_bwd(y, z, dout, w=w, group=group)
    for k in ("dy", "dz"):
        assert_close_slices(to_np(g[k]), ref[k], TOL, axes_keep=(0,), what=k)
    assert_close_slices(to_np(g["dweight"]), ref["dw"], TOL, axes_keep=(), what="dweight")


@pytest.mark.parametrize("dtype,B,L,C,pad", [("bf16", 300, 1, 4, 0), ("fp32", 260, 2, 8, 4), ("bf16", 130, 3, 260, 8),
                                             ("fp32", 260, 32, 64, 0), ("bf16", 130, 33, 252, 4), ("bf16", 27, 130, 512, 12)])
@pytest.mark.parametrize("with_state", [False, True])
def test_conv1d_silu_bwd_four_channels_and_many_blocks(dtype, B, L, C, pad, with_state):
    """The form of four channels per thread runs where its blocks of 64 threads outnumber the compute
    units (256); with fewer a thread takes one channel."""
    assert B * -(-L // 32) * -(-C // 256) > 256
    test_conv1d_silu_bwd_four_channels_per_thread(dtype, B, L, C, pad, with_state)


@pytest.mark.parametrize("rows,H", [(1, 4), (3, 4), (65, 4), (256, 1), (1000, 3), (2, 300)])
def test_dt_softplus_bwd_few_heads_and_rows(rows, H):
    """Blocks of fewer threads than the most, and halves of odd numbers of row sums."""
    test_dt_softplus_bwd_row_tiles(rows, H)


@pytest.mark.parametrize("rows", [1, 2, 17, 32, 33, 49])
def test_weight_sums_of_few_and_more_partial_rows(rows):
    """One block of 16 rows, one row in the last, and one, two, three and four partial rows to add."""
    test_gated_rmsnorm_bwd_register_pieces("bf16", rows, 264, 264)
