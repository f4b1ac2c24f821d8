"""The attention kernels on the fp32 matrix instructions, forward and backward,
at the edges of their tiles: 16 tokens of a wave in several chunks, blocks of 64
tokens cut by the end of the sequence, every N, chunk sizes around 16 and 64,
and both block shapes of the memory side (one memory of up to 64 rows per
block; as many memories as the registers hold when that leaves two blocks per
CU), against the oracle with the metrics of the other attention tests."""
import numpy as np
import pytest

import oracle
from paper_2608_02032_amd import synth
from tests.helpers import TOL, assert_close_slices, assert_lse_close, f32_dev, to_np
from tests import test_gpu_sma_bwd as MB
from tests.test_gpu_parity import run_sma, sma_case

pytestmark = pytest.mark.gpu

# B, L, H, G, N, S, dtype, z_per_head
SHAPES = [
    (1, 66, 2, 1, 16, 5, "fp32", True),      # a wave spans four chunks
    (2, 129, 3, 1, 32, 17, "fp32", False),   # chunks of 16 tokens and one
    (1, 127, 4, 2, 64, 63, "bf16", True),
    (1, 193, 2, 2, 128, 65, "bf16", False),
    (1, 257, 3, 1, 128, 64, "fp32", True),   # fp32 storage at a tuned chunk size
    (1, 65, 2, 1, 64, 64, "fp32", True),     # one token with a memory
    (32, 256, 4, 1, 64, 16, "fp32", True),   # full memory blocks: four memories
    (8, 200, 4, 1, 128, 12, "fp32", True),   # ... two memories of 128 rows, the last block half empty
    (64, 100, 4, 1, 16, 5, "fp32", True),    # ... sixteen memories
    (64, 120, 4, 1, 32, 7, "bf16", True),    # ... eight memories
]


@pytest.mark.parametrize("c", SHAPES, ids=lambda c: "B%d_L%d_H%d_G%d_N%d_S%d_%s" % c[:7])
def test_sma_f32_forward_and_backward(c):
    B, L, H, G, N, S, dtype, zh = c
    w = synth.Workload("f32_%d_%d" % (N, S), B, L, H, 64, N, S, dtype, ngroups=G, z_per_head=zh)
    print("\n[gpu-case] sma f32 %s" % (w,), flush=True)
    d, mem, y_ssd, dy = MB.bwd_case(w, seed=L)
    y, lse = run_sma(w, d, mem, y_ssd)
    y_ref, lse_ref = oracle.sma(d["q"], d["e"], d["Cm"], mem, d["z"], y_ssd, S)
    # fp32 sums whatever the storage; outputs are rounded to it
    assert_close_slices(to_np(y), y_ref, TOL[dtype] if dtype == "fp32" else 2.0 ** -8, what="y")
    assert_lse_close(to_np(lse), lse_ref, "fp32")
    np.testing.assert_array_equal(to_np(y)[:, :S], y_ssd[:, :S].astype(np.float64))
    got = MB.run_gpu(w, d, mem, y_ssd, dy)
    MB.check(w, got, d, mem, dy)


@pytest.mark.parametrize("N,dtype", [(16, "bf16"), (16, "fp32"), (32, "fp32"), (64, "fp32"), (128, "fp32")])
@pytest.mark.parametrize("S", [9, 30, 100])
def test_forward_split_and_whole(N, dtype, S):
    """The forward's two forms on either side of the line between them (one block
    of 64 tokens per CU): 200 tokens are four blocks per (b, h), the last 16-token
    one half empty, with none to 22 memories over the four waves; both against
    the oracle, and against each other on the sequences they share."""
    import torch

    cus = torch.cuda.get_device_properties(0).multi_processor_count
    B, L, H = cus // 4 + 1, 200, 1
    w = synth.Workload("split_%d_%d" % (N, S), B, L, H, 64, N, S, dtype, ngroups=1, z_per_head=True)
    print("\n[gpu-case] sma forms %s" % (w,), flush=True)
    d, mem, y_ssd = sma_case(w, seed=S + N)
    y, lse = run_sma(w, d, mem, y_ssd)
    few = synth.Workload("few", B - 1, L, H, 64, N, S, dtype, ngroups=1, z_per_head=True)
    y1, lse1 = run_sma(few, {k: v[:B - 1] if getattr(v, "ndim", 0) > 1 else v for k, v in d.items()}, mem[:B - 1], y_ssd[:B - 1])
    y_ref, lse_ref = oracle.sma(d["q"], d["e"], d["Cm"], mem, d["z"], y_ssd, S)
    tol = TOL[dtype] if dtype == "fp32" else 2.0 ** -8
    assert_close_slices(to_np(y), y_ref, tol, what="whole")
    assert_close_slices(to_np(y1), y_ref[:-1], tol, what="split")
    assert_lse_close(to_np(lse), lse_ref, "fp32")
    assert_lse_close(to_np(lse1), lse_ref[:-1], "fp32")
    assert_close_slices(to_np(y1), to_np(y)[:-1], tol, what="split against whole")


@pytest.mark.parametrize("N,S", [(32, 17), (64, 100), (128, 32)])
def test_bf16_forward_rounds_no_operand(N, S):
    """bf16 storage outside the bf16 kernels' shapes: the logits carry fp32 roundings only.
    With one memory attended the log-sum-exp is the logit, whose terms have a
    root mean square of sqrt(P) = 8 in all; 16 independent roundings of 2^-24 of it
    are 8 x 4 x 2^-24 = 1.9e-6, and twice that is the bound.  (An Ebar of 16 bits
    alone gives 8 x 2^-17 / sqrt(6) = 2.5e-5.)"""
    L = 2 * S
    w = synth.Workload("round_%d" % N, 3, L, 4, 64, N, S, "bf16", ngroups=2)
    print("\n[gpu-case] sma logits %s" % (w,), flush=True)
    d, mem, y_ssd = sma_case(w, seed=N)
    rng = np.random.default_rng(N)
    qw, ew = (rng.uniform(0.5, 1.5, n).astype(np.float32) for n in (N, 64))
    for kw in ({}, dict(q_norm_w=qw, e_norm_w=ew)):
        _, lse = run_sma(w, d, mem, y_ssd, **{k: f32_dev(v) for k, v in kw.items()})
        _, ref = oracle.sma(d["q"], d["e"], d["Cm"], mem, d["z"], y_ssd, S, **kw)
        rms = float(np.sqrt(np.mean((to_np(lse)[:, S:] - ref[:, S:]) ** 2)))
        print("  rms of the logits' error %.3e" % rms, flush=True)
        assert rms <= 2 * 8 * 4 * 2.0 ** -24


@pytest.mark.parametrize("zh", [True, False])
@pytest.mark.parametrize("N,S,dtype", [(32, 17, "bf16"), (32, 32, "bf16"), (64, 17, "bf16"), (64, 32, "bf16"),
                                       (128, 17, "bf16"), (128, 32, "bf16"), (16, 30, "bf16"), (64, 30, "fp32")])
def test_forward_options(N, S, dtype, zh):
    """normalize = 0, and norm weights with y in place of y_ssd, for one gate per head and
    one per token, over a last block of 64 tokens cut to 22; at N 16 and in fp32 with
    more such blocks than CUs, past which the whole-block form runs."""
    import torch

    many = torch.cuda.get_device_properties(0).multi_processor_count // 4 + 1
    w = synth.Workload("opts_%d_%d" % (N, S), many if N == 16 or dtype == "fp32" else 1, 214, 2, 64, N, S, dtype,
                       ngroups=2, z_per_head=zh)
    print("\n[gpu-case] sma options %s" % (w,), flush=True)
    d, mem, y_ssd = sma_case(w, seed=S + N)
    rng = np.random.default_rng(N)
    qw, ew = (rng.uniform(0.5, 1.5, n).astype(np.float32) for n in (N, 64))
    for inplace, kw in ((False, dict(normalize=False)), (True, dict(q_norm_w=qw, e_norm_w=ew))):
        y, lse = run_sma(w, d, mem, y_ssd, inplace=inplace,
                         **{k: f32_dev(v) if k != "normalize" else v for k, v in kw.items()})
        y_ref, lse_ref = oracle.sma(d["q"], d["e"], d["Cm"], mem, d["z"], y_ssd, S, **kw)
        assert_close_slices(to_np(y), y_ref, TOL[dtype] if dtype == "fp32" else 2.0 ** -8, what="y %s" % sorted(kw))
        assert_lse_close(to_np(lse), lse_ref, "fp32")
        np.testing.assert_array_equal(to_np(y)[:, :S], y_ssd[:, :S].astype(np.float64))


@pytest.mark.parametrize("N,S,dtype", [(16, 16, "fp32"), (64, 16, "fp32"), (64, 5, "fp32")])
def test_weights_carry_no_rounding_of_a_scaled_logit(N, S, dtype):
    """With 1/sqrt(N) a power of two a logit is its dot product's rounding alone,
    and a weight exp(l - max) takes one more of the difference.  Logits scaled by
    log2(e) before the difference are rounded at their own size as well, and dC,
    whose terms cancel, shows it: 5.9e-7 to 7.9e-7 against 3.2e-7 to 4.6e-7.  The
    bound lies between."""
    import torch
    w = synth.Workload("logits", 2, 500, 4, 64, N, S, dtype)
    print("\n[gpu-case] sma logits %s" % (w,), flush=True)
    d, mem, y_ssd, dy = MB.bwd_case(w, seed=N + S)
    got = MB.run_gpu(w, d, mem, y_ssd, dy)
    ref = oracle.sma_bwd(d["q"], d["e"], d["Cm"], mem, d["z"], dy, S)["dC"]
    err = float(np.linalg.norm(got["dC"] - ref) / np.linalg.norm(ref))
    print("  dC 2-norm rel err %.2e" % err, flush=True)
    assert err <= 5.2e-7
