"""The score kernel of the bf16 attention backward, whose two half sums meet a
step late: one step per workgroup, one memory per head with several heads (the
sums of one head meet after the next head's tiles have arrived), tokens past
the end, both block shapes, with and without the query residual that RMSNorm
weights bring in."""
import numpy as np
import pytest

from paper_2608_02032_amd import synth
from tests.helpers import f32_dev
from tests import test_gpu_sma_bwd as MB

pytestmark = pytest.mark.gpu

# L, H, N, S, heads per block
SHAPES = [
    (65, 1, 64, 64, 1),     # one token, one step
    (130, 4, 32, 64, 4),    # heads change at every step, then every two
    (257, 2, 128, 256, 2),  # blocks of 128 tokens, one token
    (511, 4, 64, 128, 4),
    (320, 4, 128, 64, 4),
]


@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("c", SHAPES, ids=lambda c: "L%d_H%d_N%d_S%d" % c[:4])
def test_scores_a_step_late(c, weighted, monkeypatch):
    L, H, N, S, hpb = c
    w = synth.Workload("late_%d_%d" % (N, S), 2, L, H, 64, N, S, "bf16")
    print("\n[gpu-case] sma bwd steps %s" % (w,), flush=True)
    monkeypatch.setenv("DART_SMA_HEADS_PER_BLOCK", str(hpb))
    d, mem, y_ssd, dy = MB.bwd_case(w, seed=L)
    if not weighted:
        MB.check(w, MB.run_gpu(w, d, mem, y_ssd, dy), d, mem, dy)
        return
    rng = np.random.default_rng(N)
    qw = (1.0 + 0.2 * rng.standard_normal(N)).astype(np.float32)
    ew = (1.0 + 0.2 * rng.standard_normal(64)).astype(np.float32)
    got = MB.run_gpu(w, d, mem, y_ssd, dy, q_norm_w=f32_dev(qw), e_norm_w=f32_dev(ew))
    MB.check(w, got, d, mem, dy, q_norm_w=qw, e_norm_w=ew)
