"""The scan backward on the fp32 matrix instructions at the edges of its pieces
(at most 64 tokens, nested with the memory chunks): chunks one token longer than
a piece, chunks of several pieces with a short last one, several short chunks
in a piece, chunk sizes that leave a piece ragged, every N, with and without
the optional inputs, against the oracle's reverse recurrence."""
import pytest

from paper_2608_02032_amd import synth
from tests import test_gpu_scan_bwd as SB

pytestmark = pytest.mark.gpu

# B, L, H, G, N, S, dtype
SHAPES = [
    (1, 131, 2, 1, 16, 65, "fp32"),     # pieces of 64 and 1 token
    (2, 700, 3, 1, 32, 300, "fp32"),    # five pieces a chunk, the last of 44; a partial last chunk
    (1, 200, 4, 2, 64, 5, "fp32"),      # twelve chunks in a piece of 60 tokens
    (1, 190, 2, 1, 128, 63, "bf16"),
    (1, 97, 6, 3, 128, 1, "fp32"),
    (2, 64, 16, 1, 64, 16, "fp32"),     # one piece
    (9, 1030, 8, 1, 64, 64, "fp32"),    # several heads per block
    (3, 520, 16, 2, 128, 128, "fp32"),
]


@pytest.mark.parametrize("c", SHAPES, ids=lambda c: "B%d_L%d_H%d_G%d_N%d_S%d_%s" % c)
@pytest.mark.parametrize("extras", [True, False])
def test_scan_f32_backward(c, extras):
    B, L, H, G, N, S, dtype = c
    w = synth.Workload("f32_%d_%d" % (N, S), B, L, H, 64, N, S, dtype, ngroups=G)
    SB.run_case(w, seed=L + S, with_dmem=True, with_dhl=extras, with_h0=extras, mcap=w.nchunks + 2 if extras else 0)
