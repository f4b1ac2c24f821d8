"""The scan and its backward on the fp32 matrix instructions at the edges of its pieces
(at most 64 tokens, nested with the memory chunks): chunks one token longer than
a piece, chunks of several pieces with a short last one, several short chunks
in a piece, chunk sizes that leave a piece ragged, every N, with and without
the optional inputs, against the oracle's recurrence and its reverse."""
import numpy as np
import pytest

import oracle
from paper_2608_02032_amd import dart, synth
from tests.helpers import assert_close_slices, f32_dev, to_dev, to_np
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


@pytest.mark.parametrize("c", SHAPES, ids=lambda c: "B%d_L%d_H%d_G%d_N%d_S%d_%s" % c)
def test_scan_f32_forward(c):
    import torch
    B, L, H, G, N, S, dtype = c
    w = synth.Workload("f32_%d_%d" % (N, S), B, L, H, 64, N, S, dtype, ngroups=G)
    print("\n[gpu-case] scan f32 %s" % (w,), flush=True)
    d = synth.forward_inputs(w, seed=L)
    h0 = (np.random.default_rng(L).standard_normal((B, H, N, 64)) * 0.05).astype(np.float32)
    x, Bm, Cm = (to_dev(d[k], dtype) for k in ("x", "Bm", "Cm"))
    M = w.nchunks
    mem = torch.full((B, M + 1, H, N, 64), 7.0, dtype=x.dtype, device="cuda")
    y, _, hl = dart.ssd_chunk_scan(x, f32_dev(d["dt"]), f32_dev(d["A"]), Bm, Cm, S, h0=f32_dev(h0), mem=mem)
    torch.cuda.synchronize()
    y_ref, hl_ref = oracle.ssd_recurrence(d["x"], d["dt"], d["A"], d["Bm"], d["Cm"], h0)
    mem_ref = oracle.chunk_memories(d["x"], d["dt"], d["A"], d["Bm"], S)
    # fp32 sums whatever the storage; outputs are rounded to it
    tol = 1e-5 if dtype == "fp32" else 2.0 ** -8
    assert_close_slices(to_np(y), y_ref, tol, what="y_ssd")
    assert_close_slices(to_np(mem)[:, :M], mem_ref, tol, axes_keep=(0, 1, 2), what="mem")
    assert_close_slices(to_np(hl), hl_ref, 1e-5, axes_keep=(0, 1), what="h_last")
    assert np.all(to_np(mem)[:, M:] == 7.0)


@pytest.mark.parametrize("N,S", [(16, 16), (64, 5), (128, 32), (64, 64)])
def test_strong_decays_keep_their_precision(N, S):
    """Decays of e^-0.8 to e^-1.6 a token: sums over a tile reach 37 (log2), the decays between
    tokens that still count are a few, and must not carry the rounding of the
    sums (2^-24 of 37 is 1.5e-6 of a decay).  A memory and an output are then a few
    tokens' terms with about four roundings of 2^-24 each, in the 2-norm over
    all of them at most their sum."""
    import torch
    w = synth.Workload("decays", 2, 200, 2, 64, N, S, "fp32")
    print("\n[gpu-case] scan decays %s" % (w,), flush=True)
    d = synth.forward_inputs(w, seed=N + S)
    rng = np.random.default_rng(S)
    dt = rng.uniform(0.05, 0.1, d["dt"].shape).astype(np.float32)
    A = np.full(2, -16.0, dtype=np.float32)
    y, mem, _ = dart.ssd_chunk_scan(*(f32_dev(v) for v in (d["x"], dt, A, d["Bm"], d["Cm"])), S)
    torch.cuda.synchronize()
    y_ref, _ = oracle.ssd_recurrence(d["x"], dt, A, d["Bm"], d["Cm"])
    for what, got, ref in (("mem", mem, oracle.chunk_memories(d["x"], dt, A, d["Bm"], S)), ("y", y, y_ref)):
        err = float(np.linalg.norm(to_np(got) - ref) / np.linalg.norm(ref))
        print("  %s 2-norm rel err %.2e" % (what, err), flush=True)
        assert err <= 4 * 2.0 ** -24, what


@pytest.mark.parametrize("N,S,dtype", [(16, 16, "fp32"), (64, 16, "fp32"), (128, 32, "fp32"), (64, 5, "fp32")])
def test_gradient_of_C_keeps_the_precision_of_short_sums(N, S, dtype):
    """dC_s is 64 products over p with the entering state and up to 64 over the piece's tokens.  Formed of
    sums of 8, a result carries about 4 roundings of its chains, 3 of the tree
    over them and 3 of the factors (2^-24, 2.5e-8 in the root mean square each: 8e-8)
    beside the state's own 9e-8: 1.2e-7 in all, 1.9e-7 in one chain.  The bound
    lies between."""
    import torch
    w = synth.Workload("dC", 2, 500, 4, 64, N, S, dtype)
    print("\n[gpu-case] scan dC %s" % (w,), flush=True)
    d = synth.forward_inputs(w, seed=N + S)
    dy = np.random.default_rng(S).standard_normal((2, 500, 4, 64)).astype(np.float32)
    got = dart.ssd_bwd(*(f32_dev(d[k]) for k in ("x", "dt", "A", "Bm", "Cm")), S, f32_dev(dy))
    torch.cuda.synchronize()
    ref = oracle.ssd_bwd(d["x"], d["dt"], d["A"], d["Bm"], d["Cm"], S, dy)["dC"]
    err = float(np.linalg.norm(to_np(got["dC"]) - ref) / np.linalg.norm(ref))
    print("  dC 2-norm rel err %.2e" % err, flush=True)
    assert err <= 1.5e-7
