"""An infinity or NaN in one token's inputs reaches what depends on that token and
nothing else, where the kernels multiply whole tiles of tokens and memories by
factors that are zero for the pairs that do not belong together: tokens before
it in its tile, memories of other chunks in its piece."""
import numpy as np
import pytest

import oracle
from paper_2608_02032_amd import dart, synth
from tests.helpers import assert_close_slices, f32_dev, to_dev, to_np

pytestmark = pytest.mark.gpu

BAD = [float("nan"), float("inf")]


def same_finite(got, ref, tol, what):
    """Finite where the reference is, and close to it there."""
    got = np.asarray(got, dtype=np.float64)
    fin = np.isfinite(ref)
    assert np.array_equal(np.isfinite(got), fin), "%s: %d of %d entries differ in being finite" % (
        what, int((np.isfinite(got) != fin).sum()), fin.size)
    scale = np.abs(ref[fin]).max()
    assert np.abs(got[fin] - ref[fin]).max() <= tol * scale, what


@pytest.mark.parametrize("N,S,dtype", [(16, 16, "fp32"), (64, 6, "fp32"), (32, 17, "bf16"), (128, 32, "fp32"),
                                       (16, 100, "bf16"), (64, 64, "fp32")])
@pytest.mark.parametrize("bad", BAD)
def test_scan_keeps_a_token_to_itself_and_later_ones(N, S, dtype, bad):
    import torch
    B, L, H, t0 = 2, 90, 4, 37
    w = synth.Workload("nonfinite_%d_%d" % (N, S), B, L, H, 64, N, S, dtype, ngroups=2)
    print("\n[gpu-case] scan %s %s" % (bad, w), flush=True)
    clean = synth.forward_inputs(w, seed=N + S)
    # fp32 sums whatever the storage; outputs are rounded to it
    tol = 1e-5 if dtype == "fp32" else 2.0 ** -8
    for name, at in (("x", (0, t0, 1, 7)), ("Bm", (0, t0, 0, 3)), ("Cm", (1, t0, 1, 2))):
        d = dict(clean)
        d[name] = clean[name].copy()
        d[name][at] = bad
        x, Bm, Cm = (to_dev(d[k], dtype) for k in ("x", "Bm", "Cm"))
        y, mem, hl = dart.ssd_chunk_scan(x, f32_dev(d["dt"]), f32_dev(d["A"]), Bm, Cm, S)
        torch.cuda.synchronize()
        with np.errstate(all="ignore"):
            y_ref, hl_ref = oracle.ssd_recurrence(d["x"], d["dt"], d["A"], d["Bm"], d["Cm"])
            mem_ref = oracle.chunk_memories(d["x"], d["dt"], d["A"], d["Bm"], S)
        same_finite(to_np(y), y_ref, tol, "y (%s)" % name)
        same_finite(to_np(mem), mem_ref, tol, "mem (%s)" % name)
        same_finite(to_np(hl), hl_ref, 1e-5, "h_last (%s)" % name)


def test_scan_of_an_infinite_decay():
    """A = -inf forgets everything at every token: y_t = C_t dt_t B_t x_t."""
    import torch
    w = synth.Workload("decay", 1, 70, 2, 64, 16, 16, "fp32")
    d = synth.forward_inputs(w, seed=5)
    A = np.asarray(d["A"], dtype=np.float32).copy()
    A[1] = -np.inf
    y, mem, hl = dart.ssd_chunk_scan(*(f32_dev(v) for v in (d["x"], d["dt"], A, d["Bm"], d["Cm"])), 16)
    torch.cuda.synchronize()
    A[1] = -1e6  # e^(dt A) is zero in 64 bits too
    y_ref, hl_ref = oracle.ssd_recurrence(d["x"], d["dt"], A, d["Bm"], d["Cm"])
    assert_close_slices(to_np(y), y_ref, 1e-5, what="y")
    assert_close_slices(to_np(mem), oracle.chunk_memories(d["x"], d["dt"], A, d["Bm"], 16), 1e-5, axes_keep=(0, 1, 2), what="mem")
    assert_close_slices(to_np(hl), hl_ref, 1e-5, axes_keep=(0, 1), what="h_last")
