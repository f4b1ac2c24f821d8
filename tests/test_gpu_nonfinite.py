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


def ssd_bwd(d, S, dtype, dy, dmem):
    import torch
    x, Bm, Cm, g = (to_dev(v, dtype) for v in (d["x"], d["Bm"], d["Cm"], dy))
    out = dart.ssd_bwd(x, f32_dev(d["dt"]), f32_dev(d["A"]), Bm, Cm, S, g, dmem=f32_dev(dmem))
    torch.cuda.synchronize()
    return {k: to_np(v) for k, v in out.items()}


@pytest.mark.parametrize("N,S,dtype", [(16, 16, "fp32"), (64, 6, "fp32"), (32, 17, "bf16"), (128, 32, "fp32"),
                                       (16, 100, "bf16"), (64, 64, "fp32")])
@pytest.mark.parametrize("bad", BAD)
def test_scan_backward_keeps_a_token_to_what_depends_on_it(N, S, dtype, bad):
    """One entry of batch row 0 is not finite: the gradients that do not depend on it are those
    without it (dx does not depend on x, dB not on B, dC not on C; through the
    state, dx and dB of a token depend on dy and C of the tokens from it on, dC on
    x and B of the tokens up to it; a memory's gradient reaches its own chunk)."""
    B, L, H, t0 = 2, 90, 4, 37
    w = synth.Workload("nonfinite_%d_%d" % (N, S), B, L, H, 64, N, S, dtype, ngroups=2)
    print("\n[gpu-case] scan bwd %s %s" % (bad, w), flush=True)
    d = synth.forward_inputs(w, seed=N + S)
    rng = np.random.default_rng(N)
    dy = synth.to_storage(rng.standard_normal((B, L, H, 64)).astype(np.float32), dtype)
    dmem = rng.standard_normal((B, -(-L // S), H, N, 64)).astype(np.float32)
    ref = ssd_bwd(d, S, dtype, dy, dmem)
    t = np.arange(L)
    c0, c1 = t0 // S * S, t0 // S * S + S
    own = (t >= c0) & (t < c1)
    always, never = t >= 0, t < 0
    # input, entry, and the tokens whose dx, dB, dC may change
    for name, at, may in (("x", (0, t0, 1, 7), (never, t == t0, t >= t0)),
                          ("Bm", (0, t0, 0, 3), (t == t0, never, t >= t0)),
                          ("Cm", (0, t0, 0, 2), (t <= t0, t <= t0, never)),
                          ("dy", (0, t0, 1, 7), (t <= t0, t <= t0, t == t0)),
                          ("dmem", (0, t0 // S, 1, 3, 9), (own, own, never)),
                          ("x", (0, L - 1, 0, 0), (never, t == L - 1, t == L - 1)),
                          ("Cm", (0, 70, 0, 1), (t <= 70, t <= 70, never))):
        e = dict(d, dy=dy, dmem=dmem)
        e[name] = e[name].copy()
        e[name][at] = bad
        got = ssd_bwd(e, S, dtype, e["dy"], e["dmem"])
        for k, m in zip(("dx", "dB", "dC"), may):
            np.testing.assert_allclose(got[k][1], ref[k][1], rtol=0, atol=1e-5 * np.abs(ref[k]).max())
            clean = got[k][0][~m]
            assert np.isfinite(clean).all(), "%s of other tokens (%s)" % (k, name)
            # the same sums in another order where the tile is summed token by token
            np.testing.assert_allclose(clean, ref[k][0][~m], rtol=0, atol=1e-5 * np.abs(ref[k]).max())
            assert not m.any() or not np.isfinite(got[k][0][m]).all(), "%s (%s)" % (k, name)


@pytest.mark.parametrize("N,S,dtype,B", [(16, 5, "fp32", 1), (64, 17, "fp32", 1), (32, 20, "bf16", 1), (128, 40, "bf16", 1),
                                         (16, 5, "bf16", 300), (64, 12, "fp32", 90), (128, 12, "fp32", 90)])
@pytest.mark.parametrize("bad", BAD)
def test_attention_keeps_a_memory_to_the_tokens_after_it(N, S, dtype, B, bad):
    """A memory that is not finite reaches the tokens of later chunks only, and a
    token the gradients of the memories before its chunk only (both forms of the
    forward and of the memory side: few and many sequences)."""
    import torch
    from tests import test_gpu_sma_bwd as MB
    L, H = 90, 2
    w = synth.Workload("nonfinite_%d_%d" % (N, S), B, L, H, 64, N, S, dtype)
    print("\n[gpu-case] attention %s %s" % (bad, w), flush=True)
    d, mem, y_ssd, dy = MB.bwd_case(w, seed=N)
    q, e, Cm, z, ys, g = (to_dev(v, dtype) for v in (d["q"], d["e"], d["Cm"], d["z"], y_ssd, dy))
    t, j0 = np.arange(L), 1
    chunk = t // S

    def run(mem, g):
        y, lse = dart.sma_fwd(q, e, Cm, mem, z, ys, S)
        out = dart.sma_bwd(q, e, Cm, mem, z, lse, g, S)
        torch.cuda.synchronize()
        return dict({k: to_np(v) for k, v in out.items()}, y=to_np(y), lse=to_np(lse))

    m0 = to_dev(mem, dtype)
    ref = run(m0, g)
    bm = m0.clone()
    bm[0, j0, 1, 3, 9] = bad
    got = run(bm, g)
    for k in ("y", "lse", "dq", "de", "dC", "dz"):
        np.testing.assert_array_equal(got[k][0][chunk <= j0], ref[k][0][chunk <= j0], err_msg=k)
        np.testing.assert_array_equal(got[k][1:], ref[k][1:], err_msg=k)
        assert not np.isfinite(got[k][0][chunk > j0]).all(), k
    # dy of one token: the memories of its chunk and after do not see it
    t0 = 2 * S + 1
    bg = g.clone()
    bg[0, t0, 1, 5] = bad
    got = run(m0, bg)
    np.testing.assert_array_equal(got["dmem"][0, t0 // S:], ref["dmem"][0, t0 // S:])
    np.testing.assert_array_equal(got["dmem"][1:], ref["dmem"][1:])
    assert not np.isfinite(got["dmem"][0, :t0 // S]).all()
    others = t != t0
    for k in ("dq", "de", "dC", "dz"):
        np.testing.assert_array_equal(got[k][0][others], ref[k][0][others], err_msg=k)


@pytest.mark.parametrize("C", [4, 5])
def test_convolution_backward_ends_with_the_sequence(C):
    """Inputs whose products overflow only past the last token, in the forms of four channels per
    thread (260 blocks) and of one."""
    import torch
    B, L = 260, 6
    print("\n[gpu-case] conv bwd end C %d" % C, flush=True)
    x = torch.zeros(B, L, C, device="cuda")
    x[:, -1] = 3e38
    w = torch.tensor([1.0, 1.0, 4.0, 0.1], device="cuda").repeat(C, 1)
    g = dart.conv1d_silu_bwd(x, w, torch.ones(B, L, C, device="cuda"), bias=torch.zeros(C, device="cuda"))
    torch.cuda.synchronize()
    # SiLU'(0) = 1/2 for the tokens before the last, SiLU'(3e37) = 1 for it
    du = torch.tensor([0.5] * 5 + [1.0, 0, 0, 0], device="cuda")
    ref = w[0, 3] * du[:6] + w[0, 2] * du[1:7] + w[0, 1] * du[2:8] + w[0, 0] * du[3:]
    torch.testing.assert_close(g["din"], ref[None, :, None].expand(B, L, C), rtol=1e-6, atol=0)
