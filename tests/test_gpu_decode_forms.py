"""The decode step's two forms -- one launch (at most sixteen memories and no
more (batch, head) pairs than compute units) and stream plus merge -- on either
side of the line, uniform and ragged, with a token that closes its chunk, one
that opens one, no memory at all, a row outside the step, and more splits than
a merging wave has lanes, against the oracle's step."""
import numpy as np
import pytest

import oracle
from paper_2608_02032_amd import dart, synth
from tests.helpers import TOL, assert_close_slices, f32_dev, to_dev, to_np

pytestmark = pytest.mark.gpu

# B, H, N, S, dtype, positions (one, or one per row)
CASES = [
    (2, 4, 128, 16, "bf16", 0),
    (1, 3, 16, 4, "fp32", 63),          # 15 memories, closes its chunk
    (2, 2, 64, 8, "bf16", 128),         # 16 memories, opens a chunk
    (2, 2, 64, 8, "bf16", 136),         # 17: stream and merge
    (1, 2, 32, 1, "fp32", 600),         # 75 splits of 8
    (130, 2, 16, 4, "bf16", 20),        # more pairs than compute units
    (5, 4, 128, 16, "bf16", (0, 15, 200, -1, 256)),   # 16 memories at most
    (5, 4, 32, 16, "fp32", (300, 15, 31, 272, 2)),    # up to 18
]


@pytest.mark.parametrize("c", CASES, ids=lambda c: "B%d_H%d_N%d_S%d_%s_%s" % (c[:5] + (str(c[5]).replace(", ", "-").strip("()"),)))
def test_decode_step_forms(c):
    import torch
    B, H, N, S, dtype, pos = c
    print("\n[gpu-case] decode %s" % (c,), flush=True)
    rows = list(pos) if isinstance(pos, tuple) else [pos] * B
    top = max(rows)
    rng = np.random.default_rng(top + N)
    Mcap = top // S + 1
    mem = synth.synthetic_memories(rng, B, Mcap, H, N, 64, dtype)
    d = synth.decode_inputs(B, H, 64, N, dtype, seed=top)
    hs = (rng.standard_normal((B, H, N, 64)) * 0.02).astype(np.float32)
    ca = (rng.standard_normal((B, H, N, 64)) * 0.005).astype(np.float32)
    dev = {k: to_dev(d[k], dtype) for k in ("x", "Bm", "Cm", "q", "e", "z")}
    args = (dev["x"], f32_dev(d["dt"]), f32_dev(d["A"]), dev["Bm"], dev["Cm"], dev["q"], dev["e"], dev["z"])
    h_t, a_t, m_t = f32_dev(hs), f32_dev(ca), to_dev(mem, dtype)
    y0 = torch.full_like(dev["x"], 3.0)
    if isinstance(pos, tuple):
        y = dart.decode_step_ragged(torch.tensor(rows, device="cuda"), top, *args, h_t, a_t, m_t, S, y=y0)
    else:
        y = dart.decode_step(pos, *args, h_t, a_t, m_t, S, y=y0)
    torch.cuda.synchronize()
    for b, p in enumerate(rows):
        s = slice(b, b + 1)
        if p < 0:  # takes no part
            assert np.all(to_np(y)[s] == 3.0)
            np.testing.assert_array_equal(to_np(h_t)[s], hs[s].astype(np.float64))
            continue
        hr, cr, mr = hs[s].astype(np.float64), ca[s].astype(np.float64), mem[s].astype(np.float64)
        yr = oracle.decode_step(p, d["x"][s], d["dt"][s], d["A"], d["Bm"][s], d["Cm"][s], d["q"][s], d["e"][s],
                                d["z"][s], hr, cr, mr, S)
        assert_close_slices(to_np(y)[s], yr, TOL[dtype], axes_keep=(0, 1), what="y row %d" % b)
        assert_close_slices(to_np(h_t)[s], hr, 1e-5, axes_keep=(0, 1), what="h_state")
        assert_close_slices(to_np(a_t)[s], cr, 1e-5, axes_keep=(0, 1), what="chunk_acc")
        assert_close_slices(to_np(m_t)[s], mr, 2.0 ** -8 if dtype == "bf16" else 1e-5, axes_keep=(0, 1, 2), what="cache")


def test_forced_split_size_takes_the_step_in_splits():
    """DART_DECODE_MPS forces the memories per split also where one launch would do
    (it is read once, so in a process of its own)."""
    import os
    import subprocess
    import sys
    code = ("import torch\nfrom paper_2608_02032_amd import dart\n"
            "f = lambda *s: torch.zeros(*s, device='cuda')\n"
            "dart.profile_enable(True)\n"
            "dart.decode_step(100, f(1, 2, 64), f(1, 2) + 0.1, f(2) - 1, f(1, 1, 16), f(1, 1, 16), f(1, 1, 16), f(1, 1, 64),\n"
            "                 f(1, 2), f(1, 2, 16, 64), f(1, 2, 16, 64), f(1, 9, 2, 16, 64), 12)\n"
            "torch.cuda.synchronize()\nprint(sorted(dart.profile_read()))\n")
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    out = {}
    for mps in ("", "8"):
        r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=100, cwd=root,
                           env=dict(os.environ, DART_DECODE_MPS=mps))
        assert r.returncode == 0, r.stderr
        out[mps] = r.stdout
    assert "k_decode_one" in out[""] and "k_decode_partial" not in out[""]
    assert "k_decode_partial" in out["8"] and "k_decode_one" not in out["8"]
