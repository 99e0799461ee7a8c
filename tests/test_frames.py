"""Backward where the running key frame rises by far more than float32's range
inside the rows a sweep walks together.

Large keys (scaled by a power of two) have log-features hundreds of powers of
two below an ordinary key's, so the frame jumps at the first ordinary token
after them.  Every gradient row is held to the bars of the backward tests
against a float64 reference taken in each row's own frame.
"""

import numpy as np
import pytest
import torch

from paper_2608_09307_amd import linsimp as L
from paper_2608_09307_amd.workloads import WORKLOADS, Workload, make_inputs

from helpers import ROW_TOL, UNIT_ROUNDOFF, backward_in_frames, f64, oracle_backward, rel_l2, row_max_rel

DEV = "cuda:0"
NAMES = ("dq", "dk", "dv", "dr", "du")
TOL = {"f32": 1e-4, "bf16": 2e-2}


def test_reference_is_the_oracle_where_both_hold():
    wl = Workload("frames", 1, 2, 45, 16, 16, 24, 20, "f32", "fwdbwd", seed=70)
    x = make_inputs(wl)
    scales = {}
    ref = oracle_backward(x, wl.w, [(0, 1)], scales=scales)[(0, 1)]
    grads, scale = backward_in_frames(x, 0, 1, wl.w)
    for nm, g, e in zip(NAMES, grads, ref):
        assert rel_l2(g, e) < 1e-10, nm
    assert rel_l2(scale, scales[(0, 1)]) < 1e-10


@pytest.mark.gpu
@pytest.mark.parametrize("D,m,n,w,dt,scales", [
    (128, 128, 130, 64, "bf16", ((1, 8),)),             # the sequence opens with a large key
    (64, 64, 130, 40, "bf16", ((40, 8),)),              # the rise inside a later chunk
    (128, 256, 100, 64, "bf16", ((33, 8),)),            # two feature blocks, just past a chunk's edge
    (64, 128, 97, 33, "bf16", ((7, 32), (20, 16), (50, 8))),   # three rises, two in one chunk
    (64, 64, 170, 100, "bf16", ((5, 16), (70, 8))),     # four anchor tiles a row
    (32, 32, 100, 20, "f32", ((10, 16), (45, 8))),      # one anchor tile a row
    (64, 64, 70, 64, "f32", ((32, 8),)),                # at a chunk's edge
])
def test_backward_far_frames(D, m, n, w, dt, scales):
    wl = Workload("frames", 1, 2, n, D, D, m, w, dt, "fwdbwd", seed=71)
    print(f"[frames] {wl} {scales}", flush=True)
    x = make_inputs(wl, device=DEV)
    lo = 0
    for hi, s in scales:
        x["k"][:, :, lo:hi] *= s
        lo = hi
    args = (x["q"], x["k"], x["v"], x["r"], x["u"], x["omega"], w)
    out, stats = L.fwd(*args)
    grads = L.bwd(*args, out, stats, x["dO"])
    torch.cuda.synchronize()
    refs = [backward_in_frames(x, 0, h, w) for h in range(2)]
    # dk: a large key has one feature far above its others, and while it alone
    # fills the state the gradient of its features cancels; the rounding of the
    # terms (two unit roundoffs of their absolute sum, as in the backward tests)
    # is allowed on top of the row bar, and the rows stand for the whole tensor
    slack = 2 * UNIT_ROUNDOFF[dt] * np.stack([t for _, t in refs])
    for gi, nm in enumerate(NAMES):
        got, exp = f64(grads[gi][0]), np.stack([r[gi] for r, _ in refs])
        assert np.all(np.isfinite(got)), nm
        err, rows = rel_l2(got, exp), row_max_rel(got, exp, slack=slack if nm == "dk" else None)
        print(f"      {nm} {err:.2e} row {rows:.2e}", flush=True)
        assert nm == "dk" or err <= TOL[dt], nm
        assert rows <= ROW_TOL[dt], nm


@pytest.mark.gpu
def test_backward_stress64k_every_head_finite():
    """x4 keys in 5% of the positions, the first token's among them."""
    wl = WORKLOADS["stress64k_m256"].replace(n=2048)
    x = make_inputs(wl, device=DEV)
    x["k"][:, :, 0] *= 1.0 if bool(x["boost_mask"][0, 0]) else wl.boost
    args = (x["q"], x["k"], x["v"], x["r"], x["u"], x["omega"], wl.w)
    out, stats = L.fwd(*args)
    for nm, g in zip(NAMES, L.bwd(*args, out, stats, x["dO"])):
        assert bool(torch.isfinite(g.float()).all()), nm
