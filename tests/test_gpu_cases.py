"""The timing cases' calls against their own 64-bit values: the smaller listed
cases and a fixed sample of drawn ones (every shape, dtype, window and option the
cases declare), through the same entry points, row by row.

A whole-tensor error moves little when one row, tile or head is lost, so every
row of every output is held to the bar of the parity tests (helpers.row_max_rel)
and every (sequence, head) to the case's own relative error.  dk is judged per
(sequence, head) only: a key whose gradient cancels between much larger terms
has no scale of its own.
"""

import importlib.util
import os
import random

import numpy as np
import pytest
import torch

from helpers import ROW_TOL, f64, row_max_rel

pytestmark = pytest.mark.gpu


def _cases():
    path = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "perf", "cases.py")
    spec = importlib.util.spec_from_file_location("timing_cases", path)
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    return mod


CASES = _cases()


def _cost(c):
    return c["B"] * c["H"] * c["n"] * c.get("T", 1) * c["D"] * c["m"]


def _sample():
    rng = random.Random(20)
    small = [c for c in CASES.listed() if _cost(c) <= 1 << 28]
    drawn = [c for c in (CASES.draw(rng) for _ in range(120)) if _cost(c) <= 1 << 27]
    return small + drawn[:36]


def _id(c):
    return c.get("name") or "-".join(str(c[k]) for k in ("op", "B", "H", "n", "D", "m", "w", "dtype"))


@pytest.mark.parametrize("case", _sample(), ids=_id)
def test_case_against_64_bits(case):
    print(f"[case] {case}", flush=True)
    got = CASES.run(CASES.prepare(case, 5))
    exp = CASES.exact(case, 5)
    torch.cuda.synchronize()
    if isinstance(got, dict):
        pairs = [(nm, got[nm], exp[nm]) for nm in got]
    elif isinstance(got, (list, tuple)):
        names = ("out", "dq", "dk", "dv", "dr", "du", "dtau", "dgate")
        pairs = list(zip(names, got, exp))
    else:
        pairs = [("out", got, exp)]
    tol, row_tol = CASES.tolerance(case)["rel"], ROW_TOL[case["dtype"]]
    for nm, g, e in pairs:
        if e is None:
            continue
        g, e = f64(g), e.detach().cpu().numpy()
        assert g.shape == e.shape and np.all(np.isfinite(g)), nm
        if nm == "rho":                                       # a log2 frame: absolute
            assert np.abs(g - e).max() <= (1e-5 if case["dtype"] == "f32" else 1e-3), nm
            continue
        heads = g.reshape(-1, *g.shape[2:]) if g.ndim > 2 else g[None]
        ref = e.reshape(heads.shape)
        axes = tuple(range(1, heads.ndim))
        err = np.sqrt(((heads - ref) ** 2).sum(axes)) / np.maximum(np.sqrt((ref ** 2).sum(axes)), 1e-30)
        rows = None
        if g.ndim == 4 and nm != "dk":
            # (dq of a sequence's first row is zero by definition: what is there is the
            # rounding of the bf16 output its two terms were formed from)
            first = 1 if nm == "dq" else 0
            rows = row_max_rel(heads[:, first:], ref[:, first:])
        print(f"      {nm} head {err.max():.2e}" + (f" row {rows:.2e}" if rows is not None else ""), flush=True)
        assert err.max() <= tol, (nm, err.max())
        assert rows is None or rows <= row_tol, (nm, "row", rows)
