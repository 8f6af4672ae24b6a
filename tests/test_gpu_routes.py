"""Both sides of the rules that choose a kernel by a call's size: rows are independent, so a call
that one side takes has to give what two calls on half its rows give, which the other side
takes (the rules themselves: test_routes.py).
"""
import numpy as np
import pytest
import torch

import bdlm_inputs as bi
import paper_2607_02805_amd as bd
from tests.gpu_util import DEV
from tests.test_gpu_conv import conv_params

pytestmark = pytest.mark.gpu


def inputs(rows, H, N, T, dtype, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)

    def r(*s):
        return torch.randn(*s, generator=g, device=DEV)
    v = {"x": r(rows, T, H, 64).to(dtype), "B": (r(rows, T, 1, N) * 0.5).to(dtype), "C": (r(rows, T, 1, N) * 0.5).to(dtype),
         "dt": (torch.rand(rows, T, H, generator=g, device=DEV) * 0.1 + 1e-3).to(dtype)}
    return v, {"A": -torch.rand(H, generator=g, device=DEV) * 8 - 0.5, "D": r(H), "Dr": r(H)}


def call(kind, v, w, p, pool, conv):
    """The outputs (None: none) of one call; states and rows are updated in place."""
    rows = v["x"].shape[0]
    act, nc, nb = (v["x"], v["dt"], p["A"], v["B"], v["C"]), np.zeros(rows, np.int64), np.zeros(rows, np.int64)
    if kind == "window":
        return bd.scan_full_window(*act, p["D"], p["Dr"])
    if kind == "step":
        return bd.scan_block_step(*act, p["D"], p["Dr"], pool)
    if kind == "commit":
        return bd.commit_boundary(*act, p["D"], p["Dr"], pool, nc, nb, y_clean=True)
    if kind == "sep":
        return bd.scan_block_step_sep((*act, p["D"]), (w["x"], w["dt"], p["A"], w["B"], w["C"], p["Dr"]), pool)
    if kind in ("prefill", "states"):
        return bd.prefill(*act, p["D"], pool, nc, nb, y_fwd=True if kind == "prefill" else None)
    cw, cb, rows3 = conv
    if kind == "conv_step":
        return bd.conv_block_step(*act, p["D"], p["Dr"], cw, cb, rows3, pool)
    return bd.conv_commit_boundary(*act, p["D"], p["Dr"], cw, cb, rows3, pool, nc, nb, y_clean=True)


BF, F32 = torch.bfloat16, torch.float32


@pytest.mark.parametrize("kind,rows,H,N,T,dtype", [
    ("window", 24, 32, 16, 1030, BF), ("window", 24, 32, 32, 1030, BF),       # both branches at once | twice
    ("step", 84, 32, 16, 300, BF), ("commit", 84, 32, 32, 293, BF),
    ("sep", 18, 32, 16, 200, BF), ("sep", 16, 32, 32, 150, BF), ("sep", 26, 32, 64, 193, BF),
    ("states", 64, 32, 16, 250, BF), ("states", 32, 32, 128, 250, F32),       # one launch | two
    ("prefill", 26, 32, 32, 330, BF), ("prefill", 50, 32, 16, 200, BF),       # pairs of heads
    ("prefill", 10, 32, 128, 530, F32), ("prefill", 8, 32, 16, 1100, BF),     # segments
    ("conv_step", 32, 32, 32, 7, F32), ("conv_step", 8, 32, 128, 19, F32), ("conv_commit", 32, 32, 16, 3, F32),
])
def test_halves_agree(kind, rows, H, N, T, dtype):
    print("route", kind, rows, H, N, T, dtype, flush=True)
    v, p = inputs(rows, H, N, T, dtype, 1)
    w, _ = inputs(rows, H, N, T, dtype, 2) if kind == "sep" else (v, None)
    g = torch.Generator(device=DEV).manual_seed(3)
    pool = torch.randn(rows, H, N // 4, 64, 4, generator=g, device=DEV) * 0.5
    cw, cb = (torch.from_numpy(t).to(DEV) for t in conv_params(bi.Workload("t", 1, H, 64, N, 1, T, 0, True, 1, 5), 6))
    cache = torch.randn(rows, 3, cw.shape[0], generator=g, device=DEV)
    whole = [pool.clone(), cache.clone()]
    y = call(kind, v, w, p, whole[0], (cw, cb, whole[1]))
    parts = []
    for a, b in ((0, rows // 2), (rows // 2, rows)):
        h, c = pool[a:b].clone(), cache[a:b].clone()
        yh = call(kind, {k: t[a:b] for k, t in v.items()}, {k: t[a:b] for k, t in w.items()}, p, h, (cw, cb, c))
        parts.append((yh, h, c))

    def err(got, want):
        return float((got.double() - want.double()).norm() / want.double().norm())
    # outputs of bf16 inputs: two-term bf16 splits leave up to 2^-18 of a product; states, three-term
    # splits, and fp32: sums of some hundred fp32 terms, 2^-24 each
    if y is not None:
        assert torch.isfinite(y).all()
        assert err(y, torch.cat([q[0] for q in parts])) <= (2.0 ** -18 if dtype == BF else 2.0 ** -20)
    assert err(whole[0], torch.cat([q[1] for q in parts])) <= 2.0 ** -20
    assert torch.equal(whole[1], torch.cat([q[2] for q in parts]))
