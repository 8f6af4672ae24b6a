"""Values at the ends of the range: a huge negative value before the convolution's SiLU (which
is 0 there), and infinities and NaN in one element of an input.  Such an element spoils what
depends on it and nothing else: every other output is bit for bit that of a clean call, and
what the oracle says is not finite is not finite.  Convolution blocks (bdlm_mix.hip and the
block kernel's staging), masked blocks (bdlm_maskw.hip among them) and sequences."""
import numpy as np
import pytest
import torch

import bdlm_inputs as bi
import oracle
from tests.gpu_util import DEV, REL_TOL, from_pool, pool_dev, rel_err, to_dev
from tests.test_gpu_conv import conv_params, oracle_step, say
from tests.test_gpu_strides import acts, inputs

pytestmark = pytest.mark.gpu


def put(a, idx, value):
    """value at a[idx] of stored bytes (fp32, or bf16 bit patterns)."""
    a[idx] = value if a.dtype != np.uint16 else np.float32(value).view(np.uint32) >> np.uint32(16)


@pytest.mark.parametrize("N,L,bf16", [(128, 33, True), (64, 200, True), (16, 5, False), (32, 100, False), (128, 20, True)])
@pytest.mark.parametrize("value", [-1e4, -2e30, -1e38])
def test_silu_of_a_huge_negative_value(N, L, bf16, value):
    import paper_2607_02805_amd as bd
    H = 4
    w, d = inputs(2, H, 1, N, L, bf16, 17000 + N)
    cw, cb = conv_params(w, 17001)
    cw = np.abs(cw) * np.float32(0.5)
    for t in range(0, L, 7):
        put(d["x"], (0, t, 1, t % 64), value)
        put(d["C"], (1, t, 0, t % N), value)
    cache = np.zeros((2, 3, cw.shape[0]), np.float32)
    pool = bi.random_state(w, 2, 6, 0.5).astype(np.float64)
    say("SiLU of huge negatives", dict(N=N, L=L, bf16=bf16, value=value))
    v = to_dev(d)
    h, cp = pool_dev(pool), torch.from_numpy(cache).to(DEV)
    nc, nb = np.zeros(2, np.int64), np.zeros(2, np.int64)
    y = bd.conv_commit_boundary(*acts(v), v["D_rev"], torch.from_numpy(cw).to(DEV), torch.from_numpy(cb).to(DEV), cp, h,
                                nc, nb, y_clean=True)
    torch.cuda.synchronize()
    with np.errstate(all="ignore"):
        y_ref, fin = oracle_step(d, cw, cb, cache.astype(np.float64), pool, None)
        *_, s_ref = oracle.block_step(fin, pool, parts=True, final_state=True)
    assert rel_err(y, y_ref) <= REL_TOL
    assert rel_err(from_pool(h), s_ref) <= REL_TOL


BAD = [(k, v) for k in ("x", "dt", "B", "C") for v in (np.inf, -np.inf, np.nan)]


def spoil(d, what, value, t):
    """A copy of d with one value of row 1 replaced, and the part of y [B, L, H, 64] and of the
    states [B, H, 64, N] that depends on it."""
    B, L, H, _ = d["x"].shape
    bad = {k: a.copy() for k, a in d.items()}
    y, s = np.zeros((B, L, H, 64), bool), np.zeros((B, H, 64, d["B"].shape[3]), bool)
    G = d["B"].shape[2]
    g = slice((G - 1) * (H // G), H)                       # the last group's heads
    if what == "x":
        put(bad["x"], (1, t, H - 1, 7), value)
        y[1, :, H - 1, 7] = s[1, H - 1, 7] = True
    elif what == "dt":
        put(bad["dt"], (1, t, H - 1), value)
        y[1, :, H - 1] = s[1, H - 1] = True
    elif what == "B":
        put(bad["B"], (1, t, G - 1, 3), value)
        y[1, :, g] = s[1, g] = True
    else:
        put(bad["C"], (1, t, G - 1, 3), value)
        y[1, max(t - 3, 0):t + 4, g] = True                # (the convolutions reach three tokens)
    return bad, y, s


def check(run, ref, d, what, value, t):
    """run(inputs) -> (y, states or None) on the GPU, ref(inputs) -> the same from the oracle."""
    bad, ydep, sdep = spoil(d, what, value, t)
    y0, s0 = run(d)
    y1, s1 = run(bad)
    assert np.array_equal(y0[~ydep], y1[~ydep])
    with np.errstate(all="ignore"):
        yr, sr = ref(bad)
    assert not np.isfinite(y1[~np.isfinite(yr)]).any()
    if s0 is not None:
        assert np.array_equal(s0[~sdep], s1[~sdep])
        assert not np.isfinite(s1[~np.isfinite(sr)]).any()


@pytest.mark.parametrize("what,value", BAD)
@pytest.mark.parametrize("G,N,L,bf16", [(1, 128, 40, True), (2, 64, 200, True), (2, 16, 30, False)])
def test_convolution_blocks(G, N, L, bf16, what, value):
    import paper_2607_02805_amd as bd
    w, d = inputs(2, 4, G, N, L, bf16, 17100 + N)
    cw, cb = conv_params(w, 17101)
    cache = np.random.Generator(np.random.PCG64(5)).standard_normal((2, 3, cw.shape[0])).astype(np.float32)
    pool = bi.random_state(w, 2, 6, 0.5).astype(np.float64)
    say("convolution of", dict(G=G, N=N, L=L, bf16=bf16, what=what, value=value))

    def run(d):
        v, h, cp = to_dev(d), pool_dev(pool), torch.from_numpy(cache).to(DEV)
        nc, nb = np.zeros(2, np.int64), np.zeros(2, np.int64)
        y = bd.conv_commit_boundary(*acts(v), v["D_rev"], torch.from_numpy(cw).to(DEV), torch.from_numpy(cb).to(DEV),
                                    cp, h, nc, nb, y_clean=True)
        return y.cpu().numpy(), from_pool(h)

    def ref(d):
        y, fin = oracle_step(d, cw, cb, cache.astype(np.float64), pool, None)
        return y, oracle.block_step(fin, pool, parts=True, final_state=True)[-1]
    check(run, ref, d, what, value, L // 2)


@pytest.mark.parametrize("what,value", BAD)
@pytest.mark.parametrize("B,H,G,N,L", [(2, 4, 2, 128, 100), (9, 29, 1, 128, 96), (9, 29, 1, 64, 150), (2, 4, 1, 32, 300)])
def test_long_blocks(B, H, G, N, L, what, value):
    import paper_2607_02805_amd as bd
    w, d = inputs(B, H, G, N, L, True, 17200 + N)
    _, r = inputs(B, H, G, N, L, True, 17300 + N)
    pool = bi.random_state(w, B, 6, 0.5).astype(np.float64)
    vr = to_dev(r)
    say("long blocks of", dict(B=B, H=H, G=G, N=N, L=L, what=what, value=value))

    def run(d):
        v, h = to_dev(d), pool_dev(pool)
        nc, nb = np.zeros(B, np.int64), np.zeros(B, np.int64)
        y = bd.commit_boundary(*acts(v), v["D_rev"], h, nc, nb, y_clean=True)
        return y.cpu().numpy(), from_pool(h)

    def ref(d):
        y, *_, s = oracle.block_step(d, pool, parts=True, final_state=True)
        return y, s
    check(run, ref, d, what, value, L // 2)

    def run_sep(d):
        v = to_dev(d)
        return bd.scan_block_step_sep(acts(v), acts(vr)[:5] + (vr["D_rev"],), pool_dev(pool)).cpu().numpy(), None

    def ref_sep(d):
        return (oracle.block_step(d, pool, parts=True)[1] +
                oracle.block_step(r, np.zeros_like(pool), parts=True)[2]), None
    check(run_sep, ref_sep, d, what, value, L // 2)


@pytest.mark.parametrize("what,value", BAD)
@pytest.mark.parametrize("B,H,G,N,T", [(2, 4, 2, 128, 330), (24, 32, 1, 64, 100)])
def test_sequences(B, H, G, N, T, what, value):
    import paper_2607_02805_amd as bd
    w, d = inputs(B, H, G, N, T, True, 17400 + N)
    pool = bi.random_state(w, B, 6, 0.5).astype(np.float64)
    say("sequences of", dict(B=B, H=H, G=G, N=N, T=T, what=what, value=value))

    def run(d):
        v, h = to_dev(d), pool_dev(pool)
        nc, nb = np.zeros(B, np.int64), np.zeros(B, np.int64)
        y = bd.prefill(*acts(v), h, nc, nb, y_fwd=True)
        return y.cpu().numpy(), from_pool(h)

    def ref(d):
        s, y = oracle.scan_forward(d, pool, want_y=True)
        return y, s
    check(run, ref, d, what, value, T // 2)

    def run_full(d):
        v = to_dev(d)
        return bd.scan_full_window(*acts(v), v["D_rev"]).cpu().numpy(), None
    check(run_full, lambda d: (oracle.full_window(d), None), d, what, value, T // 2)
