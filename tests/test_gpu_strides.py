"""GPU parity on inputs that are views: slices of one fused projection (batch-major and
sequence-major), head-major tensors, and tensors expanded over the tokens (token stride 0), on
the kernels that plan their loads by the strides.  Outputs at 4-byte-aligned addresses, which
the calls here accept.  Oracle on the same values made contiguous; bar as in gpu_util.py."""
import numpy as np
import pytest
import torch

import bdlm_inputs as bi
import oracle
from tests.gpu_util import DEV, REL_TOL, from_pool, pool_dev, rel_err, to_dev
from tests.test_gpu_conv import conv_params, oracle_step, say
from tests.test_gpu_seq16 import unaligned

pytestmark = pytest.mark.gpu


def lay(d, kind):
    """The values of d (numpy: x, dt, B, C, ...) on the GPU as views of layout `kind`."""
    v = to_dev(d)
    x, dt, Bm, Cm = v["x"], v["dt"], v["B"], v["C"]
    b, L, H, _ = x.shape
    G, N = Bm.shape[2:]
    if kind in ("fused", "sequence-major"):
        HP, GN = H * 64, G * N
        row = (HP + 2 * GN + H + 8 + 7) // 8 * 8                       # 8 columns of something else
        p = torch.full((b, L, row) if kind == "fused" else (L, b, row), float("nan"), dtype=x.dtype, device=DEV)
        p = p if kind == "fused" else p.transpose(0, 1)
        cut = {"x": (8, HP, (H, 64)), "B": (8 + HP, GN, (G, N)), "C": (8 + HP + GN, GN, (G, N))}
        for k, (o, n, s) in cut.items():
            p[..., o:o + n].unflatten(2, s).copy_(v[k])
            v[k] = p[..., o:o + n].unflatten(2, s)
        o = 8 + HP + 2 * GN
        p[..., o:o + H].copy_(dt)
        v["dt"] = p[..., o:o + H]
    elif kind == "head-major":
        for k in ("x", "B", "C"):
            v[k] = v[k].transpose(1, 2).contiguous().transpose(1, 2)
    else:                                                              # "expanded x", "expanded dt", ...
        for k in kind.split()[1:]:
            d[k] = np.repeat(d[k][:, :1], L, axis=1)
            v[k] = to_dev({k: d[k][:, :1].copy()})[k].expand(v[k].shape)
    return v


VIEWS = ("fused", "sequence-major", "head-major")
EXPANDED = ("expanded x", "expanded dt", "expanded B C", "expanded x dt B C")


def acts(v):
    return v["x"], v["dt"], v["A"], v["B"], v["C"], v["D"]


def inputs(B, H, G, N, L, bf16, seed):
    w = bi.Workload("t", B, H, 64, N, G, L, 0, bf16, 1, seed)
    d = bi.block_inputs(w, 0)
    d["D_rev"] = (d["D"] * 0.5).astype(np.float32)
    return w, d


@pytest.mark.parametrize("kind", VIEWS + EXPANDED)
@pytest.mark.parametrize("B,H,G,N,T,bf16", [(24, 32, 1, 64, 100, True), (2, 4, 2, 128, 330, True),
                                            (2, 6, 1, 16, 601, True), (2, 3, 1, 32, 290, False)])
def test_sequences(B, H, G, N, T, bf16, kind):
    import paper_2607_02805_amd as bd
    w, d = inputs(B, H, G, N, T, bf16, 16000 + H + N)
    say("sequence views", dict(B=B, H=H, G=G, N=N, T=T, bf16=bf16, kind=kind))
    v = lay(d, kind)
    y = unaligned((B, T, H, 64))
    bd.scan_full_window(*acts(v), v["D_rev"], y=y)
    torch.cuda.synchronize()
    assert rel_err(y, oracle.full_window(d)) <= REL_TOL
    pool = bi.random_state(w, B, 3, 0.5).astype(np.float64)
    s_ref, y_ref = oracle.scan_forward(d, pool, want_y=True)
    for want_y in (True, False):
        h, nc, nb = pool_dev(pool), np.zeros(B, np.int64), np.zeros(B, np.int64)
        y = unaligned((B, T, H, 64)) if want_y else None
        bd.prefill(*acts(v), h, nc, nb, y_fwd=y)
        torch.cuda.synchronize()
        assert rel_err(from_pool(h), s_ref) <= REL_TOL
        if want_y:
            assert rel_err(y, y_ref) <= REL_TOL


@pytest.mark.parametrize("kind", VIEWS + EXPANDED)
@pytest.mark.parametrize("B,H,N,L,K,bf16", [(2, 4, 64, 32, 9, True), (2, 3, 16, 20, 15, True), (2, 3, 128, 16, 18, False)])
def test_boundary_states(B, H, N, L, K, bf16, kind):
    import paper_2607_02805_amd as bd
    w, d = inputs(B, H, 1, N, L * K, bf16, 16200 + H + N)
    say("block states of views", dict(B=B, H=H, N=N, L=L, K=K, bf16=bf16, kind=kind))
    v = lay(d, kind)
    got, y = bd.block_boundary_states(*acts(v), L, y_fwd=True)
    torch.cuda.synchronize()
    got = from_pool(got).reshape(B, K, H, 64, N)
    s, ys = np.zeros((B, H, 64, N)), []
    for k in range(K):
        if k:
            assert rel_err(got[:, k], s) <= REL_TOL
        s, yk = oracle.scan_forward(bi.slice_tokens(d, k * L, (k + 1) * L), s, want_y=True)
        ys.append(yk)
    assert rel_err(y, np.concatenate(ys, 1)) <= REL_TOL


@pytest.mark.parametrize("kind", VIEWS + EXPANDED)
@pytest.mark.parametrize("B,H,G,N,L,bf16", [
    (2, 4, 2, 128, 100, True), (2, 3, 1, 64, 200, True), (9, 29, 1, 128, 96, True), (9, 29, 1, 64, 150, True),
    (2, 3, 1, 32, 300, True), (2, 3, 1, 64, 90, False)])
def test_blocks(B, H, G, N, L, bf16, kind):
    import paper_2607_02805_amd as bd
    w, d = inputs(B, H, G, N, L, bf16, 16400 + H + N)
    _, r = inputs(B, H, G, N, L, bf16, 16500 + H + N)
    pool = bi.random_state(w, B, 3, 0.5).astype(np.float64)
    say("block views", dict(B=B, H=H, G=G, N=N, L=L, bf16=bf16, kind=kind))
    v, vr = lay(d, kind), lay(r, kind)
    h, nc, nb = pool_dev(pool), np.zeros(B, np.int64), np.zeros(B, np.int64)
    y = unaligned((B, L, H, 64))
    bd.scan_block_step_sep(acts(v), acts(vr)[:5] + (vr["D_rev"],), h, y=y)
    yc = bd.commit_boundary(*acts(v), v["D_rev"], h, nc, nb, y_clean=True)
    torch.cuda.synchronize()
    y_ref, yf, _, s_ref = oracle.block_step(d, pool, parts=True, final_state=True)
    _, _, yr = oracle.block_step(r, np.zeros_like(pool), parts=True)
    assert rel_err(y, yf + yr) <= REL_TOL
    assert rel_err(yc, y_ref) <= REL_TOL
    assert rel_err(from_pool(h), s_ref) <= REL_TOL


@pytest.mark.parametrize("kind", VIEWS + EXPANDED)
@pytest.mark.parametrize("H,G,N,L,bf16", [(4, 1, 128, 33, True), (8, 2, 64, 200, True), (4, 1, 16, 20, False),
                                          (4, 1, 32, 130, False), (4, 1, 128, 20, True), (4, 1, 64, 300, True)])
def test_convolution_blocks(H, G, N, L, bf16, kind):
    import paper_2607_02805_amd as bd
    w, d = inputs(2, H, G, N, L, bf16, 16600 + H + N)
    cw, cb = conv_params(w, 16601)
    cache = np.random.Generator(np.random.PCG64(5)).standard_normal((2, 3, cw.shape[0])).astype(np.float32)
    pool = bi.random_state(w, 2, 6, 0.5).astype(np.float64)
    say("convolution of views", dict(H=H, G=G, N=N, L=L, bf16=bf16, kind=kind))
    v = lay(d, kind)
    cwd, cbd = torch.from_numpy(cw).to(DEV), torch.from_numpy(cb).to(DEV)
    cp, h = torch.from_numpy(cache).to(DEV), pool_dev(pool)
    y_ref, fin = oracle_step(d, cw, cb, cache.astype(np.float64), pool, None)
    *_, s_ref = oracle.block_step(fin, pool, parts=True, final_state=True)
    rows = cache.astype(np.float64)
    oracle.conv(d, cw, cb, rows, commit=True)
    y, yc = unaligned((2, L, H, 64)), unaligned((2, L, H, 64))
    nc, nb = np.zeros(2, np.int64), np.zeros(2, np.int64)
    bd.conv_block_step(*acts(v), v["D_rev"], cwd, cbd, cp, h, y=y)
    bd.conv_commit_boundary(*acts(v), v["D_rev"], cwd, cbd, cp, h, nc, nb, y_clean=yc)
    torch.cuda.synchronize()
    assert rel_err(y, y_ref) <= REL_TOL
    assert rel_err(yc, y_ref) <= REL_TOL
    assert rel_err(from_pool(h), s_ref) <= REL_TOL
    np.testing.assert_array_equal(cp.cpu().numpy(), rows.astype(np.float32))
