"""GPU parity of the convolution-state step and commit on the Gram and head kernels
(bdlm_mix.hip: blocks of up to 256 tokens that the block kernel's staging does not take),
at the edges of their tiles: lengths around 16-token tiles, 32-token pairs, 64-, 128- and
256-token blocks, every dstate, both storage types, several groups, slot maps, decays that
underflow within a pair of tiles, and a shape whose tiles do not fit in the workspace (which
takes the convolution kernel and the scan kernels).  Oracle and bar as in test_gpu_conv.py.
"""
import numpy as np
import pytest
import torch

import bdlm_inputs as bi
import oracle
from tests.gpu_util import DEV, REL_TOL, from_pool, pool_dev, rel_err, to_dev
from tests.test_gpu_conv import conv_params, oracle_step, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,N,L,bf16,G,fast,want_y", [
    (4, 128, 33, True, 1, False, True), (3, 16, 64, True, 1, True, True),
    (6, 64, 65, False, 2, False, True), (5, 32, 128, True, 1, False, False),
    (4, 128, 129, False, 1, True, True), (8, 64, 255, True, 2, False, True),
    (26, 128, 256, True, 1, False, True), (4, 32, 256, True, 1, True, True),
    (4, 16, 160, True, 1, False, False), (4, 128, 17, False, 1, False, True),
    (4, 128, 64, True, 1, True, True),
    (2, 128, 256, True, 2, False, True),       # one head per group: the tiles do not fit
])
def test_conv_long_blocks(H, N, L, bf16, G, fast, want_y):
    import paper_2607_02805_amd as bd
    w = bi.Workload("t", 2, H, 64, N, G, L, 0, bf16, 1, 12000 + H + N + L)
    d, c = bi.block_inputs(w, 0), bi.commit_inputs(w)
    d["D_rev"] = (d["D"] * 0.5).astype(np.float32)
    c["D_rev"] = d["D_rev"]
    if fast:     # a token's decay reaches 2^-60: products of decays underflow
        for v in (d, c):
            v["dt"] = bi.to_bf16_bits(bi.bf16_bits_to_f32(v["dt"]) * np.float32(300.0)) if bf16 \
                else v["dt"] * np.float32(300.0)
    cw, cb = conv_params(w, 12100 + L)
    cache = np.random.Generator(np.random.PCG64(5)).standard_normal((4, 3, cw.shape[0])).astype(np.float32)
    pool = bi.random_state(w, 4, 6, 0.5).astype(np.float64)
    cwd, cbd = torch.from_numpy(cw).to(DEV), torch.from_numpy(cb).to(DEV)
    cp, h = torch.from_numpy(cache).to(DEV), pool_dev(pool)
    say("conv block", dict(H=H, N=N, L=L, bf16=bf16, G=G, fast=fast))
    v = to_dev(d)
    y = bd.conv_block_step(v["x"], v["dt"], v["A"], v["B"], v["C"], v["D"], v["D_rev"], cwd, cbd, cp, h,
                           slot_idx=[3, 3])
    torch.cuda.synchronize()
    y_ref, _ = oracle_step(d, cw, cb, cache.astype(np.float64), pool, [3, 3])
    e = rel_err(y, y_ref)

    slots = [2, 0]
    y_ref, fin = oracle_step(c, cw, cb, cache.astype(np.float64), pool, slots)
    *_, s_ref = oracle.block_step(fin, pool, slot_idx=slots, parts=True, final_state=True)
    cache_ref = cache.astype(np.float64)
    oracle.conv(c, cw, cb, cache_ref, slot_idx=slots, commit=True)
    nc, nb = np.zeros(4, np.int64), np.zeros(4, np.int64)
    v = to_dev(c)
    yc = bd.conv_commit_boundary(v["x"], v["dt"], v["A"], v["B"], v["C"], v["D"], v["D_rev"], cwd, cbd, cp,
                                 h, nc, nb, 0, slot_idx=slots, y_clean=True if want_y else None)
    torch.cuda.synchronize()
    got = from_pool(h)
    es = rel_err(got[slots], s_ref)
    ey = rel_err(yc, y_ref) if want_y else 0.0
    say("  rel err step", e, "state", es, "clean y", ey)
    assert max(e, es, ey) <= REL_TOL
    np.testing.assert_array_equal(got[[1, 3]], pool[[1, 3]].astype(np.float32))   # untouched slots
    np.testing.assert_array_equal(cp.cpu().numpy(), cache_ref.astype(np.float32))
    assert nc.tolist() == [L, 0, L, 0] and nb.tolist() == [1, 0, 1, 0]


@pytest.mark.parametrize("N,L,bf16", [(128, 33, True), (128, 64, True), (128, 16, False), (16, 16, False),
                                      (128, 100, False), (64, 256, True)])
def test_error_of_fp32_products(N, L, bf16):
    """Products of fp32 operands run as six products of bf16 terms; their sums must not round
    more often than fp32 products would.  A rounding to fp32 of a value of its own size has a
    relative rms of about 2.6e-8.  An output's operands (x, B and C after the convolution, the
    state, the weights) and its own sums of at most eight 32-index products contribute a dozen
    to two dozen of them, in quadrature below 1.25e-7 of the 2-norm.  A state's are about half a
    dozen (6.5e-8), and per pair of tiles passed the decay's own error, which all of a head's
    state shares: the hardware exponential's unit in the last place and the rounding of its
    argument, 4e-8.  Six additions per 32 indices at the sum's size come to 1.5e-7 for outputs
    at dstate 128 and to 1.1e-7 to 2.0e-7 for states of 16 to 100 tokens."""
    import paper_2607_02805_amd as bd
    H = 6
    w = bi.Workload("t", 2, H, 64, N, 1, L, 0, bf16, 1, 12600 + N + L)
    d = bi.block_inputs(w, 0)
    # B and C of unit size, as before a convolution: the prefix term is most of the output
    r = np.random.Generator(np.random.PCG64(12601))
    for k in ("B", "C"):
        v = r.standard_normal(d[k].shape).astype(np.float32)
        d[k] = bi.to_bf16_bits(v) if bf16 else v
    cw, cb = conv_params(w, 12602)
    cache = r.standard_normal((2, 3, cw.shape[0])).astype(np.float32)
    pool = bi.random_state(w, 2, 6, 0.5).astype(np.float64)
    y_ref, fin = oracle_step(d, cw, cb, cache.astype(np.float64), pool, None)
    *_, s_ref = oracle.block_step(fin, pool, parts=True, final_state=True)
    v, h = to_dev(d), pool_dev(pool)
    nc, nb = np.zeros(2, np.int64), np.zeros(2, np.int64)
    y = bd.conv_commit_boundary(v["x"], v["dt"], v["A"], v["B"], v["C"], v["D"], v["D_rev"],
                                torch.from_numpy(cw).to(DEV), torch.from_numpy(cb).to(DEV),
                                torch.from_numpy(cache).to(DEV), h, nc, nb, y_clean=True)

    def err(a, ref):
        return float(np.linalg.norm(a.astype(np.float64) - ref) / np.linalg.norm(ref))
    ey, es = err(y.cpu().numpy(), y_ref), err(from_pool(h), s_ref)
    say("error of fp32 products", dict(N=N, L=L, bf16=bf16), "outputs", ey, "states", es)
    assert ey <= 1.25e-7 and es <= (6.5e-8 ** 2 + (L + 31) // 32 * 4e-8 ** 2) ** 0.5


@pytest.mark.parametrize("H,N,L,bf16,G", [(4, 128, 256, True, 1), (6, 64, 200, False, 2), (3, 16, 65, True, 1),
                                          (4, 32, 64, False, 1), (4, 128, 17, False, 1)])
def test_commit_without_outputs_forms_the_same_states(H, N, L, bf16, G):
    """Without outputs only the diagonal workgroups of the Gram kernel run, and the head kernel
    reads the split B alone: the states and cached rows are those of a commit with outputs, bit
    for bit, whatever the workspace held."""
    import paper_2607_02805_amd as bd
    w = bi.Workload("t", 3, H, 64, N, G, L, 0, bf16, 1, 12200 + N + L)
    v = to_dev(bi.commit_inputs(w))
    cw, cb = (torch.from_numpy(t).to(DEV) for t in conv_params(w, 12300 + L))
    ws = torch.full((3 * L * (2 * H * 64 + 4 * G * N + H) * 4 + 256,), 0xff, dtype=torch.uint8, device=DEV)
    got = []
    for want_y in (False, True):
        cp = torch.from_numpy(np.random.Generator(np.random.PCG64(6)).standard_normal((3, 3, cw.shape[0]))
                              .astype(np.float32)).to(DEV)
        h = pool_dev(bi.random_state(w, 3, 6, 0.5))
        say("conv commit", dict(H=H, N=N, L=L, bf16=bf16, G=G, want_y=want_y))
        bd.conv_commit_boundary(v["x"], v["dt"], v["A"], v["B"], v["C"], v["D"], v["D_rev"], cw, cb, cp, h,
                                np.zeros(3, np.int64), np.zeros(3, np.int64), 0,
                                y_clean=True if want_y else None, workspace=ws)
        torch.cuda.synchronize()
        got.append((h, cp))
    assert torch.isfinite(got[0][0]).all()
    for a, b in zip(*got):
        assert torch.equal(a, b)
