"""GPU parity of the windowed masked kernel (bdlm_maskw.hip) at the edges of its tiles, windows
and rules: separate reverse inputs on blocks around 64, 128 and 256 tokens at every dstate, on
few and on many workgroups, and one input set where windows take the step and the commit
(more workgroups than compute units; dstate 128 to 128 tokens, dstate 64 beyond).  Oracle and
bar as in test_gpu_variants.py."""
import numpy as np
import pytest
import torch

import bdlm_inputs as bi
import oracle
from tests.gpu_util import REL_TOL, commit, from_pool, pool_dev, rel_err, step, to_dev
from tests.test_gpu_variants import say, sep_inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch,H,N,L,G,slotted", [
    (2, 3, 16, 65, 1, False), (2, 4, 16, 256, 2, True), (2, 3, 32, 127, 1, True), (2, 4, 32, 129, 1, False),
    (2, 4, 64, 128, 2, False), (2, 3, 64, 255, 1, True), (2, 4, 128, 65, 1, True), (2, 4, 128, 144, 1, False),
    (2, 4, 128, 256, 2, True), (1, 26, 128, 96, 1, False), (9, 29, 16, 70, 1, False), (9, 29, 128, 241, 1, True),
    (9, 29, 64, 129, 1, False), (9, 29, 32, 161, 1, False), (9, 29, 128, 113, 1, False)])
def test_separate_reverse_inputs(batch, H, N, L, G, slotted):
    import paper_2607_02805_amd as bd
    w = bi.Workload("t", batch, H, 64, N, G, L, 0, True, 1, 15000 + H + N + L)
    fwd, rev = sep_inputs(w, 15100 + L)
    pool = bi.random_state(w, batch + 1, 7, 0.5).astype(np.float64)
    slots = np.arange(batch, 0, -1).astype(np.int32) if slotted else np.arange(batch).astype(np.int32)
    vf, vr = to_dev(fwd), to_dev(rev)
    h = pool_dev(pool)
    before = from_pool(h).copy()
    say("windowed, separate reverse inputs", dict(batch=batch, H=H, N=N, L=L, G=G, slotted=slotted))
    y = bd.scan_block_step_sep((vf["x"], vf["dt"], vf["A"], vf["B"], vf["C"], vf["D"]),
                               (vr["x"], vr["dt"], vr["A"], vr["B"], vr["C"], vr["D_rev"]),
                               h, slot_idx=slots if slotted else None)
    torch.cuda.synchronize()
    _, yf, _ = oracle.block_step(fwd, pool[slots], parts=True)
    _, _, yr = oracle.block_step(rev, np.zeros_like(pool[slots]), parts=True)
    assert rel_err(y, yf + yr) <= REL_TOL
    np.testing.assert_array_equal(from_pool(h), before)


@pytest.mark.parametrize("N,L,slotted", [(128, 65, True), (128, 128, False), (64, 129, False), (64, 256, True)])
@pytest.mark.parametrize("want_y", [True, False])
def test_one_input_set(N, L, slotted, want_y):
    batch, H = 9, 29                                   # 261 workgroups
    w = bi.Workload("t", batch, H, 64, N, 1, L, 0, True, 1, 15200 + N + L)
    d, c = bi.block_inputs(w, 0), bi.commit_inputs(w)
    pool = bi.random_state(w, batch + 1, 8, 0.5).astype(np.float64)
    slots = np.arange(batch, 0, -1).astype(np.int32) if slotted else np.arange(batch).astype(np.int32)
    arg = slots if slotted else None
    h = pool_dev(pool)
    say("windowed, one input set", dict(N=N, L=L, slotted=slotted, want_y=want_y))
    y = step(to_dev(d), h, slot_idx=arg)
    nc, nb = np.zeros(batch + 1, np.int64), np.zeros(batch + 1, np.int64)
    yc = commit(to_dev(c), h, nc, nb, 0, slot_idx=arg, y_clean=True if want_y else None)
    torch.cuda.synchronize()
    assert rel_err(y, oracle.block_step(d, pool, slot_idx=slots)) <= REL_TOL
    y_ref, *_, s_ref = oracle.block_step(c, pool, slot_idx=slots, parts=True, final_state=True)
    if want_y:
        assert rel_err(yc, y_ref) <= REL_TOL
    got = from_pool(h)
    assert rel_err(got[slots], s_ref) <= REL_TOL
    rest = [i for i in range(batch + 1) if i not in slots]
    np.testing.assert_array_equal(got[rest], from_pool(pool_dev(pool))[rest])


@pytest.mark.parametrize("N", [16, 32])
@pytest.mark.parametrize("H,L", [(4, 256), (32, 200)])
def test_separate_inputs_repeat(N, H, L):
    """Thirty calls on the same inputs are equal bit for bit, with two workgroups on a CU (the
    outputs' stores once let four lanes of sixteen go wrong now and then)."""
    import paper_2607_02805_amd as bd
    w = bi.Workload("t", 448 // H, H, 64, N, 1, L, 0, True, 1, 9100 + N + L)
    f, r = to_dev(bi.block_inputs(w, 0)), to_dev(bi.block_inputs(w, 1))
    h = pool_dev(bi.random_state(w, 448 // H, 6, 0.5))
    fwd = (f["x"], f["dt"], f["A"], f["B"], f["C"], f["D"])
    rev = (r["x"], r["dt"], f["A"], r["B"], r["C"], f["D_rev"])
    first = bd.scan_block_step_sep(fwd, rev, h)
    for _ in range(29):
        assert torch.equal(bd.scan_block_step_sep(fwd, rev, h), first)
