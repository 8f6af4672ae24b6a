"""GPU parity of the bf16 sequence kernels where their dispatch changes: two heads per
workgroup (768 row-heads and more) and one, one segment per row-head (with its launch straight
from and to the cache) and several, chunks and segments that end ragged, every dstate; and
outputs at a 4-byte-aligned address (the stores are 16 bytes wide).  Oracle on the heads of
the first and last rows and the rows of the first and last heads; bar as in gpu_util.py.
"""
import numpy as np
import pytest
import torch

import bdlm_inputs as bi
import oracle
from tests.gpu_util import DEV, REL_TOL, edge_cover, from_pool, host_slice, pick, pool_dev, rel_err, to_dev

pytestmark = pytest.mark.gpu


def unaligned(shape):
    """A contiguous float32 tensor whose first element sits 4 bytes past a 16-byte boundary."""
    n = int(np.prod(shape))
    return torch.full((n + 1,), float("nan"), device=DEV)[1:].view(shape)


def draw(B, H, N, T, seed):
    w = bi.Workload("t", B, H, 64, N, 1, 32, T, True, 1, seed)
    d = bi.tokens_device(w, T, seed, DEV)
    hp = bi.head_params(w)
    hp["D_rev"] = (hp["D"] * 0.5).astype(np.float32)
    return w, d, hp, to_dev(hp)


@pytest.mark.parametrize("B,H,N,T", [(24, 32, 128, 100), (24, 32, 64, 65), (24, 32, 32, 256), (24, 32, 16, 70),
                                     (48, 16, 128, 600),        # several segments, two heads
                                     (24, 33, 128, 64), (3, 5, 128, 700), (2, 2, 64, 1)])
def test_full_window(B, H, N, T):
    import paper_2607_02805_amd as bd
    w, d, hp, v = draw(B, H, N, T, 13000 + H + N + T)
    y = unaligned((B, T, H, 64))
    bd.scan_full_window(d["x"], d["dt"], v["A"], d["B"], d["C"], v["D"], v["D_rev"], y=y)
    torch.cuda.synchronize()
    assert torch.isfinite(y).all()
    for rows, heads in edge_cover(B, H):
        assert rel_err(pick(y, rows, heads), oracle.full_window(host_slice(d, rows, heads, hp))) <= REL_TOL


@pytest.mark.parametrize("B,H,N,T,want_y", [(24, 32, 128, 130, True), (24, 32, 64, 64, True), (24, 32, 16, 333, True),
                                            (24, 32, 32, 33, True),    # two heads, one segment
                                            (8, 33, 128, 300, True), (16, 17, 64, 100, True),   # one head
                                            (17, 32, 128, 520, True),  # several segments
                                            (3, 4, 128, 250, False), (2, 3, 16, 1, False)])
def test_prefill(B, H, N, T, want_y):
    import paper_2607_02805_amd as bd
    w, d, hp, v = draw(B, H, N, T, 13500 + H + N + T)
    pool = bi.random_state(w, B + 2, 3, 0.5)
    slots = np.random.RandomState(T).permutation(B + 2)[:B].astype(np.int32)
    h = pool_dev(pool)
    nc, nb = np.zeros(B + 2, np.int64), np.zeros(B + 2, np.int64)
    y = unaligned((B, T, H, 64)) if want_y else None
    bd.prefill(d["x"], d["dt"], v["A"], d["B"], d["C"], v["D"], h, nc, nb, slot_idx=slots, y_fwd=y)
    torch.cuda.synchronize()
    got = torch.from_numpy(from_pool(h))
    for rows, heads in edge_cover(B, H):
        s0 = pool[slots[rows]][:, heads].astype(np.float64)
        s_ref, y_ref = oracle.scan_forward(host_slice(d, rows, heads, hp), s0, want_y=True)
        assert rel_err(pick(got[torch.from_numpy(slots).long()], rows, heads, 1), s_ref) <= REL_TOL
        if want_y:
            assert rel_err(pick(y, rows, heads), y_ref) <= REL_TOL
    left = sorted(set(range(B + 2)) - set(slots.tolist()))
    np.testing.assert_array_equal(got[left].numpy(), pool[left])
    assert nc[slots].tolist() == [T] * B


@pytest.mark.parametrize("B,H,N,L,K", [(24, 32, 128, 32, 5), (16, 17, 64, 16, 7), (24, 32, 32, 20, 6)])
def test_boundary_states_in_one_segment(B, H, N, L, K):
    """Enough row-heads for one segment each: no segment states, no workspace traffic."""
    import paper_2607_02805_amd as bd
    w, d, hp, v = draw(B, H, N, L * K, 13900 + H + N)
    st, y = bd.block_boundary_states(d["x"], d["dt"], v["A"], d["B"], d["C"], v["D"], L, y_fwd=True)
    torch.cuda.synchronize()
    got = torch.from_numpy(from_pool(st).reshape(B, K, H, 64, N))
    for rows, heads in edge_cover(B, H):
        part = host_slice(d, rows, heads, hp)
        s, ys = np.zeros((len(rows), len(heads), 64, N)), []
        for k in range(K):
            assert rel_err(pick(got[:, k], rows, heads, 1), s) <= REL_TOL if k else True
            s, yk = oracle.scan_forward(bi.slice_tokens(part, k * L, (k + 1) * L), s, want_y=True)
            ys.append(yk)
        assert rel_err(pick(y, rows, heads), np.concatenate(ys, 1)) <= REL_TOL
    assert not got[:, 0].any()


def test_reverse_weights_after_a_strong_decay():
    """A token whose decay is 2^-131072 leaves sums whose unit in the last place is 2^-6; the
    tokens after it decay by 1.5 such units each.  The weight of a later token on an earlier one of
    its tile is 2^(difference of two sums); each sum is rounded once, so the exponent is within one
    unit (half a unit more for the weights' own roundings, far less than that)."""
    import paper_2607_02805_amd as bd
    log2e, a = np.float32(1.4426950408889634), np.float32(-0.6931472)
    for _ in range(8):
        if a * log2e == np.float32(-1):
            break
        a = np.nextafter(a, np.float32(-1 if a * log2e > -1 else 0))
    assert a * log2e == np.float32(-1)
    T, N, unit = 64, 16, 2.0 ** -6
    for j in (40, 47, 58, 63):
        x, dt = torch.zeros(1, T, 1, 64), torch.full((1, T, 1), 1.5 * unit)
        x[0, j], dt[0, 0] = 1.0, 131072.0
        B, C = torch.zeros(1, T, 1, N), torch.zeros(1, T, 1, N)
        B[..., 0] = C[..., 0] = 1.0
        v = [t.to(torch.bfloat16).to(DEV) for t in (x, dt, B, C)]
        z = torch.zeros(1, device=DEV)
        y = bd.scan_full_window(v[0], v[1], torch.tensor([float(a)], device=DEV), v[2], v[3], z, z)
        t = np.arange(j // 16 * 16, j)
        got = np.log2(y[0, t, 0, 0].double().cpu().numpy() / (1.5 * unit))
        off = np.abs(got + 1.5 * unit * (j - t)) / unit
        print("exponents off by units", off.round(2).tolist(), flush=True)
        assert off.max() <= 1.25
