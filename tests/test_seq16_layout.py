"""The LDS layouts of the bf16 sequence kernels (bdlm_seq16.hip), written out from the source:
every image index is taken once, a transpose read of B or x hands each lane its operand
element, and the access patterns meet distinct banks (no GPU)."""
import pytest


def c_at(N, t, c):
    if N == 128:
        return t * 16 + (c ^ (4 * (t & 3) + ((t >> 2) & 3)))
    if N == 64:
        return t * 8 + (c ^ (4 * ((t >> 1) & 1) + ((t >> 2) & 3)))
    if N == 32:
        return t * 4 + (c ^ ((t >> 2) & 3))
    return t * 2 + (c ^ ((t >> 3) & 1))


def b_at(N, t, q, a):
    qn = N // 16
    return t * (N // 4) + ((q ^ ((t // (8 // qn)) & (qn - 1))) * 4) + (a ^ (2 * ((t >> 3) & 1)))


def x_at(t, c):
    return t * 8 + (c ^ (2 * ((t >> 1) & 3)) ^ ((t >> 3) & 1))


def n_of(N, q, grp, r):
    """Dstate index of row 4 grp + r of state tile q."""
    return 32 * (q >> 1) + 8 * grp + 4 * (q & 1) + r if N >= 32 else 4 * grp + r


def staged_b(N):
    """Slot (8-byte quads) -> (token, first dstate of the quad), as the staging writes it."""
    at = {}
    for t in range(64):
        for c in range(N // 8):
            for d in range(2):
                slot = b_at(N, t, 2 * (c >> 2) + d, c & 3) if N >= 32 else b_at(N, t, 0, 2 * c + d)
                assert slot not in at
                at[slot] = (t, 8 * c + 4 * d)
    assert sorted(at) == list(range(64 * N // 4))
    return at


def tr_source(lane, r):
    """The lane and element that a transpose read hands to element r of ``lane``."""
    g, s = lane >> 4, lane & 15
    return 16 * g + 4 * r + (s >> 2), s & 3


@pytest.mark.parametrize("N", [16, 32, 64, 128])
def test_images_and_operands(N):
    assert sorted(c_at(N, t, c) for t in range(64) for c in range(N // 8)) == list(range(8 * N))
    assert sorted(x_at(t, c) for t in range(64) for c in range(8)) == list(range(512))
    at = staged_b(N)
    for jt in range(4):
        for q in range(N // 16):
            for lane in range(64):
                for r in range(4):
                    src, e = tr_source(lane, r)
                    tok = 16 * jt + 4 * (src >> 4) + ((src & 15) >> 2)
                    t, n0 = at[b_at(N, tok, q, src & 3)]
                    col = lane & 15
                    assert t == 16 * jt + 4 * (lane >> 4) + r
                    assert n0 + e == n_of(N, q, col >> 2, col & 3)
        for w in range(4):
            for lane in range(64):
                for r in range(4):
                    src, e = tr_source(lane, r)
                    tok, a = 16 * jt + 4 * (src >> 4) + ((src & 15) >> 2), src & 3
                    assert tok == 16 * jt + 4 * (lane >> 4) + r
                    assert 8 * (2 * w + (a >> 1)) + 4 * (a & 1) + e == 16 * w + (lane & 15)
    # a pair of state tiles is one 16-byte piece of a row of C, and B's two quads agree with it
    for u in range(N // 32):
        for grp in range(4):
            for d in range(2):
                assert n_of(N, 2 * u + d, grp, 0) == 8 * (4 * u + grp) + 4 * d
                assert at[b_at(N, 5, 2 * u + d, grp)] == (5, n_of(N, 2 * u + d, grp, 0))


@pytest.mark.parametrize("N", [64, 128])
def test_banks(N):
    """64 banks of 4 bytes: 32 lanes by 8 bytes, or 16 lanes by 16 bytes, meet each at most once."""
    for half in range(2):
        lanes = range(32 * half, 32 * half + 32)
        tr = [(4 * (l >> 4) + ((l & 15) >> 2), l & 3) for l in lanes]
        for q in range(N // 16):
            assert len({b_at(N, t, q, a) % 32 for t, a in tr}) == 32
            assert len({b_at(N, l & 15, q, l >> 4) % 32 for l in lanes}) == 32
        for w in range(4):
            assert len({(2 * x_at(t, 2 * w + (a >> 1)) + (a & 1)) % 32 for t, a in tr}) == 32
            assert len({(2 * x_at(l & 15, 2 * w + (l >> 5)) + ((l >> 4) & 1)) % 32 for l in lanes}) == 32
    for c in range(N // 8):
        assert len({c_at(N, t, c) % 16 for t in range(16)}) == 16


def m_at(full, mt, jt):
    h = mt >> 1
    return ((2 * mt if full else h * (h + 1) + (mt & 1) * (h + 1)) + (jt >> 1)) * 256 + (jt & 1)


@pytest.mark.parametrize("full", [True, False])
def test_weighted_tiles_do_not_overlap(full):
    """Each tile's hi quads at m_at + 2 lane and lo quads 128 further on, in 8-byte units."""
    seen = set()
    for mt in range(4):
        for jt in range(4 if full else mt + 1):
            for lane in range(64):
                for z in range(2):
                    slot = m_at(full, mt, jt) + 2 * lane + 128 * z
                    assert slot not in seen and slot < (8 if full else 6) * 256
                    seen.add(slot)
