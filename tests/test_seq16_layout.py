"""The LDS of the bf16 sequence kernels (bdlm_seq16.hip), written out from the source: every
image index is taken once, a transpose read of B or x hands each lane its operand element,
images are staged to and read from distinct banks by a model of 64 banks, and the accesses
of a chunk, barrier interval by barrier interval, do not race (no GPU)."""
import pytest

from tests.test_lds_model import new_model


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


def by_bank(slots, nbytes):
    """The most accesses of ``nbytes`` that one bank sees when a wave's are served 256 bytes at a
    time over 64 banks of 4 bytes (slots: lane by lane, in units of nbytes)."""
    n = 256 // nbytes
    return max(sum(s % n == b for s in slots[i:i + n]) for i in range(0, 64, n) for b in range(n))


@pytest.mark.parametrize("N", [16, 32, 64, 128])
def test_banks(N):
    """Each bank once, but for two patterns: staging B at dstate 16, and the weighted tiles, whose
    two source tiles lie side by side (8 bytes every 16).  The GPU's counters show more
    conflicts than this model: 17 to 28 % of the kernels' LDS cycles at dstate 128."""
    CH, lanes = N // 8, range(64)
    for d in range(2):
        b = [b_at(N, l // CH, 2 * ((l % CH) >> 2) + d, (l % CH) & 3) if N >= 32 else b_at(N, l // CH, 0, 2 * (l % CH) + d)
             for l in lanes]
        assert by_bank(b, 8) == (1 if N >= 32 else 2)
    assert by_bank([c_at(N, l // CH, l % CH) for l in lanes], 16) == 1
    assert by_bank([x_at(l >> 3, l & 7) for l in lanes], 16) == 1
    tr = [(4 * (l >> 4) + ((l & 15) >> 2), l & 3) for l in lanes]
    for jt in range(4):
        for q in range(N // 16):
            assert by_bank([b_at(N, 16 * jt + t, q, a) for t, a in tr], 8) == 1
            assert by_bank([b_at(N, 16 * jt + (l & 15), q, l >> 4) for l in lanes], 8) == 1
        for w in range(4):
            assert by_bank([2 * x_at(16 * jt + t, 2 * w + (a >> 1)) + (a & 1) for t, a in tr], 8) == 1
            assert by_bank([2 * x_at(16 * jt + (l & 15), 2 * w + (l >> 5)) + ((l >> 4) & 1) for l in lanes], 8) == 1
        for u in range(N // 32):
            assert by_bank([c_at(N, 16 * jt + (l & 15), 4 * u + (l >> 4)) for l in lanes], 16) == 1
    assert by_bank([m_at(True, 1, 0) + 2 * l for l in lanes], 8) == 2


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


# ---- the accesses of a chunk (as in test_lds_model.py)
def tok_of(lane):
    return 4 * (lane >> 4) + ((lane & 15) >> 2)


def stage(m, N, hpw, with_c):
    nt, CH = 256 * hpw, N // 8
    for tid in range(nt):
        for k in range(max(1, 64 * CH // nt)):
            t, c = tid // CH + nt // CH * k, tid % CH
            if t >= 64:
                continue
            for d in range(2):
                at = b_at(N, t, 2 * (c >> 2) + d, c & 3) if N >= 32 else b_at(N, t, 0, 2 * c + d)
                m.access(tid, "W", 1 + d, "sB", at * 8, 8, tag=("sB", t, 8 * c + 4 * d))
                if with_c:
                    m.access(tid, "W", 3, "sC", c_at(N, t, c) * 16 + 8 * d, 8, tag=("sC", t, 8 * c + 4 * d))
        for k in range(2):
            t, c = ((tid & 255) >> 3) + 32 * k, tid & 7
            for d in range(2):
                m.access(tid, "W", 4, f"sX{tid >> 8}", x_at(t, c) * 16 + 8 * d, 8, tag=("sX", t, 8 * c + 4 * d))


def decays(m, hpw, names):
    for h in range(hpw):
        for lane in range(64):
            for a in names:
                m.access(256 * h + lane, "W", 5, f"{a}{h}", lane * 4, 4, tag=(a, lane))


def read4(m, tid, instr, a, h, i):
    for r in range(4):
        m.access(tid, "R", instr, f"{a}{h}", 4 * (i + r), 4, tag=(a, i + r))


def read_x(m, tid, instr):
    lane, w, h = tid & 63, (tid >> 6) & 3, tid >> 8
    for jt in range(4):
        t, a = 16 * jt + tok_of(lane), lane & 3
        m.access(tid, "R", instr, f"sX{h}", 16 * x_at(t, 2 * w + (a >> 1)) + 8 * (a & 1), 8,
                 tag=("sX", t, 16 * w + 4 * a))


def read_b(m, tid, instr, N):
    lane = tid & 63
    for q in range(N // 16):
        for jt in range(4):
            t, a = 16 * jt + tok_of(lane), lane & 3
            m.access(tid, "R", instr, "sB", 8 * b_at(N, t, q, a), 8, tag=("sB", t, n_of(N, q, a, 0)))


def seg_state_model(N, both):
    names = ("Ws", "Wr") if both else ("Ws",)
    m = new_model({"sB": 128 * N, "sX0": 8192, "sTot": 16, "Ws0": 256, "Wr0": 256})
    m.barrier()                                # kernel start / the previous chunk's last barrier
    stage(m, N, 1, False)
    decays(m, 1, names)
    m.access(0, "W", 6, "sTot", 0, 4, tag="tot")
    m.barrier()
    for tid in range(256):
        m.access(tid, "R", 10, "sTot", 0, 4, tag="tot")
        read_x(m, tid, 11)
        for jt in range(4):
            for a in names:
                read4(m, tid, 12, a, 0, 16 * jt + 4 * ((tid & 63) >> 4))
        read_b(m, tid, 13, N)
    m.barrier()
    return m


FWD, BOTH, PRE = 0, 1, 2


def products(mode, hpw, wv):
    """(row tile, source tile, first head, end of heads) of wave wv's products."""
    if mode == BOTH:
        tpw = 4 // hpw
        return [(wv & 3, tpw * (wv >> 2) + i, 0, hpw) for i in range(tpw)]
    out = []
    for i in range(2):                         # kFwd runs with two heads only
        kt, h0, h1 = (wv, 0, 2) if i == 0 else (8 + ((wv >> 1) & 1), wv & 1, (wv & 1) + 1 if wv < 4 else 0)
        if kt >= 10:
            kt, h1 = 0, 0
        mt = 0 if kt < 1 else (1 if kt < 3 else (2 if kt < 6 else 3))
        out.append((mt, kt - mt * (mt + 1) // 2, h0, h1))
    return out


def seg_out_model(N, hpw, mode, barrier_over=True):
    gram, full = mode != PRE, mode == BOTH
    over = hpw == 2 and full and N == 128
    names = ("Ec", "Ws", "Cs") + (("Dt", "La", "Lb") if gram else ()) + (("Ex", "Ua", "Ub") if full else ())
    arrays = {"sB": 128 * N, "sC": 128 * N}
    for h in range(hpw):
        arrays[f"sX{h}"] = 8192
        arrays[f"sM{h}"] = (8 if full else 6) * 2048 if gram else 16
        for a in names:
            arrays[f"{a}{h}"] = 256
    m_of = (lambda h: "sC" if h == 0 else "sM0") if over else (lambda h: f"sM{h}")
    m = new_model(arrays)
    m.barrier()
    stage(m, N, hpw, True)
    decays(m, hpw, names)
    m.barrier()

    def weigh(tid):
        lane = tid & 63
        col, grp = lane & 15, lane >> 4
        for mt, jt, h0, h1 in products(mode, hpw, tid >> 6):
            t, j = 16 * mt + col, 16 * jt + 4 * grp
            for h in range(h0, h1):
                def one(a, i):
                    m.access(tid, "R", 21, f"{a}{h}", 4 * i, 4, tag=(a, i))
                if jt != mt:
                    below = jt < mt
                    lo, hi = min(mt, jt), max(mt, jt)
                    if hi > lo + 1:
                        one("Cs", 16 * hi - 1)
                        one("Cs", 16 * lo + 15)
                    one("La" if below else "Ua", t)
                    read4(m, tid, 21, "Lb" if below else "Ub", h, j)
                else:
                    for a in ("Cs", "Dt") + (("Ex",) if full else ()):
                        read4(m, tid, 21, a, h, j)
                    one("Cs", t)
                for z in range(2):
                    m.access(tid, "W", 22, m_of(h), 8 * (m_at(full, mt, jt) + 2 * lane + 128 * z), 8,
                             tag=("M", h, mt, jt, lane, z))

    def c_read(tid, mt, u):                    # 16 bytes: 32 dstates of token 16 mt + col (N = 16: 8)
        col, grp = tid & 15, (tid & 63) >> 4
        t = 16 * mt + col
        if N == 16:
            m.access(tid, "R", 20, "sC", 16 * c_at(N, t, grp >> 1) + 8 * (grp & 1), 8, tag=("sC", t, 4 * grp))
            return
        for d in range(2):
            m.access(tid, "R", 20, "sC", 16 * c_at(N, t, 4 * u + grp) + 8 * d, 8, tag=("sC", t, n_of(N, 2 * u + d, grp, 0)))

    for tid in range(256 * hpw):
        col, grp, h = tid & 15, (tid & 63) >> 4, tid >> 8
        if gram:
            for mt, jt, _, _ in products(mode, hpw, tid >> 6):
                for q in range(N // 16):
                    m.access(tid, "R", 20, "sB", 8 * b_at(N, 16 * jt + col, q, grp), 8,
                             tag=("sB", 16 * jt + col, n_of(N, q, grp, 0)))
                for u in range(max(1, N // 32)):
                    c_read(tid, mt, u)
            if not over:
                weigh(tid)
        for mt in range(4):
            for u in range(max(1, N // 32)):
                c_read(tid, mt, u)
            m.access(tid, "R", 20, f"Ec{h}", 4 * (16 * mt + col), 4, tag=("Ec", 16 * mt + col))
    if over:
        if barrier_over:
            m.barrier()                        # every wave has read C
        for tid in range(256 * hpw):
            weigh(tid)
    if gram:
        m.barrier()                            # M published
    for tid in range(256 * hpw):
        lane, w, h = tid & 63, (tid >> 6) & 3, tid >> 8
        col, grp = lane & 15, lane >> 4
        read_x(m, tid, 30)
        if gram:
            for mt in range(4):
                for jt in range(4 if full else mt + 1):
                    for z in range(2):         # (the quad of a tile above the diagonal is not used)
                        m.access(tid, "R", 31, m_of(h), 8 * m_at(full, mt, jt - (jt & 1)) + 16 * lane + 1024 * z + 8 * (jt & 1),
                                 8, tag=("M", h, mt, jt, lane, z))
                t, p = 16 * mt + col, 16 * w + 4 * grp
                m.access(tid, "R", 32, f"sX{h}", 16 * x_at(t, 2 * w + (grp >> 1)) + 8 * (grp & 1), 8, tag=("sX", t, p))
        m.access(tid, "R", 33, f"Cs{h}", 4 * 63, 4, tag=("Cs", 63))
        for jt in range(4):
            read4(m, tid, 33, "Ws", h, 16 * jt + 4 * grp)
        read_b(m, tid, 34, N)
    m.barrier()                                # LDS is rewritten by the next chunk
    return m


@pytest.mark.parametrize("N", [16, 32, 64, 128])
@pytest.mark.parametrize("both", [False, True])
def test_seg_state_accesses(N, both):
    assert seg_state_model(N, both).check() == []


@pytest.mark.parametrize("N", [16, 32, 64, 128])
@pytest.mark.parametrize("hpw,mode", [(1, BOTH), (2, BOTH), (2, FWD), (1, PRE)])
def test_seg_out_accesses(N, hpw, mode):
    assert seg_out_model(N, hpw, mode).check() == []


def test_tiles_in_place_of_c_need_their_barrier():
    """dstate 128, two heads: head 0's weighted tiles overwrite C.  Without the barrier before
    them the model finds waves that still read it."""
    assert seg_out_model(128, 2, BOTH, barrier_over=False).check() != []
