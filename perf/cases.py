"""The work a program has this library do, as cases that can be timed and checked.

A case is one call sequence of a Mamba layer (or a stack of them) as a block-diffusion
decoder, a prefill or a training forward makes it: denoising steps and commits of the
active block, the mixer with its convolution and gated normalisation, steps whose reverse
branch has inputs of its own, prefills, full windows and the all-block training forward.
Layer shapes are those of the 87M and 350M models and of the paper's widths (14 and 26
heads), and odd ones between them; head dimension 64 throughout.

Inputs follow the distributions of ``bdlm_inputs.py`` and are drawn on the GPU.  States
are drawn at the scale a long prefix leaves behind (see ``_states``).
"""
import math

import numpy as np
import torch

import paper_2607_02805_amd as bd

P = 64            # head dimension
EPS = 1e-5        # of the gated normalisation


def _case(kind, batch, heads, dstate, block, *, groups=1, dtype="bf16", length=0, steps=1,
          layers=1, slots=False, outputs=True, fused=False, **name):
    return dict(kind=kind, batch=batch, heads=heads, dstate=dstate, groups=groups, block=block,
                dtype=dtype, length=length, steps=steps, layers=layers, slots=slots,
                outputs=outputs, fused=fused, **name)


def listed():
    return [
        # the smallest call: one step of a tiny fp32 layer, where only launch and host
        # latency count
        _case("step", 1, 4, 16, 16, dtype="fp32", name="step_tiny_fp32"),
        # one layer of the 87M model in an eager decode loop: a denoising step, then the
        # commit of the finished block
        _case("cycle", 8, 24, 64, 32, outputs=False, name="cycle_87m_b8_l32"),
        # the 350M model's Mamba layers through one block: 8 denoising steps and a commit per
        # layer, replayed from a HIP graph (how decoding runs, and the headline's launches)
        _case("stack", 16, 32, 128, 32, steps=8, layers=24, outputs=False,
              name="stack_350m_b16_l32"),
        # a denoising step of a large serving batch
        _case("step", 128, 32, 128, 32, name="step_350m_b128_l32"),
        # the paper's block length at its 350M width: a step and a commit with the clean
        # block's outputs
        _case("cycle", 16, 26, 128, 256, name="cycle_paper_b16_l256"),
        # the whole mixer around the scan: step with the convolution, gated normalisation,
        # commit with the convolution rows
        _case("mixer", 16, 32, 128, 32, name="mixer_350m_b16_l32"),
        # the same at the paper's block length
        _case("mixer", 16, 26, 128, 256, name="mixer_paper_b16_l256"),
        # a reverse branch with projections of its own at the paper's block length
        _case("sep", 16, 26, 128, 256, name="sep_paper_b16_l256"),
        # a long prompt through one layer: the states into the cache, the outputs on through
        # the gated normalisation to the next layer
        _case("prefill", 16, 32, 128, 0, length=16384, name="prefill_350m_b16_16k"),
        # a ragged fp32 prompt into chosen slots of a cache
        _case("prefill", 3, 24, 64, 0, length=5003, dtype="fp32", slots=True,
              name="prefill_fp32_b3_5003"),
        # the full-sequence bidirectional scan that the cache replaces
        _case("window", 4, 32, 128, 0, length=65536, name="window_350m_b4_65k"),
        # the training forward of one layer: every block noised, from its clean prefix's state
        _case("train", 8, 32, 128, 32, length=8192, name="train_350m_b8_8k_l32"),
    ]


def _log(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))))


def draw(rng):
    """One more case: the kinds and ranges of the listed ones."""
    kind = rng.choice(["step", "step", "cycle", "cycle", "stack", "mixer", "mixer", "sep",
                       "prefill", "prefill", "window", "train"])
    heads, dstate = rng.choice([(4, 16), (rng.randint(3, 12), 32), (24, 64), (14, 128), (26, 128),
                                (32, 128), (32, 128), (rng.randint(8, 32), 64)])
    groups = 2 if heads % 2 == 0 and rng.random() < 0.15 else 1
    dtype = "fp32" if rng.random() < 0.2 else "bf16"
    block = rng.choice([16, 32, 32, 64, 128, 256, 256, rng.randint(1, 64), rng.randint(65, 256)])
    batch = _log(rng, 1, 128)
    kw = dict(groups=groups, dtype=dtype, slots=rng.random() < 0.3)
    if kind == "step":
        return _case(kind, min(batch, max(1, 4096 // block)), heads, dstate, block, **kw)
    if kind == "cycle":
        fused = rng.random() < 0.4
        block = min(block, 64) if fused else block
        return _case(kind, min(batch, max(1, 4096 // block)), heads, dstate, block, fused=fused,
                     steps=rng.choice([1, 2, 4]), outputs=rng.random() < 0.5, **kw)
    if kind == "stack":
        kw["dtype"] = "bf16"
        return _case(kind, _log(rng, 1, 16), heads, dstate, min(block, 64),
                     steps=rng.choice([1, 4, 8]), layers=rng.choice([12, 24]), outputs=False, **kw)
    if kind in ("mixer", "sep"):
        return _case(kind, min(batch, max(1, 4096 // block)), heads, dstate, block, **kw)
    # token-heads of one call, at most those of the listed cases (fp32 activations take the
    # slower fp32 matrix rate: an eighth)
    share = 8 if dtype == "fp32" else 1
    if kind == "prefill":
        length = _log(rng, 200, 32768)
        most = 16 * 16384 * 32 // share
        return _case(kind, max(1, min(batch, most // (length * heads))), heads, dstate, 0,
                     length=length, outputs=rng.random() < 0.7, **kw)
    kw["slots"] = False
    if kind == "window":
        length = _log(rng, 500, 65536)
        most = 4 * 65536 * 32 // share
        return _case(kind, max(1, min(batch, 64, most // (length * heads))), heads, dstate, 0,
                     length=length, **kw)
    block = min(block, 64)
    nblk = _log(rng, 4, max(4, min(512, 8192 // block)))
    most = 8 * 8192 * 32 // share
    return _case("train", max(1, min(batch, most // (nblk * block * heads), 8 * 256 // nblk)), heads,
                 dstate, block, length=nblk * block, outputs=rng.random() < 0.7, **kw)


# ------------------------------------------------------------------ inputs
def _dtype(case):
    return torch.float32 if case["dtype"] == "fp32" else torch.bfloat16


def _gen(seed, device):
    g = torch.Generator(device=device)
    g.manual_seed(int(seed))
    return g


def _randn(shape, g):
    return torch.randn(shape, generator=g, device=g.device, dtype=torch.float32)


def _heads(case, g):
    H = case["heads"]
    A = -torch.exp(torch.rand(H, generator=g, device=g.device) * math.log(16.0))
    D = _randn((H,), g)
    return A, D


def _tokens(case, lead, T, g):
    """(x, dt, B, C) of ``lead`` x T tokens in the case's storage type."""
    H, G, N, dty = case["heads"], case["groups"], case["dstate"], _dtype(case)
    x = _randn((*lead, T, H, P), g).to(dty)
    dt = torch.nn.functional.softplus(0.5 * _randn((*lead, T, H), g) - 4.6).to(dty)
    B = (_randn((*lead, T, G, N), g) / math.sqrt(N)).to(dty)
    C = (_randn((*lead, T, G, N), g) / math.sqrt(N)).to(dty)
    return x, dt, B, C


def _states(case, lead, A, g):
    """States in the pool layout at the scale of a long prefix: an element sums
    dt x B over tokens weighted by the decay, so its variance is about dt / (2 |A| N)."""
    H, N = case["heads"], case["dstate"]
    std = torch.sqrt(0.011 / (2.0 * -A * N))
    return _randn((*lead, *bd.pool_shape(1, H, N)[1:]), g) * std.view(H, 1, 1, 1)


def _slot_map(case, seed):
    if not case["slots"]:
        return None, case["batch"]
    nslots = case["batch"] + 3
    return np.random.RandomState(seed % (1 << 31)).permutation(nslots)[:case["batch"]].astype(
        np.int32), nslots


def _inputs(case, seed, device):
    """Everything a pass reads, as torch tensors."""
    g = _gen(seed, device)
    bsz, kind = case["batch"], case["kind"]
    A, D = _heads(case, g)
    s = {"A": A, "D": D, "D_rev": D.clone()}
    s["slots"], nslots = _slot_map(case, seed)
    if kind == "stack":
        n = case["layers"]
        s["noised"] = _tokens(case, (n, case["steps"], bsz), case["block"], g)
        s["clean"] = _tokens(case, (n, bsz), case["block"], g)
        s["h"] = _states(case, (n, nslots), A, g)
        return s
    if kind in ("step", "cycle", "mixer", "sep"):
        s["noised"] = [_tokens(case, (bsz,), case["block"], g) for _ in range(case["steps"])]
        s["clean"] = _tokens(case, (bsz,), case["block"], g)
        s["h"] = _states(case, (nslots,), A, g)
    elif kind == "prefill":
        s["clean"] = _tokens(case, (bsz,), case["length"], g)
        s["h"] = _states(case, (nslots,), A, g)
    else:
        s["clean"] = _tokens(case, (bsz,), case["length"], g)
    if kind == "train":
        s["noised"] = [_tokens(case, (bsz,), case["length"], g)]
    if kind == "sep":
        s["rev_heads"] = _heads(case, g)
        s["rev"] = _tokens(case, (bsz,), case["block"], g)
    if kind == "mixer":
        ch = bd.conv_channels(case["heads"], case["groups"], case["dstate"])
        s["conv_w"] = _randn((ch, 4), g) * 0.5
        s["conv_b"] = _randn((ch,), g) * 0.1
        s["conv"] = _randn((nslots, 3, ch), g)
    if kind == "mixer" or (kind == "prefill" and case["outputs"]):
        T = case["block"] or case["length"]
        ch = case["heads"] * P
        s["z"] = _randn((bsz, T, ch), g).to(_dtype(case))
        s["norm_w"] = 1.0 + 0.1 * _randn((ch,), g)
    return s


def _cache(case, s):
    cache = bd.Cache(s["h"].shape[-5], case["heads"], case["dstate"],
                     ngroups=case["groups"] if case["kind"] == "mixer" else 0)
    cache.h = s["h"]
    if case["kind"] == "mixer":
        cache.conv = s["conv"]
    return cache


def _y(case, lead=()):
    return torch.empty((*lead, case["batch"], case["block"], case["heads"], P), device="cuda")


def prepare(case, seed):
    s = _inputs(case, seed, "cuda")
    s["case"] = case
    kind = case["kind"]
    if kind in ("step", "cycle", "mixer", "sep", "prefill"):
        s["cache"] = _cache(case, s)
    if kind in ("step", "cycle", "mixer", "sep"):
        s["y"] = _y(case)
        s["y_clean"] = _y(case) if case["outputs"] else None
    if kind == "mixer":
        s["out"] = torch.empty_like(s["y"])
    if kind == "stack":
        _capture(case, s)
    return s


def _capture(case, s):
    """The whole stack's block cycle as one HIP graph, as a decoder keeps it."""
    n, slots = case["layers"], s["slots"]
    s["y"] = _y(case, (n,))
    caches = []
    for i in range(n):
        c = bd.Cache(s["h"].shape[1], case["heads"], case["dstate"])
        c.h = s["h"][i]
        caches.append(c)
    s["caches"] = caches

    def block():
        for k in range(case["steps"]):
            for i in range(n):
                x, dt, B, C = (t[i, k] for t in s["noised"])
                caches[i].step(x, dt, s["A"], B, C, s["D"], s["D_rev"], y=s["y"][i], slot_idx=slots)
        for i in range(n):
            x, dt, B, C = (t[i] for t in s["clean"])
            caches[i].commit(x, dt, s["A"], B, C, s["D"], s["D_rev"], slot_idx=slots)

    s["graph"] = torch.cuda.CUDAGraph()
    with torch.cuda.graph(s["graph"]):
        block()


# ------------------------------------------------------------------ one pass
def run(s):
    case = s["case"]
    kind, slots = case["kind"], s["slots"]
    A, D, Dr = s["A"], s["D"], s["D_rev"]
    if kind == "stack":
        s["graph"].replay()
        return s["y"], s["h"]
    if kind == "window":
        x, dt, B, C = s["clean"]
        return bd.scan_full_window(x, dt, A, B, C, D, Dr)
    if kind == "train":
        return bd.all_block_forward(s["clean"], s["noised"][0], A, D, Dr, case["block"],
                                    want_clean_y=case["outputs"])
    cache = s["cache"]
    if kind == "prefill":
        x, dt, B, C = s["clean"]
        y = cache.prefill(x, dt, A, B, C, D, slot_idx=slots, y_fwd=True if case["outputs"] else None)
        if y is None:
            return cache.h
        return bd.gated_rmsnorm(y, s["z"], s["norm_w"], EPS), y, cache.h
    x, dt, B, C = s["noised"][0]
    if kind == "step":
        return cache.step(x, dt, A, B, C, D, Dr, y=s["y"], slot_idx=slots)
    if kind == "sep":
        Ar, Drr = s["rev_heads"]
        xr, dtr, Br, Cr = s["rev"]
        return bd.scan_block_step_sep((x, dt, A, B, C, D), (xr, dtr, Ar, Br, Cr, Drr), cache.h,
                                      y=s["y"], slot_idx=slots)
    if kind == "mixer":
        cw, cb = s["conv_w"], s["conv_b"]
        y = cache.conv_step(x, dt, A, B, C, D, Dr, cw, cb, y=s["y"], slot_idx=slots)
        out = bd.gated_rmsnorm(y, s["z"], s["norm_w"], EPS, out=s["out"])
        xc, dtc, Bc, Cc = s["clean"]
        yc = cache.conv_commit(xc, dtc, A, Bc, Cc, D, Dr, cw, cb, slot_idx=slots,
                               y_clean=s["y_clean"])
        return out, y, yc, cache.h, cache.conv
    # cycle: the denoising steps, then the commit; fused: the commit with the next block's
    # first step, then the other steps
    noised, (xc, dtc, Bc, Cc) = s["noised"], s["clean"]
    if case["fused"]:
        y, yc = bd.commit_step(s["clean"], noised[0], A, D, Dr, cache.h, cache.n_committed,
                               cache.n_blocks, slot_idx=slots, y_clean=s["y_clean"], y_next=s["y"])
        for x, dt, B, C in noised[1:]:
            y = cache.step(x, dt, A, B, C, D, Dr, y=s["y"], slot_idx=slots)
    else:
        for x, dt, B, C in noised:
            y = cache.step(x, dt, A, B, C, D, Dr, y=s["y"], slot_idx=slots)
        yc = cache.commit(xc, dtc, A, Bc, Cc, D, Dr, slot_idx=slots, y_clean=s["y_clean"])
    return (y, cache.h) if yc is None else (y, cache.h, yc)


# ------------------------------------------------------------------ what a pass needs
def _scan_work(case, tokens, states_read, states_written, y, dirs, entering=1):
    """Bytes and operations of scanning ``tokens`` (over all batch rows) once: inputs once,
    outputs (if ``y``) once, states once; per token and head the decay, the outer product
    into the state and the contraction with C, in each direction."""
    H, G, N = case["heads"], case["groups"], case["dstate"]
    e = 4 if case["dtype"] == "fp32" else 2
    nbytes = tokens * (H * P * e + H * e + 2 * G * N * e) + (tokens * H * P * 4 if y else 0)
    nbytes += (states_read + states_written) * H * P * N * 4
    return nbytes, tokens * H * dirs * (4 + (2 if y else 0)) * P * N


def work(case):
    bsz, L, T, kind = case["batch"], case["block"], case["length"], case["kind"]
    H, G, N = case["heads"], case["groups"], case["dstate"]
    e = 4 if case["dtype"] == "fp32" else 2
    norm = bsz * (L or T) * H * P * (4 + e) + H * P * 4   # z in, normalised out, weights
    parts = []
    if kind in ("step", "cycle", "stack", "mixer", "sep"):
        n = case["layers"] * case["steps"]
        parts += [_scan_work(case, bsz * L, bsz, 0, True, 2)] * n
    if kind in ("cycle", "stack", "mixer"):
        two = 2 if case["outputs"] else 1
        parts += [_scan_work(case, bsz * L, bsz, bsz, case["outputs"], two)] * case["layers"]
    if kind == "sep":
        b, f = _scan_work(case, bsz * L, 0, 0, False, 0)
        parts.append((b, f))
    if kind == "mixer":
        ch = bd.conv_channels(H, G, N)
        parts.append((norm + 2 * ch * 5 * 4 + bsz * ch * 9 * 4, 2 * bsz * L * ch * 2 * 10))
    if kind == "prefill":
        parts.append(_scan_work(case, bsz * T, bsz, bsz, case["outputs"], 1))
        if case["outputs"]:
            parts.append((norm, bsz * T * H * P * 8))
    if kind == "window":
        parts.append(_scan_work(case, bsz * T, 0, 0, True, 2))
    if kind == "train":
        blocks = bsz * (T // L)
        parts.append(_scan_work(case, bsz * T, 0, blocks, case["outputs"], 1))
        parts.append(_scan_work(case, bsz * T, 0, 0, True, 2))
    return {"bytes": float(sum(p[0] for p in parts)), "flops": float(sum(p[1] for p in parts))}


def tolerance(case):
    # every product has fp32 terms (split into two or three bf16 terms, or fp32 MFMA) and
    # every sum is fp32: against fp64 the largest seen over these ranges are 5.4e-7 in 2-norm
    # and 1e-5 in one value (the states a 256-token commit leaves); about four times those
    return {"rel": 2e-6, "max": 4e-5}


# ------------------------------------------------------------------ in 64 bits
def _to_rows(pool):
    """Pool layout [..., H, N/4, 64, 4] -> fp64 [..., H, 64, N]."""
    p = pool.double().transpose(-3, -2)
    return p.reshape(*p.shape[:-2], p.shape[-2] * 4).contiguous()


def _to_pool(rows):
    *lead, p, n = rows.shape
    return rows.reshape(*lead, p, n // 4, 4).transpose(-3, -2).contiguous()


def _scan64(tok, A, skip, S0, chunk=64, reverse=False, entering=False):
    """The scan of one batch row in fp64, chunk by chunk: y [T, H, 64], the final state
    [H, 64, N] and, if asked, the states entering every chunk.  S0: [H, 64, N] or None."""
    x, dt, B, C = tok
    T, H, _ = x.shape
    G, N = B.shape[1:]
    if reverse:
        x, dt, B, C = (t.flip(0) for t in (x, dt, B, C))
    n = -(-T // chunk)

    def cut(t):   # [T, ...] -> [n, chunk, ...] in fp64, zeros past the end
        t = t.double()
        if n * chunk != T:
            t = torch.cat([t, t.new_zeros((n * chunk - T, *t.shape[1:]))])
        return t.reshape(n, chunk, *t.shape[1:])

    xc = cut(x).transpose(1, 2).contiguous()                  # [n, H, c, P]
    d = cut(dt).transpose(1, 2).contiguous()                  # [n, H, c]
    Bc, Cc = (cut(t).transpose(1, 2).contiguous() for t in (B, C))   # [n, G, c, N]
    cs = torch.cumsum(d * A.double().view(1, H, 1), -1)       # [n, H, c]
    tot = cs[..., -1]
    gram = torch.matmul(Cc, Bc.transpose(-1, -2).contiguous())      # [n, G, c, c]
    per = H // G
    Bh, Ch = Bc.repeat_interleave(per, 1), Cc.repeat_interleave(per, 1)
    low = torch.ones(chunk, chunk, dtype=torch.bool, device=x.device).tril()
    M = torch.where(low, cs.unsqueeze(-1) - cs.unsqueeze(-2), -torch.inf).exp_()
    M *= d.unsqueeze(-2)
    M *= gram.repeat_interleave(per, 1)
    y = torch.matmul(M, xc)
    del M, gram
    wx = xc * ((tot.unsqueeze(-1) - cs).exp() * d).unsqueeze(-1)
    U = torch.matmul(wx.transpose(-1, -2).contiguous(), Bh)   # [n, H, P, N]
    S = torch.zeros(H, P, N, dtype=torch.float64, device=x.device) if S0 is None else S0.clone()
    keep = tot.exp().view(n, H, 1, 1)
    for k in range(n):                                        # U[k] becomes the state entering k
        u = U[k].clone()
        U[k] = S
        S = S * keep[k] + u
    y += torch.matmul(Ch * cs.exp().unsqueeze(-1), U.transpose(-1, -2).contiguous())
    y = y.transpose(1, 2).reshape(n * chunk, H, P)[:T] + x.double() * skip.double().view(1, H, 1)
    return (y.flip(0) if reverse else y), S, (U if entering else None)


def _rows(tok, b):
    return tuple(t[b] for t in tok)


def _block64(tok, A, D, Dr, h, slots, rev=None):
    """A step (or commit) of every batch row: y and the states after the block."""
    ys, hs = [], []
    for b in range(tok[0].shape[0]):
        row = _rows(tok, b)
        yf, S, _ = _scan64(row, A, D, h[b if slots is None else int(slots[b])])
        rtok, rA, rD = (row, A, Dr) if rev is None else (_rows(rev[0], b), rev[1], rev[2])
        ys.append(yf + _scan64(rtok, rA, rD, None, reverse=True)[0])
        hs.append(S)
    return torch.stack(ys), torch.stack(hs)


def _stored(h, new, slots):
    """The pool's rows after the batch rows' new states (or rows) went to their slots."""
    out = h.clone()
    idx = torch.arange(len(new)) if slots is None else torch.from_numpy(np.asarray(slots)).long()
    out[idx.to(out.device)] = new
    return out


def _conv64(tok, w, b, rows, slots):
    """Width-4 depthwise convolution and SiLU in fp64: (forward, reverse) x, B, C and the
    rows that a commit keeps."""
    x, dt, B, C = tok
    bsz, L, H, _ = x.shape
    G, N = B.shape[2:]
    u = torch.cat([t.double().reshape(bsz, L, -1) for t in (x, B, C)], -1)
    old = rows.double() if slots is None else rows.double()[torch.from_numpy(slots).long().to(u.device)]
    ext = torch.cat([old[:bsz], u, torch.zeros_like(old[:bsz])], 1)
    w, b = w.double(), b.double()
    fwd = b + sum(w[:, k] * ext[:, k:k + L] for k in range(4))
    rev = b + sum(w[:, k] * ext[:, 6 - k:6 - k + L] for k in range(4))

    def back(v):
        v = v * torch.sigmoid(v)
        return (v[..., :H * P].reshape(bsz, L, H, P), dt,
                v[..., H * P:H * P + G * N].reshape(bsz, L, G, N),
                v[..., H * P + G * N:].reshape(bsz, L, G, N))

    return back(fwd), back(rev), ext[:, L:L + 3]


def _norm64(y, z, w):
    z = z.double()
    g = y.reshape(z.shape) * z * torch.sigmoid(z)
    out = w.double() * g * torch.rsqrt(g.square().mean(-1, keepdim=True) + EPS)
    return out.reshape(y.shape)


def exact(case, seed, device="cuda"):
    s = _inputs(case, seed, device)
    kind, slots = case["kind"], s["slots"]
    A, D, Dr = s["A"], s["D"], s["D_rev"]
    bsz, L = case["batch"], case["block"]
    if kind == "window":
        return torch.stack([_scan64(_rows(s["clean"], b), A, D, None)[0]
                            + _scan64(_rows(s["clean"], b), A, Dr, None, reverse=True)[0]
                            for b in range(bsz)])
    if kind == "train":
        y, yc, st = [], [], []
        K = case["length"] // L
        for b in range(bsz):
            yf, _, ent = _scan64(_rows(s["clean"], b), A, D, None, chunk=L, entering=True)
            yc.append(yf)
            st.append(_to_pool(ent).float())   # the values fp32 states hold
            tok = tuple(t[b].reshape(K, L, *t.shape[2:]) for t in s["noised"][0])
            y.append(torch.cat([_block64(_rows_of(tok, k), A, D, Dr, ent[k:k + 1], None)[0][0]
                                for k in range(K)]))
        out = torch.stack(y), torch.cat(st)
        return (*out, torch.stack(yc)) if case["outputs"] else out
    if kind == "stack":
        ys, hs = [], []
        for i in range(case["layers"]):
            h = _to_rows(s["h"][i])
            tok = tuple(t[i, case["steps"] - 1] for t in s["noised"])
            ys.append(_block64(tok, A, D, Dr, h, slots)[0])
            S = _block64(tuple(t[i] for t in s["clean"]), A, D, Dr, h, slots)[1]
            hs.append(_to_pool(_stored(h, S, slots)))
        return torch.stack(ys), torch.stack(hs)
    h = _to_rows(s["h"])
    if kind == "prefill":
        ys, hs = [], []
        for b in range(bsz):
            y, S, _ = _scan64(_rows(s["clean"], b), A, D, h[b if slots is None else int(slots[b])])
            ys.append(y if case["outputs"] else None)
            hs.append(S)
        pool = _to_pool(_stored(h, torch.stack(hs), slots))
        if not case["outputs"]:
            return pool
        y = torch.stack(ys)
        del ys
        out = torch.stack([_norm64(y[b:b + 1], s["z"][b:b + 1], s["norm_w"])[0] for b in range(bsz)])
        return out, y, pool
    if kind == "step":
        return _block64(s["noised"][0], A, D, Dr, h, slots)[0]
    if kind == "sep":
        Ar, Drr = s["rev_heads"]
        return _block64(s["noised"][0], A, D, Dr, h, slots, (s["rev"], Ar, Drr))[0]
    if kind == "mixer":
        cw, cb, rows = s["conv_w"], s["conv_b"], s["conv"]
        f, r, _ = _conv64(s["noised"][0], cw, cb, rows, slots)
        y = _block64(f, A, D, Dr, h, slots, (r, A, Dr))[0]
        f, r, kept = _conv64(s["clean"], cw, cb, rows, slots)
        yc, S = _block64(f, A, D, Dr, h, slots, (r, A, Dr))
        return (_norm64(y, s["z"], s["norm_w"]), y, yc, _to_pool(_stored(h, S, slots)),
                _stored(rows.double(), kept, slots))
    yc, S = _block64(s["clean"], A, D, Dr, h, slots)
    after = _stored(h, S, slots)
    y = _block64(s["noised"][-1], A, D, Dr, after if case["fused"] else h, slots)[0]
    return (y, _to_pool(after), yc) if case["outputs"] else (y, _to_pool(after))


def _rows_of(tok, k):
    return tuple(t[k:k + 1] for t in tok)
