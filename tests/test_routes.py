"""The dispatch rules of libbdlm, asked of the built library on the CPU: a call is sent to a
kernel only where that kernel can address every byte of it.

The rules are C++ functions of the library; a shim compiled here against its internal header
fills their argument structure.
"""
import ctypes
import os
import random
import subprocess

import pytest

import paper_2607_02805_amd as bd

SHIM = r"""
#include "bdlm_launch.h"
#include "bdlm_seq.h"
using namespace bdlm;
static LaunchArgs args(const int64_t *v) {
    LaunchArgs a = {};
    a.batch = v[0]; a.nheads = v[1]; a.ngroups = v[2]; a.L = v[3]; a.dstate = v[4]; a.bf16 = v[5];
    a.xs_t = v[6]; a.dts_t = v[7]; a.bcs_t = v[8];
    return a;
}
extern "C" int masked(const int64_t *v) { return long_masked_fits(args(v)); }
extern "C" int windows(const int64_t *v) { return masked_windows_fit(args(v)); }
extern "C" int mix(const int64_t *v) { return mix_fits(args(v)); }
// (L: tokens per block, 0 for a prefill; xs_t: tokens in all; the last value: outputs wanted)
extern "C" int one_seg(const int64_t *v) {
    LaunchArgs a = args(v);
    float y;
    a.y = v[9] ? &y : nullptr;
    return one_segment(a, v[6], v[3]);
}
extern "C" int sep(const int64_t *v) { return sep_windows_fit(args(v)); }
extern "C" int two(const int64_t *v) { return seq_two_passes(args(v), v[3]); }
extern "C" int pairs(const int64_t *v) {   // v[3]: segments
    SeqArgs k = {};
    k.heads_per_group = v[1] / v[2];
    k.nseg = v[3];
    return seq16_forward(v[4], k, v[0] * v[1] * v[3]);
}
extern "C" int pays(const int64_t *v) { return mix_pays(args(v), v[9]); }   // (v[9]: a commit)
extern "C" int in_one(const int64_t *v) { return prefill_in_one(args(v), v[3]); }
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    bd.lib()
    d = tmp_path_factory.mktemp("routes")
    src, so = d / "shim.cpp", d / "shim.so"
    src.write_text(SHIM)
    csrc = os.path.join(os.path.dirname(bd.LIB_PATH), "csrc")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__",
                    "-isystem", "/opt/rocm/include", f"-I{csrc}",
                    f"-I{os.path.dirname(bd.HEADER_PATH)}", str(src), "-o", str(so),
                    f"-L{os.path.dirname(bd.LIB_PATH)}", "-l:libbdlm.so",
                    f"-Wl,-rpath,{os.path.dirname(bd.LIB_PATH)}"], check=True)
    lib = ctypes.CDLL(str(so))

    def ask(rule, batch, H, G, L, N, bf16, xs_t=None, dts_t=None, bcs_t=None, last=0):
        v = (ctypes.c_int64 * 10)(batch, H, G, L, N, bf16, xs_t or H * 64, dts_t or H, bcs_t or G * N, last)
        return bool(getattr(lib, rule)(v))
    return ask


RANGE = 0x7fffffff          # bytes of the buffer resources that the block kernels load through


def last_byte(H, L, N, es, xs_t, dts_t, bcs_t):
    """The furthest byte of a block that a workgroup addresses from its (row, head)'s base."""
    return max((L - 1) * xs_t * es + 64 * es, (L - 1) * bcs_t * es + N * es, (L - 1) * dts_t * es + es,
               (L - 1) * H * 256 + 256)


@pytest.mark.parametrize("L", [65, 96, 128, 129, 200, 256])
@pytest.mark.parametrize("N", [16, 32, 64, 128])
def test_masked_kernels_take_only_what_they_address(rules, L, N):
    """Token strides up to 16 MiB are accepted; 256 of them span 4 GiB."""
    r = random.Random(100 * L + N)
    for _ in range(400):
        st = [8 * r.randint(128, 1 << 20) for _ in range(3)]
        if r.random() < 0.5:                              # about the limit
            k = r.randrange(3)
            st[k] = 8 * (((1 << 31) // (2 * L) + r.randint(-64, 64)) // 8)
        H = r.choice([1, 4, 26, 300, 8192, 33000, 65536])
        last = last_byte(H, L, N, 2, *st)
        took = rules("masked", 1, H, 1, L, N, 1, *st)
        assert took == (last <= RANGE)
        assert not rules("windows", 1, H, 1, L, N, 1, *st) or took


@pytest.mark.parametrize("L", [65, 128, 256])
def test_masked_kernels_keep_the_strides_of_a_projection(rules, L):
    for H, G, N in ((1, 1, 16), (32, 1, 128), (26, 2, 64), (128, 8, 128)):
        row = 2 * H * 64 + 2 * G * N + H
        assert rules("masked", 16, H, G, L, N, 1, row, row, row)


def test_convolution_blocks_launch_within_32_bits(rules):
    """The Gram kernel's grid counts (row, group)s, up to 20 blocks of 512 threads each; a
    launch holds fewer than 2^32 threads (the convolution and scan kernels take the rest)."""
    r = random.Random(7)
    took = 0
    for _ in range(4000):
        G = r.choice([1, 8, 64])
        batch = 1 << r.randint(0, 22) if r.random() < 0.5 else r.randint(1, 1 << 22)
        hpg = r.randint(1, 8)
        L = r.choice([33, 64, 65, 128, 129, 192, 193, 256])
        if batch * G * hpg > 1 << 22:
            continue
        if rules("mix", batch, G * hpg, G, L, r.choice([16, 128]), r.choice([0, 1])):
            nb = (L + 63) // 64
            took += 1
            assert batch * G * nb * (nb + 1) * 512 < 1 << 32, (batch, G, hpg, L)
    assert took > 500
    assert rules("mix", 10922, 192, 64, 129, 16, 1)
    assert not rules("mix", 10923, 192, 64, 129, 16, 1)      # 699,072 (row, group)s of 12 blocks


@pytest.mark.parametrize("units", [64, 96, 128, 160, 200, 224, 256, 300, 320, 384, 448, 512, 576, 640, 768, 1024, 2048])
def test_one_segment_fills_the_chip(rules, units):
    """fp32 at dstate 128 one workgroup fills a CU: pairs whose rounds leave more than a quarter
    of the chip idle (two fifths without outputs) run in several segments."""
    rounds = -(-units // 256) * 256
    for L in (0, 32, 48, 64):
        assert rules("one_seg", units, 1, 1, L, 128, 0, xs_t=4096, last=1) == (2 * units >= 256 and rounds <= 1.33 * units)
        if L:
            assert rules("one_seg", units, 1, 1, L, 128, 0) == (2 * units >= 256 and rounds <= 1.67 * units)
    if units < 231:                                      # 0.45 of two workgroups per CU
        assert not any(rules("one_seg", units, 1, 1, L, N, bf, last=y)
                       for L in (0, 20, 48, 64) for N in (16, 64) for bf in (0, 1) for y in (0, 1))


def test_one_segment_of_short_blocks(rules):
    """Blocks that fill little of a chunk, with outputs (16 and 32 tokens share chunks), and
    small states on a third of the chip."""
    for N, bf in ((16, 1), (32, 0)):
        assert not rules("one_seg", 256, 1, 1, 48, N, bf, last=1)
        for L in (16, 32, 64):
            assert rules("one_seg", 256, 1, 1, L, N, bf, last=1)
        assert rules("one_seg", 256, 1, 1, 48, N, bf) and rules("one_seg", 640, 1, 1, 48, N, bf, last=1)
        assert rules("one_seg", 256, 1, 1, 0, N, bf, xs_t=1024, last=1)
        assert not rules("one_seg", 256, 1, 1, 0, N, bf, xs_t=1025, last=1)
        assert rules("one_seg", 512, 1, 1, 0, N, bf, xs_t=1025, last=1)
    assert rules("one_seg", 256, 1, 1, 48, 64, 1, last=1)
    assert not rules("one_seg", 832, 1, 1, 12, 16, 1, last=1)
    assert rules("one_seg", 832, 1, 1, 12, 16, 1) and rules("one_seg", 1024, 1, 1, 12, 16, 1, last=1)


# (dstate, bf16) -> [(row-heads, tokens up to which a prefill without outputs is one launch)]
IN_ONE = {(128, 0): [(64, 128), (256, 256), (512, 256), (1024, 128), (4096, 128)], (64, 0): [(64, 256), (4096, 256)],
          (32, 0): [(64, 320), (4096, 320)], (16, 0): [(64, 256), (4096, 256)], (128, 1): [(64, 640), (4096, 640)],
          (64, 1): [(2048, 384)], (32, 1): [(2048, 384)], (16, 1): [(1024, 256), (2048, 128)]}


@pytest.mark.parametrize("N,bf16", IN_ONE)
def test_prefill_without_outputs(rules, N, bf16):
    """Longer prompts run as the states pass and the combination, as they did before."""
    for units, most in IN_ONE[N, bf16]:
        assert rules("in_one", units, 1, 1, most, N, bf16) and not rules("in_one", units, 1, 1, most + 1, N, bf16)
    quads = 64 * N // 4                                  # threads of the combination per row-head
    for units in (((1 << 32) - 1) // quads, (1 << 32) // quads):
        assert rules("in_one", units, 1, 1, 2000, N, bf16) == (units * quads >= 1 << 32)


@pytest.mark.parametrize("N", [16, 32, 64, 128])
def test_separate_reverse_inputs(rules, N):
    """Beyond 128 tokens the windows pay for 256: three quarters of them at least, and fewer
    row-heads the smaller the state."""
    for units in (1, 32, 256, 257, 512, 513, 768, 769, 1024, 2047, 2048, 4096):
        took = {L: rules("sep", 1, units, 1, L, N, 1) for L in (65, 128, 129, 192, 193, 256, 257)}
        assert took[65] and took[128] and not took[257]
        assert took[129] == took[192] == (N >= 32 and units <= 256)
        few = units <= {16: 512, 32: 512, 64: 768, 128: 256}[N]
        assert took[193] == took[256] == (few or (32 <= N <= 64 and units >= 2048))
        assert not rules("sep", 1, units, 1, 256, N, 0)                        # fp32
        assert not rules("sep", 1, units, 1, 256, N, 1, xs_t=8 << 20)          # past 2 GiB


@pytest.mark.parametrize("N", [16, 32, 64, 128])
def test_both_branches_of_large_calls(rules, N):
    """Small states and activations beyond the caches: a forward and a reverse pass."""
    for units in (1, 96, 512, 4096):
        T = -(-(3 << 18) // units)
        assert rules("two", units, 1, 1, T, N, 1) == (N <= 32)
        assert not rules("two", units, 1, 1, T - 1, N, 1)


@pytest.mark.parametrize("N", [16, 32, 64, 128])
def test_forward_outputs_in_pairs_of_heads(rules, N):
    """Small states: only where pairs take one round and single heads two."""
    for rows, segs in ((23, 1), (24, 1), (25, 1), (32, 1), (33, 1), (64, 1), (28, 1), (14, 2), (7, 8)):
        grid = 32 * rows * segs
        took = rules("pairs", rows, 32, 1, segs, N, 1)
        assert took == (grid >= 768 and (N >= 64 or (segs == 1 and 768 < grid <= 1024)))
        assert not rules("pairs", rows, 32, 32, segs, N, 1)      # one head per group


@pytest.mark.parametrize("N", [16, 32, 64, 128])
def test_short_convolution_blocks(rules, N):
    """The Gram and head kernels work on 64 tokens: many row-heads of a few fp32 tokens, and at
    dstate 128 steps of any number, stay with the convolution and block kernels."""
    for units in (1, 16, 128, 129, 1023, 1024, 2047, 2048, 4096):
        def pays(commit, L):
            return rules("pays", units, 1, 1, L, N, 0, last=commit)
        for L in (33, 64, 65, 256):
            assert pays(0, L) and pays(1, L)
        for L in (1, 8, 16):                             # rows are a grid dimension there
            assert rules("pays", 65536, units, 1, L, N, 0) and rules("pays", 65536, units, 1, L, N, 0, last=1)
        for L in (1, 4, 5, 8, 9, 12, 13, 16, 17, 32):
            assert pays(1, L) == (L > 4 or units < 1024)
            if N == 128:
                assert pays(0, L) == (units > 128 if L > 16 else L > 8 and units >= 2048)
            else:
                assert pays(0, L) == (units < 1024 or L > (12 if N == 16 and units >= 2048 else 8))
