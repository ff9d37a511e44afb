"""Which kernel form a call takes, by size, type and cut: the host side of the
library (csrc/attn_api.cpp) built with a host compiler alone and linked with
launchers that launch nothing and report the form they were asked for
(tests/sanitize_launch_stub.cpp).  The GPU tests check results, which are the
same in every form; here each rule is pinned on both sides of its lines, and
the GPU tests' own shapes at the forms they are meant for."""
import ctypes
import subprocess
from pathlib import Path

import pytest

import paper_2609_33586_amd as pkg

ROOT = Path(__file__).resolve().parent.parent
CSRC = ROOT / "paper_2609_33586_amd" / "csrc"
BF16, FP8 = pkg.ATTN_BF16, pkg.ATTN_FP8_E4M3
DTD = [(BF16, 128), (FP8, 128), (BF16, 64), (FP8, 64)]
ADDRESS = 0x100000  # 16-byte aligned, never dereferenced


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    lib = tmp_path_factory.mktemp("dispatch") / "libh15attn_host.so"
    subprocess.run(["g++", "-std=c++17", "-O1", "-fPIC", "-shared", "-ffp-contract=off", f"-I{ROOT / 'include'}",
                    f"-I{CSRC}", str(CSRC / "attn_api.cpp"), str(ROOT / "tests" / "sanitize_launch_stub.cpp"), "-o",
                    str(lib)], check=True)
    L = ctypes.CDLL(str(lib))
    P, I, F, O = ctypes.c_void_p, ctypes.c_int, ctypes.c_float, ctypes.POINTER(pkg.attn_opts)
    L.attn_fwd_ex.argtypes = [P] * 5 + [I] * 6 + [F, I, I, O]
    L.attn_decode.argtypes = [P] * 5 + [I] * 8 + [F, I, I, I, P, ctypes.c_size_t, O]
    return L


def opts(tau=0.0):
    return ctypes.byref(pkg.attn_opts(1.0, 1.0, 1.0, None, tau, 0))


def layout(L, dt, d, heads, S, causal, mode=pkg.ATTN_EXP_H15, tau=0.0):
    a = ADDRESS
    rc = L.attn_fwd_ex(a, a, a, a, None, 1, heads, heads, S, d, int(causal), 0.1, dt, mode, opts(tau))
    assert rc == pkg.ATTN_ELAUNCH
    return ("wide", "compact", "paired")[L.h15_stub_layout()]


def decode_form(L, dt, d, B=1, Hq=8, Hkv=2, Sq=1, Sk=1000, split=0, mode=1):
    """(keys of a wave and round, K through LDS) of a decode call."""
    a = ADDRESS
    rc = L.attn_decode(a, a, a, a, None, B, Hq, Hkv, Sq, Sk, Sk, d, 1, 0.1, dt, mode, split, a, 1 << 40, opts())
    assert rc == pkg.ATTN_ELAUNCH
    return L.h15_stub_unit(), L.h15_stub_k_lds()


@pytest.mark.parametrize("dt,d", DTD)
def test_decode_units_by_tiles_of_a_part(host, dt, d):
    # a round of units of 64 keys covers two tiles: parts of one and of three
    # tiles would leave waves without keys
    for sk, split, tiles in ((1, 0, 1), (100, 0, 1), (128, 0, 1), (129, 0, 2), (256, 0, 2), (257, 0, 3), (384, 0, 3),
                             (385, 0, 4), (512, 0, 4), (640, 0, 5), (4096, 128, 1), (4100, 256, 2), (4100, 384, 3),
                             (4096, 512, 4), (300, 384, 3), (300, 1024, 3)):
        want = 32 if tiles in (1, 3) or (tiles == 2 and (dt, d) == (BF16, 128)) else 64
        for B in (1, 200):
            unit, k_lds = decode_form(host, dt, d, B=B, Sk=sk, split=split)
            assert unit == want, (sk, split, B)
            assert k_lds == (0 if unit == 64 and (dt, d) == (BF16, 128) and B * 2 * host.h15_stub_parts() > 256 else 1)


@pytest.mark.parametrize("dt,d", DTD)
def test_decode_k_path_by_workgroups(host, dt, d):
    # BF16 d = 128 reads K into registers from more workgroups than compute units on
    for B, Hkv, Hq, Sq, sk, split, groups in ((128, 2, 8, 1, 1000, 0, 256), (257, 1, 4, 1, 1000, 0, 257),
                                              (16, 4, 4, 1, 4096, 1024, 256), (16, 4, 4, 1, 4097, 1024, 320),
                                              (33, 2, 16, 9, 1000, 0, 198), (43, 2, 16, 9, 1000, 0, 258)):
        nrb = -(-Hq // Hkv * Sq // 32)
        assert B * Hkv * nrb * max(1, -(-sk // split) if split else 1) == groups
        want = 0 if groups > 256 and (dt, d) == (BF16, 128) else 1
        assert decode_form(host, dt, d, B=B, Hq=Hq, Hkv=Hkv, Sq=Sq, Sk=sk, split=split) == (64, want), (B, groups)


EXACT, H15, SQ8, POT = pkg.ATTN_EXP_EXACT, pkg.ATTN_EXP_H15, pkg.ATTN_EXP_SQ8, pkg.ATTN_EXP_ROWMAX_POT


def other(dt, S, heads):
    """The layout of a call that is not paired."""
    return "wide" if dt == FP8 or (S > 2048 and heads * -(-S // 256) >= 512) else "compact"


@pytest.mark.parametrize("dt,d", DTD)
def test_paired_from_some_tiles_on(host, dt, d):
    # up to 256 blocks of 128 rows: causal from four tiles, else from five
    for mode in (EXACT, H15, SQ8):
        for S, causal, paired in ((128, True, False), (384, True, False), (481, True, True), (512, True, True),
                                  (1024, True, True), (512, False, False), (513, False, True), (1024, False, True)):
            want = "paired" if paired else other(dt, S, 4)
            assert layout(host, dt, d, 4, S, causal, mode) == want, (S, causal, mode)
    assert layout(host, dt, d, 4, 512, True, H15, tau=8.0 if dt == BF16 else 0.0) == "paired"


def test_paired_ragged_last_block(host):
    # BF16 d = 128, causal: a last block of 96 rows or fewer needs more tiles
    for mode, tiles in ((EXACT, 5), (H15, 7), (SQ8, 7)):
        for t in range(4, 10):
            for r in (1, 64, 96):
                want = "paired" if t >= tiles else "compact"
                assert layout(host, BF16, 128, 4, (t - 1) * 128 + r, True, mode) == want, (mode, t, r)
            for r in (97, 127, 128):
                assert layout(host, BF16, 128, 4, (t - 1) * 128 + r, True, mode) == "paired", (mode, t, r)
        for dt, d in ((FP8, 128), (BF16, 64), (FP8, 64)):
            assert layout(host, dt, d, 4, 385, True, mode) == "paired"
    # all keys visible: the exact control at five tiles, more than 240 blocks
    assert layout(host, BF16, 128, 48, 600, False, EXACT) == "paired"
    assert layout(host, BF16, 128, 49, 600, False, EXACT) == "compact"
    assert layout(host, BF16, 128, 49, 600, False, H15) == "paired"
    assert layout(host, BF16, 128, 41, 700, False, EXACT) == "paired"


@pytest.mark.parametrize("dt,d", DTD)
def test_layouts_by_blocks(host, dt, d):
    # blocks of 128 rows: 256 and 257 (and one row more), the second line for
    # long causal rows, and the compact layout's own lines
    for heads, S, causal, paired in ((64, 512, True, True), (65, 512, True, False), (32, 1024, False, True),
                                     (33, 1024, False, False), (44, 1024, True, True), (45, 1024, True, False),
                                     (32, 2048, True, True), (33, 2048, True, False), (32, 2047, True, False),
                                     (8, 8192, True, True), (9, 8192, True, False), (16, 4096, True, True),
                                     (16, 4096, False, False), (1, 32768, False, True), (1, 32769, False, False)):
        want = "paired" if paired else other(dt, S, heads)
        assert layout(host, dt, d, heads, S, causal) == want, (heads, S, causal)
    assert layout(host, dt, d, 64, 2048, True) == ("compact" if dt == BF16 else "wide")
    assert layout(host, dt, d, 64, 2049, True) == "wide"
    assert layout(host, dt, d, 31, 4096, True) == ("compact" if dt == BF16 else "wide")
    assert layout(host, dt, d, 32, 4096, True) == "wide"
    if dt == BF16:
        for heads, S in ((1, 40), (4, 1024), (64, 4096)):
            assert layout(host, dt, d, heads, S, True, POT) == "wide"


def test_paired_test_shapes_are_paired(host):
    # the shapes of test_gpu_paired.py, but for the ones it names
    from test_gpu_paired import FULL
    for dt, d in DTD:
        for S, causal in FULL:
            for mode in (EXACT, H15, SQ8):
                small = (dt, d) == (BF16, 128) and (S == 385 or (S == 641 and mode != EXACT))
                assert layout(host, dt, d, 2, S, causal, mode) == ("compact" if small else "paired"), (dt, d, S, mode)
        for S in (520, 700, 900):
            for causal in (True, False):
                small = (dt, d) == (BF16, 128) and causal and S < 900
                assert layout(host, dt, d, 2, S, causal) == ("compact" if small else "paired")
                assert layout(host, dt, d, 64, S, causal) == other(dt, S, 64)
        assert layout(host, dt, d, 4, 900, True) == layout(host, dt, d, 4, 900, False) == "paired"


def test_many_head_test_shapes(host):
    # the shapes of test_gpu_layouts.py, test_gpu_tau.py and the write guards
    import test_gpu_layouts as gl
    import test_gpu_parity as gp
    import test_gpu_tau as gt
    for dt, hq, S, d in gl.MANY:
        for causal in (True, False):
            for mode in (EXACT, H15, SQ8):
                want = "wide" if dt == FP8 or S == 2060 else "compact"
                assert layout(host, dt, d, hq, S, causal, mode) == want, (dt, hq, S, d)
    for dt, B, hq, hkv, S in gl.GROUPED:
        assert B * hkv % 8 == 0
        want = "wide" if dt == FP8 or S == 2100 else "compact"
        assert layout(host, dt, 128, B * hq, S, True) == layout(host, dt, 128, B * hq, S, False) == want
    for dt, hq, S in gl.LONG:
        for mode in (EXACT, H15):
            assert layout(host, dt, 128, hq, S, True, mode) == layout(host, dt, 128, hq, S, False, mode) == "paired"
    for (hq, S, d), want in zip(gt.LAYOUTS, ("compact", "compact", "wide", "paired")):
        for causal in (True, False):
            assert layout(host, BF16, d, hq, S, causal, H15, tau=8.0) == want, (hq, S, d)
    for dt, B, hq, hkv, S, d in gp.GUARD_SHAPES[-4:]:
        for mode in (EXACT, H15):
            assert layout(host, dt, d, B * hq, S, True, mode) == layout(host, dt, d, B * hq, S, False, mode) == "paired"
    for B, hq, hkv, sq, sk, split in gl.REGISTER_K:
        assert decode_form(host, BF16, 128, B=B, Hq=hq, Hkv=hkv, Sq=sq, Sk=sk, split=split) == (64, 0)
