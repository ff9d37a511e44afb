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
    L.attn_decode.argtypes = [P] * 5 + [I] * 8 + [F, I, I, I, P, ctypes.c_size_t, O]
    return L


def opts(tau=0.0):
    return ctypes.byref(pkg.attn_opts(1.0, 1.0, 1.0, None, tau, 0))


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
