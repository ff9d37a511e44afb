"""Decode at the edges of its work split: a wave takes 64 keys a round and a
workgroup of four waves two 128-key tiles, or 32 keys and one tile in parts of
one and three tiles (BF16 at d = 128 also of two), row blocks are grouped eight
units (batch, KV head, part) at a time, the merge reads its parts 32 at a time,
and BF16 at d = 128 reads K through LDS up to 256 workgroups.  O within 2e-2
(BF16) or 6e-2 (FP8) max|V| of the oracle in every row; the exact control's
LSE to 1e-3; H15's weights and P bit for bit, and its LSE to the fp32
summation bound, against the oracle fed the GPU's logits (its LSE against the
oracle's own logits says nothing here: with few keys one weight beside a
rounding boundary moves it by up to half a weight's share)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2609_33586_amd as pkg
from paper_2609_33586_amd import synth
from parity_helpers import (ALL_MODES, APPROX, BF16, EXACT, FP8, H15, ORACLE_MODE, TOL, assert_close, dev_tensors,
                            say, scale_of, vmax)
from test_gpu_decode import check_probe

pytestmark = pytest.mark.gpu

CASES = [(1, 2, 2, 1, sk, 0) for sk in (63, 64, 65, 128, 191, 256, 257, 513)]  # units, tiles, rounds
CASES += [(1, 8, 1, 4, 385, 128), (1, 8, 1, 5, 300, 0)]  # one full row block; one of 32 rows and one of 8
CASES += [(3, 8, 1, 9, 700, 256), (2, 8, 4, 17, 260, 0)]  # 9 units of 3 row blocks (one unit beyond eight); 8 of 2
CASES += [(1, 4, 1, 1, 33 * 128, 128), (1, 4, 1, 2, 65 * 128 - 5, 128)]  # 33 and 65 parts
CASES += [(16, 4, 4, 1, 520, 128), (16, 4, 4, 1, 512, 128)]  # 320 and 256 workgroups


@pytest.mark.parametrize("dt,d", [(BF16, 128), (FP8, 128), (BF16, 64), (FP8, 64)])
@pytest.mark.parametrize("B,Hq,Hkv,Sq,Sk,split", CASES)
def test_decode_edges(B, Hq, Hkv, Sq, Sk, split, dt, d):
    inp = synth.make_decode_inputs(B, Hq, Hkv, Sq, Sk + 3, d, dt, sharp=True, seed=2100 + Sk + Sq)
    q, k, v = dev_tensors(inp)
    for mode in (EXACT, H15):
        say(f"decode edges B={B} Hq={Hq} Hkv={Hkv} Sq={Sq} Sk={Sk} split={split} dtype={dt} d={d} mode={mode}")
        o = torch.full((B, Hq, Sq, d), float("nan"), dtype=torch.bfloat16, device="cuda:0")
        lse = torch.full((B, Hq, Sq), float("nan"), dtype=torch.float32, device="cuda:0")
        pkg.attn_decode(q, k, v, Sk=Sk, causal=True, scale=scale_of(d), exp_mode=mode, split_keys=split,
                        descale=inp.descale, out=o, lse=lse)
        torch.cuda.synchronize()
        o_ref, lse_ref = oracle.decode(inp.q, inp.k, inp.v, Sk=Sk, dtype=dt, causal=True, scale=scale_of(d),
                                       mode=ORACLE_MODE[mode], split_keys=split, descale=inp.descale, Bc=128)
        o = o.float().cpu().numpy().astype(np.float64)
        if mode == EXACT:
            assert_close(inp, o, lse.cpu().numpy().astype(np.float64), o_ref, lse_ref, "decode edges", mode)
        else:
            assert np.max(np.abs(o - o_ref)) <= TOL[dt] * vmax(inp)
            assert bool(torch.isfinite(lse).all())
            check_probe(inp, Sk, True, scale_of(d), mode, split, ((0, 0, 0), (B - 1, Hq - 1, Sq - 1)))


# parts of one to four tiles (units of 32 keys: one tile, three tiles and, at
# BF16 d = 128, two), whole and ragged, one part and several
SHORT = [(70, 0), (128, 0), (200, 0), (256, 0), (330, 0), (384, 0), (512, 0), (1000, 128), (900, 256), (1100, 384)]


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("dt,d", [(BF16, 128), (FP8, 128), (BF16, 64), (FP8, 64)])
@pytest.mark.parametrize("Sk,split", SHORT)
def test_decode_short_parts(Sk, split, dt, d, causal):
    # 36 query rows of a KV head: a full block of rows and a ragged one, and
    # rows that see no key of the last part.  Every weight's bits at two rows.
    B, Hq, Hkv, Sq = 1, 24, 2, 3
    inp = synth.make_decode_inputs(B, Hq, Hkv, Sq, Sk + 2, d, dt, sharp=True, seed=2900 + Sk)
    q, k, v = dev_tensors(inp)
    for mode in ALL_MODES:
        say(f"decode short parts Sk={Sk} split={split} dtype={dt} d={d} causal={causal} mode={mode}")
        o = torch.full((B, Hq, Sq, d), float("nan"), dtype=torch.bfloat16, device="cuda:0")
        pkg.attn_decode(q, k, v, Sk=Sk, causal=causal, scale=scale_of(d), exp_mode=mode, split_keys=split,
                        descale=inp.descale, out=o)
        torch.cuda.synchronize()
        o_ref, _ = oracle.decode(inp.q, inp.k, inp.v, Sk=Sk, dtype=dt, causal=causal, scale=scale_of(d),
                                 mode=ORACLE_MODE[mode], split_keys=split, descale=inp.descale, Bc=128)
        assert np.max(np.abs(o.float().cpu().numpy().astype(np.float64) - o_ref)) <= TOL[dt] * vmax(inp)
        check_probe(inp, Sk, causal, scale_of(d), mode, split, ((0, 0, 0), (0, Hq - 1, Sq - 1)))


@pytest.mark.parametrize("Sk,split", [(128, 0), (256, 0), (300, 0), (700, 384)])
def test_decode_short_parts_float_clamp(Sk, split):
    # FP8 with unit descales: the exponent bound passes 2^15, so the weights
    # are clamped in FP32 (forms of their own at FP8)
    rng = np.random.default_rng(2950)
    x = [rng.integers(-3, 4, shape).astype(np.float32) for shape in ((1, 8, 2, 128), (1, 2, Sk, 128), (1, 2, Sk, 128))]
    inp = synth.Inputs(*(synth.e4m3_codes(a) for a in x), (1.0, 1.0, 1.0), FP8)
    for mode in APPROX:
        check_probe(inp, Sk, True, scale_of(128), mode, split, ((0, 0, 0), (0, 7, 1)))


@pytest.mark.parametrize("dt,d", [(BF16, 128), (FP8, 128), (BF16, 64), (FP8, 64)])
@pytest.mark.parametrize("Sk,split", [(100, 0), (128, 0), (256, 0), (384, 0), (512, 0), (1100, 0), (1000, 128),
                                      (1100, 384)])
def test_decode_nan_query_gives_nan(Sk, split, dt, d):
    # a query row that holds NaN has no score that compares: O is NaN in that row,
    # in every form and weight, and every other row keeps its bits
    inp = synth.make_decode_inputs(1, 8, 2, 3, Sk, d, dt, sharp=True, seed=2970 + Sk)
    bad = np.array(inp.q)
    bad[0, 5, 1] = 0x7FC0 if dt == BF16 else 0x7F
    q, k, v = dev_tensors(inp)
    qn = dev_tensors(synth.Inputs(bad, inp.k, inp.v, inp.descale, dt))[0]
    for mode in ALL_MODES:
        say(f"decode nan query Sk={Sk} split={split} dtype={dt} d={d} mode={mode}")
        kw = dict(causal=True, scale=scale_of(d), exp_mode=mode, split_keys=split, descale=inp.descale)
        o, lse = pkg.attn_decode(q, k, v, **kw)
        on, ln = pkg.attn_decode(qn, k, v, **kw)
        torch.cuda.synchronize()
        assert bool(torch.isnan(on[0, 5, 1].float()).all()) and not bool(torch.isfinite(ln[0, 5, 1]))
        on[0, 5, 1], ln[0, 5, 1] = o[0, 5, 1], lse[0, 5, 1]
        assert torch.equal(on.view(torch.int16), o.view(torch.int16)) and torch.equal(ln, lse)
