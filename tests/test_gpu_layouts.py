"""The wide and the compact forward layouts and the decode kernel with K in
registers at sizes of several tiles: few heads take the paired layout, and few
sequences read K through LDS, so the shapes here have many (test_dispatch.py
pins the form of each).  And the paired layout on long rows.  Sampled rows
against the oracle, weights and P bit for bit at probe rows."""
import functools

import numpy as np
import pytest
import torch

import paper_2609_33586_amd as pkg
import test_gpu_decode as dec
from paper_2609_33586_amd import synth
from parity_helpers import (ALL_MODES, APPROX, BF16, EXACT, FP8, H15, TOL, assert_close, check_probe, dev_tensors,
                            oracle_run, say, scale_of)

pytestmark = pytest.mark.gpu


def sampled(inp, causal, mode, rows, what):
    B, Hq, S, d = inp.q.shape
    q, k, v = dev_tensors(inp)
    o = torch.full((B, Hq, S, d), float("nan"), dtype=torch.bfloat16, device="cuda:0")
    lse = torch.full((B, Hq, S), float("nan"), dtype=torch.float32, device="cuda:0")
    pkg.attn_fwd_ex(q, k, v, causal=causal, scale=scale_of(d), exp_mode=mode, descale=inp.descale, out=o, lse=lse)
    torch.cuda.synchronize()
    assert bool(torch.isfinite(o.float()).all()) and bool(torch.isfinite(lse).all())
    o_ref, lse_ref = oracle_run(inp, causal, scale_of(d), mode, rows=rows)
    assert_close(inp, o.view(-1, d).float().cpu().numpy().astype(np.float64)[rows],
                 lse.view(-1).cpu().numpy().astype(np.float64)[rows], o_ref, lse_ref, what, mode, causal=causal,
                 sc=scale_of(d), rows=rows)


# FP8 wide and BF16 compact (five tiles, ending at a tile's half and inside
# the second half; six), BF16 wide (17 tiles)
MANY = [(FP8, 72, 576, 128), (FP8, 72, 610, 128), (FP8, 72, 610, 64), (BF16, 72, 576, 128), (BF16, 72, 610, 128),
        (BF16, 72, 700, 64), (BF16, 64, 2060, 128), (BF16, 64, 2060, 64)]


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("dt,Hq,S,d", MANY)
def test_wide_and_compact_layouts(dt, Hq, S, d, causal):
    inp = synth.make_inputs(1, Hq, 2, S, d, dt, sharp=True, seed=3100 + S)
    rows = np.unique(np.concatenate([np.arange(0, Hq * S, 997), np.arange(Hq * S - 3, Hq * S)]))
    for mode in ALL_MODES:
        say(f"many heads dtype={dt} Hq={Hq} S={S} d={d} causal={causal} mode={mode}")
        sampled(inp, causal, mode, rows, "many heads")
        check_probe(inp, S, d, dt, causal, mode, scale_of(d), ((0, 1, S - 4, 4), (0, Hq - 1, 254, 4)))


@pytest.mark.parametrize("causal", [False, True])
def test_float_clamp_in_the_wide_layout(causal):
    # FP8 with unit descales: the exponent bound passes 2^15
    S, d = 610, 128
    rng = np.random.default_rng(3200)
    x = [rng.integers(-3, 4, (1, h, S, d)).astype(np.float32) for h in (72, 2, 2)]
    inp = synth.Inputs(*(synth.e4m3_codes(a) for a in x), (1.0, 1.0, 1.0), FP8)
    for mode in APPROX:
        check_probe(inp, S, d, FP8, causal, mode, scale_of(d), ((0, 0, S - 4, 4), (0, 71, 300, 4)))


# B * Hkv a multiple of 8: the XCD-grouped workgroup orders
GROUPED = [(FP8, 2, 48, 8, 700), (BF16, 2, 48, 8, 700), (BF16, 2, 32, 4, 2100)]


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("dt,B,Hq,Hkv,S", GROUPED)
def test_grouped_orders_of_the_wide_and_compact_layouts(dt, B, Hq, Hkv, S, causal):
    inp = synth.make_inputs(B, Hq, Hkv, S, 128, dt, sharp=True, seed=3300 + S)
    n = B * Hq * S
    rows = np.unique(np.concatenate([np.arange(0, n, S + 61), [S - 1, S, n - 1]]))
    sampled(inp, causal, H15, rows, "grouped order")


# 65 and 129 tiles, the last of them ragged
LONG = [(BF16, 3, 8200), (FP8, 3, 8200), (FP8, 1, 16400)]


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("dt,Hq,S", LONG)
def test_paired_layout_on_long_rows(dt, Hq, S, causal):
    inp = synth.make_inputs(1, Hq, 1, S, 128, dt, sharp=True, seed=3400 + S)
    n = Hq * S
    rows = np.unique(np.concatenate([np.arange(0, n, 1531), [S - 9, S - 8, n - 1]]))
    for mode in (EXACT, H15):
        say(f"paired long dtype={dt} Hq={Hq} S={S} causal={causal} mode={mode}")
        sampled(inp, causal, mode, rows, "paired long")
        check_probe(inp, S, 128, dt, causal, mode, scale_of(128), ((0, Hq - 1, S - 9, 3), (0, 0, S // 2, 2)))


# BF16 d = 128 with more than 256 workgroups of several rounds: eight tiles in
# one part, five and three in two; a full and a ragged block of rows
REGISTER_K = [(40, 16, 8, 3, 1000, 0), (40, 16, 8, 3, 1000, 640), (20, 64, 8, 5, 900, 0)]


@functools.lru_cache(maxsize=1)
def register_k_inputs(B, Hq, Hkv, Sq, Sk):
    return synth.make_decode_inputs(B, Hq, Hkv, Sq, Sk + 24, 128, BF16, sharp=True, seed=3500 + Sq)


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("B,Hq,Hkv,Sq,Sk,split", REGISTER_K)
def test_decode_with_k_in_registers(B, Hq, Hkv, Sq, Sk, split, causal):
    inp = register_k_inputs(B, Hq, Hkv, Sq, Sk)
    inp.k[:, :, Sk:] = 0x7FC0  # NaN beyond the cache's length
    inp.v[:, :, Sk:] = 0x7FC0
    q, k, v = dev_tensors(inp)
    n = B * Hq * Sq
    rows = np.unique(np.concatenate([np.arange(0, n, 37), [n - 1]]))
    vm = float(np.max(np.abs(synth.bf16_decode(inp.v[:, :, :Sk]))))
    for mode in ALL_MODES:
        say(f"decode K in registers B={B} Sq={Sq} Sk={Sk} split={split} causal={causal} mode={mode}")
        o = torch.full((B, Hq, Sq, 128), float("nan"), dtype=torch.bfloat16, device="cuda:0")
        pkg.attn_decode(q, k, v, Sk=Sk, causal=causal, scale=scale_of(128), exp_mode=mode, split_keys=split, out=o)
        torch.cuda.synchronize()
        assert bool(torch.isfinite(o.float()).all())
        o_ref, _ = dec.ref(inp, Sk, causal, scale_of(128), mode, split, rows=rows)
        err = np.abs(o.view(-1, 128).float().cpu().numpy().astype(np.float64)[rows] - np.asarray(o_ref).reshape(-1, 128))
        assert np.max(err) <= TOL[BF16] * vm
        dec.check_probe(inp, Sk, causal, scale_of(128), mode, split, ((0, 0, 0), (B - 1, Hq - 1, Sq - 1)))
