"""The paired forward layout (grids that leave compute units idle: two waves a
row, even and odd key tiles) at the edges of its range: four to nine key
tiles, ragged last tiles and row blocks, every weight, the conditional
rescale, and the borders of the rule that picks it.  Full outputs against the
oracle with the bars of test_gpu_parity.py, weights and P bit for bit at probe
rows, and the same heads in a batch large enough for the other layouts: equal
probe weights, O within a quarter of the bar."""
import numpy as np
import pytest
import torch

import oracle
import paper_2609_33586_amd as pkg
from paper_2609_33586_amd import synth
from parity_helpers import (ALL_MODES, BF16, EXACT, FP8, H15, ORACLE_MODE, TOL, assert_close,
                            dev_tensors, say, scale_of, vmax)

pytestmark = pytest.mark.gpu


def close(inp, o, lse, o_ref, lse_ref, mode, causal, d):
    assert_close(inp, o.float().cpu().numpy().astype(np.float64), lse.cpu().numpy().astype(np.float64), o_ref, lse_ref,
                 "paired", mode, causal=causal, sc=scale_of(d))


# (at BF16 d = 128 the causal calls of 385 rows, and of 641 with a lattice
# weight, take the compact layout: their last blocks have one row)
FULL = [(385, True), (490, True), (512, True), (513, False), (640, False), (641, True), (777, True), (895, False),
        (1025, True)]


@pytest.mark.parametrize("dt,d", [(BF16, 128), (FP8, 128), (BF16, 64), (FP8, 64)])
@pytest.mark.parametrize("S,causal", FULL)
def test_paired_full_parity(S, causal, dt, d):
    inp = synth.make_inputs(1, 2, 1, S, d, dt, sharp=True, seed=2300 + S)
    q, k, v = dev_tensors(inp)
    for mode in ALL_MODES if S in (385, 490) else (EXACT, H15):
        say(f"paired S={S} causal={causal} dtype={dt} d={d} mode={mode}")
        o = torch.full((1, 2, S, d), float("nan"), dtype=torch.bfloat16, device="cuda:0")
        lse = torch.full((1, 2, S), float("nan"), dtype=torch.float32, device="cuda:0")
        pkg.attn_fwd_ex(q, k, v, causal=causal, scale=scale_of(d), exp_mode=mode, descale=inp.descale, out=o, lse=lse)
        torch.cuda.synchronize()
        o_ref, lse_ref = oracle.attn(inp.q, inp.k, inp.v, dtype=dt, causal=causal, scale=scale_of(d),
                                     mode=ORACLE_MODE[mode], descale=inp.descale, Bc=pkg.attn_tile_bc())
        close(inp, o, lse, o_ref, lse_ref, mode, causal, d)


@pytest.mark.parametrize("dt,d", [(BF16, 128), (FP8, 128), (BF16, 64), (FP8, 64)])
@pytest.mark.parametrize("S", [520, 700, 900])
def test_paired_equals_the_other_layouts(S, dt, d):
    # two heads alone take the paired layout; the same two heads at the front
    # of 64 (more than 256 blocks of 128 rows) take the wide or the compact one
    inp = synth.make_inputs(1, 64, 64, S, d, dt, sharp=True, seed=2400 + S)
    q, k, v = dev_tensors(inp)
    few = [x[:, :2].contiguous() for x in (q, k, v)]
    sc = scale_of(d)
    for causal in (True, False):
        for mode in (EXACT, H15):
            say(f"paired against wide S={S} causal={causal} dtype={dt} d={d} mode={mode}")
            kw = dict(causal=causal, scale=sc, exp_mode=mode, descale=inp.descale)
            o1, l1 = pkg.attn_fwd_ex(*few, **kw)
            o2, l2 = pkg.attn_fwd_ex(q, k, v, **kw)
            assert float((o1.float() - o2[:, :2].float()).abs().max()) <= TOL[dt] * vmax(inp) / 4
            assert float((l1 - l2[:, :2]).abs().max()) <= 1e-5
            a = pkg.attn_fwd_probe(*few, b=0, h=1, row0=S - 40, nrows=40, **kw)
            b = pkg.attn_fwd_probe(q, k, v, b=0, h=1, row0=S - 40, nrows=40, **kw)
            torch.cuda.synchronize()
            assert all(torch.equal(x, y) for x, y in zip(a[2:], b[2:]))
            assert torch.equal(a[0].view(torch.int16), o1.view(torch.int16)) and torch.equal(a[1], l1)


@pytest.mark.parametrize("per_wave", [False, True])
@pytest.mark.parametrize("causal", [False, True])
def test_paired_conditional_rescale(causal, per_wave):
    S, d = 900, 128
    rng = np.random.default_rng(2500)
    q, k, v = (rng.standard_normal((1, h, S, d)).astype(np.float32) for h in (4, 2, 2))
    k *= (0.3 + 2.5 * np.arange(S, dtype=np.float32) / S)[None, None, :, None]  # the maximum keeps rising
    inp = synth.Inputs(synth.bf16_bits(q), synth.bf16_bits(k), synth.bf16_bits(v), (1.0, 1.0, 1.0), BF16)
    for mode in (EXACT, H15):
        say(f"paired tau causal={causal} per_wave={per_wave} mode={mode}")
        o, lse = pkg.attn_fwd_ex(*dev_tensors(inp), causal=causal, scale=scale_of(d), exp_mode=mode, tau=8.0,
                                 tau_per_wave=per_wave)
        torch.cuda.synchronize()
        o_ref, lse_ref = oracle.attn(inp.q, inp.k, inp.v, dtype=BF16, causal=causal, scale=scale_of(d),
                                     mode=ORACLE_MODE[mode], Bc=pkg.attn_tile_bc(), tau=8.0,
                                     tau_group=32 if per_wave else 1)
        assert_close(inp, o.float().cpu().numpy().astype(np.float64), lse.cpu().numpy().astype(np.float64), o_ref,
                     lse_ref, "paired tau", mode, flat_lse=True)


@pytest.mark.parametrize("Hq,Hkv,S,causal", [(64, 8, 512, True), (65, 5, 512, True), (32, 8, 2048, True),
                                             (51, 3, 600, False), (52, 4, 600, False), (44, 4, 1024, True),
                                             (45, 9, 1024, True)])
def test_paired_rule_borders(Hq, Hkv, S, causal):
    # 256 and 260 blocks, 512 blocks of 2048 rows, 255 and 260 with every key
    # visible, 352 and 360 blocks of 1024 rows
    for dt in (BF16, FP8):
        inp = synth.make_inputs(1, Hq, Hkv, S, 128, dt, sharp=True, seed=2600 + Hq)
        say(f"paired borders Hq={Hq} S={S} causal={causal} dtype={dt}")
        o, lse = pkg.attn_fwd_ex(*dev_tensors(inp), causal=causal, scale=scale_of(128), exp_mode=H15,
                                 descale=inp.descale)
        torch.cuda.synchronize()
        rows = np.unique(np.concatenate([np.arange(0, Hq * S, 509), np.arange(Hq * S - 130, Hq * S)]))
        o_ref, lse_ref = oracle.attn(inp.q, inp.k, inp.v, dtype=dt, causal=causal, scale=scale_of(128),
                                     mode=ORACLE_MODE[H15], descale=inp.descale, Bc=pkg.attn_tile_bc(), rows=rows)
        assert_close(inp, o.float().cpu().numpy().astype(np.float64).reshape(-1, 128)[rows],
                     lse.cpu().numpy().astype(np.float64).reshape(-1)[rows], o_ref, lse_ref, "borders", H15,
                     causal=causal, sc=scale_of(128), rows=rows)
