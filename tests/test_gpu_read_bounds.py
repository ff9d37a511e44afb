"""Copies of ragged tiles and of tiles beyond the last read nothing outside
the operands: Q, K and V (or the cache) as views into larger buffers filled
with NaN on both sides give the same bits as in buffers of their own, in every
forward layout and in decode with one part and with several.  (A V row read
from outside would meet a weight of zero and turn its whole row of O into
NaN.)"""
import pytest
import torch

import paper_2609_33586_amd as pkg
from paper_2609_33586_amd import synth
from parity_helpers import BF16, EXACT, FP8, H15, dev_tensors, say, scale_of

pytestmark = pytest.mark.gpu

GUARD = 1 << 20  # bytes on either side


def guarded(t):
    raw = t.contiguous().view(torch.uint8).reshape(-1)
    nan = torch.full((2 * GUARD + raw.numel(),), 0x7F if t.element_size() == 1 else 0xFF, dtype=torch.uint8,
                     device=t.device)
    nan[GUARD:GUARD + raw.numel()] = raw
    return nan[GUARD:GUARD + raw.numel()].view(t.dtype).view(t.shape)


def same(a, b):
    torch.cuda.synchronize()
    assert torch.equal(a[0].view(torch.int16), b[0].view(torch.int16)) and torch.equal(a[1], b[1])


# (heads, S): paired with an odd and an even number of tiles, one tile, the
# wide and the compact layout with ragged tails
@pytest.mark.parametrize("dt,d", [(BF16, 128), (FP8, 128), (BF16, 64), (FP8, 64)])
@pytest.mark.parametrize("Hq,S", [(2, 777), (2, 1025), (2, 40), (2, 300), (72, 520), (64, 2060)])
def test_forward_reads_stay_inside_operands(Hq, S, dt, d):
    inp = synth.make_inputs(1, Hq, 2, S, d, dt, sharp=False, seed=2700 + S)
    q, k, v = dev_tensors(inp)
    for causal in (True, False):
        for mode in (EXACT, H15) + ((pkg.ATTN_EXP_ROWMAX_POT,) if dt == BF16 else ()):
            say(f"read bounds forward Hq={Hq} S={S} dtype={dt} d={d} causal={causal} mode={mode}")
            kw = dict(causal=causal, scale=scale_of(d), exp_mode=mode, descale=inp.descale)
            same(pkg.attn_fwd_ex(guarded(q), guarded(k), guarded(v), **kw), pkg.attn_fwd_ex(q, k, v, **kw))


@pytest.mark.parametrize("dt,d", [(BF16, 128), (FP8, 128), (BF16, 64), (FP8, 64)])
@pytest.mark.parametrize("B,Hkv,Sk,cap,split", [(1, 2, 1000, 1000, 0), (1, 2, 1000, 1024, 384), (1, 2, 9, 9, 0),
                                                (1, 2, 203, 203, 128), (20, 4, 650, 650, 128)])
def test_decode_reads_stay_inside_the_cache(B, Hkv, Sk, cap, split, dt, d):
    inp = synth.make_decode_inputs(B, 8, Hkv, 2, cap, d, dt, sharp=False, seed=2800 + Sk)
    q, k, v = dev_tensors(inp)
    for mode in (EXACT, H15):
        say(f"read bounds decode B={B} Sk={Sk} cap={cap} split={split} dtype={dt} d={d} mode={mode}")
        kw = dict(causal=True, scale=scale_of(d), exp_mode=mode, descale=inp.descale, Sk=Sk, split_keys=split)
        clean = pkg.attn_decode(q, k, v, **kw)
        k2, v2 = guarded(k), guarded(v)
        for x in (k2, v2):  # the cache's rows beyond Sk
            x.view(torch.uint8)[:, :, Sk:] = 0x7F if dt == FP8 else 0xFF
        same(pkg.attn_decode(guarded(q), k2, v2, **kw), clean)
