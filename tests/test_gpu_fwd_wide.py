"""GPU parity of the forward kernel with 64 query rows per wavefront (block 128 / d 128, more than 256 query
blocks, where nothing else is chosen), where it can go wrong: list lengths around its software pipeline, the
ragged last tile, lists that do not ascend, references that have to be moved."""

import numpy as np
import pytest
import torch

import oracle
from oracle import global_tokens as og
from paper_2508_10774_amd import binding, synth
from tests import util
from tests.test_gpu_global import _run_fwd_g

pytestmark = pytest.mark.gpu

HEADS, NB = 43, 6        # 258 query blocks


def _inputs(L, seed, d=128, heads=HEADS):
    """A few distinct heads, repeated: the oracle looks at the first of them only."""
    base = [synth.make_iid((1, 2, L, d), seed, s) for s in range(3)]
    at = np.arange(heads) % 2
    return base, [util.dev_bf16(x[:, at]) for x in base]


def _check(p, base, mask, o, lse, heads=(0, 1)):
    qf, kf, vf = (synth.bf16_bits_to_f32(x) for x in base)
    for h in heads:
        want, wl = oracle.attn_fwd(qf[0, h], kf[0, h], vf[0, h], mask[h], p.block, p.scale if p.scale else None)
        util.assert_close_bf16(util.host_f32(o[0, h]), want, f"O[{h}]")
        got = lse[h].cpu().numpy()
        fin = np.isfinite(wl)
        assert np.array_equal(np.isneginf(got), np.isneginf(wl))
        assert np.abs(got[fin] - wl[fin]).max() <= util.LSE_ABS


@pytest.mark.parametrize("tail", [1, 32, 33, 95, 97, 128])
def test_rows_of_every_length_with_the_ragged_block(tail):
    L = (NB - 1) * 128 + tail
    print(f"case L={L}", flush=True)
    p = binding.Params(B=1, H=HEADS, L=L, d=128, block=128)
    base, (q, k, v) = _inputs(L, L)
    mask = np.zeros((HEADS, NB, NB), np.uint8)
    for i in range(NB):
        mask[0::2, i, NB - i:] = 1       # rows of 0 .. 5 blocks, all with the last one
        mask[1::2, i, :i + 1] = 1        # rows of 1 .. 6
    o, lse = util.run_fwd(p, q, k, v, util.lists_from_mask(p, mask, with_csc=False))
    _check(p, base, mask, o, lse)


@pytest.mark.parametrize("tail", [1, 100, 128])
def test_dense_four_wavefronts_share_the_tiles(tail):
    """Without lists 256 query rows take each copy of a tile: the last workgroup has 128 or 256 rows, few of them
    real.  (Not the bits of a call with full lists: there a row starts with its own block, here with two.)"""
    for nb in (NB, NB + 1):
        L = (nb - 1) * 128 + tail
        print(f"case L={L}", flush=True)
        p = binding.Params(B=1, H=HEADS, L=L, d=128, block=128)
        base, (q, k, v) = _inputs(L, L)
        mask = np.ones((HEADS, nb, nb), np.uint8)
        o, lse = util.run_fwd(p, q, k, v, {"row_ptr": None, "col_idx": None})
        _check(p, base, mask, o, lse)


@pytest.mark.parametrize("tail", [5, 128])
def test_a_list_that_does_not_ascend_names_the_same_keys(tail):
    L = (NB - 1) * 128 + tail
    p = binding.Params(B=1, H=HEADS, L=L, d=128, block=128)
    base, (q, k, v) = _inputs(L, 3)
    mask = np.zeros((HEADS, NB, NB), np.uint8)
    for i in range(NB):
        mask[:, i, i:] = 1
    bufs = util.lists_from_mask(p, mask, with_csc=False)
    rp = bufs["row_ptr"].cpu().numpy().reshape(HEADS, NB + 1)
    ci = bufs["col_idx"].cpu().numpy().reshape(HEADS, NB * NB).copy()
    for h in range(HEADS):
        for i in range(NB):
            ci[h, rp[h, i]:rp[h, i + 1]] = np.roll(ci[h, rp[h, i]:rp[h, i + 1]], h + 1)
    bufs["col_idx"].copy_(torch.from_numpy(ci).view(bufs["col_idx"].shape))
    o, lse = util.run_fwd(p, q, k, v, bufs)
    _check(p, base, mask, o, lse)


@pytest.mark.parametrize("order", ["up", "down", "mixed"])
def test_logits_that_grow_past_the_reference(order):
    """Blocks of keys whose logits are hundreds apart: the reference of the exponentials has to follow them upwards
    (far more than the 2^30 that a tile may exceed it by), and stays where it is downwards."""
    L = NB * 128 - 20
    p = binding.Params(B=1, H=HEADS, L=L, d=128, block=128)
    base, _ = _inputs(L, 9)
    qf, kf = (synth.bf16_bits_to_f32(x).copy() for x in base[:2])
    gain = {"up": [0, 1, 2, 3, 4, 5], "down": [5, 4, 3, 2, 1, 0], "mixed": [1, 0, 4, 0, 2, 5]}[order]
    qf[..., 0] = 16.0
    for j, g in enumerate(gain):
        kf[:, :, 128 * j + 37:128 * (j + 1), 0] = 60.0 * g      # from the middle of a tile on; 60 * 16 / sqrt(128) = 85
        kf[:, :, 128 * j:128 * j + 37, 0] = 60.0 * g - 3.0
    base = [synth.f32_to_bf16_bits(qf), synth.f32_to_bf16_bits(kf), base[2]]
    q, k, v = (util.dev_bf16(x[:, np.arange(HEADS) % 2]) for x in base)
    mask = np.ones((HEADS, NB, NB), np.uint8)
    mask[1::2, :, 5] = 0
    for bufs, m in ((util.lists_from_mask(p, mask, with_csc=False), mask),
                    ({"row_ptr": None, "col_idx": None}, np.ones_like(mask))):
        o, lse = util.run_fwd(p, q, k, v, bufs)
        _check(p, base, m, o, lse)


@pytest.mark.parametrize("n,tail", [(128, 128), (100, 17), (5, 65)])
def test_pooled_tokens_behind_the_rows_own_list(n, tail):
    L = (NB - 1) * 128 + tail
    print(f"case L={L} n={n}", flush=True)
    p = binding.Params(B=1, H=HEADS, L=L, d=128, block=128)
    base, (q, k, v) = _inputs(L, n)
    mask = np.zeros((HEADS, NB, NB), np.uint8)
    for i in range(NB):
        mask[0::2, i, NB - i:] = 1       # the first query block sees the pooled tokens only
        mask[1::2, i, :i + 1] = 1
    o, lse, _, _, _ = _run_fwd_g(p, n, q, k, v, util.lists_from_mask(p, mask, with_csc=False))
    qf, kf, vf = (synth.bf16_bits_to_f32(x) for x in base)
    for h in (0, 1):
        want, wl = og.attn_fwd_g(qf[0, h], kf[0, h], vf[0, h], mask[h], 128, n)
        util.assert_close_bf16(util.host_f32(o)[0, h], want, f"O[{h}]")
        assert np.abs(lse[h].cpu().numpy() - wl).max() <= util.LSE_ABS


@pytest.mark.parametrize("d,heads,L", [(128, 12, 4030), (128, 12, 4097), (64, 8, 8100), (64, 15, 8197), (64, 8, 8064)])
def test_block_64_without_lists(d, heads, L):
    """Long dense calls of block 64 take the workgroups of 256 rows too: a last workgroup of 1, 5, 128 and more rows."""
    print(f"case L={L} d={d}", flush=True)
    p = binding.Params(B=1, H=heads, L=L, d=d, block=64)
    base, (q, k, v) = _inputs(L, L, d, heads)
    mask = np.ones((heads, p.Nb, p.Nb), np.uint8)
    o, lse = util.run_fwd(p, q, k, v, {"row_ptr": None, "col_idx": None})
    _check(p, base, mask, o, lse, heads=(1,))
    even = [x[:, 0::2] for x in (o, lse.view(1, heads, L))]
    assert all(torch.equal(x, x[:, :1].expand_as(x)) for x in even)
