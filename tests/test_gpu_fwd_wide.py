"""GPU parity of the forward kernel with 64 query rows per wavefront, forced here, where it can go wrong: list
lengths around its software pipeline, the ragged last tile, lists that do not ascend, references that have to be
moved; and the rule that chooses between it and the other kernels."""

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
LOCK_STEP, PING_PONG, WIDE = 1, 2, 4


def own_choice(test):
    """A test about the library's choice of the kernel."""
    test.own_choice = True
    return test


@pytest.fixture(autouse=True)
def wide_kernel(request):
    """Calls of these sizes belong to other kernels: every test runs the wide one, unless it is about the choice."""
    binding.asa_test_force_fwd_kernel(0 if getattr(request.function, "own_choice", False) else WIDE)
    yield
    binding.asa_test_force_fwd_kernel(0)


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
    binding.asa_test_force_fwd_kernel(LOCK_STEP)     # (the wide kernel did run: these are other bits)
    assert not torch.equal(o, util.run_fwd(p, q, k, v, util.lists_from_mask(p, mask, with_csc=False))[0])


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


# The calls that the wide kernel has: lists, no lists, pooled tokens behind lists, and blocks of 64 without lists at both
# head sizes
CALLS = {"short lists": (128, 128, 42, 6), "lists": (128, 128, 33, 8), "dense": (128, 128, 43, 6),
         "pooled": (128, 128, 43, 6), "block 64, d 128": (64, 128, 12, 64), "block 64, d 64": (64, 64, 8, 128)}


def _run(call, L, q, k, v, mask, heads):
    block, d = CALLS[call][:2]
    p = binding.Params(B=1, H=heads, L=L, d=d, block=block)
    if call == "pooled":
        o, lse, _, _, _ = _run_fwd_g(p, 128, q, k, v, util.lists_from_mask(p, mask, with_csc=False))
        return p, o, lse
    bufs = util.lists_from_mask(p, mask, with_csc=False) if "lists" in call else {"row_ptr": None, "col_idx": None}
    return (p, *util.run_fwd(p, q, k, v, bufs))


@pytest.mark.parametrize("call", list(CALLS))
def test_infinite_values_stay_infinite(call):
    """An infinite element of V gives that infinity in its channel, in every row that sees the key (as P > 0 does), and
    changes nothing else: in the first tiles of a row, where the rounding of P is made up for, in later ones and in the last."""
    block, d, heads, nb = CALLS[call]
    L = nb * block - 30
    print(f"case {call} L={L}", flush=True)
    (qb, kb, vb), (q, k, v) = _inputs(L, 21, d, heads)
    mask = np.ones((heads, nb, nb), np.uint8)
    if call in ("short lists", "pooled"):
        mask[:, 1::2, 0] = 0
    at = {0: 40, 1: 2 * block + 33, 2: L - 1}         # channel: key
    vf = synth.bf16_bits_to_f32(vb).copy()
    for c, key in at.items():
        v[:, :, key, c] = float("inf") if c != 1 else -float("inf")
        vf[..., c] = 0.0
    p, o, lse = _run(call, L, q, k, v, mask, heads)
    o = util.host_f32(o)
    qf, kf = (synth.bf16_bits_to_f32(x) for x in (qb, kb))
    for h in (0, 1):
        if call == "pooled":                          # (every row sees the pooled infinities)
            seen = {c: np.ones(L, bool) for c in at}
            want, wl = og.attn_fwd_g(qf[0, h], kf[0, h], vf[0, h], mask[h], block, 128)
        else:
            seen = {c: np.repeat(mask[h, :, key // block], block)[:L] > 0 for c, key in at.items()}
            want, wl = oracle.attn_fwd(qf[0, h], kf[0, h], vf[0, h], mask[h], block, None)
        for c, rows in seen.items():
            assert (o[0, h, rows, c] == (np.inf if c != 1 else -np.inf)).all(), f"channel {c}"
            assert np.isfinite(o[0, h, ~rows, c]).all()
        util.assert_close_bf16(o[0, h, :, 3:], want[:, 3:], f"O[{h}]")
        assert np.abs(lse[h].cpu().numpy() - wl).max() <= util.LSE_ABS


@pytest.mark.parametrize("call", list(CALLS))
def test_large_values_do_not_overflow_on_the_way(call):
    """Logits that grow by 2^25 from the first keys of a row to the last, V at 2^106: P relative to the row maximum has sums that
    fit, P relative to an early logit does not."""
    block, d, heads, nb = CALLS[call]
    L = nb * block - 30
    print(f"case {call} L={L}", flush=True)
    (qb, kb, vb), _ = _inputs(L, 22, d, heads)
    qf, kf = (synth.bf16_bits_to_f32(x).copy() for x in (qb, kb))
    qf[..., 0] = 4.0
    kf[..., 0] = 0.0
    kf[:, :, L - 50:, 0] = np.float32(25 * np.log(2) * d ** 0.5 / 4)
    qb, kb = synth.f32_to_bf16_bits(qf), synth.f32_to_bf16_bits(kf)
    qf, kf, vf = (synth.bf16_bits_to_f32(x) for x in (qb, kb, vb))
    of_head = np.arange(heads) % 2
    q, k, v = (util.dev_bf16(x[:, of_head]) for x in (qb, kb, vb))
    v = v * 2.0 ** 106                                # (a power of two: the same bits at another exponent)
    mask = np.ones((heads, nb, nb), np.uint8)
    p, o, _ = _run(call, L, q, k, v, mask, heads)
    o = util.host_f32(o).astype(np.float64) / 2.0 ** 106
    for h in (0, 1):
        if call == "pooled":
            want, _ = og.attn_fwd_g(qf[0, h], kf[0, h], vf[0, h], mask[h], block, 128)
        else:
            want, _ = oracle.attn_fwd(qf[0, h], kf[0, h], vf[0, h], mask[h], block, None)
        util.assert_close_bf16(o[0, h], want, f"O[{h}]")


@pytest.mark.parametrize("call", list(CALLS))
def test_a_first_tile_without_a_finite_logit(call):
    """The first block of a row has logits of minus infinity only (a product that overflows fp32), all others far below zero:
    the first reference must not stay above them."""
    block, d, heads, nb = CALLS[call]
    L = nb * block - 30
    print(f"case {call} L={L}", flush=True)
    (qb, kb, vb), _ = _inputs(L, 23, d, heads)
    qf, kf = (synth.bf16_bits_to_f32(x).copy() for x in (qb, kb))
    qf[..., 0] = 2.0 ** 64
    kf[..., 0] = -2.0 ** -52                          # -2^12 / sqrt(d): 370 (d 128) and 510 (d 64)
    kf[:, :, :block, 0] = -2.0 ** 70
    qb, kb = synth.f32_to_bf16_bits(qf), synth.f32_to_bf16_bits(kf)
    of_head = np.arange(heads) % 2
    q, k, v = (util.dev_bf16(x[:, of_head]) for x in (qb, kb, vb))
    mask = np.ones((heads, nb, nb), np.uint8)
    if call != "lists":
        mask[:, np.arange(1, nb), np.arange(1, nb)] = 0
    if "block 64" in call or call == "dense":
        mask[:] = 1                                   # (the rows of the first block start with it)
    p, o, lse = _run(call, L, q, k, v, mask, heads)
    o = util.host_f32(o)
    qf, kf, vf = (synth.bf16_bits_to_f32(x) for x in (qb, kb, vb))
    for h in (0, 1):
        if call == "pooled":
            want, wl = og.attn_fwd_g(qf[0, h], kf[0, h], vf[0, h], mask[h], block, 128)
        else:
            want, wl = oracle.attn_fwd(qf[0, h], kf[0, h], vf[0, h], mask[h], block, None)
        util.assert_close_bf16(o[0, h], want, f"O[{h}]")
        assert np.abs(lse[h].cpu().numpy() - wl).max() <= util.LSE_ABS


@own_choice
@pytest.mark.parametrize("heads,nb", [(4, 64), (60, 32), (33, 8)])
def test_the_timing_hook_covers_both_kernels_of_a_pair(heads, nb):
    """The ping-pong, the wide and the lock-step kernel do the work of the call; the first two stand beside a launch that
    finds none."""
    p = binding.Params(B=1, H=heads, L=nb * 128, d=128, block=128)
    _, (q, k, v) = _inputs(p.L, 5, 128, heads)
    bufs = util.lists_from_mask(p, np.ones((heads, nb, nb), np.uint8), with_csc=False)
    o, lse = torch.empty_like(q), torch.empty((heads, p.L), dtype=torch.float32, device="cuda")
    ws = binding.alloc_workspace(binding.asa_fwd_workspace_bytes(p))
    share = []
    for _ in range(5):
        ev = [torch.cuda.Event(enable_timing=True) for _ in range(4)]
        for e in ev:
            e.record()                                # (creates the handles)
        for _ in range(10):                           # the host runs ahead of these
            binding.asa_attn_fwd(p, q, k, v, bufs["row_ptr"], bufs["col_idx"], o, lse, ws)
        ev[0].record()
        binding.asa_set_kernel_timing(ev[1], ev[2])
        binding.asa_attn_fwd(p, q, k, v, bufs["row_ptr"], bufs["col_idx"], o, lse, ws)
        ev[3].record()
        torch.cuda.synchronize()
        share.append(ev[1].elapsed_time(ev[2]) / ev[0].elapsed_time(ev[3]))
    assert max(share) <= 1.01 and sorted(share)[2] >= 0.5, share


# block 128 / d 128: what, heads, blocks per head, tiles per row, the kernel that the library chooses
CHOICES = [
    ("lists", 4, 64, 17, LOCK_STEP), ("lists", 4, 64, 18, PING_PONG),                # up to 256 query blocks
    ("lists", 8, 64, 17, LOCK_STEP), ("lists", 8, 64, 18, PING_PONG),                # 512: two rounds, maybe uneven
    ("fixed budget", 8, 64, 17, LOCK_STEP), ("fixed budget", 8, 64, 18, WIDE),       # 512 of one length
    ("fixed budget", 9, 64, 18, PING_PONG), ("fixed budget", 28, 64, 18, PING_PONG),  # 576, 1792: an odd number of rounds
    ("lists", 28, 64, 18, PING_PONG), ("lists", 29, 64, 18, WIDE), ("lists", 29, 64, 17, LOCK_STEP),    # 1792, 1856
    ("prefix", 29, 64, 18, PING_PONG), ("prefix, budget", 29, 64, 18, WIDE),
    ("lists", 16, 17, 17, LOCK_STEP), ("fixed budget", 29, 17, 17, LOCK_STEP),       # no slab can reach 18
    ("dense", 4, 64, 64, PING_PONG), ("dense", 8, 64, 64, WIDE), ("dense", 9, 64, 64, PING_PONG),
    ("dense", 28, 64, 64, PING_PONG), ("dense", 29, 64, 64, WIDE), ("dense", 36, 64, 64, WIDE),
    ("dense", 30, 13, 13, WIDE), ("dense", 38, 13, 13, LOCK_STEP),                   # 494 blocks, but 266 times 256 rows
    ("dense", 37, 7, 7, LOCK_STEP), ("dense", 33, 8, 8, WIDE), ("dense", 11, 24, 24, PING_PONG), ("dense", 12, 23, 23, WIDE),
    ("dense", 10, 47, 47, PING_PONG), ("dense", 18, 47, 47, WIDE), ("dense", 10, 48, 48, WIDE),
    ("pooled", 4, 64, 8, PING_PONG), ("pooled", 8, 64, 8, PING_PONG), ("pooled, budget", 8, 64, 8, WIDE),
    ("pooled", 12, 64, 8, PING_PONG), ("pooled", 13, 64, 8, WIDE), ("pooled, prefix", 13, 64, 8, PING_PONG),
    ("pooled", 33, 8, 8, WIDE), ("pooled", 90, 8, 4, WIDE), ("pooled", 30, 9, 8, PING_PONG),
]


@own_choice
@pytest.mark.parametrize("what,heads,nb,tiles,kernel", CHOICES)
def test_both_sides_of_the_lines_between_the_kernels(what, heads, nb, tiles, kernel):
    """Which kernel ran shows in the last bits: the library's choice equals one forced kernel and differs from the others."""
    budget = dict(r_min=(tiles - 0.5) / nb, r_max=(tiles - 0.5) / nb) if "budget" in what else {}
    p = binding.Params(B=1, H=heads, L=nb * 128 - 5, d=128, block=128, n_prefix_dense=100 if "prefix" in what else 0, **budget)
    print(f"case {what} {heads} x {nb} blocks of {tiles} tiles", flush=True)
    _, (q, k, v) = _inputs(p.L, 31, 128, heads)
    mask = np.zeros((nb, nb), np.uint8)
    for i in range(nb):
        mask[i, (i + np.arange(tiles)) % nb] = 1
    mask = np.broadcast_to(mask, (heads, nb, nb))
    bufs = {"row_ptr": None, "col_idx": None} if what == "dense" else util.lists_from_mask(p, mask, with_csc=False)
    out = []
    for which in (0, LOCK_STEP, PING_PONG, WIDE):
        binding.asa_test_force_fwd_kernel(which)
        o = _run_fwd_g(p, 128, q, k, v, bufs)[0] if "pooled" in what else util.run_fwd(p, q, k, v, bufs)[0]
        assert torch.isfinite(o).all()
        out.append(o)
    same = [torch.equal(out[0], x) for x in out[1:]]
    if "pooled" in what:                             # (has no lock-step kernel: that switch is the ping-pong one again)
        assert same[1:] == [kernel == PING_PONG, kernel == WIDE]
    else:
        assert same == [kernel == x for x in (LOCK_STEP, PING_PONG, WIDE)], same


@own_choice
@pytest.mark.parametrize("d,heads,L,wide", [
    (128, 12, 4000, True), (128, 12, 3999, False),       # 192 workgroups of 256 rows: three quarters of a round
    (128, 11, 4096, False), (128, 24, 4000, True), (128, 23, 4090, False),
    (64, 8, 8000, True), (64, 8, 7999, False),           # 256
    (64, 7, 8192, False), (64, 15, 8192, True), (64, 14, 8192, False),    # 15 sixteenths
])
def test_block_64_without_lists_on_both_sides_of_the_line(d, heads, L, wide):
    print(f"case L={L} d={d} heads={heads}", flush=True)
    p = binding.Params(B=1, H=heads, L=L, d=d, block=64)
    _, (q, k, v) = _inputs(L, 33, d, heads)
    out = []
    for which in (0, WIDE):
        binding.asa_test_force_fwd_kernel(which)
        out.append(util.run_fwd(p, q, k, v, {"row_ptr": None, "col_idx": None})[0])
    assert torch.isfinite(out[0]).all()
    assert torch.equal(*out) == wide


@pytest.mark.parametrize("lists", [False, True])
@pytest.mark.parametrize("gain", [1.0, 1.5, 2.0, 3.0])
def test_error_no_larger_than_with_the_running_maximum(gain, lists):
    """Noise of growing logits, where many keys of a row pass the reference of its start: O + o_lo is no further from
    64 bits than with the ping-pong kernel, whose running maximum makes each of them exact as it comes.  (2 %: what the two
    figures scatter by, sums over 2 x 2 400 x 128 roundings of which a few per cent of the keys decide.)"""
    nb, heads = 19, 2
    L = nb * 128 - 32
    print(f"case gain={gain} lists={lists}", flush=True)
    (qb, kb, vb), (_, k, v) = _inputs(L, 41, 128, heads)
    qb = synth.f32_to_bf16_bits(synth.bf16_bits_to_f32(qb) * np.float32(gain))
    q = util.dev_bf16(qb)
    p = binding.Params(B=1, H=heads, L=L, d=128, block=128)
    mask = np.ones((heads, nb, nb), np.uint8)
    bufs = util.lists_from_mask(p, mask, with_csc=False) if lists else {"row_ptr": None, "col_idx": None}
    qf, kf, vf = (synth.bf16_bits_to_f32(x) for x in (qb, kb, vb))
    want = np.stack([oracle.attn_fwd(qf[0, h], kf[0, h], vf[0, h], mask[h], 128, None)[0] for h in range(heads)])
    error = {}
    for which in (WIDE, PING_PONG):
        binding.asa_test_force_fwd_kernel(which)
        o, _, o_lo = util.run_fwd(p, q, k, v, bufs, with_lo=True)
        got = util.host_f32(o)[0].astype(np.float64) + util.host_f32(o_lo)[0]
        error[which] = np.linalg.norm(got - want) / np.linalg.norm(want)
    print(f"    wide {error[WIDE]:.3e} ping-pong {error[PING_PONG]:.3e}")
    assert error[WIDE] <= 1.02 * error[PING_PONG]
