"""GPU parity: block-sparse attention forward vs the CPU oracle, through the C ABI."""

import numpy as np
import pytest
import torch

import oracle
from paper_2508_10774_amd import binding, synth
from tests import util

pytestmark = pytest.mark.gpu


FORCED = {"auto": 0, "lockstep": 1, "pingpong": 2, "wide": 4}


def picks_its_kernel(test):
    """A test that is about the choice of the kernel, or forces one itself: runs once."""
    test.picks_its_kernel = True
    return test


def equal_bits_without_lists(test):
    """A test that a dense call has the bits of one with full lists: not so with the wide kernel, whose
    workgroups of 256 rows start with two blocks of their own where those with lists start with one."""
    test.equal_bits_without_lists = True
    return test


def pytest_generate_tests(metafunc):
    once = getattr(metafunc.function, "picks_its_kernel", False)
    all_but = {"wide"} if getattr(metafunc.function, "equal_bits_without_lists", False) else set()
    metafunc.parametrize("kernel_choice", ["auto"] if once else [x for x in FORCED if x not in all_but], indirect=True)


@pytest.fixture(autouse=True)
def kernel_choice(request):
    """Every other test of this module runs four times: with the library's own choice of forward kernel
    (at the small sizes here the pipelined one), with the lock-step kernel,
    which production calls reach at larger sizes, with the ping-pong kernel, which block 128 / d 128 has, and
    with the wide kernel, which that shape has and block 64 without lists (where a shape has not got it, its own
    choice runs again)."""
    binding.asa_test_force_fwd_kernel(FORCED[request.param])
    yield request.param
    binding.asa_test_force_fwd_kernel(0)


def _case(B, H, L, d, block, seed):
    shape = (B, H, L, d)
    q, k, v = (synth.make_iid(shape, seed, s) for s in range(3))
    return q, k, v


def _check_fwd(p, qb, kb, vb, mask, heads=None, qblocks=None):
    bufs = util.lists_from_mask(p, mask, with_csc=False)
    o, lse = util.run_fwd(p, util.dev_bf16(qb), util.dev_bf16(kb), util.dev_bf16(vb), bufs)
    o = util.host_f32(o)
    lse = lse.cpu().numpy()
    qf, kf, vf = (synth.bf16_bits_to_f32(x) for x in (qb, kb, vb))
    scale = p.scale if p.scale else None
    worst = (0.0, 0.0)
    for b in range(p.B):
        for h in (heads if heads is not None else range(p.H)):
            s = b * p.H + h
            want, wl = oracle.attn_fwd(qf[b, h], kf[b, h], vf[b, h], mask.reshape(-1, p.Nb, p.Nb)[s],
                                       p.block, scale, qblocks)
            rows = ~np.isnan(wl)
            e = util.assert_close_bf16(o[b, h][rows], want[rows], f"O[{b},{h}]")
            worst = max(worst, e)
            fin = np.isfinite(wl[rows])
            assert np.abs(lse[s][rows][fin] - wl[rows][fin]).max() <= util.LSE_ABS
            assert np.array_equal(np.isneginf(lse[s][rows]), np.isneginf(wl[rows]))
    return worst


@pytest.mark.parametrize("B,H,L,d,block,dens", [
    (1, 2, 1024, 64, 64, 0.4),      # several tiles, exact multiple
    (1, 2, 1000, 128, 128, 0.5),    # ragged tail: last block 104 valid
    (2, 2, 300, 64, 128, 0.6),      # block 128 with d 64, tail 44
    (1, 3, 520, 128, 64, 0.5),      # block 64 with d 128, tail 8
    (1, 1, 64, 64, 64, 1.0),        # a single block
    (1, 1, 1, 128, 128, 1.0),       # a single token
])
def test_fwd_random_masks(B, H, L, d, block, dens):
    print(f"case B={B} H={H} L={L} d={d} block={block} dens={dens}", flush=True)
    p = binding.Params(B=B, H=H, L=L, d=d, block=block)
    qb, kb, vb = _case(B, H, L, d, block, seed=L + d)
    mask = synth.random_block_mask(p.Nb, dens, seed=L, slabs=B * H)
    _check_fwd(p, qb, kb, vb, mask)


def test_fwd_all_blocks_kept_is_dense_attention():
    p = binding.Params(B=1, H=2, L=640, d=128, block=128)
    qb, kb, vb = _case(1, 2, 640, 128, 128, seed=3)
    mask = np.ones((2, p.Nb, p.Nb), np.uint8)
    bufs = util.lists_from_mask(p, mask, with_csc=False)
    o, _ = util.run_fwd(p, util.dev_bf16(qb), util.dev_bf16(kb), util.dev_bf16(vb), bufs)
    qf, kf, vf = (torch.from_numpy(synth.bf16_bits_to_f32(x).astype(np.float64)) for x in (qb, kb, vb))
    want = torch.nn.functional.scaled_dot_product_attention(qf, kf, vf).numpy()
    util.assert_close_bf16(util.host_f32(o), want, "dense O")


@equal_bits_without_lists
@pytest.mark.parametrize("L,d,block", [(640, 128, 128), (1000, 64, 64), (333, 128, 64)])
def test_fwd_dense_specialisation_needs_no_lists(L, d, block):
    """row_ptr = col_idx = NULL: every key block.  Same tiles in the same order as a full mask's
    lists, so bit-identical to that call; and equal to plain soft-max attention."""
    print(f"case dense L={L} d={d} block={block}", flush=True)
    p = binding.Params(B=1, H=2, L=L, d=d, block=block)
    qb, kb, vb = _case(1, 2, L, d, block, seed=11)
    q, k, v = (util.dev_bf16(x) for x in (qb, kb, vb))
    full = util.lists_from_mask(p, np.ones((2, p.Nb, p.Nb), np.uint8), with_csc=False)
    o_ref, lse_ref = util.run_fwd(p, q, k, v, full)
    o, lse = util.run_fwd(p, q, k, v, {"row_ptr": None, "col_idx": None})
    assert torch.equal(o.view(torch.int16), o_ref.view(torch.int16))
    assert torch.equal(lse, lse_ref)
    qf, kf, vf = (torch.from_numpy(synth.bf16_bits_to_f32(x).astype(np.float64)) for x in (qb, kb, vb))
    want = torch.nn.functional.scaled_dot_product_attention(qf, kf, vf).numpy()
    util.assert_close_bf16(util.host_f32(o), want, "dense O")


@picks_its_kernel
def test_fwd_single_stage_kernel_is_still_correct():
    """The kernel that takes over for slabs of 4 GiB and more, forced by its switch."""
    binding.asa_test_force_fwd_kernel(1)
    p = binding.Params(B=1, H=2, L=1000, d=128, block=128)
    qb, kb, vb = _case(1, 2, 1000, 128, 128, seed=5)
    mask = synth.random_block_mask(p.Nb, 0.5, seed=5, slabs=2)
    _check_fwd(p, qb, kb, vb, mask)
    p = binding.Params(B=1, H=1, L=520, d=64, block=64)
    qb, kb, vb = _case(1, 1, 520, 64, 64, seed=6)
    _check_fwd(p, qb, kb, vb, synth.random_block_mask(p.Nb, 0.6, seed=6, slabs=1))


@picks_its_kernel
@pytest.mark.parametrize("L,d,block", [(1024, 64, 64), (520, 128, 64), (300, 64, 128)])
def test_fwd_forcing_the_ping_pong_kernel_where_there_is_none_changes_nothing(L, d, block):
    p = binding.Params(B=1, H=2, L=L, d=d, block=block)
    qb, kb, vb = _case(1, 2, L, d, block, seed=L)
    bufs = util.lists_from_mask(p, synth.random_block_mask(p.Nb, 0.5, seed=L, slabs=2), with_csc=False)
    q, k, v = (util.dev_bf16(x) for x in (qb, kb, vb))
    o, lse = util.run_fwd(p, q, k, v, bufs)
    binding.asa_test_force_fwd_kernel(2)
    o2, lse2 = util.run_fwd(p, q, k, v, bufs)
    assert torch.equal(o.view(torch.int16), o2.view(torch.int16)) and torch.equal(lse, lse2)


@picks_its_kernel
@pytest.mark.parametrize("heads,r", [(4, None), (6, None), (10, 0.5)])
def test_fwd_each_slab_goes_to_the_kernel_that_suits_its_lists(heads, r):
    """Block 128 / d 128 with lists: a kernel for long and one for short rows are launched, and each takes the (batch, head) slabs
    that are long / short for it.  Head 0 keeps 32 of 40 blocks per row, head 1 keeps 6, head 2 sits just below the
    switch-over (17 per row), head 3 just above (18), then from the start again; every row must come from exactly one.
    160 query blocks: ping-pong and pipelined; 240: ping-pong and lock-step; 400 with a fixed budget: wide and lock-step."""
    L, base_heads = 128 * 40 - 9, 4
    base = _case(1, base_heads, L, 128, 128, seed=77)
    at = np.arange(heads) % base_heads
    p = binding.Params(B=1, H=heads, L=L, d=128, block=128, **({} if r is None else dict(r_min=r, r_max=r)))
    mask = np.zeros((base_heads, p.Nb, p.Nb), np.uint8)
    rng = np.random.default_rng(7)
    for h, m in enumerate((32, 6, 17, 18)):
        for i in range(p.Nb):
            mask[h, i, rng.choice(p.Nb, size=m, replace=False)] = 1
    bufs = util.lists_from_mask(p, mask[at], with_csc=False)
    o = torch.full((1, heads, L, 128), float("nan"), dtype=torch.bfloat16, device="cuda")
    lse = torch.full((heads, L), float("nan"), dtype=torch.float32, device="cuda")
    ws = binding.alloc_workspace(binding.asa_fwd_workspace_bytes(p))
    binding.asa_attn_fwd(p, *(util.dev_bf16(x[:, at]) for x in base), bufs["row_ptr"], bufs["col_idx"], o, lse, ws)
    torch.cuda.synchronize()
    qf, kf, vf = (synth.bf16_bits_to_f32(x) for x in base)
    for h in range(heads):
        if h < base_heads:
            want, want_lse = oracle.attn_fwd(qf[0, h], kf[0, h], vf[0, h], mask[h], 128)
            util.assert_close_bf16(util.host_f32(o)[0, h], want, f"O[{h}]")
            assert np.abs(lse[h].cpu().numpy() - want_lse).max() <= util.LSE_ABS
        else:
            assert torch.equal(o[0, h].view(torch.int16), o[0, h % base_heads].view(torch.int16)) and torch.equal(lse[h], lse[h % base_heads])


@picks_its_kernel
@pytest.mark.parametrize("r", [0.5, 0.1, None])
def test_few_rows_of_any_length_whatever_the_rule_says(r):
    """Up to 192 query blocks of block 128 / d 128 the parameters of the rule choose one kernel for all rows: ping-pong from a fixed
    budget of 18 blocks on, pipelined below, both without one.  Lists that do not come from the rule are served all the
    same: rows of 0, 1, 2, 17, 18 and all 39 blocks, side by side."""
    L, H = 128 * 39 - 31, 4
    p = binding.Params(B=1, H=H, L=L, d=128, block=128, **({} if r is None else dict(r_min=r, r_max=r)))
    qb, kb, vb = _case(1, H, L, 128, 128, seed=78)
    rng = np.random.default_rng(8)
    mask = np.zeros((H, p.Nb, p.Nb), np.uint8)
    for h in range(H):
        for i in range(p.Nb):
            mask[h, i, rng.choice(p.Nb, size=(0, 1, 2, 17, 18, p.Nb)[(i + h) % 6], replace=False)] = 1
    bufs = util.lists_from_mask(p, mask, with_csc=False)
    o, lse = util.run_fwd(p, *(util.dev_bf16(x) for x in (qb, kb, vb)), bufs)
    qf, kf, vf = (synth.bf16_bits_to_f32(x) for x in (qb, kb, vb))
    for h in range(H):
        want, want_lse = oracle.attn_fwd(qf[0, h], kf[0, h], vf[0, h], mask[h], 128)
        util.assert_close_bf16(util.host_f32(o)[0, h], want, f"O[{h}]")
        got, empty = lse[h].cpu().numpy(), np.isneginf(want_lse)
        assert np.array_equal(np.isneginf(got), empty) and empty.any()
        assert np.abs(got[~empty] - want_lse[~empty]).max() <= util.LSE_ABS


def test_fwd_tiny_workload_with_oracle_mask():
    w = synth.TINY
    qb, kb, vb = synth.make_qkv(w, seed=0)
    p = binding.Params(B=w.B, H=w.H, L=w.L, d=w.d, block=w.block)
    qf, kf = synth.bf16_bits_to_f32(qb), synth.bf16_bits_to_f32(kb)
    mask, _ = oracle.build_mask(qf, kf, w.block, synth.default_sample_offsets(w.block, w.k_samples),
                                tau=0.9)
    _check_fwd(p, qb, kb, vb, mask)


def test_fwd_peaked_logits_and_custom_scale():
    # large logits (shared smooth field) stress the running-maximum rescaling
    w = synth.Workload("t", 1, 2, 128, (2, 16, 16), 0, 128, 16)
    qb, kb, vb = synth.make_qkv(w, seed=5)
    p = binding.Params(B=1, H=2, L=w.L, d=128, block=128, scale=0.05)
    mask = synth.random_block_mask(p.Nb, 0.7, seed=9, slabs=2)
    _check_fwd(p, qb, kb, vb, mask)


def test_fwd_empty_row_gives_zero_and_minus_inf():
    p = binding.Params(B=1, H=1, L=256, d=64, block=64)
    qb, kb, vb = _case(1, 1, 256, 64, 64, seed=8)
    mask = synth.random_block_mask(4, 0.5, seed=1, slabs=1)
    mask[0, 2, :] = 0
    bufs = util.lists_from_mask(p, mask, with_csc=False)
    o, lse = util.run_fwd(p, util.dev_bf16(qb), util.dev_bf16(kb), util.dev_bf16(vb), bufs)
    assert (util.host_f32(o)[0, 0, 128:192] == 0).all()
    assert torch.isneginf(lse[0, 128:192]).all()
    _check_fwd(p, qb, kb, vb, mask)


def test_fwd_strided_inputs():
    # [B, L, H, d] storage viewed as [B, H, L, d]
    B, H, L, d, block = 1, 2, 384, 64, 64
    qb, kb, vb = _case(B, H, L, d, block, seed=12)
    st = (L * H * d, d, H * d)
    p = binding.Params(B=B, H=H, L=L, d=d, block=block, q_stride=st, k_stride=st, v_stride=st,
                       o_stride=st)
    mask = synth.random_block_mask(p.Nb, 0.5, seed=2, slabs=B * H)
    bufs = util.lists_from_mask(p, mask, with_csc=False)
    tq, tk, tv = (util.dev_bf16(x).permute(0, 2, 1, 3).contiguous() for x in (qb, kb, vb))
    o = torch.zeros((B, L, H, d), dtype=torch.bfloat16, device="cuda")
    lse = torch.empty((B * H, L), dtype=torch.float32, device="cuda")
    ws = binding.alloc_workspace(binding.asa_fwd_workspace_bytes(p))
    binding.asa_attn_fwd(p, tq, tk, tv, bufs["row_ptr"], bufs["col_idx"], o, lse, ws)
    torch.cuda.synchronize()
    got = util.host_f32(o.permute(0, 2, 1, 3))
    qf, kf, vf = (synth.bf16_bits_to_f32(x) for x in (qb, kb, vb))
    for h in range(H):
        want, _ = oracle.attn_fwd(qf[0, h], kf[0, h], vf[0, h], mask[h], block)
        util.assert_close_bf16(got[0, h], want, f"strided O[{h}]")


def test_fwd_is_deterministic():
    p = binding.Params(B=1, H=2, L=1024, d=128, block=128)
    qb, kb, vb = _case(1, 2, 1024, 128, 128, seed=4)
    mask = synth.random_block_mask(p.Nb, 0.5, seed=4, slabs=2)
    bufs = util.lists_from_mask(p, mask, with_csc=False)
    args = [util.dev_bf16(x) for x in (qb, kb, vb)]
    o1, l1 = util.run_fwd(p, *args, bufs)
    o2, l2 = util.run_fwd(p, *args, bufs)
    assert torch.equal(o1.view(torch.int16), o2.view(torch.int16)) and torch.equal(l1, l2)


@pytest.mark.parametrize("block", [64, 128])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("tail", [1, 31, 32, 33, 64])
def test_fwd_list_lengths_and_tails(block, d, tail, kernel_choice):
    """Rows of 0, 1, 2, 3, ... blocks (the pipelined kernel takes four tiles of 32 keys at a time,
    blocks of 64 keys are two of them) with a last block that ends inside its first tile, at the
    end of it, inside the second one, or at a block's end."""
    Nb = 6
    L = (Nb - 1) * block + tail
    print(f"case L={L} d={d} block={block} {kernel_choice}", flush=True)
    p = binding.Params(B=1, H=2, L=L, d=d, block=block)
    qb, kb, vb = _case(1, 2, L, d, block, seed=L + d)
    mask = np.zeros((2, Nb, Nb), np.uint8)
    for i in range(Nb):
        mask[0, i, Nb - i:] = 1      # rows of 0 .. 5 blocks, every one of them with the ragged block
        mask[1, i, :i + 1] = 1       # rows of 1 .. 6
    _check_fwd(p, qb, kb, vb, mask)


@picks_its_kernel
@pytest.mark.parametrize("H,Nb", [(16, 64), (17, 64)])
def test_fwd_block_64_d_64_on_both_sides_of_the_kernel_choice(H, Nb):
    """Up to 1024 query blocks the pipelined kernel runs, beyond that the lock-step kernel."""
    L = Nb * 64 - 9
    print(f"case H={H} L={L}", flush=True)
    p = binding.Params(B=1, H=H, L=L, d=64, block=64)
    qb, kb, vb = _case(1, H, L, 64, 64, seed=H)
    _check_fwd(p, qb, kb, vb, synth.random_block_mask(Nb, 0.2, seed=H, slabs=H), heads=[0, H - 1])


@picks_its_kernel
@pytest.mark.parametrize("block,d,H,Nb,tail,lists,lock_step", [
    (128, 64, 12, 42, 119, False, False),   # 504 query blocks: pipelined workgroups all start at once
    (128, 64, 52, 10, 128, False, True),    # 520, 1 280 keys per row: lock-step from V's rows
    (128, 64, 13, 40, 33, False, True),     # 520, 5 025 keys: lock-step from the transposed copy
    (64, 128, 8, 64, 55, False, False),     # 512
    (64, 128, 19, 27, 32, False, True),     # 513, 1 696 keys
    (64, 128, 9, 57, 1, False, True),       # 513, 3 585 keys
    (64, 128, 16, 63, 55, False, False),    # 1008 of 4 023 keys: the wide kernel
    (64, 128, 17, 59, 55, False, False),    # 1003 of 3 767: two rounds, the second one nearly full
    (64, 128, 41, 25, 55, False, False),    # 1025: a second round of lock-step workgroups
    (64, 128, 53, 29, 64, False, True),     # 1537: a fourth round of pipelined ones
    (128, 64, 16, 60, 119, True, False),    # lists: pipelined whatever the number (960, 600)
    (64, 128, 20, 30, 55, True, False),
])
def test_fwd_mixed_shapes_on_both_sides_of_the_kernel_choice(block, d, H, Nb, tail, lists, lock_step):
    """Which kernel ran shows in the last bits (tiles of 64 keys or of 32): auto equals the forced lock-step
    kernel exactly where the choice falls on it.  One head against the oracle."""
    L = (Nb - 1) * block + tail
    print(f"case H={H} L={L} d={d} block={block} lists={lists}", flush=True)
    p = binding.Params(B=1, H=H, L=L, d=d, block=block)
    qb, kb, vb = _case(1, H, L, d, block, seed=H)
    q, k, v = (util.dev_bf16(x) for x in (qb, kb, vb))
    mask = np.ones((H, Nb, Nb), np.uint8)
    bufs = {"row_ptr": None, "col_idx": None}
    if lists:
        mask = synth.random_block_mask(Nb, 0.2, seed=H, slabs=H)
        bufs = util.lists_from_mask(p, mask, with_csc=False)
    o, lse = util.run_fwd(p, q, k, v, bufs)
    binding.asa_test_force_fwd_kernel(1)
    o1, lse1 = util.run_fwd(p, q, k, v, bufs)
    same = torch.equal(o.view(torch.int16), o1.view(torch.int16)) and torch.equal(lse, lse1)
    assert same == lock_step
    qf, kf, vf = (synth.bf16_bits_to_f32(x[0, H - 1]) for x in (qb, kb, vb))
    want, wl = oracle.attn_fwd(qf, kf, vf, mask[H - 1], block)
    util.assert_close_bf16(util.host_f32(o[0, H - 1]), want, "O")
    assert np.abs(lse[H - 1].cpu().numpy() - wl).max() <= util.LSE_ABS


@picks_its_kernel
@pytest.mark.parametrize("which", [0, 1, 2, 4])
@pytest.mark.parametrize("block,d", [(64, 64), (64, 128), (128, 64), (128, 128)])
def test_fwd_infinite_value_in_the_last_row_stays_infinite(block, d, which):
    """Keys past the end have probability zero and must not turn an infinite value of a real key into
    NaN (0 * inf), whatever stands in for their rows."""
    L = 2 * block + 5
    p = binding.Params(B=1, H=1, L=L, d=d, block=block)
    g = torch.Generator(device="cuda").manual_seed(1)
    q, k, v = (torch.randn(1, 1, L, d, device="cuda", generator=g).mul(0.3).bfloat16() for _ in range(3))
    v[0, 0, L - 1] = float("inf")
    bufs = util.lists_from_mask(p, np.ones((1, p.Nb, p.Nb), np.uint8), with_csc=False)
    binding.asa_test_force_fwd_kernel(which)
    o, lse = util.run_fwd(p, q, k, v, bufs)
    assert torch.isposinf(o.float()).all()
    assert torch.isfinite(lse).all()


@pytest.mark.parametrize("block,d", [(64, 64), (64, 128), (128, 64), (128, 128)])
@pytest.mark.parametrize("tail", [1, 40, 64])
def test_fwd_dense_packed_projection_with_the_low_half(block, d, tail):
    """No lists, Q, K, V as slices of one [B, L, 3, H, d] projection, O and o_lo [B, L, H, d].  O against
    plain soft-max attention; o_lo is what rounding left out of O: half a unit in its last place at most
    (2^-8 of O with 8 significant bits)."""
    B, H, L = 2, 2, 3 * block + tail
    print(f"case L={L} d={d} block={block}", flush=True)
    bits = [synth.make_iid((B, H, L, d), L, s) for s in range(3)]
    qkv = torch.stack([util.dev_bf16(x).transpose(1, 2) for x in bits], dim=2).contiguous()
    q, k, v = (qkv[:, :, i].transpose(1, 2) for i in range(3))
    o, o_lo = (torch.full((B, L, H, d), float("nan"), dtype=torch.bfloat16, device="cuda").transpose(1, 2)
               for _ in range(2))
    lse = torch.empty((B * H, L), dtype=torch.float32, device="cuda")
    p = binding.Params(B=B, H=H, L=L, d=d, block=block, q_stride=tuple(q.stride()[:3]),
                       k_stride=tuple(k.stride()[:3]), v_stride=tuple(v.stride()[:3]), o_stride=tuple(o.stride()[:3]))
    ws = binding.alloc_workspace(binding.asa_fwd_workspace_bytes(p))
    binding.asa_attn_fwd(p, q, k, v, None, None, o, lse, ws, o_lo=o_lo)
    torch.cuda.synchronize()
    qf, kf, vf = (torch.from_numpy(synth.bf16_bits_to_f32(x).astype(np.float64)) for x in bits)
    want = torch.nn.functional.scaled_dot_product_attention(qf, kf, vf).numpy()
    util.assert_close_bf16(util.host_f32(o), want, "O")
    hi, lo = util.host_f32(o).astype(np.float64), util.host_f32(o_lo).astype(np.float64)
    util.assert_close_bf16(hi + lo, want, "O + o_lo")
    assert (np.abs(lo) <= np.abs(hi) * 2.0 ** -8 + 1e-30).all() and (lo != 0).mean() > 0.9


@picks_its_kernel
@pytest.mark.parametrize("block,d,many", [(64, 64, 120), (64, 128, 110), (128, 64, 110), (128, 128, 39)])
@pytest.mark.parametrize("tail", [1, 31, 33, 64])
def test_one_and_two_groups_of_wavefronts_per_row(block, d, many, tail):
    """Few rows: two groups of wavefronts share a row, each with half of every block's keys; many rows: one group (block 128 / d 128: lock-step).  Lists of
    0 .. 5 blocks, so every remainder of the loop over four tiles; a last block whose second half may hold no key.
    The groups' parts are put together in fp32: both are as near to the oracle."""
    Nb = 5
    L = (Nb - 1) * block + tail
    base = [synth.make_iid((1, 3, L, d), block + d, s) for s in range(3)]
    rng = np.random.default_rng(tail)
    mask = np.stack([(rng.random((Nb, Nb)).argsort(axis=1) < (np.arange(Nb)[:, None] + h) % 6) for h in range(3)]).astype(np.uint8)
    qf, kf, vf = (synth.bf16_bits_to_f32(x) for x in base)
    out = []
    for heads in (3, many):
        print(f"case block={block} d={d} tail={tail} heads={heads}", flush=True)
        at = np.arange(heads) % 3
        p = binding.Params(B=1, H=heads, L=L, d=d, block=block, r_min=0.5, r_max=0.5)
        bufs = util.lists_from_mask(p, mask[at], with_csc=False)
        o, lse = util.run_fwd(p, *(util.dev_bf16(x[:, at]) for x in base), bufs)
        out.append((o, lse))
        for h in range(3):
            want, want_lse = oracle.attn_fwd(qf[0, h], kf[0, h], vf[0, h], mask[h], block)
            for copy in (h, heads - 3 + (h - (heads - 3)) % 3):
                util.assert_close_bf16(util.host_f32(o)[0, copy], want, f"O[{copy}]")
                got = lse[copy].cpu().numpy()
                empty = np.isneginf(want_lse)
                assert np.array_equal(np.isneginf(got), empty)
                assert np.abs(got[~empty] - want_lse[~empty]).max() <= 1e-3
    assert not torch.equal(out[0][0].view(torch.int16), out[1][0][:, :3].view(torch.int16))   # (two kernels ran)


@picks_its_kernel
@pytest.mark.parametrize("block,d,heads,Nb,text,r", [
    (128, 64, 60, 5, 0, (0.1, 0.5)), (64, 64, 110, 6, 0, (0.0, 1.0)), (64, 128, 60, 5, 0, (0.1, 0.5)),        # uneven rows, not all at once
    (64, 128, 93, 12, 130, (0.0, 1.0)), (128, 64, 100, 7, 20, (0.0, 1.0)), (64, 64, 40, 18, 140, (0.5, 0.5))])  # short prefix rows
def test_a_full_chip_keeps_one_group_of_wavefronts_per_row(block, d, heads, Nb, text, r):
    """What the parameters of the rule say of the rows (uneven, with a prefix) does not split rows where the chip is full without:
    the same lists with parameters that never do give the same bits (two groups would round differently)."""
    L = Nb * block - 9
    q, k, v = (util.dev_bf16(synth.make_iid((1, heads, L, d), block + d, s)) for s in range(3))
    mask = synth.random_block_mask(Nb, 0.4, seed=3, slabs=heads).reshape(heads, Nb, Nb)
    first = -(-text // block)
    mask[:, :first] = 1
    mask[:, :, :first] = 1
    out = []
    for more in (dict(r_min=r[0], r_max=r[1], n_prefix_dense=text), dict(r_min=0.5, r_max=0.5)):
        p = binding.Params(B=1, H=heads, L=L, d=d, block=block, **more)
        print(f"case block={block} d={d} heads={heads} Nb={Nb} {more}", flush=True)
        out.append(util.run_fwd(p, q, k, v, util.lists_from_mask(p, mask, with_csc=False)))
    assert torch.equal(out[0][0].view(torch.int16), out[1][0].view(torch.int16)) and torch.equal(out[0][1], out[1][1])
