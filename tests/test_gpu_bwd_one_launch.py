"""GPU parity of the backward on both sides of the choice between one launch for dK / dV and dQ and two: the
same tiles in the same order, so the gradients of a head are the same bits in a call with few heads (one launch)
and in one with many (two), with lists, without, and with pooled tokens."""

import numpy as np
import pytest
import torch

import oracle
from paper_2508_10774_amd import binding, synth
from tests import util

pytestmark = pytest.mark.gpu

NB, TAIL = 6, 21
# heads on the last and on the first side of the line: 3 (block and d alike) or 6 rounds of resident workgroups
LINE = {(64, 64): 3072, (128, 128): 768, (128, 64): 3072, (64, 128): 3072}


@pytest.mark.parametrize("with_lo", [True, False])
@pytest.mark.parametrize("lists", [True, False])
@pytest.mark.parametrize("block,d", list(LINE))
def test_a_head_has_the_same_gradients_in_one_launch_and_in_two(block, d, lists, with_lo):
    L = (NB - 1) * block + TAIL
    most = LINE[block, d] // NB
    print(f"case block={block} d={d} lists={lists} lo={with_lo}", flush=True)
    base = [synth.make_iid((1, 2, L, d), block + d, s) for s in range(4)]
    base_mask = synth.random_block_mask(NB, 0.5, seed=d, slabs=2)
    if not lists:
        base_mask[:] = 1

    def inputs(heads):
        at = np.arange(heads) % 2
        p = binding.Params(B=1, H=heads, L=L, d=d, block=block)
        bufs = (util.lists_from_mask(p, base_mask[at]) if lists else
                dict.fromkeys(("row_ptr", "col_idx", "col_ptr", "row_idx")))
        return p, bufs, [util.dev_bf16(x[:, at]) for x in base]

    p, bufs, (q, k, v, g) = inputs(2)
    o, lse, o_lo = util.run_fwd(p, q, k, v, bufs, with_lo=True)
    one = util.run_bwd(p, q, k, v, o, lse, g, bufs, o_lo=o_lo if with_lo else None)
    qf, kf, vf, gf = (synth.bf16_bits_to_f32(x) for x in base)
    for h in range(2):
        want = oracle.attn_bwd(qf[0, h], kf[0, h], vf[0, h], gf[0, h], base_mask[h], block, None)
        for got, w, name in zip(one, want, ("dQ", "dK", "dV")):
            util.assert_close_bf16(util.host_f32(got)[0, h], w, f"{name}[{h}]")
    for heads in (most, most + 1):
        p, bufs, (q, k, v, g) = inputs(heads)
        at = torch.arange(heads, device="cuda") % 2
        many = util.run_bwd(p, q, k, v, o[:, at], lse[at], g, bufs, o_lo=o_lo[:, at] if with_lo else None)
        for a, b, name in zip(many, one, ("dQ", "dK", "dV")):
            assert torch.equal(a.view(torch.int16), b[:, at].view(torch.int16)), f"{name} {heads} heads"


def test_the_same_with_pooled_tokens():
    """(Block 128 / d 128: there the pooled tokens' own sums have as many parts on both sides of the line.)"""
    block = d = 128
    L, n = (NB - 1) * block + TAIL, 32
    few, many = LINE[block, d] // NB - 1, LINE[block, d] // NB + 1
    print(f"case pooled block={block} d={d}", flush=True)
    base = [synth.make_iid((1, 2, L, d), block, s) for s in range(4)]
    base_mask = synth.random_block_mask(NB, 0.5, seed=d, slabs=2)
    grads = []
    for heads in (few, many):
        at = np.arange(heads) % 2
        p = binding.Params(B=1, H=heads, L=L, d=d, block=block)
        bufs = util.lists_from_mask(p, base_mask[at])
        q, k, v, g = (util.dev_bf16(x[:, at]) for x in base)
        G = binding.asa_global_token_count(p, n)
        kg, vg = (torch.zeros(1, heads, G, d, dtype=torch.bfloat16, device="cuda") for _ in range(2))
        ws = binding.alloc_workspace(max(binding.asa_fwd_g_workspace_bytes(p, n), binding.asa_bwd_g_workspace_bytes(p, n)))
        o, o_lo = torch.empty_like(q), torch.empty_like(q)
        lse = torch.empty((heads, L), dtype=torch.float32, device="cuda")
        binding.asa_global_tokens(p, n, k, v, kg, vg)
        binding.asa_attn_fwd_g(p, n, q, k, v, kg, vg, bufs["row_ptr"], bufs["col_idx"], o, lse, ws, o_lo=o_lo)
        out = [torch.full_like(q, float("nan")) for _ in range(3)]
        binding.asa_attn_bwd_g(p, n, q, k, v, kg, vg, o, g, lse, bufs["row_ptr"], bufs["col_idx"], bufs["col_ptr"],
                               bufs["row_idx"], *out, ws, o_lo=o_lo)
        grads.append(out)
    for a, b, name in zip(*grads, ("dQ", "dK", "dV")):
        assert torch.isfinite(a).all() and torch.isfinite(b).all()
        # (the heads repeat with period 2)
        assert torch.equal(a[:, 2:4].view(torch.int16), a[:, :2].view(torch.int16)), name
        assert torch.equal(a[:, :2].view(torch.int16), b[:, :2].view(torch.int16)), name


def _starts_early(p):
    """The rule for prefix rows: a fifth of the rows at most, as long as 1.2 times the work of a resident workgroup (whose other
    rows are taken to have the prefix columns and, with the parameters used here, half of a quarter of the blocks)."""
    resident = {(64, 64): 1024, (128, 128): 256}.get((p.block, p.d), 512)
    prefix = -(-p.n_prefix_dense // p.block)
    listed = prefix * p.Nb + (p.Nb - prefix) * min(p.Nb, prefix + (1 + max(1, p.Nb // 4)) // 2)
    return 0 < 5 * prefix <= p.Nb and 5 * p.Nb * resident > 6 * p.B * p.H * listed


@pytest.mark.parametrize("pooled", [False, True])
@pytest.mark.parametrize("block,d,heads,text,early", [
    (64, 64, 17, 1, True), (64, 64, 20, 3 * 64, True), (64, 64, 20, 3 * 64 + 1, False), (64, 128, 19, 70, True), (128, 64, 18, 300, True),
    (128, 128, 17, 129, True), (128, 128, 38, 129, True), (128, 128, 39, 129, False), (128, 64, 18, 10 ** 4, False)])
def test_rows_of_a_prefix_start_early(block, d, heads, text, early, pooled):
    """With few prefix blocks some of dQ's workgroups come before the rest of dK / dV's (more than 256 lists): every one
    runs once, whatever the number of prefix blocks, so the gradients are those of the two launches that dQ over Q takes."""
    Nb, n = 16, 32
    L = (Nb - 1) * block + TAIL
    print(f"case block={block} d={d} heads={heads} text={text} pooled={pooled}", flush=True)
    q, k, v, g = (util.dev_bf16(synth.make_iid((1, heads, L, d), block + d, s)) for s in range(4))
    p = binding.Params(B=1, H=heads, L=L, d=d, block=block, n_prefix_dense=min(text, L))
    assert heads * Nb > 256 and _starts_early(p) == early
    mask = synth.random_block_mask(Nb, 0.3, seed=text, slabs=heads).reshape(heads, Nb, Nb)
    first = -(-p.n_prefix_dense // block)
    mask[:, :first] = 1
    mask[:, :, :first] = 1
    bufs = util.lists_from_mask(p, mask)
    lists = [bufs[x] for x in ("row_ptr", "col_idx", "col_ptr", "row_idx")]
    if pooled:
        G = binding.asa_global_token_count(p, n)
        kg, vg = (torch.zeros(1, heads, G, d, dtype=torch.bfloat16, device="cuda") for _ in range(2))
        ws = binding.alloc_workspace(max(binding.asa_fwd_g_workspace_bytes(p, n), binding.asa_bwd_g_workspace_bytes(p, n)))
        o, o_lo, lse = torch.empty_like(q), torch.empty_like(q), torch.empty((heads, L), dtype=torch.float32, device="cuda")
        binding.asa_global_tokens(p, n, k, v, kg, vg)
        binding.asa_attn_fwd_g(p, n, q, k, v, kg, vg, *lists[:2], o, lse, ws, o_lo=o_lo)
    else:
        o, lse, o_lo = util.run_fwd(p, q, k, v, bufs, with_lo=True)
        ws = binding.alloc_workspace(binding.asa_bwd_workspace_bytes(p))
    out = []
    for over in (False, True):
        qq = q.clone()
        dq, dk, dv = qq if over else torch.full_like(q, float("nan")), torch.full_like(k, float("nan")), torch.full_like(v, float("nan"))
        if pooled:
            binding.asa_attn_bwd_g(p, n, qq, k, v, kg, vg, o, g, lse, *lists, dq, dk, dv, ws, o_lo=o_lo)
        else:
            binding.asa_attn_bwd(p, qq, k, v, o, g, lse, *lists, dq, dk, dv, ws, o_lo=o_lo)
        out.append([x.view(torch.int16) for x in (dq, dk, dv)])
    for a, b, name in zip(*out, ("dQ", "dK", "dV")):
        assert torch.equal(a, b), name
        assert torch.isfinite(a.view(torch.bfloat16).float()).all(), name


@pytest.mark.parametrize("with_lo", [True, False])
@pytest.mark.parametrize("block,d", list(LINE))
@pytest.mark.parametrize("pooled", [False, True])
def test_dq_in_the_place_of_an_input(block, d, with_lo, pooled):
    """dQ may be written over Q, dO or O (asa.h): dK / dV read Q and dO of every row, so that they must have ended before."""
    L, heads, n = (NB - 1) * block + TAIL, 4, 32
    print(f"case block={block} d={d} lo={with_lo} pooled={pooled}", flush=True)
    q, k, v, g = (util.dev_bf16(synth.make_iid((1, heads, L, d), block + d, s)) for s in range(4))
    p = binding.Params(B=1, H=heads, L=L, d=d, block=block)
    bufs = util.lists_from_mask(p, synth.random_block_mask(NB, 0.5, seed=d, slabs=heads))
    lists = [bufs[x] for x in ("row_ptr", "col_idx", "col_ptr", "row_idx")]
    o, o_lo = torch.empty_like(q), torch.empty_like(q)
    lse = torch.empty((heads, L), dtype=torch.float32, device="cuda")
    if pooled:
        ws = binding.alloc_workspace(max(binding.asa_fwd_g_workspace_bytes(p, n), binding.asa_bwd_g_workspace_bytes(p, n)))
        G = binding.asa_global_token_count(p, n)
        kg, vg = (torch.zeros(1, heads, G, d, dtype=torch.bfloat16, device="cuda") for _ in range(2))
        binding.asa_global_tokens(p, n, k, v, kg, vg)
        binding.asa_attn_fwd_g(p, n, q, k, v, kg, vg, *lists[:2], o, lse, ws, o_lo=o_lo)
    else:
        ws = binding.alloc_workspace(max(binding.asa_fwd_workspace_bytes(p), binding.asa_bwd_workspace_bytes(p)))
        binding.asa_attn_fwd(p, q, k, v, *lists[:2], o, lse, ws, o_lo=o_lo)

    def run(over):
        t = {"q": q.clone(), "d_o": g.clone(), "o": o.clone()}
        dq = t[over] if over else torch.empty_like(q)
        dk, dv = torch.empty_like(k), torch.empty_like(v)
        lo = o_lo if with_lo else None
        if pooled:
            binding.asa_attn_bwd_g(p, n, t["q"], k, v, kg, vg, t["o"], t["d_o"], lse, *lists, dq, dk, dv, ws, o_lo=lo)
        else:
            binding.asa_attn_bwd(p, t["q"], k, v, t["o"], t["d_o"], lse, *lists, dq, dk, dv, ws, o_lo=lo)
        return [x.view(torch.int16) for x in (dq, dk, dv)]

    want = run(None)
    for over in ("q", "d_o", "o"):
        for a, b, name in zip(run(over), want, ("dQ", "dK", "dV")):
            assert torch.equal(a, b), f"{name} with dQ over {over}"
