"""GPU parity: seeded per-block random sampling (Alg. 3 step 2 with a counter-based generator)."""

import numpy as np
import pytest
import torch

import oracle
from oracle import random_sampling as rs
from paper_2508_10774_amd import binding, synth
from tests import util

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,L,block,ks,seed", [
    (2, 1024, 64, 16, 1),
    (3, 1000, 128, 16, 0xDEADBEEF12345678),    # 64-bit seed: both key words in use
    (1, 300, 128, 5, 7),
    (1, 640, 64, 1, 3),
])
def test_offset_table_is_bit_exact(H, L, block, ks, seed):
    print(f"case H={H} L={L} block={block} k={ks} seed={seed:#x}", flush=True)
    p = binding.Params(B=1, H=H, L=L, d=64, block=block, k_samples=ks)
    table = torch.full((H, p.Nb, ks), 255, dtype=torch.uint8, device="cuda")
    binding.asa_sample_offsets(p, seed, table)
    torch.cuda.synchronize()
    want = rs.offsets_table(seed, H, p.Nb, block, ks)
    assert np.array_equal(table.cpu().numpy(), want)


@pytest.mark.parametrize("H,L,d,block,ks,tau", [
    (2, 1024, 64, 64, 16, 0.9),
    (2, 1000, 128, 128, 16, 0.8),     # ragged last block: 104 tokens, some samples fall past L
    (1, 333, 128, 64, 7, 0.95),       # fewer than 16 samples, last block 13 tokens
    (2, 77 * 64 - 30, 128, 64, 16, 0.9),   # shares of five chunks, a last one of one block
    (1, 61 * 128 - 1, 64, 128, 5, 0.9),    # of four chunks, few samples
])
def test_seeded_mask_matches_the_oracle(H, L, d, block, ks, tau):
    print(f"case H={H} L={L} d={d} block={block} k={ks} tau={tau}", flush=True)
    seed = 1234 + L
    qb, kb = (synth.make_iid((1, H, L, d), L + d, s) for s in range(2))
    p = binding.Params(B=1, H=H, L=L, d=d, block=block, k_samples=ks, tau=tau)
    bufs = binding.alloc_index_lists(p)
    gp = torch.empty((H, p.Nb, p.Nb), dtype=torch.float32, device="cuda")
    ws = binding.alloc_workspace(binding.asa_mask_seeded_workspace_bytes(p))
    binding.asa_build_mask_seeded(p, seed, util.dev_bf16(qb), util.dev_bf16(kb), bufs["mask"],
                                  bufs["row_ptr"], bufs["col_idx"], bufs["col_ptr"], bufs["row_idx"],
                                  gp, ws)
    torch.cuda.synchronize()
    table = rs.offsets_table(seed, H, p.Nb, block, ks)
    gmask = bufs["mask"].cpu().numpy()
    gp = gp.cpu().numpy()
    qf, kf = synth.bf16_bits_to_f32(qb), synth.bf16_bits_to_f32(kb)
    for h in range(H):
        P = rs.p_imp_table(qf[0, h], kf[0, h], block, table[h])
        nz = P > 1e-30
        rel = np.abs(gp[h][nz] - P[nz]) / P[nz]
        assert rel.max() <= 1e-4, f"head {h}: P_imp rel err {rel.max():.2e}"
        assert ((gp[h] == 0) == (P == 0)).all()
        want, _ = oracle.mask_rule(P.astype(np.float32), tau)
        self_rule, _ = oracle.mask_rule(gp[h], tau)
        assert np.array_equal(self_rule, gmask[h]), f"head {h}: rule on the GPU's own scores"
        e, x, failed = util.classify_mask_rows(P.astype(np.float32), want, gmask[h], tau)
        assert not failed, f"head {h}: rows {failed[:5]}"
        print(f"  head {h}: rows exact {e} excused {x}", flush=True)
    # index lists agree with the mask
    rp, ci = oracle.csr_from_mask(gmask[0])
    assert np.array_equal(bufs["row_ptr"][0].cpu().numpy(), np.asarray(rp).reshape(-1))


def test_default_build_is_unchanged_by_the_table_variant():
    # the shared-offset path still gives what it gave: compare with the oracle on one case
    H, L, d, block = 1, 512, 64, 64
    qb, kb = (synth.make_iid((1, H, L, d), 9, s) for s in range(2))
    p = binding.Params(B=1, H=H, L=L, d=d, block=block, tau=0.9)
    bufs = binding.alloc_index_lists(p)
    ws = binding.alloc_workspace(binding.asa_mask_workspace_bytes(p))
    binding.asa_build_mask(p, util.dev_bf16(qb), util.dev_bf16(kb), bufs["mask"], bufs["row_ptr"],
                           bufs["col_idx"], bufs["col_ptr"], bufs["row_idx"], None, ws)
    torch.cuda.synchronize()
    offs = synth.default_sample_offsets(block, 16)
    want, _ = oracle.build_mask(synth.bf16_bits_to_f32(qb), synth.bf16_bits_to_f32(kb), block, offs, 0.9)
    assert np.array_equal(bufs["mask"].cpu().numpy(), want.reshape(H, p.Nb, p.Nb))
