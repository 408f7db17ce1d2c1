"""The variants of the factor producers that large batches take (tables of the projection in LDS; four residues per wave
in the neighbour search) at ragged sizes just past the line, against the oracles: whole-number decisions bit-equal, sums
within half a bf16 step (the bounds of test_gpu_factor and test_gpu_knn)."""
import numpy as np
import pytest

from oracle import knn_ref
from paper_2505_11580_amd import binding
from tests.test_gpu_factor import make_tables

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,k,n_bins,n_pos,n_out,pos_mode", [(16391, 3, 5, 9, 520, 1), (5471, 2, 7, 0, 1400, 0), (8195, 1, 4, 33, 1024, 0)])
def test_projection_from_lds_tables(L, k, n_bins, n_pos, n_out, pos_mode):
    import torch
    B = 1 if n_out == 520 else 6
    rng = np.random.default_rng(L)
    e_bin, e_pos, bias = make_tables(rng, k, n_bins, n_pos, n_out)
    idx = rng.integers(-1, L, size=(B, L, k)).astype(np.int32)
    bins = np.where(idx < 0, -1, rng.integers(0, n_bins, size=(B, L, k))).astype(np.int32)
    z = torch.full((B, L, n_out), float("nan"), dtype=torch.bfloat16, device="cuda:0")
    binding.fipa_factor_project(pos_mode, torch.from_numpy(idx).cuda(), torch.from_numpy(bins).cuda(), e_bin.cuda(),
                                e_pos.cuda() if n_pos else None, torch.from_numpy(bias).cuda(), z)
    torch.cuda.synchronize()
    rows = np.unique(np.concatenate([np.arange(300), rng.integers(0, L, 300), np.arange(L - 300, L)]))
    e32 = [e_bin.float().numpy(), e_pos.float().numpy() if n_pos else None]
    for b in (0, B - 1):
        got = z[b][torch.from_numpy(rows).cuda()].float().cpu().numpy().astype(np.float64)
        # (the sampled residues' sums, slot by slot)
        want = np.tile(bias.astype(np.float64), (len(rows), 1))
        for s in range(k):
            j, bn = idx[b, rows, s], bins[b, rows, s]
            on = (j >= 0)[:, None]
            want += np.where(on, e32[0][s][np.maximum(bn, 0)], 0.0)
            if n_pos:
                half = (n_pos - 1) // 2
                code = np.minimum(j, n_pos - 1) if pos_mode == 0 else np.clip(j - rows, -half, half) + half
                want += np.where(on, e32[1][s][np.maximum(code, 0)], 0.0)
        assert np.all(np.abs(got - want) <= 2.0 ** -8 * np.abs(want) + 1e-5 * np.abs(want).max())


@pytest.mark.parametrize("B,L,k", [(3, 5470, 20), (65, 257, 7)])
def test_neighbours_four_residues_per_wave(B, L, k):
    import torch
    rng = np.random.default_rng(L)
    trans = np.cumsum(rng.standard_normal((B, L, 3)) * 2.2, axis=1).astype(np.float32)
    trans[0, 5:9] = trans[0, 4]  # equal distances
    mask = (rng.random((B, L)) > 0.2).astype(np.uint8)
    mask[-1, L // 3:] = 0
    i32 = dict(dtype=torch.int32, device="cuda:0")
    idx, bins = torch.empty(B, L, k, **i32), torch.empty(B, L, k, **i32)
    d2 = torch.empty(B, L, k, device="cuda:0")
    binding.fipa_knn_distogram(k, 16, 2.0, 22.0, torch.from_numpy(trans).cuda(), torch.from_numpy(mask).cuda(), idx, d2, bins)
    torch.cuda.synchronize()
    for b in sorted({0, B // 2, B - 1}):
        w_idx, w_d2, w_bins = knn_ref.knn_distogram(trans[b:b + 1], mask[b:b + 1], k, 16, 2.0, 22.0)
        assert np.array_equal(idx[b].cpu().numpy(), w_idx[0]) and np.array_equal(bins[b].cpu().numpy(), w_bins[0])
        assert np.array_equal(d2[b].cpu().numpy(), w_d2[0])
