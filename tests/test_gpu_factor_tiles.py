"""GPU parity of fipa_factor_project_backward at the edges of its residue tiles (32 per wave, eight waves) and row
blocks (32 table rows), with masked residues that hold NaN, against the oracle; and of fipa_factor_project with its tables in
LDS at the edges of its groups of 16 residues."""
import numpy as np
import pytest

from oracle import factor_ref
from paper_2505_11580_amd import binding
from tests.test_gpu_factor import _bf16, check, make_tables

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,L,k,n_bins,n_pos,n_out,masked", [
    (1, 1, 1, 1, 0, 8, False), (1, 31, 2, 16, 15, 64, True), (1, 33, 3, 16, 33, 72, True), (2, 257, 2, 22, 33, 128, True),
    (1, 513, 2, 30, 95, 56, False), (3, 300, 1, 16, 111, 200, True)])
def test_factor_backward_tiles(B, L, k, n_bins, n_pos, n_out, masked):
    rng = np.random.default_rng(900 + L)
    idx = rng.integers(-1, L, size=(B, L, k))
    bins = np.where(idx < 0, -1, rng.integers(0, n_bins, size=(B, L, k)))
    mask = (rng.random((B, L)) > 0.3).astype(np.uint8) if masked else None
    if masked:
        mask[:, L // 3:L // 3 + 40] = 0  # whole tiles without a valid residue
    _check_backward(rng, idx, bins, n_bins, n_pos, n_out, mask)


def _check_backward(rng, idx, bins, n_bins, n_pos, n_out, mask):
    import torch
    B, L, k = idx.shape
    d_z = _bf16(rng.standard_normal((B, L, n_out)))
    want = factor_ref.factor_project_backward(idx, bins, d_z.float().numpy(), n_bins, n_pos, 1, mask)
    scale = float(np.abs(d_z.float().numpy()).sum(axis=(0, 1)).max())
    if mask is not None:
        d_z[torch.from_numpy(mask == 0)] = float("nan")
    f = dict(dtype=torch.float32, device="cuda:0")
    got = [torch.full((k, n_bins, n_out), float("nan"), **f),
           torch.full((k, n_pos, n_out), float("nan"), **f) if n_pos else None, torch.full((n_out,), float("nan"), **f)]
    binding.fipa_factor_project_backward(1, torch.from_numpy(idx.astype(np.int32)).cuda(), torch.from_numpy(bins.astype(np.int32)).cuda(),
                                         d_z.cuda(), torch.from_numpy(mask).cuda() if mask is not None else None, *got)
    torch.cuda.synchronize()
    for g, w in zip(got, want):
        if g is not None:
            # float32 sums against float64: a few 1e-7 of the largest sum of magnitudes (the bound of test_gpu_factor)
            assert np.abs(g.cpu().numpy().astype(np.float64) - w).max() <= 2e-6 * scale


# More than 64 tiles per wave (a second and third look at the masks), the middle ones without a residue that counts, the last one not whole; three
# and two stages, the most row blocks
@pytest.mark.parametrize("k,n_bins,n_pos", [(2, 4, 5), (1, 22, 91), (1, 16, 127)])
def test_factor_backward_windows(k, n_bins, n_pos):
    B, L = 5, 7001
    rng = np.random.default_rng(n_pos)
    idx = np.clip(np.arange(L)[None, :, None] + rng.integers(-80, 81, size=(B, L, k)), -1, L - 1)
    bins = np.where(idx < 0, -1, rng.integers(0, n_bins, size=(B, L, k)))
    mask = (rng.random(B * L) > 0.3).astype(np.uint8)
    mask[64 * 8 * 32:2 * 64 * 8 * 32] = 0  # every tile of the second look
    mask[64 * 8 * 32 - 3 * 32:64 * 8 * 32 - 32] = 0
    _check_backward(rng, idx, bins, n_bins, n_pos, 72, mask.reshape(B, L))


# Batches that end within a tile: one to three residues behind the last whole word of masks, the only valid ones
@pytest.mark.parametrize("L", [1, 2, 3, 5, 39, 294, 515])
def test_factor_backward_tail(L):
    rng = np.random.default_rng(L)
    idx = rng.integers(0, L, size=(1, L, 2))
    bins = rng.integers(0, 16, size=(1, L, 2))
    mask = np.zeros((1, L), np.uint8)
    mask[0, L // 4 * 4:] = 1
    _check_backward(rng, idx, bins, 16, 9, 64, mask)


@pytest.mark.parametrize("B,L,k,n_bins,n_pos,n_out,pos_mode", [
    (1, 1920, 33, 4, 5, 520, 1), (400, 5, 2, 3, 9, 520, 1), (1, 2049, 4, 16, 0, 512, 0), (3, 691, 64, 9, 25, 488, 1)])
def test_projection_groups(B, L, k, n_bins, n_pos, n_out, pos_mode):
    rng = np.random.default_rng(L)
    idx = rng.integers(-1, L, size=(B, L, k))
    idx[-1, L // 2:] = -1  # groups without neighbours
    bins = np.where(idx < 0, -1, rng.integers(0, n_bins, size=(B, L, k)))
    check(idx, bins, *make_tables(rng, k, n_bins, n_pos, n_out), pos_mode, "groups %d x %d" % (B, L))


def _in_lds(B, L, k, n_bins, n_pos, n_out):
    """Whether the projection runs with its tables in LDS: they fit, and each workgroup has enough residues to add."""
    groups = (n_out + 31) // 32
    parts = 256 // groups if groups < 256 else 1
    return 64 * (k * (n_bins + n_pos) + 1) + 1024 * k <= 160 * 1024 and B * L >= parts * (128 if k >= 16 else 136 if k >= 6 else 200)


# One order of sums, float32 to the nearest, whichever kernel adds them: the values of a sum in that order, rounded once
@pytest.mark.parametrize("B,L,k,n_bins,n_pos,n_out,pos_mode,in_lds", [
    (1, 1920, 33, 4, 5, 520, 1, True), (800, 5, 2, 3, 9, 520, 1, True), (1, 4097, 4, 16, 0, 512, 0, True),
    (3, 691, 64, 9, 13, 488, 1, True), (2, 2000, 10, 16, 33, 512, 1, True), (1, 700, 20, 16, 65, 512, 1, False),
    (1, 2177, 10, 16, 33, 512, 0, True), (1, 2175, 10, 16, 33, 512, 0, False), (1, 3200, 3, 16, 0, 512, 1, True)])
def test_projection_order(B, L, k, n_bins, n_pos, n_out, pos_mode, in_lds):
    import torch
    from tests.test_gpu_factor import run_gpu
    assert _in_lds(B, L, k, n_bins, n_pos, n_out) == in_lds
    rng = np.random.default_rng(L + k)
    idx = rng.integers(-1, L, size=(B, L, k))
    idx[-1, L // 2:L // 2 + 40] = -1  # groups without neighbours
    bins = np.where(idx < 0, -1, rng.integers(0, n_bins, size=(B, L, k)))
    e_bin, e_pos, bias = make_tables(rng, k, n_bins, n_pos, n_out)
    half = (n_pos - 1) // 2
    code = np.minimum(idx, n_pos - 1) if pos_mode == 0 else np.clip(idx - np.arange(L)[None, :, None], -half, half) + half
    want = np.broadcast_to(bias, (B, L, n_out)).astype(np.float32)
    for s in range(k):
        for table, at in ((e_bin, bins), (e_pos, code)):
            if table is not None:
                want += np.where((idx[..., s] >= 0)[..., None], table[s].float().numpy()[np.maximum(at[..., s], 0)], np.float32(0))
    got = run_gpu(idx, bins, e_bin, e_pos, bias, pos_mode).cpu()
    assert torch.equal(got, torch.from_numpy(want).to(torch.bfloat16))
