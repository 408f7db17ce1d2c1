"""GPU parity of the fp32 mode at the edges of its tiles (16 query rows, 16 keys, 16 feature columns), for every
width class of its attention kernel and for head shapes outside AlphaFold2's, against the CPU oracle (1e-4)."""
import numpy as np
import pytest

from paper_2505_11580_amd import workloads as wl
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kw", [
    dict(L=1), dict(L=15), dict(L=16, H=1), dict(L=17, B=2), dict(L=65, cz=8, r=2), dict(L=129, cz=32, r=2, H=2),
    dict(L=70, cz=128, r=1, H=2), dict(L=40, cz=128, r=4, H=1),  # one width class each
    dict(L=300, B=3, H=12, cz=16), dict(L=257, B=6, H=12, cz=16, r=1, varlen=True, min_len=1),  # 32-row workgroups
    # generic: odd widths, scalars wider than a chunk, wide records, many query points, rows that are no multiple of 16 bytes
    dict(L=50, c=7, Pq=3, Pv=5, cz=9, r=3, H=2), dict(L=33, c=40, Pq=1, Pv=1, cz=20, r=1, H=2),
    dict(L=20, c=300, Pq=2, Pv=10, cz=50, r=1, H=1), dict(L=90, c=16, Pq=4, Pv=8, cz=12, r=2, H=2),
    dict(L=40, c=8, Pq=50, Pv=2, cz=16, r=2, H=1), dict(L=30, c=500, Pq=2, Pv=20, cz=16, r=1, H=1),
    dict(L=300, B=2, H=12, c=8, Pq=2, Pv=3, cz=8, r=2, varlen=True, min_len=100),
    # AlphaFold2's heads at widths without an exact kernel (48, 80, 96, 192, 384; 32-row workgroups in the last)
    dict(L=37, cz=16, r=3, H=2), dict(L=50, cz=80, r=1), dict(L=131, B=2, cz=32, r=3, varlen=True, min_len=20),
    dict(L=65, cz=64, r=3, H=2), dict(L=33, cz=128, r=3, H=1), dict(L=161, B=8, H=12, cz=16, r=3, varlen=True, min_len=9)])
def test_f32_shapes(kw):
    kw = dict(dict(B=1, H=4, chain=True, trans_scale=0.3), **kw)
    gu.check(wl.make_inputs(0, **kw), label="fp32 %s" % kw)


# the longest chains of the one-launch form (256 residues, 64 from r c_z = 256 on), with and without a mask, and one residue more
@pytest.mark.parametrize("kw", [
    dict(L=256, cz=16, B=2, varlen=True, min_len=30), dict(L=257, cz=32, r=2), dict(L=256, cz=128, r=1, H=2),
    dict(L=128, cz=128, r=2, H=2, B=2, varlen=True, min_len=1), dict(L=129, cz=128, r=2, H=2), dict(L=64, cz=128, r=4, H=1),
    dict(L=64, cz=64, r=4, H=5, B=2, varlen=True, min_len=3), dict(L=65, cz=64, r=4, H=5),
    dict(L=65, cz=128, r=4, H=1, B=2, varlen=True, min_len=20)])
def test_f32_one_launch_edges(kw):
    kw = dict(dict(B=1, H=3, chain=True, trans_scale=0.3), **kw)
    gu.check(wl.make_inputs(0, **kw), label="fp32 %s" % kw)


def test_f32_lse_and_far_keys():
    # log-sum-exp against the oracle, at full chain geometry (logits of several thousand) with a scattered mask
    inp = wl.make_inputs(0, L=150, H=3, cz=64, chain=True)
    inp["mask"] = (np.random.default_rng(3).random((1, 150)) < 0.7).astype(np.uint8)
    gu.check(inp, label="fp32 scattered mask, chain")
    from tests.test_gpu_f32_split import log_sum_exp
    assert gu.rel_err(gu.run_gpu(inp)["lse"], log_sum_exp(inp)) <= gu.TOL["fp32"]


# split operands: every width, one residue past a block and a tile, blocks and whole tiles without a valid residue, key ranges in one and
# several parts (fewer and more than 128 tiles), columns of one rank narrower than 64
@pytest.mark.parametrize("kw", [
    dict(L=512, cz=32, r=1, H=2), dict(L=600, cz=8, r=4, H=2, B=2, varlen=True, min_len=1),
    dict(L=384, cz=128, r=2, H=1), dict(L=417, cz=64, r=2, H=2, B=2, varlen=True, min_len=1), dict(L=513, cz=64, r=1, H=3),
    dict(L=545, cz=16, r=4, H=2, B=2, varlen=True, min_len=40), dict(L=385, cz=8, r=16, H=1), dict(L=161, B=4, H=6, cz=32, r=8),
    dict(L=170, B=8, H=12, cz=256, r=1, varlen=True, min_len=1), dict(L=520, B=3, H=12, cz=128, r=1, varlen=True, min_len=100)])
def test_f32_split_operands(kw):
    kw = dict(dict(B=1, H=4, chain=True, trans_scale=0.3), **kw)
    gu.check(wl.make_inputs(0, **kw), label="fp32 split %s" % kw)


def test_f32_split_operands_in_every_workspace():
    # the space that the query asks for, without the split key range's, and without the key blocks (fp32 matrix instructions)
    import torch
    from paper_2505_11580_amd import binding
    inp = wl.make_inputs(0, B=1, L=545, H=3, cz=64, r=2, chain=True, trans_scale=0.3)
    inp["mask"] = (np.random.default_rng(5).random((1, 545)) < 0.6).astype(np.uint8)
    desc, dev = binding.upload(inp)
    want = gu.oracle_forward_chunked(inp)
    full = binding.workspace_bytes(desc)[0]
    # 15 tiles of 128 queries, eight key ranges; key blocks of 32 residues: three planes of z2, and 17408 bytes per head
    tiles, unit, least = 15, 128 * (44 + 64) * 4, (3 * 545 * 76 * 4 + 255) // 256 * 256 + 2 * 256
    blocks = 2 * 256 + 18 * 3 * 64 * 128 + 3 * 18 * 17408
    assert full == blocks + 8 * tiles * unit
    for size in (full, full - 256, blocks + 2 * tiles * unit, blocks, blocks - 256, least):
        out = binding.alloc_outputs(desc)
        for n in gu.NAMES:
            out[n].fill_(float("nan"))
        out["workspace"] = torch.empty(size, dtype=torch.uint8, device="cuda:0")
        binding.forward(desc, dev, out)
        torch.cuda.synchronize()
        for n in gu.NAMES:
            assert gu.rel_err(out[n].cpu().numpy().astype(np.float64), want[n]) <= gu.TOL["fp32"], (size, n)
    out["workspace"] = torch.empty(least - 256, dtype=torch.uint8, device="cuda:0")
    with pytest.raises(binding.FipaError):
        binding.forward(desc, dev, out)


def test_f32_split_operands_without_a_valid_residue():
    inp = wl.make_inputs(0, B=2, L=520, H=2, cz=128, r=1, chain=True, trans_scale=0.3)
    inp["mask"] = np.ones((2, 520), np.uint8)
    want = gu.oracle_forward_chunked(inp)  # (which wants a valid key in every element)
    inp["mask"][0] = 0
    got = gu.run_gpu(inp)
    for n in gu.NAMES:
        assert not got[n][0].any(), n
        assert gu.rel_err(got[n][1], want[n][1]) <= gu.TOL["fp32"], n
    assert not got["lse"][0].any()


def _run_in(inp, size):
    import torch
    from paper_2505_11580_amd import binding
    desc, dev = binding.upload(inp)
    out = binding.alloc_outputs(desc)
    for n in gu.NAMES + ("lse",):
        out[n].fill_(float("nan"))
    out["workspace"] = torch.empty(size or binding.workspace_bytes(desc)[0], dtype=torch.uint8, device="cuda:0")
    binding.forward(desc, dev, out)
    torch.cuda.synchronize()
    return {n: out[n].cpu().numpy().astype(np.float64) for n in gu.NAMES + ("lse",)}


# Infinite operands, on split operands (in several parts, and unsplit) as on the fp32 matrix instructions, which the least workspace gives
@pytest.mark.parametrize("kw", [dict(L=530, H=4, cz=64, r=2), dict(L=710, H=2, cz=16, r=2), dict(L=385, H=2, cz=128, r=2),
                                dict(L=512, B=11, H=3, cz=32, r=2)])
def test_f32_split_operands_infinities(kw):
    kw = dict(dict(B=1, chain=False, trans_scale=0.05), **kw)
    B, L, H, cz, r = (kw[n] for n in ("B", "L", "H", "cz", "r"))
    inp = wl.make_inputs(0, **kw)
    inf, h = np.float32(np.inf), H - 1
    inp["mask"] = (np.random.default_rng(1).random((B, L)) < 0.9).astype(np.uint8)
    inp["mask"][0, [7, 9, 11, 20, 30, 40]] = 1
    inp["mask"][0, 50] = 0
    inp["q"][0, :, h, 3] = -np.abs(inp["q"][0, :, h, 3]) - 0.1
    inp["k"][0, 7, h, 3] = inf               # a logit of -inf: left out
    inp["v"][0, 9, h, 2] = inf               # an infinite sum
    inp["v_pts"][0, 11, 0, 3, 1] = -inf
    inp["q"][0, 20, 0, 1] = inf              # one row
    inp["v"][0, 30, 0, 4] = 3e38
    inp["k"][0, 40, 0, 5] = 3.4e38
    inp["v"][0, 50] = inf                    # a masked residue
    if B > 1:
        inp["z2"][B - 1, 60, 0, 5] = -inf    # a logit and a value
        inp["mask"][B - 1, 60] = 1
    least = (B * H * L * 76 * 4 + 255) // 256 * 256 + (16 * B + 255) // 256 * 256 + 256
    want, got = _run_in(inp, least), _run_in(inp, None)
    for n in gu.NAMES + ("lse",):
        w, g = want[n], got[n]
        odd = ~np.isfinite(w)
        assert np.array_equal(w[odd], g[odd], equal_nan=True) and np.isfinite(g[~odd]).all(), n
        huge = np.abs(w) > 1e30  # (3e38 weighted: to the precision of a float)
        for part in (~odd & ~huge, ~odd & huge):
            if part.any():
                assert np.abs(g[part] - w[part]).max() <= 1e-5 * np.abs(w[part]).max(), n
    assert np.isinf(got["o"][0, 0, h, 2]) and np.isfinite(got["o"][0, 0, h, :2]).all()
    assert not got["o"][0, 20, 0].any() and not got["o_pair"][0, 20, 0].any()
