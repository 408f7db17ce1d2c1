"""GPU parity of the forward that keeps its weights in memory (r c_z = 512 and 1024): edges of its tiles (32 keys, 256
queries, 128 padded rows), rows whose softmax reference is raised many times, several ranges of query rows, and the
static entry point where the scratch does not hold the weights, against the CPU oracle (2e-2, the bf16 tolerance)."""
import numpy as np
import pytest

from paper_2505_11580_amd import binding
from paper_2505_11580_amd import workloads as wl
from tests import gpu_util as gu
from tests.test_zz_no_alloc import OUT, _both

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kw", [
    dict(L=1, H=1), dict(L=31), dict(L=33, r=8), dict(L=129), dict(L=257), dict(L=257, r=8, H=1),
    dict(L=300, cz=64, r=8), dict(L=300, cz=256, r=2, H=1), dict(L=140, cz=256, r=4, H=1), dict(L=140, cz=512, r=1, H=1),
    dict(L=600, H=1, B=3, varlen=True, min_len=1), dict(L=600, r=8, H=1, B=3, varlen=True, min_len=1),
    dict(L=300, c=8, Pq=2, Pv=3)])
def test_forward_stored_weights(kw):
    inp = wl.make_inputs(3, **dict(dict(B=1, H=2, cz=128, r=4, varlen=False, trans_scale=0.3), **kw))
    gu.check(inp, label="fwd stored %s" % kw)


@pytest.mark.parametrize("r", [4, 8])
def test_forward_stored_weights_raised_references(r):
    # a chain in random order: the nearest residue of a row lies in any block, hundreds of log2 units above the first ones
    inp = wl.make_inputs(3, B=1, L=700, H=2, cz=128, r=r, varlen=False)
    perm = np.random.default_rng(5).permutation(700)
    for n in ("rot", "trans"):
        inp[n] = np.ascontiguousarray(inp[n][:, perm])
    inp["k_pts"] = np.ascontiguousarray(inp["k_pts"] * 0 + 8.0)  # keys far from their own queries
    gu.check(inp, label="fwd stored, raised references r=%d" % r)


def test_forward_stored_weights_several_ranges():
    # 192 pairs: 1024 query rows per range
    inp = wl.make_inputs(3, B=16, L=1100, H=12, cz=128, r=4, min_len=900)
    gu.check(inp, rows=wl.select_rows(inp, 12), label="fwd stored, two ranges")


def test_static_scratch_too_small_for_the_weights():
    inp = wl.make_inputs(3, B=1, L=2048, H=12, cz=128, r=4, varlen=False)
    desc, _ = binding.upload(inp)
    assert binding.workspace_bytes(desc)[0] > binding.STATIC_SCRATCH_BYTES
    ref, got = _both(inp)
    for n in OUT:
        # two roundings of the same sums: each within the bf16 tolerance of the exact result
        assert gu.rel_err(got[n], ref[n]) <= 2e-2, n
