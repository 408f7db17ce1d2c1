"""GPU parity of fipa_backward where its weights are kept in memory (r c_z = 256 and 512), at the edges of its tiles
(32 residues per block, 256 per tile, 128 per padded row group) and with more residues than the weights of one range of
queries (4096), against the CPU oracle (2e-2, the tolerance of every bf16 gradient test)."""
import pytest

from paper_2505_11580_amd import workloads as wl
from tests.test_gpu_backward import check_backward

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kw", [
    dict(L=1, H=1), dict(L=31), dict(L=33, r=4), dict(L=128, r=4), dict(L=129), dict(L=255, r=4), dict(L=257), dict(L=300, cz=64, r=8, H=1),
    dict(L=400, B=3, H=3, varlen=True, min_len=1), dict(L=300, B=5, H=1, r=4, varlen=True, min_len=20),
    dict(L=513, H=1, r=4)])
def test_backward_stored_weights(kw):
    kw = dict(dict(B=1, H=2, cz=128, r=2, trans_scale=0.3), **kw)
    check_backward(wl.make_inputs(4, **kw), "bwd stored %s" % kw)


@pytest.mark.parametrize("kw", [dict(L=4300, r=2), dict(L=4200, r=4, B=2, varlen=True, min_len=3000)])
def test_backward_two_query_ranges(kw):
    inp = wl.make_inputs(4, **dict(dict(B=1, H=1, cz=128), **kw))
    check_backward(inp, "bwd two ranges %s" % kw, samples=wl.select_rows(inp, 96))
