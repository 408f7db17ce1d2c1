"""GPU parity of fipa_module_forward (through the C ABI) against the module oracle
(oracle/module_ref.py): bf16 inputs and weights, fp32 accumulation, max|gpu - oracle| /
max|oracle| <= 2e-2 on the output representation."""
import numpy as np
import pytest

from oracle import module_ref
from paper_2505_11580_amd import binding
from paper_2505_11580_amd import workloads as wl
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu


def run_gpu_module(m):
    import torch
    desc, dev = binding.upload_module(m)
    dev["s_out"].fill_(float("nan"))
    binding.module_forward(desc, m["d_s"], dev)
    torch.cuda.synchronize()
    return dev["s_out"].cpu().numpy().astype(np.float64)


def check_module(m, label, rows=None, tol=2e-2):
    got = run_gpu_module(m)
    assert np.all(np.isfinite(got)), label
    want = module_ref.module_forward(m, rows=rows)
    if rows is not None:
        got = np.stack([got[b][rows[b]] for b in range(got.shape[0])])
    err = gu.rel_err(got, want)
    print(label, "s_out rel err %.2e" % err, flush=True)
    assert err <= tol, (label, err)


def test_module_small_shapes():
    # several row tiles with a ragged tail, d_s not a multiple of the column tile
    check_module(wl.make_module_inputs(1, d_s=48, B=2, L=200, H=4), "module L=200 d_s=48")
    check_module(wl.make_module_inputs(1, d_s=256, B=1, L=130, H=12, trans_scale=0.1), "module spread L=130 H=12")
    check_module(wl.make_module_inputs(1, d_s=64, B=1, L=96, H=2, cz=32, r=2), "module H=2 cz=32")
    # three query points: the point tensors of Eq. 1's result start at columns that are no multiples
    # of 8 and the result is 180 wide (pieces of an output row that straddle two tensors or its end)
    check_module(wl.make_module_inputs(1, d_s=64, B=1, L=70, H=2, Pq=3), "module Pq=3")
    # rank 4 (lifted width 576: the two-window attention kernel with its epilogue on the registers)
    check_module(wl.make_module_inputs(3, d_s=64, B=2, L=200, H=2, min_len=50), "module r=4 ragged")


def test_module_masked_rows_receive_the_bias():
    m = wl.make_module_inputs(1, d_s=64, B=3, L=160, H=4, varlen=True, min_len=20)
    check_module(m, "module varlen")
    got = run_gpu_module(m)
    for b, ln in enumerate(m["lengths"]):
        assert np.array_equal(got[b, int(ln):], np.broadcast_to(m["b_out"].astype(np.float64), got[b, int(ln):].shape))
    m["b_in"], m["b_out"] = None, None
    check_module(m, "module varlen, no biases")


def test_module_workload2_sampled_rows():
    m = wl.make_module_inputs(2, d_s=256)
    check_module(m, "module cfg2 sampled rows", rows=wl.select_rows(m, 48))


def test_module_rejects_unsupported_width():
    m = wl.make_module_inputs(1, d_s=40, B=1, L=64, H=4)
    with pytest.raises(binding.FipaError):
        binding.upload_module(m)


MODULE_GRADS = (("d_s", "ds"), ("d_w_in", "dw_in"), ("d_b_in", "db_in"), ("d_w_out", "dw_out"), ("d_b_out", "db_out"),
                ("d_z1", "dz1"), ("d_z2", "dz2"), ("d_gamma", "dgamma"), ("d_w_b", "dw_b"), ("d_rot", "drot"),
                ("d_trans", "dtrans"))


def check_module_backward(m, label, seed=0, tol=2e-2):
    import torch
    rng = np.random.default_rng(seed)
    d = m["dims"]
    up = rng.standard_normal((d["B"], d["L"], m["d_s"])).astype(np.float32)
    desc, dev = binding.upload_module(m)
    grads = binding.alloc_module_grads(desc, m["d_s"])
    for n, _ in MODULE_GRADS:
        grads[n].fill_(float("nan"))
    binding.module_backward(desc, m["d_s"], dev, torch.from_numpy(up).to("cuda:0"), grads)
    torch.cuda.synchronize()
    want = module_ref.module_backward(m, up)
    errs = {}
    for n, o in MODULE_GRADS:
        got = grads[n].float().cpu().numpy().astype(np.float64)
        assert np.all(np.isfinite(got)), (label, n)
        errs[n] = gu.rel_err(got, want[o])
    print(label, {k: "%.1e" % v for k, v in errs.items()}, flush=True)
    for n, _ in MODULE_GRADS:
        assert errs[n] <= tol, (label, n, errs[n])


def test_module_backward_small_shapes():
    # B*L = 130 is neither a multiple of the row tile nor of the K chunk of the weight gradients
    check_module_backward(wl.make_module_inputs(4, d_s=48, B=1, L=130, H=4, trans_scale=0.3), "module bwd L=130 d_s=48")
    check_module_backward(wl.make_module_inputs(4, d_s=64, B=2, L=96, H=2, cz=32, r=2), "module bwd B=2 L=96 cz=32")
    check_module_backward(wl.make_module_inputs(4, d_s=64, B=1, L=150, H=2, cz=128, r=4, trans_scale=0.5), "module bwd rank 4")


def test_module_backward_masked_and_without_biases():
    m = wl.make_module_inputs(4, d_s=64, B=2, L=160, H=4, varlen=True, min_len=30, trans_scale=0.5)
    check_module_backward(m, "module bwd varlen")
    m["b_in"], m["b_out"] = None, None
    check_module_backward(m, "module bwd varlen, no biases")


@pytest.mark.parametrize("d_s,kw", [
    (16, dict(B=1, L=9, H=4)), (80, dict(B=1, L=64, H=4, cz=32)), (48, dict(B=3, L=43, H=4, Pq=3)), (144, dict(B=1, L=65, H=8, Pq=3, cz=16))])
def test_module_backward_transposed_tiles(d_s, kw):
    # rows and columns at the edges of the 64 x 64 tiles; three query points: pieces of a gathered row that straddle two tensors
    # (not one residue alone: its weight is constant, d_gamma zero and without a relative error; the other gradients agree there)
    check_module_backward(wl.make_module_inputs(4, d_s=d_s, trans_scale=0.3, **kw), "module bwd d_s=%d %s" % (d_s, kw))
