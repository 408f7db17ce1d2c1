"""GPU tests of the fp32 forward on split operands (three bf16 parts of every operand, six products) on the routes that lead to it:
accuracy and log-sum-exp at every width, unsplit and with 2 to 8 key ranges, and packed, static, captured and concurrent calls."""
import threading

import numpy as np
import pytest

from paper_2505_11580_amd import binding
from paper_2505_11580_amd import workloads as wl
from tests import gpu_util as gu
from tests.test_gpu_f32_shapes import _run_in
from tests.test_gpu_graph import _replay_and_compare
from tests.test_gpu_packed import PACKED_IN, packed_forward

pytestmark = pytest.mark.gpu

NAMES = gu.NAMES + ("lse",)
# max|gpu - float64| / max|float64|: below what two parts of one operand (in the place of three) would show, evaluated in float64 at 384 to
# 640 residues -- o 1.6e-6 (q, k, z2) to 6e-6 (v), o_pts 1.0e-5 (global points), o_pair 1.1e-6, lse 5.5e-7 -- and about twice what is seen
# (5.1e-7, 3.5e-6, 5.9e-7, 3.5e-7)
TIGHT = {"o": 1e-6, "o_pts": 7e-6, "o_pair": 1e-6, "lse": 5e-7}


def _inputs(**kw):
    return wl.make_inputs(0, **dict(dict(B=1, chain=True, trans_scale=0.3), **kw))


def log_sum_exp(inp):
    """[B, H, L]: of the softmax argument of Eq. 3 over the valid keys, in float64; 0 for masked rows."""
    f = {n: np.asarray(inp[n], np.float64) for n in ("q", "k", "q_pts", "k_pts", "rot", "trans", "z1", "z2", "w_b", "gamma")}
    B, L, H, c = f["q"].shape
    mask = np.ones((B, L), bool) if inp["mask"] is None else np.asarray(inp["mask"]) != 0
    out = np.zeros((B, H, L))
    for b in range(B):
        t = f["trans"][b] - f["trans"][b].mean(0)
        Q, K = (np.einsum("lxy,lhpy->lhpx", f["rot"][b], f[n][b]) + t[:, None, None] for n in ("q_pts", "k_pts"))
        for h in range(H):
            S = f["q"][b, :, h] @ f["k"][b, :, h].T / np.sqrt(c) + (f["z1"][b] * f["w_b"][h]).reshape(L, -1) @ f["z2"][b].reshape(L, -1).T
            for p in range(Q.shape[2]):
                for x in range(3):
                    S -= 0.5 * f["gamma"][h] * inp["w_C"] * np.subtract.outer(Q[:, h, p, x], K[:, h, p, x]) ** 2
            S = inp["w_L"] * S[:, mask[b]]
            if mask[b].any():
                m = S.max(1)
                out[b, h] = np.where(mask[b], m + np.log(np.exp(S - m[:, None]).sum(1)), 0.0)
    return out


@pytest.mark.parametrize("parts,kw", [
    (1, dict(L=530, B=4, H=10, cz=16, r=2)), (1, dict(L=512, B=11, H=3, cz=32, r=2, varlen=True, min_len=40)),
    (1, dict(L=450, B=11, H=3, cz=64, r=2)), (1, dict(L=384, B=4, H=11, cz=128, r=2, varlen=True, min_len=30)),
    (2, dict(L=512, B=2, H=12, cz=64, r=1)), (2, dict(L=1000, H=12, cz=16, r=8)), (2, dict(L=400, B=3, H=10, cz=128, r=2, varlen=True, min_len=1)),
    (3, dict(L=640, H=14, cz=32, r=1)), (4, dict(L=520, B=2, H=6, cz=128, r=1, varlen=True, min_len=90)), (8, dict(L=600, H=2, cz=128, r=2)),
    (8, dict(L=710, B=2, H=2, cz=8, r=4, varlen=True, min_len=1)), (8, dict(L=590, B=2, H=2, cz=16, r=4, varlen=True, min_len=40)),
    (8, dict(L=545, B=2, H=2, cz=64, r=2, varlen=True, min_len=1))])
def test_accuracy_and_log_sum_exp(parts, kw):
    inp = _inputs(**kw)
    B, L, H = inp["q"].shape[:3]
    tiles = B * H * ((L + 127) // 128)
    assert parts == (1 if tiles > 128 else min(256 // tiles, 8))
    want = dict(gu.oracle_forward_chunked(inp), lse=log_sum_exp(inp))
    got = gu.run_gpu(inp)
    least = (B * H * L * 76 * 4 + 255) // 256 * 256 + (16 * B + 255) // 256 * 256 + 256
    assert not np.array_equal(_run_in(inp, least)["o"], got["o"])  # (the fp32 matrix instructions)
    errs = {n: gu.rel_err(got[n], want[n]) for n in NAMES}
    print("fp32 split %s" % kw, {n: "%.2e" % e for n, e in errs.items()}, flush=True)
    for n in NAMES:
        assert errs[n] <= TIGHT[n], (n, errs)


def _outputs(desc, dev, workspace=None):
    import torch
    out = binding.alloc_outputs(desc)
    if workspace is not None:
        out["workspace"] = workspace
    for n in NAMES:
        out[n].fill_(float("nan"))
    binding.forward(desc, dev, out)
    torch.cuda.synchronize()
    return out


# Chain after chain in a workspace for the longest: every chain gives the bits of its own call there
@pytest.mark.parametrize("kw", [dict(B=4, L=640, H=3, cz=64, r=2, min_len=200), dict(B=3, L=1500, H=12, cz=128, r=2, min_len=60)])
def test_packed_chains(kw):
    import torch
    inp = _inputs(**dict(kw, varlen=True))
    got, cu, lengths, ws_bytes = packed_forward(inp)
    assert max(lengths) >= 512
    H = inp["dims"]["H"]
    ws = torch.empty(ws_bytes, dtype=torch.uint8, device="cuda:0")
    for b, n in enumerate(lengths):
        one = dict(inp, mask=None, dims=dict(inp["dims"], B=1, L=n), **{x: np.ascontiguousarray(inp[x][b:b + 1, :n]) for x in PACKED_IN})
        out = _outputs(*binding.upload(one), workspace=ws)
        for name in gu.NAMES:
            assert np.array_equal(got[name][cu[b]:cu[b + 1]], out[name][0].cpu().numpy()), (b, name)
        assert np.array_equal(got["lse"][H * cu[b]:H * cu[b + 1]], out["lse"].cpu().numpy().reshape(-1)), b


@pytest.mark.parametrize("kw", [dict(B=1, L=450, H=3, cz=64, r=2), dict(B=4, L=400, H=11, cz=128, r=2, varlen=True, min_len=50)])
def test_static_scratch_and_replays(kw):
    # the same bits as with a workspace of the query's size, eagerly and from a graph; several key ranges, and none
    import torch
    desc, dev = binding.upload(_inputs(**kw))
    want, out = _outputs(desc, dev), binding.alloc_outputs(desc)

    def static():
        binding.fipa_forward_static(desc, dev["q"], dev["k"], dev["v"], dev["q_pts"], dev["k_pts"], dev["v_pts"],
                                    dev["rot"], dev["trans"], dev["z1"], dev["z2"], dev["w_b"], dev["gamma"], dev["mask"],
                                    out["o"], out["o_pts"], out["o_pair"], out["lse"])

    static()
    torch.cuda.synchronize()
    for n in NAMES:
        assert torch.equal(out[n], want[n]), n
    _replay_and_compare(static, out, "static fp32 %s" % kw)
    _replay_and_compare(lambda: binding.forward(desc, dev, out), out, "fp32 %s" % kw)


def test_two_threads_two_streams():
    import torch
    jobs = [binding.upload(_inputs(**kw)) for kw in (dict(L=700, H=5, cz=64, r=2), dict(B=2, L=520, H=6, cz=128, r=2, varlen=True, min_len=60))]
    want = [_outputs(*job) for job in jobs]
    outs = [binding.alloc_outputs(job[0]) for job in jobs]
    streams, errors = [torch.cuda.Stream(), torch.cuda.Stream()], []

    def worker(job, out, stream):
        try:
            with torch.cuda.stream(stream):
                for _ in range(20):
                    binding.forward(*job, out)
            stream.synchronize()
        except Exception as e:  # surfaced in the main thread below
            errors.append(e)

    threads = [threading.Thread(target=worker, args=x) for x in zip(jobs, outs, streams)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    assert not errors, errors
    for out, w in zip(outs, want):
        for n in NAMES:
            assert torch.equal(out[n], w[n]), n
