"""Performance cases: the calls that users of this library make, over the range of sizes they make them at.

Chains of residues with AlphaFold2's head shape (c = 16 scalars, 4 query and 8 value points per head), from the
shortest RNA to the longest proteins of the variable-length training sets; everything goes through the public
binding (`paper_2505_11580_amd.binding`), which is the C ABI with torch tensors.  Five kinds of pass:

  forward    fipa_forward, the inference call, float32 ("fp32", the accuracy mode) or bfloat16 inputs
  step       a training step of the attention core: fipa_forward and fipa_backward with FIPA_FLAG_KEEP_FORWARD
  packed     the same step on chains of different lengths stored back to back (the *_packed calls)
  module     a training step of the whole IPA module: fipa_module_forward and fipa_module_backward
  producers  pair factors from the frames: k nearest neighbours, both factor projections, both table gradients
"""
import math

import torch

from paper_2505_11580_amd import binding

C, PQ, PV = 16, 4, 8  # AlphaFold2's scalar width, query points and value points per head


def _case(kind, name=None, **kw):
    base = dict(kind=kind, B=1, L=256, H=12, cz=128, r=2, dtype="bf16", ragged=False)
    base.update(kw)
    if name is not None:
        base["name"] = name
    return base


def listed():
    return [
        # The smallest call: one short peptide in the accuracy mode, four heads.  Latency and launches.
        _case("forward", "fp32_peptide", B=1, L=64, H=4, cz=16, dtype="fp32"),
        # The accuracy mode at a real width: two chains, checked or refined in float32.
        _case("forward", "fp32_chains", B=2, L=1024, dtype="fp32"),
        # Inference on one short chain (an RNA of odd length, inside a sampling loop): latency.
        _case("forward", "fwd_short_rna", B=1, L=131),
        # Inference or evaluation on a batch of 512-residue crops.
        _case("forward", "fwd_crops", B=8, L=512),
        # The headline: two long chains of 2048 residues.
        _case("forward", "fwd_long", B=2, L=2048),
        # Factor rank 4 on a padded batch of very unequal long chains, with a mask.
        _case("forward", "fwd_rank4_ragged", B=4, L=8192, r=4, ragged=True, min_len=1024),
        # The highest factor rank (lifted width 1088), long chains.
        _case("forward", "fwd_rank8", B=2, L=2048, r=8),
        # Training on protein crops of 64 to 512 residues stored without padding.
        _case("packed", "step_packed_crops", B=32, L=512, min_len=64),
        # Training on long chains.
        _case("step", "step_long", B=2, L=4096),
        # Training at rank 4 on the ragged batch; the largest case.
        _case("step", "step_rank4_ragged", B=4, L=8192, r=4, ragged=True, min_len=1024),
        # Training of the whole module, single representation of width 256.
        _case("module", "step_module", B=2, L=2048, d_s=256),
        # The pair factors of the rank-4 batch from its frames, and the gradients of their tables.
        _case("producers", "producers_long", B=4, L=8192, r=4, ragged=True, min_len=1024, k=20, n_bins=16, n_pos=65),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the listed ranges; work is bounded by the listed case of the same kind."""
    kind = rng.choice(["fp32", "forward", "forward", "forward", "step", "packed", "module", "producers"])
    if kind == "fp32":
        L = _log_int(rng, 48, 1024)
        cz = rng.choice([16, 32, 64, 128])
        return _case("forward", B=rng.randint(1, 2), L=L, H=rng.choice([4, 8, 12]), cz=cz, r=rng.choice([1, 2]),
                     dtype="fp32", ragged=rng.random() < 0.3, min_len=max(1, L // 4))
    if kind == "forward":
        L = _log_int(rng, 100, 8192)
        cz, r = rng.choice([(128, 2), (128, 2), (128, 2), (64, 2), (32, 2), (128, 1), (128, 4), (128, 8), (64, 4)])
        most = 4 * 8192 * 8192 // (cz * r // 256 or 1)  # pairs per head
        B = max(1, min(rng.randint(1, 8), most // (L * L)))
        return _case("forward", B=B, L=L, H=rng.choice([8, 12, 12]), cz=cz, r=r, ragged=rng.random() < 0.4,
                     min_len=max(1, L // 4))
    if kind == "step":
        L = _log_int(rng, 256, 6000)
        cz, r = rng.choice([(128, 2), (128, 2), (64, 2), (128, 1), (128, 4)])
        B = max(1, min(rng.randint(1, 8), 2 * 6000 * 6000 // (L * L)))
        return _case("step", B=B, L=L, H=rng.choice([8, 12, 12]), cz=cz, r=r, ragged=rng.random() < 0.5,
                     min_len=max(1, L // 4))
    if kind == "packed":
        L = _log_int(rng, 150, 512)
        return _case("packed", B=rng.randint(4, 32), L=L, cz=rng.choice([64, 128]), r=2, min_len=max(16, L // 8))
    if kind == "module":
        L = _log_int(rng, 128, 2048)
        return _case("module", B=rng.randint(1, 4096 // L if L <= 2048 else 1) if L < 1024 else rng.randint(1, 2), L=L,
                     H=rng.choice([8, 12]), cz=128, r=rng.choice([1, 2]), d_s=rng.choice([128, 256, 384]),
                     ragged=rng.random() < 0.3, min_len=max(1, L // 4))
    L = _log_int(rng, 128, 8192)
    return _case("producers", B=rng.randint(1, 4), L=L, cz=128, r=rng.choice([1, 2, 4]), ragged=rng.random() < 0.5,
                 min_len=max(1, L // 8), k=rng.choice([10, 16, 20, 30]), n_bins=rng.choice([16, 22]),
                 n_pos=rng.choice([33, 65]))


def _lengths(case):
    """Chain lengths: L, or (ragged and packed batches) spread evenly over min_len .. L."""
    B, L = case["B"], case["L"]
    if not (case["ragged"] or case["kind"] == "packed"):
        return [L] * B
    lo = case["min_len"]
    return [lo + int((L - lo) * math.fmod((b + 1) * 0.6180339887498949, 1.0)) for b in range(B)]


def _frames(g, B, L):
    """Random rotations, and origins along a random walk of 3.8 A steps (a backbone)."""
    f = dict(device="cuda:0", generator=g)
    q = torch.randn(B, L, 4, **f)
    w, x, y, z = (q / q.norm(dim=-1, keepdim=True)).unbind(-1)
    rot = torch.stack([1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y),
                       2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x),
                       2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)], dim=-1)
    step = torch.randn(B, L, 3, **f)
    return rot.view(B, L, 3, 3).contiguous(), (3.8 * step / step.norm(dim=-1, keepdim=True)).cumsum(1).contiguous()


def prepare(case, seed):
    """Inputs, outputs and workspaces on the GPU, as a program holds them before the call."""
    B, L, H, cz, r, kind = (case[n] for n in ("B", "L", "H", "cz", "r", "kind"))
    lengths = _lengths(case)
    g = torch.Generator(device="cuda:0")
    g.manual_seed(seed)
    fp32 = case["dtype"] == "fp32"
    dt = torch.float32 if fp32 else torch.bfloat16
    f32 = dict(dtype=torch.float32, device="cuda:0")

    def normal(*shape, std=1.0, dtype=dt):
        return (std * torch.randn(*shape, device="cuda:0", generator=g)).to(dtype)

    desc = binding.make_desc(B, L, H, C, PQ, PV, cz, r, binding.FIPA_DTYPE_F32 if fp32 else binding.FIPA_DTYPE_BF16)
    rot, trans = _frames(g, B, L)
    mask = None
    if case["ragged"]:
        mask = (torch.arange(L, device="cuda:0")[None] < torch.tensor(lengths, device="cuda:0")[:, None]).to(torch.uint8)
    if kind == "producers":
        k, n_bins, n_pos, n = case["k"], case["n_bins"], case["n_pos"], r * cz
        i32 = dict(dtype=torch.int32, device="cuda:0")
        return dict(case=case, trans=trans, mask=mask,
                    idx=torch.empty(B, L, k, **i32), d2=torch.empty(B, L, k, **f32), bins=torch.empty(B, L, k, **i32),
                    sets=[dict(e_bin=normal(k, n_bins, n, std=k ** -0.5), e_pos=normal(k, n_pos, n, std=k ** -0.5),
                               bias=normal(n, dtype=torch.float32), z=torch.empty(B, L, n, dtype=dt, device="cuda:0"),
                               d_z=normal(B, L, n), d_e_bin=torch.empty(k, n_bins, n, **f32),
                               d_e_pos=torch.empty(k, n_pos, n, **f32), d_bias=torch.empty(n, **f32)) for _ in range(2)])

    std_z = r ** -0.25  # z_ij has unit variance
    dev = dict(rot=rot, trans=trans, mask=mask, z1=normal(B, L, r, cz, std=std_z), z2=normal(B, L, r, cz, std=std_z),
               w_b=normal(H, cz, std=cz ** -0.5, dtype=torch.float32),
               gamma=torch.nn.functional.softplus(normal(H, dtype=torch.float32)))
    if kind == "module":
        d_s = case["d_s"]
        n_in, n_cat = H * (3 * C + 3 * (2 * PQ + PV)), H * (cz + C + 4 * PV)
        dev.update(s=normal(B, L, d_s), w_in=normal(n_in, d_s, std=d_s ** -0.5), w_out=normal(d_s, n_cat, std=n_cat ** -0.5),
                   b_in=normal(n_in, std=0.1, dtype=torch.float32), b_out=normal(d_s, std=0.1, dtype=torch.float32),
                   s_out=torch.empty(B, L, d_s, **f32))
        grads = binding.alloc_module_grads(desc, d_s)
        dev["workspace"] = grads["workspace"]
        desc.flags = binding.FIPA_FLAG_KEEP_FORWARD
        return dict(case=case, desc=desc, dev=dev, grads=grads, up=normal(B, L, d_s, dtype=torch.float32))

    dev.update(q=normal(B, L, H, C), k=normal(B, L, H, C), v=normal(B, L, H, C), q_pts=normal(B, L, H, PQ, 3),
               k_pts=normal(B, L, H, PQ, 3), v_pts=normal(B, L, H, PV, 3))
    if kind == "forward":
        return dict(case=case, desc=desc, dev=dev, out=binding.alloc_outputs(desc))

    desc.flags = binding.FIPA_FLAG_KEEP_FORWARD
    up = dict(d_o=normal(B, L, H, C, dtype=torch.float32), d_o_pts=normal(B, L, H, PV, 3, dtype=torch.float32),
              d_o_pair=normal(B, L, H, cz, dtype=torch.float32))
    if kind == "step":
        dev.update(up)
        out, grads = binding.alloc_outputs(desc), binding.alloc_grads(desc)
        out["workspace"] = grads["workspace"]
        return dict(case=case, desc=desc, dev=dev, out=out, grads=grads)

    def pack(t):
        return torch.cat([t[b, :n] for b, n in enumerate(lengths)]).contiguous()

    cu = [0]
    for n in lengths:
        cu.append(cu[-1] + n)
    pk = {n: pack(dev[n]) for n in ("q", "k", "v", "q_pts", "k_pts", "v_pts", "rot", "trans", "z1", "z2")}
    total = cu[-1]
    out = dict(o=torch.empty(total, H, C, **f32), o_pts=torch.empty(total, H, PV, 3, **f32),
               o_pair=torch.empty(total, H, cz, **f32), lse=torch.empty(H * total, **f32))
    grads = {"d_" + n: torch.empty_like(pk[n]) for n in ("q", "k", "v", "q_pts", "k_pts", "v_pts", "z1", "z2")}
    grads.update(d_gamma=torch.empty(H, **f32), d_w_b=torch.empty(H, cz, **f32), d_rot=torch.empty(total, 3, 3, **f32),
                 d_trans=torch.empty(total, 3, **f32))
    ws = torch.empty(max(binding.packed_workspace_bytes(desc, cu)), dtype=torch.uint8, device="cuda:0")
    ins = [pk[n] for n in ("q", "k", "v", "q_pts", "k_pts", "v_pts", "rot", "trans", "z1", "z2")] + [dev["w_b"], dev["gamma"], None]
    return dict(case=case, desc=desc, cu=cu, ins=ins, up=[pack(up[n]) for n in ("d_o", "d_o_pts", "d_o_pair")],
                out=out, grads=grads, ws=ws)


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "forward":
        binding.forward(state["desc"], state["dev"], state["out"])
        return [state["out"][n] for n in ("o", "o_pts", "o_pair", "lse")]
    if kind == "step":
        binding.forward(state["desc"], state["dev"], state["out"])
        binding.backward(state["desc"], state["dev"], state["out"], state["grads"])
        return [state["out"][n] for n in ("o", "o_pts", "o_pair", "lse")] + [t for n, t in state["grads"].items() if n != "workspace"]
    if kind == "packed":
        out, grads = list(state["out"].values()), list(state["grads"].values())
        binding.fipa_forward_packed(state["desc"], state["cu"], *state["ins"], *out, state["ws"])
        binding.fipa_backward_packed(state["desc"], state["cu"], *state["ins"], *state["up"], *grads, state["ws"])
        return out + grads
    if kind == "module":
        binding.module_forward(state["desc"], case["d_s"], state["dev"])
        binding.module_backward(state["desc"], case["d_s"], state["dev"], state["up"], state["grads"])
        return [state["dev"]["s_out"]] + [t for n, t in state["grads"].items() if n != "workspace"]
    idx, bins = state["idx"], state["bins"]
    binding.fipa_knn_distogram(case["k"], case["n_bins"], 2.0, 22.0, state["trans"], state["mask"], idx, state["d2"], bins)
    outs = [idx, state["d2"], bins]
    for s in state["sets"]:
        binding.fipa_factor_project(1, idx, bins, s["e_bin"], s["e_pos"], s["bias"], s["z"])
        binding.fipa_factor_project_backward(1, idx, bins, s["d_z"], state["mask"], s["d_e_bin"], s["d_e_pos"], s["d_bias"])
        outs += [s[n] for n in ("z", "d_e_bin", "d_e_pos", "d_bias")]
    return outs


def work(case):
    """Inputs read once and outputs written once; flops of the minimal lifted widths over valid pairs."""
    B, L, H, cz, r, kind = (case[n] for n in ("B", "L", "H", "cz", "r", "kind"))
    lengths = _lengths(case)
    pairs = sum(n * n for n in lengths)
    rows = sum(lengths) if kind == "packed" else B * L
    if kind == "producers":
        k, n, t = case["k"], r * cz, case["k"] * (case["n_bins"] + case["n_pos"])
        nbytes = rows * (12 + 12 * k) + 2 * (2 * 2 * rows * n + 2 * t * n + 4 * t * n + 8 * n) + 2 * 2 * 8 * rows * k
        return dict(bytes=nbytes, flops=8 * pairs + 2 * 2 * 2 * k * rows * n)
    size = 4 if case["dtype"] == "fp32" else 2
    heads, factors, frames = H * (3 * C + 3 * (2 * PQ + PV)), 2 * r * cz, 48
    outs = 4 * H * (C + 3 * PV + cz)
    lift_qk, lift_v = C + 3 * PQ + 1 + r * cz, C + 3 * PV + r * cz
    fwd = 2 * (lift_qk + lift_v) * pairs * H
    bwd = 2 * (3 * lift_qk + 2 * lift_v) * pairs * H
    if kind == "forward":
        return dict(bytes=rows * (size * (heads + factors) + frames + outs + 4 * H), flops=fwd)
    if kind in ("step", "packed"):
        # inputs and frames, outputs, upstream gradients, gradients
        return dict(bytes=rows * (2 * size * (heads + factors) + 2 * frames + 2 * outs + 4 * H), flops=fwd + bwd)
    d_s, n_cat = case["d_s"], H * (cz + C + 4 * PV)
    weights = d_s * (heads + n_cat)
    return dict(bytes=rows * ((2 + 4 + 4 + 4) * d_s + 2 * size * factors + 2 * frames) + (2 + 4) * weights,
                flops=fwd + bwd + 3 * 2 * rows * weights)


def tolerance(case):
    """About four times the distance measured against a float64 evaluation of standard IPA on the same inputs
    (2-norm, and the largest single value): float32 3.6e-6 / 3.5e-5, bfloat16 forward 1.0e-3 / 1.5e-2, its
    gradients 3.6e-3 / 4.0e-2 (a head's d_gamma, a cancelling sum, up to 5e-3).  Pair factors are float32 sums
    rounded once to bfloat16: a sum in another order may fall on the other side of a rounding (half to one
    part in 256); neighbours, distances and bins are whole decisions and stay the same."""
    if case["kind"] == "producers":
        return {"rel": 1e-3, "max": 1e-2, "differ": 0.0}
    if case["dtype"] == "fp32":
        return {"rel": 1.5e-5, "max": 1.5e-4}
    if case["kind"] == "forward":
        return {"rel": 4e-3, "max": 6e-2}
    return {"rel": 1.5e-2, "max": 0.16}
