"""The C-ABI library loads and exports what include/fipa.h declares; host-side argument
checks answer with error codes before anything touches a device (no GPU needed)."""
import ctypes
import os
import re

import pytest

from paper_2505_11580_amd import binding

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def declared_functions():
    text = open(os.path.join(ROOT, "include", "fipa.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(fipa_[a-z_]+)\s*\(", text)))


def test_header_symbols_are_exported():
    lib = binding.lib()
    names = declared_functions()
    assert set(names) == set(binding.EXPORTS)
    for n in names:
        assert getattr(lib, n) is not None


def test_version_and_status_strings():
    assert binding.lib().fipa_version() >= 100
    for code in (0, -1, -2, -3, -4, -5):
        assert binding.status_string(code) != "unknown status"
    assert binding.status_string(-99) == "unknown status"


def test_workspace_is_affine_in_length():
    # linear memory in L (Section 2.3): equal steps in L give equal steps in bytes
    # (every width but r c_z = 1024, whose forward keeps its weights in memory)
    for dtype, r in ((binding.FIPA_DTYPE_BF16, 1), (binding.FIPA_DTYPE_BF16, 2), (binding.FIPA_DTYPE_BF16, 4), (binding.FIPA_DTYPE_F32, 2)):
        sizes = [binding.workspace_bytes(binding.make_desc(1, L, 12, 16, 4, 8, 128, r, dtype))[0]
                 for L in (1024, 2048, 3072, 4096, 8192)]
        steps = [sizes[1] - sizes[0], sizes[2] - sizes[1], sizes[3] - sizes[2], (sizes[4] - sizes[3]) // 4]
        assert len(set(steps)) == 1 and steps[0] > 0, sizes


@pytest.mark.parametrize("cz,r", [(128, 1), (128, 2), (64, 4), (128, 4), (128, 8)])
def test_workspaces_grow_with_the_length(cz, r):
    # chains that run one after the other share a workspace of the longest one's size, so no shorter chain may need more:
    # around every size at which the number of stored query rows changes
    lengths = sorted({1, 127, 128, 129, 256, 384, 4000, 4096, 4097, 9000, 20000, 65536, 100000, 1000000, 2000000}
                     | {x + e for rows in range(256, 4097, 256) for x in ((1 << 30) // rows // 128 * 128,) for e in (-256, -128, 0, 128, 256)})
    for H in (1, 12):
        last = (0, 0)
        for L in lengths:
            if H * (L + 128) >= 1 << 31:
                continue
            now = binding.workspace_bytes(binding.make_desc(1, L, H, 16, 4, 8, cz, r, binding.FIPA_DTYPE_BF16))
            assert now[0] >= last[0] and now[1] >= last[1], (H, L, now, last)
            last = now


def test_packed_chain_by_chain_workspace_holds_every_chain():
    desc = binding.make_desc(2, 262400, 1, 16, 4, 8, 128, 2, binding.FIPA_DTYPE_BF16)
    desc.flags = binding.FIPA_FLAG_PACKED_PER_CHAIN
    bwd = binding.packed_workspace_bytes(desc, [0, 262400, 524544])[1]
    for L in (262400, 262144):
        one = binding.make_desc(1, L, 1, 16, 4, 8, 128, 2, binding.FIPA_DTYPE_BF16)
        assert binding.workspace_bytes(one)[1] <= bwd, L


def test_f32_workspace_holds_the_record_of_the_kernel_that_runs():
    # AlphaFold2's heads: k | Kg | v, Vg at the widths that have an exact kernel; at any other the generic kernel's record
    # with Qg (12 floats) behind it
    B, L, H = 2, 64, 4
    for cz, r in ((16, 1), (16, 2), (64, 1), (128, 1), (128, 2), (128, 4), (16, 3), (80, 1), (32, 3), (64, 3), (128, 3), (12, 4)):
        DZ = r * cz
        record = 76 if DZ in (16, 32, 64, 128, 256, 512) else 88
        need = binding.workspace_bytes(binding.make_desc(B, L, H, 16, 4, 8, cz, r, binding.FIPA_DTYPE_F32))[0]
        assert need == B * H * L * record * 4 + 2 * 256, (cz, r, need)


def test_f32_split_workspace_asks_for_what_is_used():
    # key blocks of 32 residues (three bf16 planes of z2, 17408 bytes per head) and, up to 128 tiles of 128 queries, the sums of
    # two to eight key ranges of each: the most that a length up to the batch's takes, which is never less for a longer one
    def need(B, L, H, cz, r):
        return binding.workspace_bytes(binding.make_desc(B, L, H, 16, 4, 8, cz, r, binding.FIPA_DTYPE_F32))[0]

    def blocks(B, L, H, DZ):
        kb = (L + 31) // 32
        return 2 * 256 + B * kb * (192 * DZ + H * 17408)

    unit = 128 * (44 + 128) * 4
    assert need(1, 384, 4, 128, 2) == blocks(1, 384, 4, 256) + 12 * 6 * unit     # 12 tiles, 12 key blocks
    assert need(2, 2048, 12, 128, 2) == blocks(2, 2048, 12, 256) + 120 * 2 * unit  # at 640 residues
    assert need(12, 512, 12, 128, 2) == blocks(12, 512, 12, 256)                 # 144 tiles from the shortest chain on
    for B, H, cz, r in ((1, 12, 128, 2), (2, 12, 16, 2), (2, 8, 128, 1), (20, 12, 128, 2), (1, 4, 64, 1)):
        sizes = [need(B, L, H, cz, r) for L in range(16, 3000, 31)]
        assert sizes == sorted(sizes), (B, H, cz, r)


def test_bad_descriptions_are_rejected_on_the_host():
    lib = binding.lib()
    sz = ctypes.c_size_t(0)
    bad = binding.make_desc(1, 0, 4, 16, 4, 8, 16, 2, binding.FIPA_DTYPE_F32)
    assert lib.fipa_workspace_bytes(ctypes.byref(bad), ctypes.byref(sz), None) == binding.FIPA_ERR_INVALID_ARG
    bad = binding.make_desc(1, 64, 4, 16, 4, 8, 16, 2, 7)
    assert lib.fipa_workspace_bytes(ctypes.byref(bad), ctypes.byref(sz), None) == binding.FIPA_ERR_INVALID_ARG
    odd = binding.make_desc(1, 64, 4, 16, 4, 8, 24, 2, binding.FIPA_DTYPE_BF16)  # r*cz = 48
    assert lib.fipa_workspace_bytes(ctypes.byref(odd), ctypes.byref(sz), None) == binding.FIPA_ERR_UNSUPPORTED
    assert lib.fipa_workspace_bytes(None, ctypes.byref(sz), None) == binding.FIPA_ERR_INVALID_ARG


def test_forward_argument_checks_need_no_device():
    lib = binding.lib()
    d = binding.make_desc(1, 64, 4, 16, 4, 8, 16, 2, binding.FIPA_DTYPE_F32)
    nulls = [None] * 17
    assert lib.fipa_forward(ctypes.byref(d), *nulls, None, 0, None) == binding.FIPA_ERR_INVALID_ARG
    fake = [ctypes.c_void_p(0x1000)] * 17
    fake[12] = None  # mask may be NULL
    assert lib.fipa_forward(ctypes.byref(d), *fake, ctypes.c_void_p(0x1000), 0, None) == binding.FIPA_ERR_WORKSPACE
    mis = list(fake)
    mis[0] = ctypes.c_void_p(0x1004)
    assert lib.fipa_forward(ctypes.byref(d), *mis, ctypes.c_void_p(0x1000), 1 << 30, None) == binding.FIPA_ERR_ALIGNMENT
    with pytest.raises(binding.FipaError):
        binding.workspace_bytes(binding.make_desc(1, -5, 4, 16, 4, 8, 16, 2, 0))


def test_packed_forward_argument_checks_need_no_device():
    lib = binding.lib()
    d = binding.make_desc(3, 64, 4, 16, 4, 8, 16, 2, binding.FIPA_DTYPE_BF16)
    fake = [ctypes.c_void_p(0x1000)] * 17
    ws = ctypes.c_void_p(0x1000)

    def call(cu, size=1 << 30):
        arr = (ctypes.c_int32 * len(cu))(*cu)
        return lib.fipa_forward_packed(ctypes.byref(d), arr, *fake, ws, size, None)

    assert lib.fipa_forward_packed(ctypes.byref(d), None, *fake, ws, 1 << 30, None) == binding.FIPA_ERR_INVALID_ARG
    assert call([1, 10, 20, 30]) == binding.FIPA_ERR_INVALID_ARG      # does not start at 0
    assert call([0, 10, 5, 30]) == binding.FIPA_ERR_INVALID_ARG       # decreasing
    assert call([0, 10, 80, 90]) == binding.FIPA_ERR_INVALID_ARG      # a chain longer than desc->L
    assert call([0, 10, 20, 30], size=0) == binding.FIPA_ERR_WORKSPACE
    assert call([0, 0, 0, 0]) == binding.FIPA_OK                      # only empty chains: nothing to enqueue


def test_packed_workspace_query_and_backward_argument_checks_need_no_device():
    lib = binding.lib()
    d = binding.make_desc(4, 900, 12, 16, 4, 8, 128, 2, binding.FIPA_DTYPE_BF16)
    one = binding.make_desc(1, 900, 12, 16, 4, 8, 128, 2, binding.FIPA_DTYPE_BF16)
    even = binding.make_desc(4, 700, 12, 16, 4, 8, 128, 2, binding.FIPA_DTYPE_BF16)
    # chains of similar lengths: one set of launches, workspace of the padded batch (at the longest chain) + offsets
    fwd, bwd = binding.packed_workspace_bytes(d, [0, 700, 1300, 1900, 2500])
    pf, pb = binding.workspace_bytes(even)
    assert pf < fwd <= pf + 1024 and pb < bwd <= pb + 1024
    # one dominant chain: chain after chain, workspace of the longest chain alone (+ the per-chain gamma / w_b sums)
    fwd, bwd = binding.packed_workspace_bytes(d, [0, 900, 940, 973, 1043])
    assert fwd == binding.workspace_bytes(one)[0]
    assert binding.workspace_bytes(one)[1] < bwd <= binding.workspace_bytes(one)[1] + 4 * 4 * (12 + 12 * 128) + 1024
    # the flag forces it
    d.flags = binding.FIPA_FLAG_PACKED_PER_CHAIN
    per = binding.make_desc(1, 700, 12, 16, 4, 8, 128, 2, binding.FIPA_DTYPE_BF16)
    assert binding.packed_workspace_bytes(d, [0, 700, 1300, 1900, 2500])[0] == binding.workspace_bytes(per)[0]
    d.flags = 0
    with pytest.raises(binding.FipaError):
        binding.packed_workspace_bytes(d, [0, 950, 1000, 1100, 1200])  # a chain longer than desc->L
    fake = [ctypes.c_void_p(0x1000)] * 28
    fake[12] = None  # mask
    cu = (ctypes.c_int32 * 5)(0, 700, 1300, 1900, 2500)
    ws = ctypes.c_void_p(0x1000)
    assert lib.fipa_backward_packed(ctypes.byref(d), cu, *fake, ws, 0, None) == binding.FIPA_ERR_WORKSPACE
    assert lib.fipa_backward_packed(ctypes.byref(d), None, *fake, ws, 1 << 40, None) == binding.FIPA_ERR_INVALID_ARG
    only_rot = list(fake)
    only_rot[27] = None  # d_trans without d_rot's partner
    assert lib.fipa_backward_packed(ctypes.byref(d), cu, *only_rot, ws, 1 << 40, None) == binding.FIPA_ERR_INVALID_ARG
    f32 = binding.make_desc(4, 900, 12, 16, 4, 8, 16, 2, binding.FIPA_DTYPE_F32)
    assert lib.fipa_backward_packed(ctypes.byref(f32), cu, *fake, ws, 1 << 40, None) == binding.FIPA_ERR_UNSUPPORTED


def test_knn_distogram_argument_checks_need_no_device():
    lib = binding.lib()
    p = ctypes.c_void_p(0x1000)

    def call(B=2, L=50, k=20, n_bins=16, d_min=2.0, d_max=22.0, trans=p, idx=p):
        return lib.fipa_knn_distogram(B, L, k, n_bins, d_min, d_max, trans, None, idx, p, p, None)

    assert call(L=0) == binding.FIPA_ERR_INVALID_ARG
    assert call(k=0) == binding.FIPA_ERR_INVALID_ARG
    assert call(n_bins=1) == binding.FIPA_ERR_INVALID_ARG
    assert call(d_min=5.0, d_max=5.0) == binding.FIPA_ERR_INVALID_ARG
    assert call(d_min=-1.0) == binding.FIPA_ERR_INVALID_ARG
    assert call(trans=None) == binding.FIPA_ERR_INVALID_ARG
    assert call(k=65) == binding.FIPA_ERR_UNSUPPORTED
    assert call(idx=ctypes.c_void_p(0x1002)) == binding.FIPA_ERR_ALIGNMENT


def test_factor_project_argument_checks_need_no_device():
    lib = binding.lib()
    p = ctypes.c_void_p(0x1000)

    def call(B=2, L=50, k=20, n_bins=16, n_pos=65, pos_mode=1, n_out=256, idx=p, e_pos=p, z=p):
        return lib.fipa_factor_project(B, L, k, n_bins, n_pos, pos_mode, n_out, idx, p, p, e_pos, None, z, None)

    assert call(L=0) == binding.FIPA_ERR_INVALID_ARG
    assert call(n_bins=0) == binding.FIPA_ERR_INVALID_ARG
    assert call(pos_mode=2) == binding.FIPA_ERR_INVALID_ARG
    assert call(n_pos=64) == binding.FIPA_ERR_INVALID_ARG          # offsets need an odd number of rows
    assert call(n_pos=0) == binding.FIPA_ERR_INVALID_ARG           # a table without rows
    assert call(e_pos=None) == binding.FIPA_ERR_INVALID_ARG        # rows without a table
    assert call(z=None) == binding.FIPA_ERR_INVALID_ARG
    assert call(n_out=100) == binding.FIPA_ERR_UNSUPPORTED
    assert call(k=65) == binding.FIPA_ERR_UNSUPPORTED
    assert call(z=ctypes.c_void_p(0x1008)) == binding.FIPA_ERR_ALIGNMENT
    assert call(idx=ctypes.c_void_p(0x1002)) == binding.FIPA_ERR_ALIGNMENT


def test_factor_project_backward_argument_checks_need_no_device():
    lib = binding.lib()
    p = ctypes.c_void_p(0x1000)

    def call(B=2, L=50, k=20, n_bins=16, n_pos=65, pos_mode=1, n_out=256, d_z=p, d_e_pos=p, d_e_bin=p):
        return lib.fipa_factor_project_backward(B, L, k, n_bins, n_pos, pos_mode, n_out, p, p, d_z, None, d_e_bin, d_e_pos,
                                                None, None)

    assert call(B=0) == binding.FIPA_ERR_INVALID_ARG
    assert call(d_z=None) == binding.FIPA_ERR_INVALID_ARG
    assert call(d_e_pos=None) == binding.FIPA_ERR_INVALID_ARG
    assert call(n_pos=0) == binding.FIPA_ERR_INVALID_ARG
    assert call(n_pos=64) == binding.FIPA_ERR_INVALID_ARG
    assert call(n_out=100) == binding.FIPA_ERR_UNSUPPORTED
    assert call(n_bins=4096) == binding.FIPA_ERR_UNSUPPORTED      # the table slice does not fit LDS
    assert call(d_e_bin=ctypes.c_void_p(0x1004)) == binding.FIPA_ERR_ALIGNMENT


def test_stage_timer_argument_checks_need_no_device():
    lib = binding.lib()
    assert lib.fipa_profile_begin_every(10, 0) == binding.FIPA_ERR_INVALID_ARG
    assert lib.fipa_profile_begin_every(0, 1) == binding.FIPA_ERR_INVALID_ARG
    assert lib.fipa_profile_begin_every(5000, 1) == binding.FIPA_ERR_INVALID_ARG
    assert lib.fipa_profile_end(None, None) == binding.FIPA_ERR_INVALID_ARG  # timing is not active


def test_bench_refuses_more_than_one_gpu():
    # one GPU only: the benchmark says so instead of running on a subset
    import os
    import subprocess
    import sys
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    res = subprocess.run([sys.executable, os.path.join(root, "bench.py"), "--gpus", "2"], capture_output=True, text=True)
    assert res.returncode == 2
    assert "single-GPU" in res.stderr


def test_stored_weights_add_at_most_32_gib_to_a_workspace():
    # against what the calls take that form the weights again in every product (r c_z = 256: sizes of such a build; forward:
    # that of a call too small to store weights, times the length)
    for B, L, again in ((64, 2048, 10636756224), (64, 4096, 21273511168), (8, 16384, 10636755456), (128, 8192, 85094042112),
                        (1, 1000000, 81157169664)):
        bwd = binding.workspace_bytes(binding.make_desc(B, L, 12, 16, 4, 8, 128, 2, binding.FIPA_DTYPE_BF16))[1]
        assert again <= bwd <= again + (32 << 30), (B, L, bwd)
    for L in (65536, 262144, 1000000):
        small = binding.workspace_bytes(binding.make_desc(1, 128, 12, 16, 4, 8, 128, 8, binding.FIPA_DTYPE_BF16))[0]
        fwd = binding.workspace_bytes(binding.make_desc(1, L, 12, 16, 4, 8, 128, 8, binding.FIPA_DTYPE_BF16))[0]
        assert fwd <= (L // 128 + 1) * small + (32 << 30) + L * 128, (L, fwd)


def test_backward_asks_for_the_weights_that_it_stores():
    # where dS' alone is stored (r c_z = 128, 256): 2 bytes per query row (all, or 8192) and key, and 160 MiB at most for tiles in parts,
    # beside what is affine in the length (sizes of shapes without weights, times the length)
    for r in (1, 2):
        base = binding.workspace_bytes(binding.make_desc(2, 128, 12, 16, 4, 8, 128, r, binding.FIPA_DTYPE_BF16))[1]
        for L in (1024, 2048, 4096, 8192, 16384):
            bwd = binding.workspace_bytes(binding.make_desc(2, L, 12, 16, 4, 8, 128, r, binding.FIPA_DTYPE_BF16))[1]
            weights = 24 * min(L, 8192) * L * 2
            assert weights < bwd <= weights + (160 << 20) + L // 128 * base, (r, L, bwd)
