"""Which kernels the cases of the GPU tests reach (host only: the choice is made
from the plan's sizes), so that a change of the choice cannot leave a kernel
untested."""
import ctypes

import pytest
import torch

import paper_2407_16847_amd as splat
import test_gpu_slices as gpu

F32, BF16 = torch.float32, torch.bfloat16


def _acsr(kind, params, L):
    return splat.Acsr(splat.Pattern.named(kind, params, L), columns=True)


def _reached(call, dtype, cases, d, heads=None):
    """{(route, sets)}; cases without the heads are taken with each of `heads`."""
    out = set()
    for kind, params, L, *h in cases:
        a = _acsr(kind, params, L)
        for n in heads or h:
            out.add(splat.route(a, call, dtype, 1, n, d))
    return out


def _names(*args, **kw):
    return {r for r, _ in _reached(*args, **kw)}


@pytest.mark.parametrize("d", [64, 128])
def test_fp32_cases(d):
    assert _names("sparse_mhsa_fwd", F32, gpu.CASES, d) == {"rows", "slices"}
    for call in ("rsddmm", "rspmm"):
        assert _names(call, F32, gpu.STEPS, d) == {"rows", "slices"}
    assert _names("sparse_mhsa_unfused", F32, gpu.CHAIN, d) == {"chain", "steps"}


@pytest.mark.parametrize("d", [64, 128])
def test_fp32_column_major_cases(d):
    """The column-major R-SpMM takes the row-major call's kernel, and needs
    masks whose columns are single runs; stepped columns are addressed apart."""
    cols = [c for c in gpu.STEPS if _acsr(*c[:3]).info()["columns"] == 1]
    for kinds in ({"window", "blocked", "strided_local", "full"}, {"dilated"}):
        assert _names("rspmm", F32, [c for c in cols if c[0] in kinds], d) == {"rows", "slices"}


def test_non_finite_cases():
    for call in ("sparse_mhsa_fwd", "rspmm"):
        assert _names(call, F32, gpu.NON_FINITE, 64) == {"rows", "slices"}
    assert _names("sparse_mhsa_unfused", F32, gpu.NON_FINITE, 64) == {"chain", "steps"}
    # all four results are compared: every mask has the column-major layout
    assert all(_acsr(*c[:3]).info()["columns"] == 1 for c in gpu.NON_FINITE)


@pytest.mark.parametrize("d", [64, 128])
def test_bf16_cases(d):
    masks = [c[:3] for c in gpu.CASES[:-1]]
    for call in ("rsddmm", "rspmm"):
        assert "slices" in _names(call, BF16, masks, d, heads=[2])
        assert "tiles" in _names(call, BF16, masks, d, heads=[400])
    assert _names("sparse_mhsa_unfused", BF16, gpu.CHAIN, d) == {"chain", "steps"}
    sets = {("tiles", 1), ("tiles", 2)} | ({("tiles", 4)} if d == 64 else set())
    assert _reached("sparse_mhsa_fwd", BF16, gpu.SETS, d, heads=[3]) == sets


# launches away from the lines, with the faster side as measured (the time of
# the other in brackets, us)
MEASURED = [
    # the chain in one kernel against its steps, bf16
    ("sparse_mhsa_unfused", BF16, "window", {"w": 8}, 8192, 32, 128, "steps"),       # 137 (161)
    ("sparse_mhsa_unfused", BF16, "window", {"w": 2}, 8192, 100, 64, "steps"),       # 238 (307)
    ("sparse_mhsa_unfused", BF16, "window", {"w": 128}, 1024, 64, 64, "chain"),      # 45 (134)
    ("sparse_mhsa_unfused", BF16, "window", {"w": 8}, 8192, 1, 128, "chain"),
    ("sparse_mhsa_unfused", BF16, "window_global", {"w": 3, "n_global": 3}, 9000, 60, 64, "chain"),
    ("sparse_mhsa_unfused, column-major", BF16, "window", {"w": 8}, 8192, 32, 128, "chain"),
    ("sparse_mhsa_unfused_noalloc", BF16, "window", {"w": 4}, 12000, 57, 64, "chain"),   # 197 (209)
    ("sparse_mhsa_unfused", BF16, "window", {"w": 4}, 12000, 57, 64, "steps"),       # 209 (256)
    ("sparse_mhsa_unfused_noalloc", BF16, "dilated", {"w": 8, "dilation": 5}, 16288, 37, 128, "steps"),
    # ... and fp32, d = 128
    ("sparse_mhsa_unfused", F32, "window", {"w": 1}, 925, 19, 128, "steps"),         # 29 (41)
    ("sparse_mhsa_unfused", F32, "full", {}, 1523, 18, 128, "steps"),                # 336 (426)
    ("sparse_mhsa_unfused", F32, "window_global", {"w": 11, "n_global": 2}, 1638, 48, 128, "chain"),  # 194 (257)
    ("sparse_mhsa_unfused, column-major", F32, "full", {}, 968, 7, 128, "chain"),    # 84 (123)
    # R-SDDMM, bf16, over slices or tiles
    ("rsddmm", BF16, "full", {}, 384, 402, 64, "tiles"),                             # 58 (75)
    ("rsddmm", BF16, "full", {}, 1024, 64, 64, "slices"),                            # 70 (98)
    ("rsddmm", BF16, "window_global", {"w": 512, "n_global": 64}, 4096, 16, 64, "slices"),  # 91 (178)
    # R-SpMM, bf16, over slices or tiles; `columns` handles
    ("rspmm", BF16, "dilated", {"w": 51, "dilation": 4}, 947, 28, 64, "tiles"),      # 14.1 (19.1)
    ("rspmm", BF16, "dilated", {"w": 8, "dilation": 6}, 180, 2, 64, "tiles"),        # 5.1 (5.7)
    ("rspmm", BF16, "dilated", {"w": 40, "dilation": 3}, 4106, 3, 128, "slices"),    # 13 (27), columns
    # sets of wavefronts in the fused bf16 forward
    ("sparse_mhsa_fwd", BF16, "window_global", {"w": 3, "n_global": 27}, 686, 104, 128, "tiles:1"),
    ("sparse_mhsa_fwd", BF16, "window_global", {"w": 17, "n_global": 57}, 4217, 75, 128, "tiles:1"),
    ("sparse_mhsa_fwd", BF16, "window_global", {"w": 31, "n_global": 99}, 633, 107, 64, "tiles:1"),
    ("sparse_mhsa_fwd", BF16, "full", {}, 777, 16, 128, "tiles:2"),
    ("sparse_mhsa_fwd", BF16, "window_global", {"w": 512, "n_global": 64}, 4096, 16, 64, "tiles:4"),
]


@pytest.mark.parametrize("call,dtype,kind,params,L,heads,d,want", MEASURED)
def test_the_faster_side_is_taken(call, dtype, kind, params, L, heads, d, want):
    got, sets = splat.route(_acsr(kind, params, L), call, dtype, 1, heads, d)
    assert (f"{got}:{sets}" if ":" in want else got) == want


def test_rspmm_of_handles_without_columns():
    """One-tile groups, and a chip's slices exceeded by short full masks, take
    the tile kernel: 4.2 (5.4), 10.4 (14.4); blocked 64 the slices: 5.9 (7.7)."""
    for kind, params, L, heads, want in (("dilated", {"w": 13, "dilation": 6}, 151, 25, "tiles"),
                                         ("full", {}, 218, 113, "tiles"),
                                         ("blocked", {"block": 64}, 1024, 16, "slices")):
        a = splat.Acsr(splat.Pattern.named(kind, params, L))
        assert splat.route(a, "rspmm", BF16, 1, heads, 64) == (want, 1)


def test_argument_checks():
    a = _acsr("window", {"w": 5}, 65)
    lib, r = splat.load(), ctypes.c_int32(7)
    bad = [(None, 0, 0, 1, 1, 64, ctypes.byref(r)), (a.handle, 0, 0, 1, 1, 64, None),
           (a.handle, 6, 0, 1, 1, 64, ctypes.byref(r)), (a.handle, -1, 0, 1, 1, 64, ctypes.byref(r)),
           (a.handle, 0, 2, 1, 1, 64, ctypes.byref(r)), (a.handle, 0, 0, 0, 1, 64, ctypes.byref(r))]
    for args in bad:
        assert lib.splat_debug_route(*args, None) == 1          # INVALID_ARG
    assert lib.splat_debug_route(a.handle, 0, 0, 1, 1, 96, ctypes.byref(r), None) == 2   # UNSUPPORTED
    assert r.value == 7                                          # nothing written
    assert lib.splat_debug_route(a.handle, 0, 0, 1, 1, 64, ctypes.byref(r), None) == 0
