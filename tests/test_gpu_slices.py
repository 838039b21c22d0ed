"""The 32-row slice kernels and the choice between them and their alternatives.

Sizes where they can go wrong: tiles of fewer than 32 and of 33 .. 63 keys,
gathered tiles, slices with empty tiles, a ragged last slice, more than 64
tiles in a group, launches on both sides of the row/slice choice.  Tolerances
as in test_gpu_parity (fp32: 1e-5 of each row's largest reference value).
"""
import math

import numpy as np
import pytest
import torch

import workloads
from oracle import attention as oa
from oracle import masks as om

pytestmark = pytest.mark.gpu

F32_REL = 1e-5


def _row_err(O, ref):
    O = O.double().cpu().numpy()
    assert np.isfinite(O).all()
    num, den = np.abs(O - ref).max(axis=-1), np.abs(ref).max(axis=-1)
    assert (num[den == 0] == 0).all()
    return float((num[den > 0] / den[den > 0]).max())


def _qkv(L, d, heads, seed, dtype="f32"):
    w = workloads.Workload("slices", 1, heads, L, d, dtype, workloads.make_pattern("full"), 1.0, seed)
    return workloads.make_qkv(w)


CASES = [
    ("full", {}, 31, 3), ("full", {}, 33, 2), ("full", {}, 97, 40), ("full", {}, 128, 16),
    ("window", {"w": 5}, 65, 1), ("window", {"w": 16}, 700, 20), ("window", {"w": 150}, 321, 2),
    ("blocked", {"block": 33}, 300, 12), ("dilated", {"w": 33, "dilation": 3}, 400, 12),
    ("strided_local", {"local": 40, "stride": 33}, 500, 12),
    ("strided_local", {"local": 4, "stride": 64}, 600, 2),
    ("window_global", {"w": 3, "n_global": 1}, 4200, 1),
]
# heads enough for the fp32 R-SpMM over slices.  Which kernels the lists of this
# file reach is checked without a GPU in test_host_routes.py.
STEPS = CASES + [
    ("full", {}, 97, 120), ("blocked", {"block": 33}, 300, 100),
    ("dilated", {"w": 100, "dilation": 3}, 700, 40),
    ("strided_local", {"local": 40, "stride": 33}, 500, 100),
]
NON_FINITE = [CASES[5], CASES[6], CASES[7], CASES[8], CASES[10], STEPS[-3], STEPS[-2], STEPS[-1]]


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("kind,params,L,heads", CASES)
def test_fused_f32(gpu_lib, kind, params, L, heads, d):
    splat = gpu_lib
    print(f"[gpu] fused f32 {kind} {params} L={L} heads={heads} d={d}", flush=True)
    Q, K, V = _qkv(L, d, heads, L + d)
    M = om.dense_mask(kind, params, L)
    a = splat.Acsr(splat.Pattern.named(kind, params, L))
    for scale in (1.0 / math.sqrt(d), -0.3, 0.0):
        ref = oa.masked_attention(Q[:, :2], K[:, :2], V[:, :2], M, scale)
        O = splat.sparse_mhsa_fwd(a, Q.cuda(), K.cuda(), V.cuda(), scale)
        torch.cuda.synchronize()
        # a score's fp32 error is relative to the sum of its terms' magnitudes,
        # which |scale| * sqrt(d) scales against the default scale
        bound = F32_REL * max(1.0, abs(scale) * math.sqrt(d))
        assert _row_err(O[:, :2], ref) <= bound, scale


@pytest.mark.parametrize("where", ["K", "V"])
@pytest.mark.parametrize("value", [math.inf, -math.inf, math.nan])
@pytest.mark.parametrize("kind,params,L,heads", NON_FINITE)
def test_f32_rows_see_only_their_keys(gpu_lib, kind, params, L, heads, value, where):
    """A key with an infinity or a NaN changes only the rows that have it."""
    splat = gpu_lib
    d, scale = 64, 0.125
    print(f"[gpu] non-finite {where} {value} {kind} {params} L={L}", flush=True)
    Q, K, V = _qkv(L, d, heads, 5)
    j = L // 2
    (K if where == "K" else V)[:, :, j, 3] = value
    M = om.dense_mask(kind, params, L)
    a = splat.Acsr(splat.Pattern.named(kind, params, L), columns=True)
    Qd, Kd, Vd = Q.cuda(), K.cuda(), V.cuda()
    P = splat.row_softmax(a, splat.rsddmm(a, Qd, Kd, scale))
    outs = {"fused": splat.sparse_mhsa_fwd(a, Qd, Kd, Vd, scale),
            "steps": splat.rspmm(a, P, Vd),
            "columns": splat.rspmm_colmajor(a, splat.transpose_colmajor(a, P), Vd),
            "unfused": splat.sparse_mhsa_unfused(a, Qd, Kd, Vd, scale)[0]}
    torch.cuda.synchronize()
    clean = torch.from_numpy(~M[:, j])
    (K if where == "K" else V)[:, :, j, 3] = 0.0
    ref = oa.masked_attention(Q[:, :2], K[:, :2], V[:, :2], M, scale)
    for name, O in outs.items():
        O = O.cpu()
        assert _row_err(O[:, :2, clean], ref[:, :, clean.numpy()]) <= F32_REL, name
        if where == "V":   # the other rows: feature 3 only
            assert not torch.isfinite(O[:, :, ~clean, 3]).any(), name
            assert torch.isfinite(O[:, :, ~clean, 4:]).all(), name


# a wavefront per row (68 keys of one head), slices, and slices redone row by
# row: V of key 199, which the compared rows lack, is infinite
@pytest.mark.parametrize("kind,params,L,heads,rows,redo", [
    ("full", {}, 68, 1, 68, False), ("full", {}, 68, 64, 68, False),
    ("window", {"w": 100}, 200, 4, 99, False), ("window", {"w": 100}, 200, 4, 99, True)])
def test_fused_f32_first_scores_minus_infinity(gpu_lib, kind, params, L, heads, rows, redo):
    """Rows whose first 64 keys score -inf return the softmax over the others;
    rows whose keys all do return NaN."""
    splat = gpu_lib
    d, scale = 64, 0.125
    print(f"[gpu] fused f32 -inf scores {kind} {params} L={L} heads={heads} redo={redo}", flush=True)
    Q, K, V = _qkv(L, d, heads, 41)
    M = om.dense_mask(kind, params, L)
    seen = M.copy()
    seen[:, :64] = False
    Q[..., 0] = K[..., 0] = 0.0
    ref = oa.masked_attention(Q[:, :2], K[:, :2], V[:, :2], seen, scale)
    Q[..., 0], K[:, :, :64, 0] = 1.0, -math.inf
    if redo:
        V[:, :, 199] = math.inf
    a = splat.Acsr(splat.Pattern.named(kind, params, L))
    Qd, Kd, Vd = Q.cuda(), K.cuda(), V.cuda()
    Kn = Kd.clone()
    Kn[..., 0] = -math.inf
    none = splat.sparse_mhsa_fwd(a, Qd, Kn, Vd, scale)
    for O in (torch.empty_like(Qd), Qd):   # a tensor of its own, and Q's place
        splat.sparse_mhsa_fwd(a, Qd, Kd, Vd, scale, O=O)
        torch.cuda.synchronize()
        assert _row_err(O[:, :2, :rows], ref[:, :, :rows]) <= F32_REL
    assert torch.isnan(none).all()


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("big", [1e37, 2e36])
def test_fused_f32_large_values(gpu_lib, big, d):
    """V near fp32's end: keys that score 7 binary orders above a wavefront's
    first unit, one in the second unit of each wavefront, outgrow fp32 before
    the division by the sum (big = 2e36: only over all four), the result does
    not."""
    splat = gpu_lib
    L, heads, scale = 300, 12, 1.0 / math.sqrt(d)
    print(f"[gpu] fused f32 V up to {big} d={d}", flush=True)
    _, K, V = _qkv(L, d, heads, 31)
    Q, K = torch.ones_like(K), 1e-3 * K
    for j in (130, 170, 200, 230):
        K[:, :, j] += 7.0 * math.log(2.0) / (scale * d)
        V[:, :, j, :8] *= big / V[:, :, j, :8].abs().amax(-1, keepdim=True)
    a = splat.Acsr(splat.Pattern.full(L))
    ref = oa.masked_attention(Q[:, :2], K[:, :2], V[:, :2], om.dense_mask("full", {}, L), scale)
    Qd = Q.cuda()
    for O in (torch.empty_like(Qd), Qd):   # a tensor of its own, and Q's place
        splat.sparse_mhsa_fwd(a, Qd, K.cuda(), V.cuda(), scale, O=O)
        torch.cuda.synchronize()
        assert _row_err(O[:, :2], ref) <= F32_REL


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("heads", [1, 24])
def test_rspmm_f32_large_values(gpu_lib, heads, d):
    """Values that cancel key by key, near fp32's end: key after key the sums
    stay finite, in another order they do not.  One head takes a wavefront per
    row, 24 the slices; both layouts."""
    splat = gpu_lib
    L = 300
    print(f"[gpu] rspmm f32 V = +-3e38 heads={heads} d={d}", flush=True)
    a = splat.Acsr(splat.Pattern.full(L), columns=True)
    P = torch.ones(1, heads, a.nnz, device="cuda")
    V = torch.full((1, heads, L, d), 3e38, device="cuda")
    V[:, :, 1::2] *= -1
    O = splat.rspmm(a, P, V)
    Oc = splat.rspmm_colmajor(a, P, V)
    torch.cuda.synchronize()
    assert (O == 0).all() and (Oc == 0).all()


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("kind,params,L,heads", STEPS)
def test_steps_f32(gpu_lib, kind, params, L, heads, d):
    splat = gpu_lib
    print(f"[gpu] steps f32 {kind} {params} L={L} heads={heads} d={d}", flush=True)
    scale = 1.0 / math.sqrt(d)
    Q, K, V = _qkv(L, d, heads, L + 2 * d)
    M = om.dense_mask(kind, params, L)
    a = splat.Acsr(splat.Pattern.named(kind, params, L), columns=True)
    S = splat.rsddmm(a, Q.cuda(), K.cuda(), scale)
    P = splat.row_softmax(a, S)
    O = splat.rspmm(a, P, V.cuda())
    if a.info()["columns"] == 1:
        Oc = splat.rspmm_colmajor(a, splat.transpose_colmajor(a, P), V.cuda())
        assert torch.equal(Oc, O)
    torch.cuda.synchronize()
    ref, _, _ = oa.masked_attention(Q[:, :2], K[:, :2], V[:, :2], M, scale, want_csr=True)
    assert _row_err(O[:, :2], ref) <= F32_REL
    m = torch.from_numpy(M)
    for h in (0, heads - 1):
        x = Q[0, h].double() @ K[0, h].double().t() * scale
        mag = Q[0, h].double().abs() @ K[0, h].double().abs().t() * scale
        assert float(((S[0, h].cpu().double() - x[m]).abs() / mag[m]).max()) <= F32_REL


# (dtype, alpha): the row-major and the column-major branch; windows of few
# keys over many heads and short fp32 sequences take the chain of single steps,
# the others one kernel
CHAIN = [("full", {}, 33, 2), ("window", {"w": 5}, 65, 1), ("window", {"w": 2}, 4096, 40),
         ("window", {"w": 150}, 321, 2), ("blocked", {"block": 33}, 300, 12),
         ("dilated", {"w": 33, "dilation": 3}, 400, 12),
         ("strided_local", {"local": 40, "stride": 33}, 500, 12),
         ("strided_local", {"local": 4, "stride": 64}, 600, 2),
         ("window_global", {"w": 3, "n_global": 1}, 4200, 1)]


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("kind,params,L,heads", CHAIN)
def test_chain(gpu_lib, kind, params, L, heads, dtype, d):
    """O and the P left in S against the oracle; Pt is exactly P's column-major
    copy; the allocation-free call gives the same O."""
    splat = gpu_lib
    print(f"[gpu] chain {kind} {params} L={L} heads={heads} d={d} {dtype}", flush=True)
    scale = 1.0 / math.sqrt(d)
    Q, K, V = _qkv(L, d, heads, L + 3 * d, dtype)
    Qd, Kd, Vd = Q.cuda(), K.cuda(), V.cuda()
    M = om.dense_mask(kind, params, L)
    n = min(heads, 2)
    ref, _, Pref = oa.masked_attention(Q[:, :n], K[:, :n], V[:, :n], M, scale, want_csr=True)
    a = splat.Acsr(splat.Pattern.named(kind, params, L), columns=True)
    col = a.info()["columns"] == 1
    for alpha in (2.0, 0.0):
        S = torch.full((1, heads, a.nnz), float("nan"), device="cuda")
        Pt = torch.full_like(S, float("nan"))
        O, used = splat.sparse_mhsa_unfused(a, Qd, Kd, Vd, scale, alpha=alpha, S=S, Pt=Pt,
                                            out_dtype=torch.float32)
        torch.cuda.synchronize()
        assert used == (col and alpha == 0.0)
        if dtype == "f32":
            assert _row_err(O[:, :n], ref) <= F32_REL
        else:   # P enters the products with 16 bits, sums in fp32
            assert float(np.abs(O[:, :n].cpu().numpy() - ref).max()) <= 1e-4
        assert float(np.abs(S[:, :n].cpu().numpy() - Pref).max()) <= 1e-5
        if used:
            src = torch.from_numpy(om.colmajor_source(M))
            assert torch.equal(Pt.cpu(), S.cpu()[:, :, src])
        if heads * a.nnz * 8 + 256 <= splat.NOALLOC_SCRATCH_BYTES:
            On, _ = splat.sparse_mhsa_unfused_noalloc(a, Qd, Kd, Vd, scale, alpha=alpha,
                                                      out_dtype=torch.float32)
            torch.cuda.synchronize()
            assert torch.equal(On, O)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("noalloc", [False, True])
@pytest.mark.parametrize("onto", ["Q", "K"])
def test_chain_output_over_an_input(gpu_lib, onto, noalloc, dtype):
    """O may take the place of Q or K (the steps are done with both before O
    is written): the same result as in a tensor of its own."""
    splat = gpu_lib
    L, d, heads = 1000, 64, 16
    q, k, v = (x.cuda() for x in _qkv(L, d, heads, 21, dtype))
    a = splat.Acsr(splat.Pattern.window(L, 100))
    call = splat.sparse_mhsa_unfused_noalloc if noalloc else splat.sparse_mhsa_unfused
    ref = call(a, q, k, v, 0.125)[0]
    O = call(a, q, k, v, 0.125, O=q if onto == "Q" else k)[0]
    torch.cuda.synchronize()
    # two orders of the same sums: fp32 rounding, for bf16 one step of O's
    tol = 2.0 ** -8 if dtype == "bf16" else F32_REL
    err = (O.double() - ref.double()).abs().amax(-1) / ref.double().abs().amax(-1)
    assert float(err.max()) <= 2 * tol


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("where", ["front", "back"])
def test_chain_output_inside_scores(gpu_lib, where, dtype):
    """On the column-major branch the last step reads Pt and V only, so O may
    lie inside S: the same O as in a tensor of its own."""
    splat = gpu_lib
    L, d, heads = 1000, 64, 16
    q, k, v = (x.cuda() for x in _qkv(L, d, heads, 22, dtype))
    a = splat.Acsr(splat.Pattern.window(L, 100), columns=True)
    ref, used = splat.sparse_mhsa_unfused(a, q, k, v, 0.125, alpha=0.0)
    S = torch.empty(1, heads, a.nnz, device="cuda")
    flat = S.view(-1).view(q.dtype)
    O = (flat[:q.numel()] if where == "front" else flat[-q.numel():]).view(q.shape)
    splat.sparse_mhsa_unfused(a, q, k, v, 0.125, alpha=0.0, S=S, O=O)
    torch.cuda.synchronize()
    assert used
    tol = 2.0 ** -8 if dtype == "bf16" else F32_REL   # two orders of the same sums
    err = (O.double() - ref.double()).abs().amax(-1) / ref.double().abs().amax(-1)
    assert float(err.max()) <= 2 * tol


def test_chain_without_keys(gpu_lib):
    """An empty mask and empty rows: O = 0, nothing else is written."""
    splat = gpu_lib
    L, d = 70, 64
    Q, K, V = (x.cuda() for x in _qkv(L, d, 2, 3))
    for terms in ([], [dict(row_lo=40, lo_i=1, lo_c=-3, hi_i=1)]):
        a = splat.Acsr(splat.Pattern.from_terms(L, terms))
        for dt in (torch.float32, torch.bfloat16):
            q, k, v = (x.to(dt) for x in (Q, K, V))
            for O, _ in (splat.sparse_mhsa_unfused(a, q, k, v, 0.1),
                         splat.sparse_mhsa_unfused_noalloc(a, q, k, v, 0.1)):
                torch.cuda.synchronize()
                assert (O[:, :, :40] == 0).all()
                assert (O[:, :, 40:] == 0).all() if not terms else torch.isfinite(O).all()


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("heads", [2, 400])
@pytest.mark.parametrize("kind,params,L", [c[:3] for c in CASES[:-1]])
def test_steps_bf16(gpu_lib, kind, params, L, heads, d):
    """Two heads take the slices but for the shortest masks, 400 the 128-row tile
    kernels but for some short or thin ones."""
    splat = gpu_lib
    print(f"[gpu] steps bf16 {kind} {params} L={L} heads={heads} d={d}", flush=True)
    scale = 1.0 / math.sqrt(d)
    Q, K, V = _qkv(L, d, heads, L + 5 * d, "bf16")
    M = om.dense_mask(kind, params, L)
    a = splat.Acsr(splat.Pattern.named(kind, params, L), columns=True)
    S = torch.full((1, heads, a.nnz), float("nan"), device="cuda")
    splat.rsddmm(a, Q.cuda(), K.cuda(), scale, S=S)
    P = splat.row_softmax(a, S)
    O = splat.rspmm(a, P, V.cuda(), out_dtype=torch.float32)
    if a.info()["columns"] == 1:
        Oc = splat.rspmm_colmajor(a, splat.transpose_colmajor(a, P), V.cuda(),
                                  out_dtype=torch.float32)
        assert torch.equal(Oc, O)
    torch.cuda.synchronize()
    assert torch.isfinite(S).all() and torch.isfinite(O).all()
    m = torch.from_numpy(M)
    for h in (0, heads - 1):
        sel = slice(h, h + 1)
        ref = oa.masked_attention(Q[:, sel], K[:, sel], V[:, sel], M, scale)
        # P enters the products with 16 bits, sums in fp32
        assert float(np.abs(O[:, sel].cpu().numpy() - ref).max()) <= 1e-4
        q, k = Q[0, h].double(), K[0, h].double()
        x, mag = q @ k.t() * scale, q.abs() @ k.abs().t() * scale
        assert float(((S[0, h].cpu().double() - x[m]).abs() / mag[m]).max()) <= F32_REL


def test_binding_streams_and_outputs(gpu_lib):
    """Calls go to the current stream; an output made by the call is plain and
    contiguous whatever the class and the strides of size-1 axes of the input."""
    splat = gpu_lib
    L, d = 130, 64
    Q, K, V = (x.cuda() for x in _qkv(L, d, 3, 9, "bf16"))
    a = splat.Acsr(splat.Pattern.window(L, 20))
    ref = splat.sparse_mhsa_fwd(a, Q, K, V, 0.1)
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        torch.cuda._sleep(20_000_000)        # the inputs change only after this
        K2 = K * 0.5
        O = splat.sparse_mhsa_fwd(a, Q, K2, V, 0.2)
    side.synchronize()
    # (0.5 K) at twice the scale: the same scores to bf16's rounding of Q * scale
    assert float((O.float() - ref.float()).abs().max()) <= 2e-2
    odd = Q.as_strided(Q.shape, (7, L * d, d, 1))     # the batch axis has size 1
    assert odd.is_contiguous()
    for q in (odd, torch.nn.Parameter(Q, requires_grad=False)):
        O = splat.sparse_mhsa_fwd(a, q, K, V, 0.1)
        torch.cuda.synchronize()
        assert O.stride() == (3 * L * d, L * d, d, 1) and torch.equal(O, ref)
        assert type(O) is torch.Tensor


# groups of 7 (one set of wavefronts), 9, 13 (two), 17 and 23 tiles (four at d =
# 64), a last group of few rows, empty tiles; scores around 0, and rising with
# the key so that the sets end with references far apart
SETS = [
    ("full", {}, 448), ("full", {}, 520), ("full", {}, 777), ("full", {}, 1088),
    ("window", {"w": 500}, 1450), ("window_global", {"w": 30, "n_global": 3}, 1300),
    ("strided_local", {"local": 600, "stride": 100}, 900)]


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("rise", [0.0, 12.0])
@pytest.mark.parametrize("kind,params,L", SETS)
def test_fused_sets(gpu_lib, kind, params, L, rise, d):
    splat = gpu_lib
    print(f"[gpu] fused sets {kind} {params} L={L} rise={rise} d={d}", flush=True)
    scale = 1.0 / math.sqrt(d)
    Q, K, V = _qkv(L, d, 3, L + d, "f32")
    if rise:   # q and k along one direction u, |u|^2 * scale = 8
        u = math.sqrt(8.0 / (scale * d))
        c = torch.arange(L).float()[:, None] / L
        Q, K = 2.0 * u + 0.05 * Q, rise * c * u + 0.3 * K
    Q, K, V = (x.to(torch.bfloat16) for x in (Q, K, V))
    M = om.dense_mask(kind, params, L)
    ref = oa.masked_attention(Q, K, V, M, scale)
    a = splat.Acsr(splat.Pattern.named(kind, params, L))
    O = splat.sparse_mhsa_fwd(a, Q.cuda(), K.cuda(), V.cuda(), scale, out_dtype=torch.float32)
    Ob = splat.sparse_mhsa_fwd(a, Q.cuda(), K.cuda(), V.cuda(), scale)
    torch.cuda.synchronize()
    assert float(np.abs(O.cpu().numpy() - ref).max()) <= 2e-2
    assert float(np.abs(Ob.float().cpu().numpy() - ref).max()) <= 2e-2
