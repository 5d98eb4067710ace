"""GPU parity of the spectral corrector against the CPU oracle (Sec. 3.2; Alg. 1;
App. E).

Tolerances (relative Frobenius error of G_proj against the float64 oracle):
1e-4 for fp32 inputs, 2e-2 for bf16 inputs with fp32 accumulation.  The
prior's singular values and projectors are reported as diagnostics and
checked against looser bounds; U and V themselves are never compared (signs
and rotations inside equal singular values are not unique).
"""
import math

import numpy as np
import pytest
import torch

import workloads
from oracle import spectral as osp

pytestmark = pytest.mark.gpu

TOL = {torch.float32: 1e-4, torch.bfloat16: 2e-2}


@pytest.fixture(scope="module")
def pk():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2609_14339_amd as pk
    return pk


def _np(t):
    return t.detach().double().cpu().numpy()


def _signal_basis(spec, cid, layer, mat, r):
    """(G_anc, G_mask, U_sig[:, :r], s_sig[:r], V_sig[:, :r]) on the host."""
    gp = workloads.grad_pair(spec, cid, layer, mat, "cpu", keep_basis=True)
    return gp, gp.U_sig[:, :r].numpy(), gp.s_signal[:r].numpy(), gp.V_sig[:, :r].numpy()


# ---------------------------------------------------------------------------
# sc_correct with a given prior (U, d, V)
# ---------------------------------------------------------------------------
@pytest.mark.parametrize("cid,mat", [(1, 0), (2, 0), (2, 4), (2, 5), (3, 1)])
@pytest.mark.parametrize("alpha", [0.3, 0.0])
def test_correct_matches_oracle_with_the_signal_prior(pk, cid, mat, alpha):
    cfg = workloads.CONFIGS[cid]
    r = cfg.grad.r[0]
    gp, U, s, V = _signal_basis(cfg.grad, cid, 0, mat, r)
    d = osp.filter_weights(0.1 * s, workloads.TAU)     # the prior's s after one EMA arrival
    G = gp.G_mask
    ref = osp.correct(_np(G), U, d, V, alpha)
    Ug = torch.tensor(U, dtype=torch.float32, device="cuda")
    Vg = torch.tensor(V, dtype=torch.float32, device="cuda")
    dg = torch.tensor(d, dtype=torch.float32, device="cuda")
    out = pk.sc_correct(G.cuda(), Ug, dg, Vg, alpha)
    torch.cuda.synchronize()
    err = osp.rel_fro(_np(out), ref)
    assert err <= TOL[G.dtype], err
    if alpha == 0.0:
        # the filtered part alone carries a large share of G's energy here
        assert np.linalg.norm(ref) > 0.4 * np.linalg.norm(_np(G))


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("m,n,r", [(300, 200, 7), (200, 328, 33), (64, 64, 64), (1000, 16, 1),
                                   (129, 4104, 40)])
def test_correct_ragged_shapes(pk, dtype, m, n, r):
    U, s, V = workloads.random_orthonormal_basis(m, n, r, seed=m + n + r)
    # a gradient with a large component inside the prior plus isotropic noise
    c = workloads.gaussian((r,), seed=3).double().abs() + 0.5
    G64 = (U * c) @ V.T + 0.02 * workloads.gaussian((m, n), seed=4).double()
    G = G64.to(dtype)
    d = osp.filter_weights(s.numpy(), 0.7)
    ref = osp.correct(_np(G), U.numpy(), d, V.numpy(), 0.3)
    out = pk.sc_correct(G.cuda(), U.float().cuda(), torch.tensor(d, dtype=torch.float32).cuda(),
                        V.float().cuda(), 0.3)
    torch.cuda.synchronize()
    assert osp.rel_fro(_np(out), ref) <= TOL[dtype]


@pytest.mark.parametrize("m,n,r", [(130, 260, 64), (257, 1003, 50), (129, 515, 128), (200, 333, 190), (300, 1001, 24),
                                   (140, 452, 80), (1000, 4099, 150), (4097, 1101, 73), (513, 2049, 160)])
def test_correct_stores_widths_that_are_no_multiple_of_8(pk, m, n, r):
    """bf16 rows that are not 16-byte aligned, at every padded rank: whole
    chunks take unaligned 16-byte stores and each row's last chunk
    element-wise ones; the output starts as NaN, so an element that is not
    stored shows."""
    U, s, V = workloads.random_orthonormal_basis(m, n, r, seed=m + n + r)
    G = (((U * 0.5) @ V.T) + 0.02 * workloads.gaussian((m, n), seed=4).double()).to(torch.bfloat16)
    d = osp.filter_weights(s.numpy(), 0.7)
    ref = osp.correct(_np(G), U.numpy(), d, V.numpy(), 0.3)
    out = torch.full((m, n), float("nan"), dtype=torch.bfloat16, device="cuda")
    pk.sc_correct(G.cuda(), U.float().cuda(), torch.tensor(d, dtype=torch.float32).cuda(), V.float().cuda(), 0.3,
                  out=out)
    torch.cuda.synchronize()
    assert osp.rel_fro(_np(out), ref) <= TOL[torch.bfloat16]


@pytest.mark.parametrize("shapes,r", [(((300, 5000), (256, 2100)), 16), (((2048, 1536), (257, 9000), (511, 4096)), 72),
                                      (((1300, 3333), (200, 1024)), 40)])
def test_passes_cut_into_uneven_pieces(pk, shapes, r):
    """Small batches cut the long rows of a pass into pieces of a common
    length (last pieces shorter, any piece count), whose partials the Gram
    kernel or a reduction adds: a build and a correction against plain
    PyTorch in 64 bits from the same bf16 inputs."""
    spec = workloads.GradSpec(shapes, 24, (1.0, 10.0), (r,), torch.bfloat16, None, None)
    items, pairs = [], [workloads.grad_pair(spec, 21, 0, i, "cpu") for i in range(len(shapes))]
    for i, (m, n) in enumerate(shapes):
        U, s, V = workloads.random_orthonormal_basis(m, n, r, seed=m + n)
        items.append(dict(G=pairs[i].G_mask.cuda(), prior=(U.float().cuda(), (s / (s + 0.7)).float().cuda(),
                                                           V.float().cuda()),
                          out=torch.empty(m, n, dtype=torch.bfloat16, device="cuda"),
                          ws=pk.workspace(m, n, r, 0, torch.bfloat16)))
    pk.sc_correct_batched(items, r, workloads.ALPHA)
    torch.cuda.synchronize()
    for it in items:
        U, d, V = (_np(t) for t in it["prior"])
        assert osp.rel_fro(_np(it["out"]), osp.correct(_np(it["G"]), U, d, V, workloads.ALPHA)) <= TOL[torch.bfloat16]
    builds = []
    for i, (m, n) in enumerate(shapes):
        outs = (torch.empty(m, 24, device="cuda"), torch.empty(24, device="cuda"), torch.empty(n, 24, device="cuda"),
                torch.empty(24, device="cuda"))
        builds.append(dict(G_anc=pairs[i].G_anc.cuda(), M=torch.zeros(m, n, device="cuda"), out=outs,
                           ws=pk.workspace(m, n, 24, 16, torch.bfloat16)))
    pk.sc_build_prior_batched(builds, 24, workloads.BETA, workloads.TAU, 16, 3, seed=5)
    torch.cuda.synchronize()
    for it, gp in zip(builds, pairs):
        M = (1 - workloads.BETA) * _np(gp.G_anc)
        U0, s0, V0 = osp.top_r_svd_gram(M, 24)
        U, s, V, d = it["out"]
        assert np.max(np.abs(_np(s) - s0) / s0) < 5e-3
        assert osp.projector_distance(_np(U), U0) < 2e-2 and osp.projector_distance(_np(V), V0) < 2e-2


@pytest.mark.parametrize("m,n,r", [(17, 40, 5), (4100, 1037, 13), (16400, 515, 33), (16391, 1030, 150), (130, 9001, 100),
                                   (16384, 2048, 64), (64, 33, 32)])
def test_fp32_products_at_the_edges_of_their_tiles(pk, m, n, r):
    """The fp32 products take 16-row workgroups or, where they fill the GPU,
    64-row ones (32 beyond 144 columns), cut k among waves and workgroups, and
    mask tails of k, rows and columns; rows of odd widths are not 16-byte
    aligned.  Correction and one PowerSGD step against 64 bits."""
    U, s, V = workloads.random_orthonormal_basis(m, n, r, seed=m + n + r)
    G = (((U * 0.5) @ V.T) + 0.02 * workloads.gaussian((m, n), seed=4).double()).float()
    d = osp.filter_weights(s.numpy(), 0.7)
    ref = osp.correct(_np(G), U.numpy(), d, V.numpy(), 0.3)
    out = torch.full((m, n), float("nan"), device="cuda")
    pk.sc_correct(G.cuda(), U.float().cuda(), torch.tensor(d, dtype=torch.float32).cuda(), V.float().cuda(), 0.3,
                  out=out)
    torch.cuda.synchronize()
    assert osp.rel_fro(_np(out), ref) <= 2e-6
    Q0 = workloads.gaussian((n, r), seed=8)
    it = dict(G=G.cuda(), E=torch.zeros(m, n, device="cuda"), P=torch.empty(m, r, device="cuda"), Q=Q0.cuda(),
              out=torch.full((m, n), float("nan"), device="cuda"), ws=pk.psgd_workspace(m, n, r, torch.float32))
    pk.psgd_step([it], r, torch.float32)
    torch.cuda.synchronize()
    P, R = np.linalg.qr(_np(G) @ _np(Q0))
    P *= np.sign(np.diag(R))
    Q = _np(G).T @ P
    assert osp.rel_fro(_np(it["Q"]), Q) <= 1e-4 and osp.rel_fro(_np(it["out"]), P @ Q.T) <= 1e-4


def test_correct_in_place_and_alpha_one(pk):
    m, n, r = 512, 384, 16
    U, s, V = workloads.random_orthonormal_basis(m, n, r, seed=1)
    G = workloads.gaussian((m, n), seed=2, dtype=torch.bfloat16).cuda()
    Ug, Vg = U.float().cuda(), V.float().cuda()
    dg = torch.full((r,), 0.9, device="cuda")
    ref = pk.sc_correct(G, Ug, dg, Vg, 0.3)
    G2 = G.clone()
    pk.sc_correct(G2, Ug, dg, Vg, 0.3, out=G2)
    same = pk.sc_correct(G, Ug, dg, Vg, 1.0)
    torch.cuda.synchronize()
    assert torch.equal(G2, ref)
    assert torch.equal(same, G)                      # alpha = 1: masked-only training


# ---------------------------------------------------------------------------
# sc_build_prior (EMA + SVD + filter), then the full corrector step
# ---------------------------------------------------------------------------
def _gpu_step(pk, G_anc, G_mask, r, cfg, beta=workloads.BETA, M0=None, iters=None):
    m, n = G_anc.shape
    M = torch.zeros(m, n, device="cuda") if M0 is None else M0.clone()
    U, s, V, d = pk.sc_build_prior(G_anc.cuda(), M, r, beta, workloads.TAU, cfg.oversample,
                                   cfg.power_iters if iters is None else iters, seed=11)
    out = pk.sc_correct(G_mask.cuda(), U, d, V, workloads.ALPHA)
    torch.cuda.synchronize()
    return M, U, s, V, d, out


@pytest.mark.parametrize("cid,mat", [(1, 0), (2, 0), (2, 4), (2, 5)])
def test_build_prior_and_correct_match_oracle(pk, cid, mat):
    cfg = workloads.CONFIGS[cid]
    r = cfg.grad.r[0]
    gp = workloads.grad_pair(cfg.grad, cid, 0, mat, "cpu")
    M, U, s, V, d, out = _gpu_step(pk, gp.G_anc, gp.G_mask, r, cfg)
    Mo, Uo, so, Vo, do, ref = osp.corrected_step(np.zeros(gp.G_anc.shape), _np(gp.G_anc),
                                                 _np(gp.G_mask), workloads.BETA, r, workloads.TAU,
                                                 workloads.ALPHA)
    tol = TOL[gp.G_anc.dtype]
    assert osp.rel_fro(_np(M), Mo) < 1e-6                       # EMA, fp32 state
    assert np.max(np.abs(_np(s) - so) / so) < (1e-5 if cid == 1 else 1e-3)
    assert np.max(np.abs(_np(d) - do)) < 1e-5
    Ug, Vg = _np(U), _np(V)
    assert np.abs(Ug.T @ Ug - np.eye(r)).max() < 1e-4
    assert np.abs(Vg.T @ Vg - np.eye(r)).max() < 1e-4
    assert osp.rel_fro(_np(out), ref) <= tol
    # subspace diagnostics: randomised iteration vs the exact SVD
    assert osp.projector_distance(Ug, Uo) < (1e-4 if cid == 1 else tol)
    assert osp.projector_distance(Vg, Vo) < (1e-4 if cid == 1 else tol)


@pytest.mark.parametrize("m,n", [(200, 328), (328, 200), (70, 130), (1000, 1100)])
def test_ragged_bf16_build_ignores_workspace_padding(pk, m, n):
    """The bf16 shadow of M is kept in 64 x 64 tiles whose padding (rows past
    m, columns past n) is never written.  With the workspace filled with NaN
    bit patterns (bytes 0xFF) beforehand, a build at shapes that are not
    multiples of 64 must still match the oracle (Sec. 3.2 EMA and SVD,
    App. E filter) to the bf16 bounds: no pass may multiply padding into a
    stored output."""
    # singular values in [1, 10]: at these small shapes a [1, 100] range puts
    # the noise edge above the smallest signal value and leaves the top-12
    # subspace undetermined
    r, p, q = 12, 8, 3
    spec = workloads.GradSpec(((m, n),), r, (1.0, 10.0), (r,), torch.bfloat16, None, None)
    gp = workloads.grad_pair(spec, 9, 0, 0, "cpu")
    ws = pk.workspace(m, n, r, p, torch.bfloat16)
    ws.fill_(255)
    M = torch.zeros(m, n, device="cuda")
    U, s, V, d = pk.sc_build_prior(gp.G_anc.cuda(), M, r, workloads.BETA, workloads.TAU, p, q, seed=5, ws=ws)
    out = pk.sc_correct(gp.G_mask.cuda(), U, d, V, workloads.ALPHA)
    torch.cuda.synchronize()
    assert torch.isfinite(U).all() and torch.isfinite(V).all() and torch.isfinite(out.float()).all()
    Mo, Uo, so, Vo, do, ref = osp.corrected_step(np.zeros((m, n)), _np(gp.G_anc), _np(gp.G_mask),
                                                 workloads.BETA, r, workloads.TAU, workloads.ALPHA)
    assert osp.rel_fro(_np(M), Mo) < 1e-6
    # diagnostics: the passes see bf16(M).  At these small shapes the noise
    # edge (about 0.08) sits close to the smallest kept value (0.11), so the
    # shadow's rounding (||E||_2 ~ 2e-3) moves that value by a few 1e-3 and
    # tilts its direction by a few 1e-2; the corrected gradient is the contract
    assert np.max(np.abs(_np(s) - so) / so) < 5e-3
    assert osp.projector_distance(_np(U), Uo) < 5e-2
    assert osp.projector_distance(_np(V), Vo) < 5e-2
    assert osp.rel_fro(_np(out), ref) <= TOL[torch.bfloat16]


def test_two_arrivals_and_warm_start(pk):
    # the same anchor gradient arrives twice: M = (1 - beta^2) G_anc, so
    # s(M) = 0.19 s(G_anc); the second build starts from the first build's V
    cfg = workloads.CONFIGS[1]
    r = cfg.grad.r[0]
    g1 = workloads.grad_pair(cfg.grad, 1, 0, 0, "cpu")
    m, n = g1.G_anc.shape
    M = torch.zeros(m, n, device="cuda")
    U1, s1, V1, d1 = pk.sc_build_prior(g1.G_anc.cuda(), M, r, 0.9, 1e-3, 8, 6, seed=1)
    U2, s2, V2, d2 = pk.sc_build_prior(g1.G_anc.cuda(), M, r, 0.9, 1e-3, 8, 1, seed=2, V_warm=V1)
    torch.cuda.synchronize()
    Mo = osp.ema(osp.ema(np.zeros((m, n)), _np(g1.G_anc), 0.9), _np(g1.G_anc), 0.9)
    Uo, so, Vo = osp.top_r_svd(Mo, r)
    sg = np.linalg.svd(_np(g1.G_anc), compute_uv=False)[:r]
    assert np.allclose(so, 0.19 * sg, rtol=1e-12)
    assert osp.rel_fro(_np(M), Mo) < 1e-6
    assert np.max(np.abs(_np(s2) - so) / so) < 1e-5
    assert osp.projector_distance(_np(U2), Uo) < 1e-4
    assert osp.projector_distance(_np(V2), Vo) < 1e-4


def test_zero_prior_gives_alpha_G(pk):
    m, n, r = 96, 80, 4
    M = torch.zeros(m, n, device="cuda")
    U, s, V, d = pk.sc_build_prior(None, M, r, 0.9, 1e-3, 4, 2, seed=5)
    G = workloads.gaussian((m, n), seed=8).cuda()
    out = pk.sc_correct(G, U, d, V, 0.3)
    torch.cuda.synchronize()
    assert torch.all(s == 0) and torch.all(d == 0)
    assert torch.allclose(out, 0.3 * G, rtol=1e-6, atol=0)


@pytest.mark.parametrize("m,n,r,rank,p,q", [(120, 90, 5, 3, 8, 3), (70, 200, 6, 6, 8, 3),
                                             (257, 129, 12, 40, 24, 8)])
def test_rank_deficient_and_ragged_priors(pk, m, n, r, rank, p, q):
    U, s, V = workloads.random_orthonormal_basis(m, n, rank, seed=m * n)
    M64 = (U * s) @ V.T
    M = M64.float().cuda()
    Ug, sg, Vg, dg = pk.sc_build_prior(None, M, r, 0.9, 1e-3, p, q, seed=9)
    torch.cuda.synchronize()
    Uo, so, Vo = osp.top_r_svd(M64.numpy(), r)
    k = min(r, rank)
    assert np.allclose(_np(sg)[:k], so[:k], rtol=1e-4, atol=1e-5)
    assert np.all(_np(sg)[k:] < 1e-3 * so[0])
    assert osp.projector_distance(_np(Ug)[:, :k], Uo[:, :k]) < 1e-4
    assert osp.projector_distance(_np(Vg)[:, :k], Vo[:, :k]) < 1e-4
    G = workloads.gaussian((m, n), seed=10).cuda()
    out = pk.sc_correct(G, Ug, dg, Vg, 0.3)
    ref = osp.correct(_np(G), Uo, osp.filter_weights(so, 1e-3), Vo, 0.3)
    torch.cuda.synchronize()
    assert osp.rel_fro(_np(out), ref) < 1e-4


def test_build_prior_is_deterministic(pk):
    cfg = workloads.CONFIGS[2]
    gp = workloads.grad_pair(cfg.grad, 2, 0, 0, "cpu")
    a = _gpu_step(pk, gp.G_anc, gp.G_mask, 32, cfg)
    b = _gpu_step(pk, gp.G_anc, gp.G_mask, 32, cfg)
    for x, y in zip(a, b):
        assert torch.equal(x, y)


def test_errors_raise_before_any_work(pk):
    M = torch.zeros(64, 48, device="cuda")
    with pytest.raises(pk.AcscError) as e:
        pk.sc_build_prior(None, M, 49, 0.9, 1e-3, 4, 2)
    assert e.value.code == pk.ACSC_EINVAL
    with pytest.raises(pk.AcscError) as e:
        pk.sc_build_prior(None, M, 8, 1.5, 1e-3, 4, 2)
    small = torch.empty(16, dtype=torch.uint8, device="cuda")
    with pytest.raises(pk.AcscError) as e:
        pk.sc_build_prior(None, M, 8, 0.9, 1e-3, 4, 2, ws=small)
    assert e.value.code == pk.ACSC_ENOSPC


def test_batched_calls_equal_single_calls(pk):
    """One batched call over mixed shapes gives bit-identical results to one
    call per matrix (matrix i of the batch uses seed + i).  The (20, 300)
    matrix has k = min(r + p, m, n) = 20 rather than 24, so the batch runs as
    two groups."""
    shapes = [(256, 384), (384, 256), (20, 300), (200, 328)]
    r, p, q = 16, 8, 2
    mats = []
    for i, (m, n) in enumerate(shapes):
        gp = workloads.grad_pair(workloads.GradSpec(((m, n),), 16, (1.0, 100.0), (r,), torch.bfloat16,
                                                    None, None), 9, 0, 0, "cpu")
        mats.append(gp)
    single = []
    for i, gp in enumerate(mats):
        m, n = gp.G_anc.shape
        M = torch.zeros(m, n, device="cuda")
        U, s, V, d = pk.sc_build_prior(gp.G_anc.cuda(), M, r, 0.9, 1e-3, p, q, seed=40 + i)
        out = pk.sc_correct(gp.G_mask.cuda(), U, d, V, 0.3)
        single.append((M, U, s, V, d, out))
    items, corr = [], []
    for i, gp in enumerate(mats):
        m, n = gp.G_anc.shape
        M = torch.zeros(m, n, device="cuda")
        outs = (torch.empty(m, r, device="cuda"), torch.empty(r, device="cuda"),
                torch.empty(n, r, device="cuda"), torch.empty(r, device="cuda"))
        items.append(dict(G_anc=gp.G_anc.cuda(), M=M, out=outs,
                          ws=pk.workspace(m, n, r, p, torch.bfloat16)))
    pk.sc_build_prior_batched(items, r, 0.9, 1e-3, p, q, seed=40)
    for it, gp in zip(items, mats):
        m, n = gp.G_anc.shape
        U, s, V, d = it["out"]
        corr.append(dict(G=gp.G_mask.cuda(), prior=(U, d, V), out=torch.empty(m, n, dtype=torch.bfloat16,
                                                                               device="cuda"),
                         ws=pk.workspace(m, n, r, 0, torch.bfloat16)))
    pk.sc_correct_batched(corr, r, 0.3)
    torch.cuda.synchronize()
    for it, c, ref in zip(items, corr, single):
        got = (it["M"],) + tuple(it["out"]) + (c["out"],)
        for x, y in zip(got, ref):
            assert torch.equal(x, y)


@pytest.mark.parametrize("fused,dtype", [(False, torch.bfloat16), (True, torch.bfloat16), (False, torch.float32)])
def test_build_in_two_phases_equals_one_call(pk, fused, dtype):
    """sc_build_subspace_batched then sc_build_ritz_batched (the same
    arguments and workspaces) give bit-identical EMA state and prior to one
    sc_build_prior_batched call, with the unfused EMA (a small mixed batch,
    bf16 and fp32) and with the EMA fused with the first pass (8 x 8192 x 512,
    256 row blocks); the ritz phase leaves M alone, and both arrangements
    report a converged build."""
    if fused:
        shapes, r, p = [(8192, 512)] * 8, 32, 16
    else:
        shapes, r, p = [(256, 384), (384, 256), (200, 328)], 16, 8
    q = 2
    runs = []
    for split in (False, True):
        items = []
        for i, (m, n) in enumerate(shapes):
            gp = workloads.grad_pair(workloads.GradSpec(((m, n),), r, (1.0, 100.0), (r,), dtype,
                                                        None, None), 9, i, 0, "cpu")
            outs = (torch.empty(m, r, device="cuda"), torch.empty(r, device="cuda"),
                    torch.empty(n, r, device="cuda"), torch.empty(r, device="cuda"))
            items.append(dict(G_anc=gp.G_anc.cuda(), M=torch.zeros(m, n, device="cuda"), out=outs,
                              ws=pk.workspace(m, n, r, p, dtype)))
        args = (r, workloads.BETA, workloads.TAU, p, q)
        if split:
            pk.sc_build_subspace_batched(items, *args, seed=70, dtype=dtype)
            torch.cuda.synchronize()
            M_mid = [it["M"].clone() for it in items]
            pk.sc_build_ritz_batched(items, *args, seed=70, dtype=dtype)
            torch.cuda.synchronize()
            for it, Mm in zip(items, M_mid):
                assert torch.equal(it["M"], Mm)
        else:
            pk.sc_build_prior_batched(items, *args, seed=70, dtype=dtype)
            torch.cuda.synchronize()
        status = pk.sc_build_status([it["ws"] for it in items])
        assert all(1 <= sw <= 40 for sw, _ in status), status
        runs.append(items)
    for a, b in zip(*runs):
        assert torch.equal(a["M"], b["M"])
        for x, y in zip(a["out"], b["out"]):
            assert torch.equal(x, y)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_ritz_phase_takes_the_matrices_of_a_subspace_call_one_by_one(pk, dtype):
    """One subspace call on a batch whose last products are cut along k as the
    batch asks for (8, 1, 1 pieces in bf16; alone these matrices would be cut
    in 16, 2, 2), then a ritz call per matrix: each gives the prior that one
    call on the batch gives.  Only the fp64 Gram sums may be grouped
    differently (1e-16), so the fp32 outputs agree to a few rounding errors:
    1e-6 on the singular values, 1e-5 on U diag(s) V^T."""
    shapes, r, p = [(8192, 256), (1024, 16384), (1024, 16384)], 64, 16
    runs = []
    for split in (False, True):
        items = []
        for i, (m, n) in enumerate(shapes):
            gp = workloads.grad_pair(workloads.GradSpec(((m, n),), r, (1.0, 100.0), (r,), dtype, None, None), 9, i, 0,
                                     "cpu")
            outs = tuple(torch.zeros(*s, device="cuda") for s in ((m, r), (r,), (n, r), (r,)))
            items.append(dict(G_anc=gp.G_anc.cuda(), M=torch.zeros(m, n, device="cuda"), out=outs,
                              ws=pk.workspace(m, n, r, p, dtype)))
        args = (r, workloads.BETA, workloads.TAU, p, 2)
        if split:
            pk.sc_build_subspace_batched(items, *args, seed=70, dtype=dtype)
            for it in items:
                pk.sc_build_ritz_batched([it], *args, seed=70, dtype=dtype)
        else:
            pk.sc_build_prior_batched(items, *args, seed=70, dtype=dtype)
        torch.cuda.synchronize()
        pk.sc_build_status([it["ws"] for it in items])
        runs.append(items)
    for a, b in zip(*runs):
        (U0, s0, V0, _), (U1, s1, V1, _) = a["out"], b["out"]
        assert (s1 / s0 - 1).abs().max().item() <= 1e-6
        P0 = (U0 * s0) @ V0.t()
        assert ((U1 * s1) @ V1.t() - P0).norm().item() <= 1e-5 * P0.norm().item()


@pytest.mark.parametrize("k", [1, 3, 5, 8, 9, 16, 17, 31, 44, 61, 80, 100, 113, 128, 129, 160, 161, 189])
def test_ritz_step_at_every_block_count(pk, k):
    """The Jacobi works on blocks of four columns (odd block counts and partial
    blocks are padded with zero columns) up to order 128 and on column pairs
    beyond: with k = n the Ritz step is the whole SVD of M, compared with
    numpy's.  Bounds: fp32 M and Z = M^T Q, so about 1e-6 of the largest
    singular value; the fp32 Jacobi stops at 1e-5."""
    m, n = 260, k
    g = torch.Generator().manual_seed(k)
    q1, q2 = (torch.linalg.qr(torch.randn(s, k, generator=g, dtype=torch.float64))[0] for s in (m, n))
    s0 = torch.exp(torch.linspace(math.log(10.0), 0.0, k, dtype=torch.float64)) if k > 1 else torch.tensor([3.0]).double()
    if k > 4:
        s0[2] = s0[1]                     # a repeated value: its vectors may be any basis
    G = ((q1 * s0) @ q2.T).float()
    M = torch.zeros(m, n, device="cuda")
    ws = pk.workspace(m, n, k, 0, torch.float32)
    U, s, V, d = pk.sc_build_prior(G.cuda(), M, k, 0.0, 0.0, 0, 1, seed=1, ws=ws)
    torch.cuda.synchronize()
    pk.sc_build_status([ws])
    ref = np.linalg.svd(G.double().numpy(), compute_uv=False)
    assert np.max(np.abs(_np(s) - ref)) <= 2e-5 * ref[0]
    tol = 2e-4 if k > 128 else 2e-5
    assert osp.rel_fro(_np(U) * _np(s) @ _np(V).T, G.double().numpy()) <= tol
    for B in (_np(U), _np(V)):
        assert np.max(np.abs(B.T @ B - np.eye(k))) <= tol


@pytest.mark.parametrize("n,k,added", [(16, 16, True), (40, 13, True), (100, 30, True), (256, 48, True),
                                       (257, 48, False), (512, 17, True), (512, 32, True), (513, 32, False),
                                       (64, 50, False), (500, 72, False), (512, 144, False)])
def test_who_adds_the_gram_partials(pk, n, k, added):
    """The factorisation adds up the Gram partials (one per 32 rows) of orders
    up to 48 with up to 16 of them and 144 KiB, where that takes less time than the
    launch that adds them otherwise.  An n x n matrix of rank k: U diag(s) V^T
    is the matrix itself (fp32 products; the fp32 Jacobi beyond order 128
    stops at 1e-5)."""
    g = torch.Generator().manual_seed(k)
    q1, q2 = (torch.linalg.qr(torch.randn(n, k, generator=g, dtype=torch.float64))[0] for _ in range(2))
    G = ((q1 * torch.exp(torch.linspace(math.log(10.0), 0.0, k, dtype=torch.float64))) @ q2.T).float()
    M = torch.zeros(n, n, device="cuda")
    ws = pk.workspace(n, n, k, 0, torch.float32)
    try:
        pk.acsc_stats_enable(True)
        U, s, V, d = pk.sc_build_prior(G.cuda(), M, k, 0.0, 0.0, 0, 1, seed=1, ws=ws)
        torch.cuda.synchronize()
        launches = pk.acsc_stats_read()
    finally:
        pk.acsc_stats_enable(False)
    pk.sc_build_status([ws])
    assert ("sc_gram_reduce" not in launches) == added
    assert osp.rel_fro(_np(U) * _np(s) @ _np(V).T, G.double().numpy()) <= (2e-4 if k > 128 else 2e-5)


@pytest.mark.parametrize("dtype,r", [(torch.float32, 8), (torch.bfloat16, 40), (torch.bfloat16, 130)])
def test_a_nan_gradient_leaves_the_next_build_alone(pk, dtype, r):
    """A NaN in the anchor gradient: the call returns, and the same workspace
    then builds a clean matrix's prior to the bits that a fresh one gives."""
    m, n = 300, 400
    g = workloads.gaussian((m, n), seed=2, dtype=dtype).cuda()
    bad = g.clone()
    bad[17, 23] = float("nan")
    ws = pk.workspace(m, n, r, 16, dtype)
    U, s, V, d = pk.sc_build_prior(bad, torch.zeros(m, n, device="cuda"), r, 0.9, 1e-3, 16, 2, seed=3, ws=ws)
    again = pk.sc_build_prior(g, torch.zeros(m, n, device="cuda"), r, 0.9, 1e-3, 16, 2, seed=3, ws=ws)
    fresh = pk.sc_build_prior(g, torch.zeros(m, n, device="cuda"), r, 0.9, 1e-3, 16, 2, seed=3)
    torch.cuda.synchronize()
    for x, y in zip(again, fresh):
        assert torch.isfinite(x).all() and torch.equal(x, y)


@pytest.mark.parametrize("m,n", [(300, 400), (1500, 400)])
@pytest.mark.parametrize("dtype,r", [(torch.float32, 8), (torch.bfloat16, 8), (torch.bfloat16, 40), (torch.bfloat16, 130)])
def test_a_nan_gradient_stays_out_of_its_batch(pk, dtype, r, m, n):
    """A NaN in one anchor gradient of a batched build spreads into that
    matrix's prior only: its neighbours (products cut and uncut, Gram
    partials added by the factorisation and before it) have the bits that
    the same batch gives with a clean gradient in its place."""
    gs = [workloads.gaussian((m, n), seed=s, dtype=dtype).cuda() for s in range(3)]
    bad = gs[1].clone()
    bad[17, 23] = float("nan")
    runs = []
    for mid in (gs[1], bad):
        items = [dict(G_anc=g, M=torch.zeros(m, n, device="cuda"), ws=pk.workspace(m, n, r, 16, dtype),
                      out=tuple(torch.zeros(*s, device="cuda") for s in ((m, r), (r,), (n, r), (r,))))
                 for g in (gs[0], mid, gs[2])]
        pk.sc_build_prior_batched(items, r, 0.9, 1e-3, 16, 2, seed=3, dtype=dtype)
        torch.cuda.synchronize()
        runs.append(items)
    for i in (0, 2):
        assert torch.equal(runs[0][i]["M"], runs[1][i]["M"])
        for x, y in zip(runs[0][i]["out"], runs[1][i]["out"]):
            assert torch.isfinite(x).all() and torch.equal(x, y)
    assert torch.isnan(runs[1][1]["M"][17, 23])


@pytest.mark.parametrize("r,p", [(16, 8), (130, 16)])
def test_build_status_reports_a_sweep_cap_and_a_missing_subspace_phase(pk, r, p, monkeypatch):
    """The Rayleigh-Ritz Jacobi (fp64 for k <= 128, fp32 above) reports its
    sweeps and residual; capped at one sweep through ACSC_JACOBI_MAX_SWEEPS
    it stops above its tolerance and sc_build_status returns ACSC_ENOCONV.
    A Rayleigh-Ritz phase run alone after a complete build, or after a
    correction reused the workspace, finds no subspace stamp and is reported
    too; a new subspace phase clears the report."""
    m, n = 512, 384
    spec = workloads.GradSpec(((m, n),), 64, (1.0, 100.0), (r,), torch.bfloat16, None, None)
    gp = workloads.grad_pair(spec, 9, 0, 0, "cpu")
    outs = (torch.empty(m, r, device="cuda"), torch.empty(r, device="cuda"),
            torch.empty(n, r, device="cuda"), torch.empty(r, device="cuda"))
    item = dict(G_anc=gp.G_anc.cuda(), M=torch.zeros(m, n, device="cuda"), out=outs,
                ws=pk.workspace(m, n, r, p, torch.bfloat16))
    args = (r, workloads.BETA, workloads.TAU, p, 2)
    pk.sc_build_prior_batched([item], *args, seed=3)
    [(sw, res)] = pk.sc_build_status([item["ws"]])
    assert 2 <= sw <= 40 and res <= (1e-5 if r + p > 128 else 1e-13), (sw, res)
    monkeypatch.setenv("ACSC_JACOBI_MAX_SWEEPS", "1")
    pk.sc_build_prior_batched([item], *args, seed=3)
    with pytest.raises(pk.AcscError) as e:
        pk.sc_build_status([item["ws"]])
    assert e.value.code == pk.ACSC_ENOCONV and "1 sweeps" in str(e.value)
    assert e.value.status[0][0] == 1
    monkeypatch.delenv("ACSC_JACOBI_MAX_SWEEPS")
    # a complete build, then the Rayleigh-Ritz phase alone on the same workspace
    pk.sc_build_prior_batched([item], *args, seed=3)
    pk.sc_build_status([item["ws"]])
    pk.sc_build_ritz_batched([item], *args, seed=3)
    with pytest.raises(pk.AcscError) as e:
        pk.sc_build_status([item["ws"]])
    assert e.value.code == pk.ACSC_ENOCONV and "without a subspace phase" in str(e.value)
    # the subspace phase, a correction reusing the workspace, then the ritz phase
    pk.sc_build_subspace_batched([item], *args, seed=3)
    U, s, V, d = outs
    pk.sc_correct(gp.G_mask.cuda(), U, d, V, workloads.ALPHA, ws=item["ws"])
    pk.sc_build_ritz_batched([item], *args, seed=3)
    with pytest.raises(pk.AcscError) as e:
        pk.sc_build_status([item["ws"]])
    assert e.value.code == pk.ACSC_ENOCONV
    pk.sc_build_subspace_batched([item], *args, seed=3)
    pk.sc_build_ritz_batched([item], *args, seed=3)
    pk.sc_build_status([item["ws"]])


def test_build_status_reports_a_fused_ema_pass_that_gave_up_a_wait(pk, monkeypatch):
    """The fused EMA pass bounds every wait for the other waves of its
    workgroup.  With ACSC_EMA_SPIN_LIMIT=0 a wait gives up at its first unmet
    check (the kernel still finishes, every access in bounds), and
    sc_build_status reports the build as ACSC_ENOCONV.  The EMA of M is each
    wave's own and stays exact; the next build with the default limit clears
    the report and is bit-identical to a build that never gave up."""
    m, n, r, p, q = 8192, 512, 32, 16, 2
    spec = workloads.GradSpec(((m, n),), 32, (1.0, 100.0), (r,), torch.bfloat16, None, None)
    pairs = [workloads.grad_pair(spec, 9, layer, 0, "cpu") for layer in range(8)]

    def make():
        return [dict(G_anc=gp.G_anc.cuda(), M=torch.zeros(m, n, device="cuda"),
                     out=(torch.empty(m, r, device="cuda"), torch.empty(r, device="cuda"),
                          torch.empty(n, r, device="cuda"), torch.empty(r, device="cuda")),
                     ws=pk.workspace(m, n, r, p, torch.bfloat16)) for gp in pairs]

    args = (r, workloads.BETA, workloads.TAU, p, q)
    ref = make()
    pk.sc_build_prior_batched(ref, *args, seed=70)
    pk.sc_build_status([it["ws"] for it in ref])
    items = make()
    monkeypatch.setenv("ACSC_EMA_SPIN_LIMIT", "0")
    pk.sc_build_prior_batched(items, *args, seed=70)
    with pytest.raises(pk.AcscError) as e:
        pk.sc_build_status([it["ws"] for it in items])
    assert e.value.code == pk.ACSC_ENOCONV and "fused EMA pass" in str(e.value)
    for it, rf in zip(items, ref):
        assert torch.equal(it["M"], rf["M"])
    monkeypatch.delenv("ACSC_EMA_SPIN_LIMIT")
    for it in items:
        it["M"].zero_()
    pk.sc_build_prior_batched(items, *args, seed=70)
    pk.sc_build_status([it["ws"] for it in items])
    torch.cuda.synchronize()
    for it, rf in zip(items, ref):
        assert torch.equal(it["M"], rf["M"])
        for x, y in zip(it["out"], rf["out"]):
            assert torch.equal(x, y)


def test_large_batch_takes_the_fused_ema_pass(pk):
    """A batch with enough row blocks to fill the GPU (8 matrices of 8192 x 512:
    256 row blocks of 256 rows) runs the anchor EMA fused with the first pass
    over the bf16 shadow.  Single calls (too few row blocks: separate EMA and
    pass, the same products in the same order) give bit-identical results;
    the EMA, the prior and the correction match the oracle to the bf16
    bounds; a second build with no new gradient keeps M and the prior."""
    m, n, r, p, q = 8192, 512, 32, 16, 2
    spec = workloads.GradSpec(((m, n),), 32, (1.0, 100.0), (r,), torch.bfloat16, None, None)
    pairs = [workloads.grad_pair(spec, 9, layer, 0, "cpu") for layer in range(8)]
    items = []
    for gp in pairs:
        outs = (torch.empty(m, r, device="cuda"), torch.empty(r, device="cuda"),
                torch.empty(n, r, device="cuda"), torch.empty(r, device="cuda"))
        items.append(dict(G_anc=gp.G_anc.cuda(), M=torch.zeros(m, n, device="cuda"), out=outs,
                          ws=pk.workspace(m, n, r, p, torch.bfloat16)))
    pk.sc_build_prior_batched(items, r, workloads.BETA, workloads.TAU, p, q, seed=70)
    corr = [dict(G=gp.G_mask.cuda(), prior=(it["out"][0], it["out"][3], it["out"][2]),
                 out=torch.empty(m, n, dtype=torch.bfloat16, device="cuda"),
                 ws=pk.workspace(m, n, r, 0, torch.bfloat16)) for it, gp in zip(items, pairs)]
    pk.sc_correct_batched(corr, r, workloads.ALPHA)
    torch.cuda.synchronize()
    for i, (it, gp) in enumerate(zip(items, pairs)):
        M = torch.zeros(m, n, device="cuda")
        single = pk.sc_build_prior(gp.G_anc.cuda(), M, r, workloads.BETA, workloads.TAU, p, q, seed=70 + i)
        torch.cuda.synchronize()
        assert torch.equal(it["M"], M)
        for x, y in zip(it["out"], single):
            assert torch.equal(x, y)
    for it, c, gp in zip(items, corr, pairs):
        Mo, Uo, so, Vo, do, ref = osp.corrected_step(np.zeros((m, n)), _np(gp.G_anc), _np(gp.G_mask),
                                                     workloads.BETA, r, workloads.TAU, workloads.ALPHA)
        U, s, V, d = it["out"]
        assert osp.rel_fro(_np(it["M"]), Mo) < 1e-6
        # the prior comes from the bf16 shadow and two power iterations; the
        # last kept value sits near the noise floor of 8192 rows, so its
        # direction is the least determined (subspaces are compared in the
        # oracle tests at the C1/C2 shapes); the corrected gradient is the
        # contract
        assert np.max(np.abs(_np(s) - so) / so) < 5e-3
        assert osp.rel_fro(_np(c["out"]), ref) <= TOL[torch.bfloat16]
    first = [tuple(x.clone() for x in it["out"]) for it in items]
    M_first = [it["M"].clone() for it in items]
    for it in items:
        it["G_anc"] = None
    pk.sc_build_prior_batched(items, r, workloads.BETA, workloads.TAU, p, q, seed=70)
    torch.cuda.synchronize()
    for it, M0, out0 in zip(items, M_first, first):
        assert torch.equal(it["M"], M0)
        for x, y in zip(it["out"], out0):
            assert torch.equal(x, y)


def test_fused_ema_pass_over_more_matrices_than_one_launch_takes(pk):
    """20 matrices of 4096 x 256 (320 row blocks: the fused EMA pass, in two
    launches of at most 16 matrices, each with its own dispatch plan) give
    the same M and prior, bit for bit, as single calls (separate EMA and
    pass, the same products in the same order)."""
    m, n, r, p, q = 4096, 256, 16, 16, 2
    spec = workloads.GradSpec(((m, n),), 16, (1.0, 100.0), (r,), torch.bfloat16, None, None)
    pairs = [workloads.grad_pair(spec, 11, layer, 0, "cpu") for layer in range(20)]
    items = []
    for gp in pairs:
        outs = (torch.empty(m, r, device="cuda"), torch.empty(r, device="cuda"),
                torch.empty(n, r, device="cuda"), torch.empty(r, device="cuda"))
        items.append(dict(G_anc=gp.G_anc.cuda(), M=torch.zeros(m, n, device="cuda"), out=outs,
                          ws=pk.workspace(m, n, r, p, torch.bfloat16)))
    pk.sc_build_prior_batched(items, r, workloads.BETA, workloads.TAU, p, q, seed=90)
    torch.cuda.synchronize()
    for i, (it, gp) in enumerate(zip(items, pairs)):
        M = torch.zeros(m, n, device="cuda")
        single = pk.sc_build_prior(gp.G_anc.cuda(), M, r, workloads.BETA, workloads.TAU, p, q, seed=90 + i)
        torch.cuda.synchronize()
        assert torch.equal(it["M"], M), i
        for x, y in zip(it["out"], single):
            assert torch.equal(x, y), i


def test_fused_ema_pass_on_ragged_shapes(pk):
    """10 matrices of 8000 x 1000 (320 row blocks: the fused EMA pass, with a
    partial last row block and a 40-column last step) give the same M and
    prior, bit for bit, as single calls (separate EMA and pass), with and
    without a new gradient."""
    m, n, r, p, q = 8000, 1000, 16, 16, 2
    spec = workloads.GradSpec(((m, n),), 16, (1.0, 100.0), (r,), torch.bfloat16, None, None)
    pairs = [workloads.grad_pair(spec, 12, layer, 0, "cpu") for layer in range(10)]
    items = []
    for gp in pairs:
        outs = (torch.empty(m, r, device="cuda"), torch.empty(r, device="cuda"),
                torch.empty(n, r, device="cuda"), torch.empty(r, device="cuda"))
        items.append(dict(G_anc=gp.G_anc.cuda(), M=torch.zeros(m, n, device="cuda"), out=outs,
                          ws=pk.workspace(m, n, r, p, torch.bfloat16)))
    singles = [torch.zeros(m, n, device="cuda") for _ in pairs]
    for arrival in range(2):
        if arrival == 1:
            for it in items:
                it["G_anc"] = None
        pk.sc_build_prior_batched(items, r, workloads.BETA, workloads.TAU, p, q, seed=40, dtype=torch.bfloat16)
        torch.cuda.synchronize()
        for i, (it, gp) in enumerate(zip(items, pairs)):
            G = gp.G_anc.cuda() if arrival == 0 else None
            single = pk.sc_build_prior(G, singles[i], r, workloads.BETA, workloads.TAU, p, q, seed=40 + i,
                                       dtype=torch.bfloat16)
            torch.cuda.synchronize()
            assert torch.equal(it["M"], singles[i]), (arrival, i)
            for x, y in zip(it["out"], single):
                assert torch.equal(x, y), (arrival, i)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_bench_counts_every_kernel_of_a_correction(pk, dtype):
    """The benchmark splits a step's kernel time into correction and build by
    the kernels' names; a G V product that is cut along k (512 x 4096) also
    launches the addition of its partials, under the correction's own name."""
    import bench
    m, n, r = 512, 4096, 16
    it = dict(G=torch.randn(m, n, device="cuda").to(dtype), ws=pk.workspace(m, n, r, 0, dtype),
              prior=(torch.randn(m, r, device="cuda"), torch.rand(r, device="cuda"), torch.randn(n, r, device="cuda")),
              out=torch.empty(m, n, dtype=dtype, device="cuda"))
    try:
        pk.acsc_stats_enable(True)
        pk.sc_correct_batched([it], r, 0.3, dtype=dtype)
        torch.cuda.synchronize()
        launches = pk.acsc_stats_read()
    finally:
        pk.acsc_stats_enable(False)
    assert "sc_gv_reduce" in launches and set(launches) <= set(bench.CORRECTION_KERNELS), launches


@pytest.mark.parametrize("m,n,count", [(3848, 4200, 9), (4248, 520, 16)])
def test_narrow_passes_at_two_workgroups_per_cu(pk, m, n, count):
    """Batches of narrow passes whose row blocks fill just over half the CUs
    (9 x 16 row blocks, cut) or a second round badly (16 x 17, whole rows)
    take two workgroups per CU.  G_proj of every matrix against its float64
    value: bf16 rounds G V's factor, U X_f and the output, 2^-9 each at most
    (the transposed form is in the PowerSGD tests)."""
    r, dev = 20, "cuda"
    g = torch.Generator(device=dev).manual_seed(m)
    items = []
    for _ in range(count):
        U, V = (torch.linalg.qr(torch.randn(s, r, generator=g, device=dev))[0].contiguous() for s in (m, n))
        d = torch.rand(r, generator=g, device=dev)
        G = (torch.randn(m, n, generator=g, device=dev) + 40 * (U @ V.t())).bfloat16()
        items.append(dict(G=G, prior=(U, d, V), out=torch.zeros_like(G), ws=pk.workspace(m, n, r, 0, torch.bfloat16)))
    pk.sc_correct_batched(items, r, workloads.ALPHA)
    for i, it in enumerate(items):
        U, d, V = (t.double() for t in it["prior"])
        G = it["G"].double()
        ref = workloads.ALPHA * G + (1 - workloads.ALPHA) * ((U * d) @ (U.t() @ (G @ V)) @ (V * d).t())
        assert (it["out"].double() - ref).norm().item() <= 3 * 2.0 ** -9 * ref.norm().item(), i


def test_stats_filter_times_only_the_named_kernel(pk):
    """acsc_stats_only: with a name set, only that kernel's launches are
    timed; the build's result does not depend on the timing."""
    cfg = workloads.CONFIGS[2]
    gp = workloads.grad_pair(cfg.grad, 2, 0, 0, "cpu")
    ref = _gpu_step(pk, gp.G_anc, gp.G_mask, 32, cfg)
    try:
        pk.acsc_stats_only("sc_gram")
        pk.acsc_stats_enable(True)
        out = _gpu_step(pk, gp.G_anc, gp.G_mask, 32, cfg)
        torch.cuda.synchronize()
        only = pk.acsc_stats_read()
        pk.acsc_stats_only(None)
        pk.acsc_stats_enable(True)
        _gpu_step(pk, gp.G_anc, gp.G_mask, 32, cfg)
        torch.cuda.synchronize()
        every = pk.acsc_stats_read()
    finally:
        pk.acsc_stats_enable(False)
        pk.acsc_stats_only(None)
    assert set(only) == {"sc_gram"}
    assert only["sc_gram"][0] == every["sc_gram"][0] > 0
    assert {"sc_jacobi", "sc_chol_inv", "sc_gram"} <= set(every)
    for x, y in zip(ref, out):
        assert torch.equal(x, y)
