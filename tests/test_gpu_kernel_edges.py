"""Kernels at the sizes where their tiles, remainders and dispatch rules change, against the
FP64 oracle: the smallest and largest of a range, one past a tile, odd and ragged."""
import numpy as np
import pytest

import modal_inputs as mi
from helpers import Case
from oracle import modal as om

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _ctx(case, prec):
    from paper_1105_2791_amd import ModalContext
    return ModalContext(case.lmax, case.ntheta, case.nphi, case.P, prec, case.q, case.cl, mask=case.mask())


# FP64 contraction: 1 to 4 column tiles of 16 modes (P 1, 16 | 17, 33 | 49, 64), row tiles that
# end inside a wave, a chunk shorter than a staged step, more chunks than pixels to fill them,
# and the chunk count that the ring coefficients' region bounds (l_max 2, P 64).
F64_CASES = [(2, 3, 6, 1, 1), (2, 3, 6, 64, 2), (9, 14, 30, 16, 3), (9, 15, 32, 17, 1), (20, 31, 64, 33, 2),
             (40, 61, 124, 49, 1), (12, 19, 40, 64, 2)]


@pytest.mark.parametrize("lmax,ntheta,nphi,P,S", F64_CASES)
def test_f64_contraction_edges(lmax, ntheta, nphi, P, S):
    case = Case("edge", lmax, ntheta, nphi, P, S, "wmap", 71)
    print(f"[case] f64 contraction lmax={lmax} {ntheta}x{nphi} P={P} S={S}", flush=True)
    a = case.alms(0, S)
    M, w = case.maps(a), case.grid.w
    mc = case.maps(case.alms(50, 2))
    V = om.pair_means(mc)
    c = _ctx(case, "f64")
    got = c.beta(a).cpu().numpy()
    st = c.linear_state()
    c.linear_reset(st)
    c.linear_accumulate(st, case.alms(50, 2))
    c.linear_finalize(st)
    hat = c.beta(a, state=st).cpu().numpy()
    for i in range(S):
        ref, mag = om.beta(M[i], w), om.beta(np.abs(M[i]), w)
        lin, lmag = om.linear_term(M[i], w, V), om.linear_term(np.abs(M[i]), w, np.abs(V))
        # forward-error scale of the sums: the FP64 bound of the other beta tests
        assert np.max(np.abs(got[i] - ref) / mag) < 1e-10
        assert np.max(np.abs(hat[i] - (ref - lin)) / (mag + lmag)) < 1e-10


# Theory side: one pair, a tile of pairs not filled and one past it (55 and 66 pairs of 64), an
# odd pair count (its last i alone), a node count that is a multiple of a stage (32 of 16) and
# ones that are not, several tiles of modes (816 of 64), and one node more than a tile (65 at l_max 43).
@pytest.mark.parametrize("lmax,P", [(1, 1), (10, 10), (11, 11), (21, 3), (6, 16), (43, 2)])
def test_theory_side_edges(lmax, P):
    from oracle import shapes as osh
    from paper_1105_2791_amd import ModalContext
    print(f"[case] theory lmax={lmax} P={P}", flush=True)
    rng = np.random.default_rng(100 * lmax + P)
    q, cl = rng.uniform(-1, 1, (P, lmax + 1)), rng.uniform(0.5, 2, lmax + 1)
    c = rng.uniform(0.5, 1.5, lmax + 1)
    terms = rng.uniform(-1, 1, (2, 3, lmax + 1))
    ctx = ModalContext(lmax, lmax + 1, 2 * lmax + 2, P, "f64", q, cl)
    z = ctx.ideal_covariance(c).cpu().numpy()
    a = ctx.alpha_separable(terms).cpu().numpy()
    # the FP64 bound of the theory tests (1e-11) on the sums of the absolute terms
    assert np.array_equal(z, z.T)
    assert np.all(np.abs(z - osh.ideal_covariance(q, c)) <= 1e-11 * osh.ideal_covariance(np.abs(q), c))
    mag = osh.alpha_separable(np.abs(terms), cl, np.abs(q))
    assert np.all(np.abs(a - osh.alpha_separable(terms, cl, q)) <= 1e-11 * mag)


# FP32 synthesis: 1 to 4 ring tiles of 16 per wave and two workgroups of rings (nrp 3, 65, 129,
# 193, 257), l_max on both sides of a 64-l chunk, lambda on the fly (fewer than three blocks of
# 64 columns) and from the table, a last column block that is not full, columns of one sky and
# of more skies than a block holds.
@pytest.mark.parametrize("lmax,ntheta,nphi,P,S", [(3, 5, 8, 2, 1), (63, 129, 130, 5, 2), (64, 130, 136, 7, 5),
                                                  (64, 257, 150, 7, 14), (130, 386, 270, 3, 33), (40, 514, 90, 6, 17),
                                                  (127, 128, 256, 1, 100)])
def test_f32_synthesis_edges(lmax, ntheta, nphi, P, S):
    case = Case("edge", lmax, ntheta, nphi, P, S, "wmap", 72)
    print(f"[case] f32 synthesis lmax={lmax} {ntheta}x{nphi} P={P} S={S}", flush=True)
    a = case.alms(0, S)
    c = _ctx(case, "f32")
    out = torch.full((S, P, ntheta, nphi), float("nan"), dtype=torch.float32, device="cuda")
    got = c.filter_maps(a, out=out).cpu().numpy()
    ref = case.maps(a)
    # the FP32 bound of the map tests, per sky and mode
    rms = np.sqrt(np.mean(ref * ref, axis=(2, 3)))
    assert np.all(np.max(np.abs(got - ref), axis=(2, 3)) <= 1e-5 * rms)


# Adjoint of the FP32 and FP64 contexts: 1, 2 and 3 row tiles of 16 modes (P 16 | 17 | 33), l on
# both sides of a block of 128, ring counts that are and are not a multiple of a 16-ring stage,
# with and without an equator ring, columns past one block of 32, a last chunk of few pairs.
@pytest.mark.parametrize("lmax,ntheta,nphi,P,S,prec", [(3, 5, 8, 1, 1, "f32"), (127, 129, 256, 2, 3, "f32"),
                                                       (128, 161, 270, 16, 1, "f32"), (20, 32, 44, 17, 2, "f32"),
                                                       (17, 27, 54, 33, 1, "f32"), (130, 135, 264, 3, 11, "f64")])
def test_adjoint_edges(lmax, ntheta, nphi, P, S, prec):
    case = Case("edge", lmax, ntheta, nphi, P, S, "wmap", 73)
    print(f"[case] adjoint {prec} lmax={lmax} {ntheta}x{nphi} P={P} S={S}", flush=True)
    a = case.alms(0, S)
    rng = np.random.default_rng(lmax)
    cot = rng.standard_normal((S, P * (P + 1) * (P + 2) // 6))
    V = om.pair_means(case.maps(case.alms(50, 2)))
    c = _ctx(case, prec)
    st = c.linear_state()
    c.linear_reset(st)
    c.linear_accumulate(st, case.alms(50, 2))
    c.linear_finalize(st)
    got = c.beta_vjp(a, cot, state=st).cpu().numpy()
    tol = 1e-5 if prec == "f32" else 1e-10   # the bounds of the other gradient tests
    for i in range(S):
        ref = om.vjp(a[i], case.cl, case.q, case.grid, V, cot[i])[0]
        assert np.linalg.norm(got[i] - ref) <= tol * np.linalg.norm(ref)


# Ring transforms compiled in (nphi 1536, 3072, 6016) and a general one (1440), both directions,
# with ring groups of 8 that are not full, l_max far below and at the ring's limit.
@pytest.mark.parametrize("lmax,ntheta,nphi", [(20, 21, 1536), (767, 770, 1536), (20, 21, 3072), (20, 27, 6016),
                                              (20, 21, 1440)])
def test_ring_transform_edges(lmax, ntheta, nphi):
    P = 2
    case = Case("edge", lmax, ntheta, nphi, P, 1, "wmap", 74)
    print(f"[case] ring transforms lmax={lmax} {ntheta}x{nphi}", flush=True)
    a = case.alms(0, 1)
    c = _ctx(case, "f32")
    out = torch.full((1, P, ntheta, nphi), float("nan"), dtype=torch.float32, device="cuda")
    got = c.filter_maps(a, out=out).cpu().numpy()[0]
    ref = case.maps(a)[0]
    rms = np.sqrt(np.mean(ref * ref, axis=(1, 2)))
    assert np.all(np.max(np.abs(got - ref), axis=(1, 2)) <= 1e-5 * rms)
    cot = np.random.default_rng(5).standard_normal((1, 4))
    g = c.beta_vjp(a, cot).cpu().numpy()[0]
    gref = om.vjp(a[0], case.cl, case.q, case.grid, None, cot[0])[0]
    assert np.linalg.norm(g - gref) <= 1e-5 * np.linalg.norm(gref)


# FP64 linear algebra: n = P (P + 1) (P + 2) / 6 modes that end inside a 16-block, a 64 or 128 tile
# (35, 165), on none of them (4, 1), odd and even row lengths, one block column and several,
# sample counts on both sides of a 16-sample stage.  Tolerances: sums of N products agree to
# N eps of their absolute sum; the estimator to the condition number (below 100 here) times n eps.
@pytest.mark.parametrize("P,N", [(1, 1), (2, 17), (5, 33), (8, 16), (9, 165), (10, 250), (11, 40)])
@pytest.mark.parametrize("centered", [False, True])
def test_covariance_and_cholesky_edges(P, N, centered):
    case = Case("edge", 4, 6, 12, P, 1, "wmap", 73)
    c = _ctx(case, "f64")
    n = P * (P + 1) * (P + 2) // 6
    print(f"[case] linalg n={n} N={N} centered={centered}", flush=True)
    rng = np.random.default_rng(100 * P + N)
    b = rng.standard_normal((N, n)) + 0.5
    if not centered or N > 1:
        Z = c.covariance_sample(b, centered=centered).cpu().numpy()
        d = b - b.mean(0) if centered else b
        scale = 6.0 * (N - 1 if centered else N)
        bound = 4 * N * np.finfo(float).eps * (np.abs(d).T @ np.abs(d)) / scale
        if centered:
            bound += 4 * N * np.finfo(float).eps * np.abs(b).max() ** 2
        assert np.all(np.abs(Z - d.T @ d / scale) <= bound)
        assert np.array_equal(Z, Z.T)
    A = np.eye(n) + b.T @ b / (n + N)
    assert np.linalg.cond(A) < 100
    alpha, beta = rng.standard_normal(n), rng.standard_normal((3, n))
    E, s2, Lg = c.fnl(A, alpha, beta, want_L=True)
    ref = np.linalg.cholesky(A)
    tol = 100 * n * np.finfo(float).eps
    assert np.linalg.norm(Lg.cpu().numpy() - ref) <= tol * np.linalg.norm(ref)
    y = np.linalg.solve(A, alpha)
    assert abs(s2 * (alpha @ y) - 6.0) <= 6.0 * tol
    assert np.abs(E - beta @ y / (alpha @ y)).max() <= tol * np.abs(beta).sum(1).max()


# The first pivot that fails, wherever it lies in its 16-row block and its 64-row panel.
@pytest.mark.parametrize("bad", [0, 15, 16, 63, 64, 130, 164])
def test_cholesky_reports_first_bad_pivot(bad):
    from paper_1105_2791_amd import ModalError
    c = _ctx(Case("edge", 4, 6, 12, 9, 1, "wmap", 73), "f64")
    A = np.eye(165) * 2.0
    A[bad, bad] = -1.0
    if bad < 164:
        A[164, 164] = 0.0
    with pytest.raises(ModalError, match=rf"pivot {bad}\b"):
        c.fnl(A, np.ones(165), np.ones((1, 165)))


# Split synthesis: ring counts whose south rings are stored in pairs (even), one by one (odd, with
# the equator ring) and with a last pair cut by the ring count (2 mod 4), one and several blocks
# of 256 north rings, l_max on both sides of a chunk of 64 l, column blocks that are not full,
# pairs of several skies in a block; lambda from the table and from the recurrence.
@pytest.mark.parametrize("prec", ["bf16x3", "f16x3"])
@pytest.mark.parametrize("table", [True, False])
@pytest.mark.parametrize("lmax,ntheta,nphi,P,S", [(3, 5, 8, 2, 1), (63, 66, 130, 5, 2), (64, 129, 136, 7, 5),
                                                  (130, 514, 270, 3, 11), (40, 517, 90, 6, 6), (127, 128, 256, 1, 33)])
def test_split_synthesis_edges(lmax, ntheta, nphi, P, S, table, prec):
    from paper_1105_2791_amd import ModalContext
    case = Case("edge", lmax, ntheta, nphi, P, S, "wmap", 74)
    print(f"[case] split synthesis {prec} lmax={lmax} {ntheta}x{nphi} P={P} S={S} table={table}", flush=True)
    a = case.alms(0, S)
    c = ModalContext(lmax, ntheta, nphi, P, prec, case.q, case.cl, mask=case.mask(), lambda_table=table)
    out = torch.full((S, P, ntheta, nphi), float("nan"), dtype=torch.float32, device="cuda")
    got = c.filter_maps(a, out=out).cpu().numpy()
    ref = case.maps(a)
    tol = 1e-4 if prec == "bf16x3" else 1e-5   # the bounds of the map tests
    rms = np.sqrt(np.mean(ref * ref, axis=(2, 3)))
    assert np.all(np.max(np.abs(got - ref), axis=(2, 3)) <= tol * rms)


# Trispectrum update: one tile of 128 pairs and several (P 15 | 16 | 23 | 33), pairs that end inside
# a tile, 1, 2, 8 and 16 pixel chunks, pixel counts off a multiple of 4, skies alone and in
# pairs, with and without the pair means (whose own product fills or opens a pair).  Against FP64
# sums of the library's own maps: each operand is kept to 2^-17, their low parts' product
# (2^-18) is dropped and the FP32 chains round up to 100 times, which makes 2.6e-5 of the sums of
# the absolute terms; the bound is 4e-5 of them.
@pytest.mark.parametrize("lmax,ntheta,nphi,P,S", [(3, 5, 8, 1, 1), (20, 45, 90, 15, 2), (20, 64, 136, 16, 3),
                                                  (30, 130, 260, 23, 1), (40, 181, 370, 12, 5), (10, 40, 130, 33, 2)])
def test_trispectrum_edges(lmax, ntheta, nphi, P, S):
    from oracle import trispectrum as otr
    case = Case("edge", lmax, ntheta, nphi, P, S, "wmap", 75)
    print(f"[case] trispectrum lmax={lmax} {ntheta}x{nphi} P={P} S={S}", flush=True)
    a, mc = case.alms(0, S), case.alms(60, 2)
    c = _ctx(case, "bf16x3")
    st = c.linear_state()
    c.linear_reset(st)
    c.linear_accumulate(st, mc)
    c.linear_finalize(st)
    M = c.filter_maps(a).cpu().numpy().astype(np.float64).reshape(S, P, -1)
    V = om.pair_means(c.filter_maps(mc).cpu().numpy().astype(np.float64)).reshape(P * (P + 1) // 2, -1)
    w = np.broadcast_to(np.asarray(case.grid.w), (ntheta, nphi)).reshape(-1)
    pid = otr._pair_index(P)
    q = np.array(otr.quad_list(P))
    pair = np.array([[pid[(min(i, j), max(i, j))] for j in range(P)] for i in range(P)])
    pa, pb = np.triu_indices(P)
    order = pair[pa, pb]
    for state, Vs in ((None, 0.0 * V), (st, V)):
        got = c.trispectrum(a, state=state).cpu().numpy()
        for s in range(S):
            MM = np.empty_like(V)
            MM[order] = M[s][pa] * M[s][pb]
            A, B = MM - 3 * Vs, np.abs(MM) + 3 * np.abs(Vs)
            K = (A * w) @ A.T - 6 * ((Vs * w) @ Vs.T)
            Kabs = (B * np.abs(w)) @ B.T + 6 * ((np.abs(Vs) * np.abs(w)) @ np.abs(Vs).T)
            parts = [(pair[q[:, i], q[:, j]], pair[q[:, k], q[:, l]]) for i, j, k, l in ((0, 1, 2, 3), (0, 2, 1, 3), (0, 3, 1, 2))]
            ref = sum(K[x, y] for x, y in parts) / 3
            bound = 4e-5 * sum(Kabs[x, y] for x, y in parts) / 3
            assert np.all(np.abs(got[s] - ref) <= bound), (s, state is None, np.max(np.abs(got[s] - ref) / bound))


# Adjoint of the bf16 contexts: l_max on both sides of a block of 256 l, ring counts with 16-byte
# (even) and 8-byte (odd) aligned pairs, an equator ring alone in its pair, ring counts off a chunk of 32,
# the smallest grids, columns past a block of 64.
@pytest.mark.parametrize("lmax,ntheta,nphi,P,S", [(2, 3, 6, 1, 1), (2, 4, 6, 2, 1), (30, 33, 64, 7, 10),
                                                  (255, 259, 512, 2, 2), (256, 258, 514, 3, 1)])
def test_bf16_adjoint_edges(lmax, ntheta, nphi, P, S):
    case = Case("edge", lmax, ntheta, nphi, P, S, "wmap", 76)
    print(f"[case] bf16 adjoint lmax={lmax} {ntheta}x{nphi} P={P} S={S}", flush=True)
    a = case.alms(0, S)
    cot = np.random.default_rng(lmax).standard_normal((S, P * (P + 1) * (P + 2) // 6))
    got = _ctx(case, "bf16x3").beta_vjp(a, cot).cpu().numpy()
    for i in range(S):
        ref = om.vjp(a[i], case.cl, case.q, case.grid, None, cot[i])[0]
        assert np.linalg.norm(got[i] - ref) <= 1e-4 * np.linalg.norm(ref)   # the map bound of these contexts


# Linear term in harmonic space: workgroup counts on both sides of 128 (2 pairs and 16 waves below, 8
# and 4 from there), pair counts off a multiple of 2 and of 8, l_max on both sides of an l tile
# of 64 and below the 16 waves, more maps than a workgroup takes.
@pytest.mark.parametrize("lmax,ntheta,nphi,P,S", [(2, 3, 6, 1, 1), (9, 14, 30, 2, 9), (63, 66, 130, 5, 3),
                                                  (64, 66, 130, 10, 12), (64, 66, 130, 10, 80)])
@pytest.mark.parametrize("prec", ["f32", "f64"])
def test_linear_apply_edges(lmax, ntheta, nphi, P, S, prec):
    case = Case("edge", lmax, ntheta, nphi, P, S, "wmap", 77)
    print(f"[case] linear apply {prec} lmax={lmax} P={P} S={S}", flush=True)
    a, mc = case.alms(0, S), case.alms(200, 2)
    c = _ctx(case, prec)
    st = c.linear_state()
    c.linear_reset(st)
    c.linear_accumulate(st, mc)
    c.linear_finalize(st)
    got = c.linear_apply(st, a).cpu().numpy()
    V = om.pair_means(case.maps(mc))
    tol = 1e-5 if prec == "f32" else 1e-10   # the bounds of the linear-term tests
    for i in {0, S // 2, S - 1}:
        ref = om.linear_term(case.maps(a[i:i + 1])[0], case.grid.w, V)
        assert np.abs(got[i] - ref).max() <= tol * np.abs(ref).max()


# The modes of the linear term: one to four tiles of 16 modes (P 16 | 17, 33, 49), l in a single
# block of 32, at its edge and in blocks for every wave and more, rows off a multiple of 16.
@pytest.mark.parametrize("lmax,ntheta,nphi,P,S", [(30, 33, 64, 16, 1), (31, 33, 64, 17, 2), (32, 34, 66, 33, 1),
                                                  (9, 14, 30, 49, 1), (129, 131, 260, 4, 2), (160, 162, 322, 3, 1)])
def test_linear_modes_edges(lmax, ntheta, nphi, P, S):
    case = Case("edge", lmax, ntheta, nphi, P, S, "wmap", 78)
    print(f"[case] linear modes lmax={lmax} P={P} S={S}", flush=True)
    a, mc = case.alms(0, S), case.alms(200, 2)
    c = _ctx(case, "f64")
    st = c.linear_state()
    c.linear_reset(st)
    c.linear_accumulate(st, mc)
    c.linear_finalize(st)
    got = c.linear_apply(st, a).cpu().numpy()
    V = om.pair_means(case.maps(mc))
    for i in range(S):
        ref = om.linear_term(case.maps(a[i:i + 1])[0], case.grid.w, V)
        assert np.abs(got[i] - ref).max() <= 1e-10 * np.abs(ref).max()   # the bound of the linear-term tests


# FP32 synthesis of skies so large that the last of a block's 32 skies (P 1) lies past 32-bit byte
# offsets from the first: each sky of a batch equals the sky alone (columns do not mix), bit for bit.
def test_f32_synthesis_offsets_past_32_bits():
    from paper_1105_2791_amd import ModalContext
    lmax, ntheta, nphi, S = 5884, 5885, 12288, 32
    assert 8 * (S - 1) * (lmax + 1) * (lmax + 2) // 2 > 2**32
    print(f"[case] f32 synthesis lmax={lmax} {ntheta}x{nphi} P=1 S={S}", flush=True)
    c = ModalContext(lmax, ntheta, nphi, 1, "f32", np.ones((1, lmax + 1)), np.ones(lmax + 1))
    g = torch.Generator(device="cuda").manual_seed(3)
    a = torch.view_as_complex(torch.randn((S, c.nalm, 2), generator=g, device="cuda"))
    got = c.filter_maps(a)
    for s in (0, 30, 31):
        assert torch.equal(got[s:s + 1], c.filter_maps(a[s:s + 1]))


# A state finalised over each form of the ring transform that scales and weights its rows as they are
# loaded: plans of at most 16, 24, 32 and 48 points per lane run from their arguments (nphi 1440, 2560,
# 4096, 3840) and the compiled ones (1536, 3072, 6016).  Both what it writes: the pair means in place
# and, through the linear term, their harmonic transform.
@pytest.mark.parametrize("nphi", [1440, 1536, 2560, 3072, 3840, 4096, 6016])
@pytest.mark.parametrize("prec", ["f32", "bf16x3"])
def test_finalized_state_of_each_ring_transform(nphi, prec):
    lmax, ntheta, P, S = 20, 27, 3, 2
    case = Case("edge", lmax, ntheta, nphi, P, S, "wmap", 79)
    print(f"[case] finalised state {prec} {ntheta}x{nphi}", flush=True)
    a, mc = case.alms(0, S), case.alms(60, 3)
    c = _ctx(case, prec)
    st = c.linear_state()
    c.linear_reset(st)
    c.linear_accumulate(st, mc)
    c.linear_finalize(st)
    Mmc = case.maps(mc)
    V, rms = om.pair_means(Mmc), np.sqrt(np.mean(Mmc**2, axis=(0, 2, 3)))
    pa, pb = np.triu_indices(P)
    tol = 1e-5 if prec == "f32" else 1e-4   # the map bounds: twice them for a product of two maps
    err = np.abs(c.pair_means(st).cpu().numpy() - V).reshape(len(pa), -1).max(1)
    assert np.all(err <= 2 * tol * rms[pa] * rms[pb])
    got = c.linear_apply(st, a).cpu().numpy()
    for i in range(S):
        ref = om.linear_term(case.maps(a[i:i + 1])[0], case.grid.w, V)
        assert np.abs(got[i] - ref).max() <= tol * np.sqrt(np.mean(ref**2))


# Maps written over the a_lm they are formed from, which lie at the start, in the middle or at the end
# of their memory: what separate memory gives, bit for bit.
@pytest.mark.parametrize("prec", ["f32", "f64", "bf16x3"])
@pytest.mark.parametrize("where", [0.0, 0.4, 1.0])
def test_maps_over_their_own_alm(prec, where):
    lmax, ntheta, nphi, P, S = 64, 130, 136, 7, 14
    case = Case("edge", lmax, ntheta, nphi, P, S, "wmap", 80)
    print(f"[case] maps over alm {prec} at {where}", flush=True)
    c = _ctx(case, prec)
    a = torch.as_tensor(case.alms(0, S)).to("cuda", c.complex_dtype)
    ref = c.filter_maps(a)
    out = torch.zeros_like(ref)
    room = out.numel() - 2 * a.numel()
    at = int(where * room) // 64 * 64
    inside = torch.view_as_complex(out.view(-1)[at:at + 2 * a.numel()].view(-1, 2)).view(S, c.nalm)
    inside.copy_(a)
    assert torch.equal(c.filter_maps(inside, out=out), ref)


# The covariance's two tiles: 64 rows (1771 modes, 210 tiles of 128 rows) and 128 (2024 modes, 272), odd
# and even row lengths, sample counts off a stage of 16.  Against FP64 within the bound above,
# and the modes that both hold are the same bit for bit.
@pytest.mark.parametrize("N", [17, 200])
def test_covariance_tile_forms(N):
    print(f"[case] covariance tiles N={N}", flush=True)
    b = np.random.default_rng(N).standard_normal((N, 2024)) + 0.5
    Z = {}
    for P, n in ((21, 1771), (22, 2024)):
        d = np.ascontiguousarray(b[:, :n])
        Z[n] = _ctx(Case("edge", 4, 6, 12, P, 1, "wmap", 73), "f64").covariance_sample(d).cpu().numpy()
        bound = 4 * N * np.finfo(float).eps * (np.abs(d).T @ np.abs(d)) / (6.0 * N)
        assert np.all(np.abs(Z[n] - d.T @ d / (6.0 * N)) <= bound)
        assert np.array_equal(Z[n], Z[n].T)
    assert np.array_equal(Z[2024][:1771, :1771], Z[1771])


# A mode of infinite variance has no weight: the estimator of the other modes, wherever it lies.
@pytest.mark.parametrize("mode", [0, 15, 16, 63, 64, 130, 164])
def test_cholesky_infinite_pivot(mode):
    n = 165
    print(f"[case] infinite pivot {mode}", flush=True)
    rng = np.random.default_rng(mode)
    b = rng.standard_normal((2 * n, n))
    A = np.eye(n) + b.T @ b / n
    alpha, beta = rng.standard_normal(n), rng.standard_normal((2, n))
    keep = np.arange(n) != mode
    y = np.linalg.solve(A[np.ix_(keep, keep)], alpha[keep])
    A[mode, mode] = np.inf
    E, s2 = _ctx(Case("edge", 4, 6, 12, 9, 1, "wmap", 73), "f64").fnl(A, alpha, beta)
    tol = 100 * n * np.finfo(float).eps   # as the factor of the other modes above
    assert abs(s2 * (alpha[keep] @ y) - 6.0) <= 6.0 * tol
    assert np.abs(E - beta[:, keep] @ y / (alpha[keep] @ y)).max() <= tol * np.abs(beta).sum(1).max()


# Backward error of the factor over nine 128-wide block columns: an entry's old value meets a rounded
# sum once per block column, half an eps of sqrt(A_ii A_jj) each at most, and as much again for
# the sums themselves.
@pytest.mark.parametrize("seed", [0, 1])
def test_cholesky_backward_error(seed):
    P, n = 18, 1140
    print(f"[case] cholesky backward error n={n}", flush=True)
    rng = np.random.default_rng(seed)
    b = rng.standard_normal((n + n // 4, n)) * np.exp(rng.uniform(-3, 3, n))
    A = b.T @ b / len(b)
    A = (A + A.T) / 2
    _, _, L = _ctx(Case("edge", 4, 6, 12, P, 1, "wmap", 73), "f64").fnl(A, np.ones(n), np.ones((1, n)), want_L=True)
    L = L.cpu().numpy()
    d = np.sqrt(np.diag(A))
    assert np.abs((A - L @ L.T) / np.outer(d, d)).max() <= (n / 128 + 1) * np.finfo(float).eps


# A sky's results do not depend on the batch it comes in, bit for bit: batches on both sides of where
# the linear term changes its split (8 and 160 skies: 14 and 280 workgroups of 8 pairs), where the
# FP32 synthesis takes its table and where a second block of skies begins.
@pytest.mark.parametrize("prec", ["f32", "f64", "bf16x3", "f16x3"])
@pytest.mark.parametrize("lmax,ntheta,nphi,P,S", [(64, 66, 130, 10, 160), (150, 152, 304, 13, 31)])
def test_batch_independence(lmax, ntheta, nphi, P, S, prec):
    case = Case("edge", lmax, ntheta, nphi, P, S, "wmap", 81)
    print(f"[case] batch independence {prec} lmax={lmax} P={P} S={S}", flush=True)
    c = _ctx(case, prec)
    a = torch.as_tensor(case.alms(0, S)).to("cuda", c.complex_dtype)
    st = c.linear_state()
    c.linear_reset(st)
    c.linear_accumulate(st, a[:2])
    c.linear_finalize(st)
    lin, hat = c.linear_apply(st, a), c.beta(a, state=st)
    for lo, hi in ((0, 1), (S // 2, S // 2 + 8), (S - 10, S)):
        assert torch.equal(c.linear_apply(st, a[lo:hi]), lin[lo:hi])
        assert torch.equal(c.beta(a[lo:hi], state=st), hat[lo:hi])


# Adjoint of the bf16 contexts with two and four blocks of 128 l per m, whose order turns with m, the
# last of them empty for most m, and with two blocks of columns.
@pytest.mark.parametrize("lmax,ntheta,nphi,P,S", [(128, 130, 260, 13, 5), (385, 387, 772, 1, 1)])
def test_bf16_adjoint_block_order(lmax, ntheta, nphi, P, S):
    case = Case("edge", lmax, ntheta, nphi, P, S, "wmap", 82)
    print(f"[case] bf16 adjoint blocks lmax={lmax} {ntheta}x{nphi} P={P} S={S}", flush=True)
    a = case.alms(0, S)
    cot = np.random.default_rng(lmax).standard_normal((S, P * (P + 1) * (P + 2) // 6))
    got = _ctx(case, "bf16x3").beta_vjp(a, cot).cpu().numpy()
    for i in {0, S - 1}:
        ref = om.vjp(a[i], case.cl, case.q, case.grid, None, cot[i])[0]
        assert np.linalg.norm(got[i] - ref) <= 1e-4 * np.linalg.norm(ref)   # the map bound of these contexts


# Workspaces hold what their call uses and no more: their sizes by region, and results with a buffer
# of exactly that size, whose neighbourhood stays untouched.  Ring transforms with a register-pass
# plan (a state's rows are weighted as they are loaded: no plane of them) and the general one.
@pytest.mark.parametrize("prec,nphi", [("f32", 96), ("bf16x3", 96), ("f32", 94), ("f64", 96)])
def test_workspaces_hold_what_is_used(prec, nphi):
    from paper_1105_2791_amd import _lib as L
    lmax, ntheta, P, S = 32, 48, 12, 2
    case = Case("edge", lmax, ntheta, nphi, P, S, "wmap", 83)
    print(f"[case] workspaces {prec} {ntheta}x{nphi}", flush=True)
    c = _ctx(case, prec)
    rb, npairs, planes = c.real_dtype.itemsize, P * (P + 1) // 2, min(P * (P + 1) // 2, 64)
    F, maps, Lrow = S * P * ((ntheta + 7) // 8) * 8 * (lmax + 1) * 2 * rb, S * P * ntheta * nphi * rb, S * npairs * P * 8
    X = S * npairs * (lmax + 1) * 8

    def size(*regions):
        return sum((b + 255) // 256 * 256 for b in regions)
    part = c.workspace_size(L.OP_BETA, S) - size(F, maps, X, Lrow)
    assert part > 0 and part % Lrow < 256   # the contraction's chunks alone, [S][chunk][pairs][P]
    lam, Gh = c.nalm * ((ntheta + 1) // 2) * rb, planes * ntheta * (lmax + 1) * 2 * rb
    general = prec == "f64" or nphi == 94
    assert c.workspace_size(L.OP_LINEAR_FINALIZE, 1) == size(lam, *([planes * ntheta * nphi * rb] if general else []), Gh)

    a, mc = case.alms(0, S), case.alms(60, 3)
    guard = 4096

    def run():
        st = c.linear_state()
        c.linear_reset(st)
        c.linear_accumulate(st, mc)
        c.linear_finalize(st)
        return c.beta(a, state=st), c.beta(a), c.beta_loo(mc[:2], st)
    ref = run()
    bufs = []

    def exact(op, n):
        need = c.workspace_size(op, n)
        t = torch.full((need + 2 * guard,), 255, dtype=torch.uint8, device="cuda")
        bufs.append((t, need))
        return t[guard:guard + need]
    c.workspace = exact
    got = run()
    for x, y in zip(got, ref):
        assert torch.equal(x, y)
    for t, need in bufs:
        assert bool((t[:guard] == 255).all()) and bool((t[guard + need:] == 255).all())


# Ring transforms run from their plan's arguments, both directions: rings of two pixels (no pass), last
# passes of every radix (8: nphi 16, 4: 8, 2: 20 x 2, 3: 6, 5: 30), strides that are and are not powers of
# two, rounds of 3 and of 4 spectrum elements, and plans of up to 16, 24, 32 and 48 points per lane.
@pytest.mark.parametrize("nphi", [2, 6, 8, 16, 20, 30, 54, 200, 720, 1536, 1600, 2048, 2400, 2700, 3000, 3600, 4050, 4096])
def test_ring_transform_plans(nphi):
    lmax, P = min(12, (nphi - 1) // 2), 2
    ntheta = lmax + 2
    case = Case("edge", lmax, ntheta, nphi, P, 1, "wmap", 84)
    print(f"[case] ring plan {ntheta}x{nphi}", flush=True)
    if lmax < 2:
        case.__dict__.update(cl=np.ones(lmax + 1), q=np.linspace(0.5, 1.0, P * (lmax + 1)).reshape(P, lmax + 1))
    a = case.alms(0, 1)
    c = _ctx(case, "f32")
    out = torch.full((1, P, ntheta, nphi), float("nan"), dtype=torch.float32, device="cuda")
    got, ref = c.filter_maps(a, out=out).cpu().numpy()[0], case.maps(a)[0]
    rms = np.sqrt(np.mean(ref * ref, axis=(1, 2)))
    assert np.all(np.max(np.abs(got - ref), axis=(1, 2)) <= 1e-5 * rms)
    cot = np.random.default_rng(5).standard_normal((1, 4))
    g = c.beta_vjp(a, cot).cpu().numpy()[0]
    gref = om.vjp(a[0], case.cl, case.q, case.grid, None, cot[0])[0]
    assert np.linalg.norm(g - gref) <= 1e-5 * np.linalg.norm(gref)
