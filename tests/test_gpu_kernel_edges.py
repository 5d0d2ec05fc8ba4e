


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
