"""The adjoint's greedy steps: a set whose Gram is not positive definite is
reported from whichever checkpoint segment it lies in; sets of rows that nearly
repeat lose no more accuracy than factor solves do; Grams in many column chunks
(wide matrices) give the same bits however many sets go together.

Bars: FP64 1e-10 relative to the oracle's adjoint; for rows that nearly repeat the
distance from the adjoint in 80-bit arithmetic may be at most 8 times the FP64 oracle's, which solves with the factor at every step (the
two differ in summation order only, so their distances are of one size)."""
import numpy as np
import pytest

import oracle as O

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2510_02156_amd as P  # noqa: E402
from tests.gpu_util import dev, host  # noqa: E402


def raises_not_spd(f):
    try:
        f()
    except P.RorBkError as e:
        assert e.code == P.RORBK_ERR_NOT_SPD
        return True
    return False


# Every row of a "kind" is one vector with its signs flipped, so all have the
# same squared norm a, and each row stands twice in the matrix: the greedy pair
# [[a, a], [a, a]] at lambda = 0 has the second pivot a - a (a / a), zero or a
# rounding of either sign.  The forward step and the adjoint add a's terms in
# different orders, so a vector can be found whose pivot is positive in one and
# not in the other.
N_COLS, PAIRS = 200, 6


def kind_rows(seed, rows):
    rng = np.random.default_rng(seed)
    v = rng.standard_normal(N_COLS)
    return v * rng.choice([-1.0, 1.0], (rows, N_COLS))


def pair_system(rows, seed):
    A = np.vstack([rows, rows])
    return P.Solver(dev(A), 2, 0.0), dev(A @ np.random.default_rng(seed).standard_normal(N_COLS))


def outcome(sol, b, iters, every=0):
    """(forward failed, backward failed) of one recorded solve."""
    if raises_not_spd(lambda: sol.solve(b, seed=2, tol=0.0, max_iters=iters, record=not every,
                                        checkpoint_every=every)):
        return True, True
    g = dev(np.ones(N_COLS))
    return False, raises_not_spd(lambda: sol.backward(g))


def failure(sol, b, iters):
    try:
        sol.solve(b, seed=2, tol=0.0, max_iters=iters)
    except P.RorBkError as e:
        assert e.code == P.RORBK_ERR_NOT_SPD
        return str(e)
    return ""


def find_kind(alone_ok):
    """Seed of a vector that passes in the greedy step fused with the next
    iteration's sampled ones and, as alone_ok says, passes or fails in the
    greedy step of the last iteration, which adds its terms as the adjoint does."""
    for s in range(3000):
        sol, b = pair_system(kind_rows(s, PAIRS), s)
        if ("iteration 0" not in failure(sol, b, 2)) and (failure(sol, b, 1) == "") == alone_ok:
            return s
    return None


def test_failing_set_in_any_checkpoint_segment():
    sp, sf = find_kind(True), find_kind(False)
    print("kinds", sp, sf, flush=True)
    if sp is None or sf is None:
        pytest.skip("no vector whose pivot changes sign between the two sums")
    half = PAIRS // 2
    rows = np.vstack([kind_rows(sp, half), kind_rows(sf, half)])
    hits = 0
    for s in range(400):
        sol, b = pair_system(rows[np.random.default_rng(s).permutation(PAIRS)], s)
        for iters in (3, 4):
            fwd, back = outcome(sol, b, iters)
            if fwd:
                continue
            for every in (1, 2, 3):
                assert outcome(sol, b, iters, every) == (False, back), (s, iters, every)
            hits += back
        if hits > 20:
            break
    print("failing adjoints", hits, flush=True)
    assert hits > 0


def adjoint_80bit(A, br, lam, tau, I, g):
    L = np.longdouble
    A, g = A.astype(L), g.astype(L)
    off = O.partition(len(A), br)
    gb = np.zeros(len(A), L)
    for it in range(len(I) - 1, -1, -1):
        for S in [I[it]] + [np.arange(off[t], off[t + 1]) for t in tau[3 * it:3 * it + 3][::-1]]:
            As = A[S]
            M, z = As @ As.T + L(lam) * np.eye(len(S), dtype=L), As @ g
            low = np.zeros_like(M)
            for k in range(len(S)):                 # L D L^T
                low[k + 1:, k] = M[k + 1:, k] / M[k, k]
                M[k + 1:, k + 1:] -= np.outer(low[k + 1:, k], M[k, k + 1:])
                z[k + 1:] -= low[k + 1:, k] * z[k]
            y = z / np.diag(M)
            for k in range(len(S) - 2, -1, -1):
                y[k] -= low[k + 1:, k] @ y[k + 1:]
            gb[S] += y
            g = g - As.T @ y
    return gb, g


@pytest.mark.parametrize("br,m,csr", [(20, 400, False), (64, 640, False), (65, 650, False),
                                      (100, 1000, False), (160, 1280, False), (64, 640, True),
                                      (160, 1280, True)])
def test_accuracy_on_rows_that_nearly_repeat(br, m, csr):
    n, lam, iters = 330, 1e-6 * br, 12
    rng = np.random.default_rng(br)
    B = rng.standard_normal((m // 2, n))
    if csr:
        B *= rng.random((m // 2, n)) < 0.2
    A = np.vstack([B, B + 1e-4 * rng.standard_normal((m // 2, n)) * (B != 0)])
    b, g = A @ rng.standard_normal(n), rng.standard_normal(n)
    ref = O.solve(A, br, lam, b, seed=5, max_iters=iters)
    if csr:
        rows, cols = np.nonzero(A)
        sol = P.Solver(None, br, lam, rowptr=dev(np.searchsorted(rows, np.arange(m + 1)), torch.int64),
                       colidx=dev(cols, torch.int32), values=dev(A[rows, cols]), shape=(m, n))
    else:
        sol = P.Solver(dev(A), br, lam)
    sol.set_replay(ref["tau"], ref["I"], iters)
    sol.solve(dev(b), tol=0.0, max_iters=iters, replay=True, record=True)
    got = [host(t) for t in sol.backward(dev(g))]
    orc = O.backward(A, br, lam, ref["tau"], ref["I"], iters, False, g)
    want = adjoint_80bit(A, br, lam, np.asarray(ref["tau"]).reshape(-1), ref["I"], g)
    for what, x, o, w in zip(("dL/db", "dL/dx0"), got, orc, want):
        e, eo = (float(np.linalg.norm(v - w) / np.linalg.norm(w)) for v in (x, o))
        print(f"near repeats br={br} csr={csr} {what}: {e:.1e}, oracle {eo:.1e}", flush=True)
        assert e <= 8 * eo


@pytest.mark.parametrize("br,n,iters", [(1, 5001, 65), (10, 5001, 65), (33, 17000, 9),
                                        (64, 5002, 9), (100, 20000, 5), (161, 5001, 3)])
def test_wide_matrices_in_batches_of_any_size(br, n, iters):
    m, lam = 3 * br + 5, 1e-2
    rng = np.random.default_rng(br)
    A, g = rng.standard_normal((m, n)), rng.standard_normal(n)
    b = A @ rng.standard_normal(n)
    sol = P.Solver(dev(A), br, lam)
    sol.solve(dev(b), seed=4, tol=0.0, max_iters=iters, record=True)
    rec = sol.record()
    got = sol.backward(dev(g))
    want = O.backward(A, br, lam, rec["tau"], rec["I"], iters, False, g)
    print(f"wide adjoint br={br} n={n}", flush=True)
    for x, w in zip(got, want):
        assert np.linalg.norm(host(x) - w) < 1e-10 * np.linalg.norm(w)
    for every in (1, 2, 4):
        sol.solve(dev(b), seed=4, tol=0.0, max_iters=iters, checkpoint_every=every)
        assert all(torch.equal(x, y) for x, y in zip(sol.backward(dev(g)), got)), every
