"""A block whose stored inverse overflows (pivots of 2^-1020 are accepted, sums
of their reciprocals are not finite) leaves the steps of the other blocks alone,
whose kernels read a few columns past their own inverses.

Bar: 1e-10 relative to the same steps in FP64 on the host (well conditioned
blocks of 20 rows)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2510_02156_amd as P  # noqa: E402
from tests.gpu_util import dev, host, rel  # noqa: E402

B, BAD = 20, 3   # rows per block, the block that overflows


@pytest.mark.parametrize("kind,n", [("dense", 60), ("dense", 5000), ("csr", 60)])
def test_overflowing_inverse_stays_in_its_block(kind, n):
    m, iters = 6 * B, 4
    rng = np.random.default_rng(n)
    A = rng.standard_normal((m, n))
    A[BAD * B:(BAD + 1) * B] = 0.0
    for i in range(B):                      # s e_0, s (e_0 + e_i): every pivot s^2
        A[BAD * B + i, 0] = A[BAD * B + i, i] = 2.0 ** -510
    b = A @ rng.standard_normal(n)
    tau = np.array([0, 1, 2] * iters, dtype=np.int32)
    I = np.stack([np.arange(4 * B, 5 * B, dtype=np.int32)] * iters)
    if kind == "csr":
        rows, cols = np.nonzero(A)
        sol = P.Solver(None, B, 0.0, rowptr=dev(np.searchsorted(rows, np.arange(m + 1)), torch.int64),
                       colidx=dev(cols, torch.int32), values=dev(A[rows, cols]), shape=(m, n))
    else:
        sol = P.Solver(dev(A), B, 0.0)
    assert np.isinf(sol.block_inverse(BAD)).any() and np.isfinite(sol.block_inverse(BAD - 1)).all()
    sol.set_replay(tau, I, iters)
    print(f"overflowing neighbour {kind} n={n}", flush=True)
    x, _ = sol.solve(dev(b), tol=0.0, max_iters=iters, replay=True, record=True)
    want = np.zeros(n)
    sets = [S for it in range(iters) for S in (np.arange(B), np.arange(B, 2 * B),
                                               np.arange(2 * B, 3 * B), I[it])]
    for S in sets:
        want = want + A[S].T @ np.linalg.solve(A[S] @ A[S].T, b[S] - A[S] @ want)
    assert rel(host(x), want) < 1e-10
    g = rng.standard_normal(n)
    gb, gx0 = sol.backward(dev(g))
    for S in sets[::-1]:
        g = g - A[S].T @ np.linalg.solve(A[S] @ A[S].T, A[S] @ g)
    assert np.isfinite(host(gb)).all()
    assert np.linalg.norm(host(gx0) - g) < 1e-10 * np.sqrt(n)


@pytest.mark.parametrize("br", [1, 2])
@pytest.mark.parametrize("csr", [False, True])
def test_one_row_blocks_of_any_norm(br, csr):
    """Blocks of one row: every positive squared norm is accepted, also one
    whose reciprocal overflows (a last row of 2^-520 here)."""
    m, n = 2 * br + 1, 40                       # the last block has one row for br = 1
    A = np.random.default_rng(br).standard_normal((m, n))
    if br == 1:
        A[-1] = 0.0
        A[-1, 3] = 2.0 ** -520
    if csr:
        rows, cols = np.nonzero(A)
        sol = P.Solver(None, br, 0.0, rowptr=dev(np.searchsorted(rows, np.arange(m + 1)), torch.int64),
                       colidx=dev(cols, torch.int32), values=dev(A[rows, cols]), shape=(m, n))
    else:
        sol = P.Solver(dev(A), br, 0.0)
    off = sol.setup_arrays()["offsets"]
    for t in range(sol.k):
        G = A[off[t]:off[t + 1]] @ A[off[t]:off[t + 1]].T
        with np.errstate(divide="ignore", over="ignore"):
            want = 1.0 / G if len(G) == 1 else np.linalg.inv(G)
        np.testing.assert_allclose(sol.block_inverse(t), want, rtol=1e-13)
    zero = A.copy()
    zero[-1] = 0.0
    with pytest.raises(P.RorBkError) as e:
        P.Solver(dev(zero), br, 0.0)
    assert e.value.code == P.RORBK_ERR_NOT_SPD
