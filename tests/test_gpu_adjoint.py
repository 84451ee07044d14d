"""The adjoint's greedy steps: a set whose Gram is not positive definite is
reported from whichever checkpoint segment it lies in."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2510_02156_amd as P  # noqa: E402
from tests.gpu_util import dev  # noqa: E402


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
