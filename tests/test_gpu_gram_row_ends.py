"""Grams of rows of every alignment and length (the block Grams of the setup,
the greedy Gram and the Grams of the chain form): rows shorter than one 16-byte
vector, rows that end inside a wave's step, at its end and one element past it.

The stored inverse H of a block is held against (A_t A_t^T + lam I) in FP64:
||H M - I|| is at most a few times b cond(M) 2^-53, cond(M) <= 1e4 with the lam
taken here, so 1e-9 (wide blocks of few columns: the Gram of the columns).  Solves are held
against the FP64 oracle on the stored values with its selections: 1e-10, 1e-4
with FP32 vectors."""
import numpy as np
import pytest

import oracle as O

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2510_02156_amd as P  # noqa: E402
from tests.gpu_util import bf16_tensor, bf16_values, dev, host, rel  # noqa: E402


@pytest.mark.parametrize("storage", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("br", [1, 11, 33, 64, 120, 200])
@pytest.mark.parametrize("n", [1, 3, 7, 9, 63, 129, 515, 1030, 2311, 4095])
def test_grams_at_row_ends(storage, br, n):
    m, iters = 5 * br + 2, 3
    lam = 0.01 * (n + br)
    rng = np.random.default_rng(1000 * br + n)
    A = rng.standard_normal((m, n))
    if storage == "bf16":
        At, v = bf16_tensor(A), bf16_values(A)
    else:
        At = dev(A, torch.float64 if storage == "f64" else torch.float32)
        v = host(At).astype(np.float64)
    vec = torch.float64 if storage == "f64" else torch.float32
    b = host(dev(v @ rng.standard_normal(n), vec)).astype(np.float64)
    print(f"row ends {storage} br={br} n={n}", flush=True)
    sol = P.Solver(At, br, lam)
    off = sol.setup_arrays()["offsets"]
    for t in (0, len(off) - 2):
        H = np.asarray(sol.block_inverse(t))
        At_ = v[off[t]:off[t + 1]]
        M = At_.T @ At_ if sol.column_form else At_ @ At_.T
        M[np.diag_indices_from(M)] += lam
        assert np.linalg.cond(M) < 1e4
        assert np.linalg.norm(H @ M - np.eye(len(M))) < 1e-9
    ref = O.solve(v, br, lam, b, seed=9, max_iters=iters)
    sol.set_replay(ref["tau"], ref["I"], iters)
    x, _ = sol.solve(dev(b, vec), tol=0.0, max_iters=iters, replay=True)
    assert rel(host(x), ref["x"]) < (1e-10 if storage == "f64" else 1e-4)
