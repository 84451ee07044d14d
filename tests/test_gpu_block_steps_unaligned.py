"""Block steps of 65 to 161 rows on rows of every alignment (the forms of the
step with the most rows per thread), forward and adjoint, against the FP64
oracle on the stored values with its selections.

Bars: FP64 1e-10, FP32 and BF16 storage 1e-4 relative."""
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
@pytest.mark.parametrize("br", [65, 72, 100, 136, 160, 161])
@pytest.mark.parametrize("n", [770, 1021, 1024, 9001])
def test_steps_of_large_blocks_on_any_alignment(storage, br, n):
    m, lam, iters = 5 * br, 1e-2, 5
    rng = np.random.default_rng(n + br)
    A = rng.standard_normal((m, n))
    if storage == "bf16":
        At, v = bf16_tensor(A), bf16_values(A)
    else:
        At = dev(A, torch.float64 if storage == "f64" else torch.float32)
        v = host(At).astype(np.float64)
    vec = torch.float64 if storage == "f64" else torch.float32
    bar = 1e-10 if storage == "f64" else 1e-4
    b = host(dev(v @ rng.standard_normal(n), vec)).astype(np.float64)
    g = host(dev(rng.standard_normal(n), vec)).astype(np.float64)
    ref = O.solve(v, br, lam, b, seed=6, max_iters=iters)
    print(f"steps {storage} br={br} n={n}", flush=True)
    sol = P.Solver(At, br, lam)
    sol.set_replay(ref["tau"], ref["I"], iters)
    x, _ = sol.solve(dev(b, vec), tol=0.0, max_iters=iters, replay=True, record=True)
    assert rel(host(x), ref["x"]) < bar
    gb, gx0 = sol.backward(dev(g, vec))
    rb, rx0 = O.backward(v, br, lam, ref["tau"], ref["I"], iters, False, g)
    assert rel(host(gb), rb) < bar
    assert np.linalg.norm(host(gx0) - rx0) < bar * np.linalg.norm(g)
