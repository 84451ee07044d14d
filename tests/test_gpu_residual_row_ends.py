"""The residual on rows of any alignment: rows shorter than a 16-byte vector, rows
that end inside a slice of 64 lanes, at its end and one element past it, half a
vector past 16-byte alignment, with few rows (one per wave) and with many.

Bars: the products are summed in the vector type (each lane in column order,
then a six-level butterfly; the segments in FP64), then r is rounded to it: at
most n + 8 roundings of terms whose magnitudes sum to |A||x| + |b|."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2510_02156_amd as P  # noqa: E402
from tests.gpu_util import bf16_tensor, bf16_values, dev, host  # noqa: E402


@pytest.mark.parametrize("storage", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("m,n", [(5, 1), (7001, 1), (7001, 3), (40, 127), (9001, 129), (300, 204),
                                 (9003, 204), (6001, 513), (200, 601), (9001, 1023), (50, 1025),
                                 (7003, 604), (300, 2049), (5001, 2049), (90, 4101), (70, 7468)])
def test_residual_at_row_ends(storage, m, n):
    rng = np.random.default_rng(31 * m + n)
    A = rng.standard_normal((m, n))
    if storage == "bf16":
        At, v = bf16_tensor(A), bf16_values(A)
    else:
        At = dev(A, torch.float64 if storage == "f64" else torch.float32)
        v = host(At).astype(np.float64)
    vec = torch.float64 if storage == "f64" else torch.float32
    x = host(dev(rng.standard_normal(n), vec)).astype(np.float64)
    b = host(dev(rng.standard_normal(m), vec)).astype(np.float64)
    print(f"residual {storage} {m}x{n}", flush=True)
    r, _, _ = P.Solver(At, 2, 1e-1).residual(dev(b, vec), dev(x, vec))
    eps = 2.0 ** -53 if storage == "f64" else 2.0 ** -24
    # the reference itself is summed in FP64
    bound = (n + 8) * (eps + 2.0 ** -53) * 1.01 * (np.abs(v) @ np.abs(x) + np.abs(b))
    assert np.all(np.abs(host(r) - (b - v @ x)) <= bound)
