"""Device memory of closed handles: given back by ror_bk_trim and at the pool's
bounds (the bounds themselves: test_block_pool.py), and handles made and closed
by two threads at once, each on its own stream."""
import threading

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2510_02156_amd as P  # noqa: E402
from tests.gpu_util import DEV, dev  # noqa: E402

MB = 1 << 20


def free_bytes():
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


def test_trim_gives_the_memory_of_closed_handles_back():
    A = torch.randn(160000, 16, dtype=torch.float64, device=DEV)
    P.ror_bk_trim()
    before = free_bytes()
    sol = P.Solver(A, 160, 1e-1)      # 1000 blocks of 160 rows: 205 MB
    held = before - free_bytes()
    assert held > 200 * MB
    sol.close()
    idle = before - free_bytes()
    assert idle > 200 * MB                    # kept for the next handle
    again = P.Solver(A, 160, 1e-1)
    assert before - free_bytes() <= held + 16 * MB
    again.close()
    P.ror_bk_trim()
    assert before - free_bytes() < 16 * MB
    P.ror_bk_trim()                           # nothing left: no error


def test_handles_of_two_threads():
    rng = np.random.default_rng(0)
    sizes = [(600, 130, 20), (2000, 200, 100), (900, 1100, 64), (640, 64, 160)]
    cases = []
    for m, n, br in sizes:
        A = rng.standard_normal((m, n))
        cases.append((dev(A), dev(A @ rng.standard_normal(n)), br))

    def once(A, b, br):
        sol = P.Solver(A, br, 1e-1)
        x = sol.solve(b, seed=5, tol=0.0, max_iters=8, record=True)[0]
        gb, gx = sol.backward(x)
        sol.close()
        return x, gb, gx

    want = [once(*c) for c in cases]
    torch.cuda.synchronize()
    errors = []

    def work(k):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                for i in range(24):
                    j = (i * (k + 1) + k) % len(cases)
                    got = once(*cases[j])
                    torch.cuda.current_stream().synchronize()
                    if not all(torch.equal(a, b) for a, b in zip(got, want[j])):
                        errors.append((k, i, j))
                    if i % 10 == 9:
                        P.ror_bk_trim()
        except Exception as e:   # noqa: BLE001
            errors.append((k, repr(e)))

    ts = [threading.Thread(target=work, args=(k,)) for k in range(2)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not errors, errors
