"""Device memory of closed handles: given back by ror_bk_trim and at the pool's
bounds (the bounds themselves: test_block_pool.py), handles made and closed by
two threads at once, each on its own stream, and handles that go on after a call
that asked for more memory than there is."""
import threading

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2510_02156_amd as P  # noqa: E402
from paper_2510_02156_amd import binding  # noqa: E402
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


@pytest.mark.parametrize("iters", [1 << 36, 1537228672809129301, (1 << 63) - 1])
@pytest.mark.parametrize("record,every", [(False, 0), (True, 0), (False, 1)])
def test_handle_after_running_out_of_memory(iters, record, every):
    """12 bytes of draws an iteration: 0.8 TB, 2^64 - 4 bytes (which round up to
    2^64) and more than 64 bits hold."""
    A = torch.randn(300, 70, dtype=torch.float64, device=DEV)
    b = A.sum(1)
    sol, other = P.Solver(A, 20, 1e-1), P.Solver(A, 20, 1e-1)
    sol.solve(b, seed=1, tol=0.0, max_iters=3, record=record, checkpoint_every=every)
    with pytest.raises(P.RorBkError) as e:
        sol.solve(b, seed=1, tol=0.0, max_iters=iters, record=record, checkpoint_every=every)
    assert e.value.code == P.RORBK_ERR_OOM
    got = sol.solve(b, seed=1, tol=0.0, max_iters=9, record=record, checkpoint_every=every)[0]
    want = other.solve(b, seed=1, tol=0.0, max_iters=9, record=record, checkpoint_every=every)[0]
    assert torch.equal(got, want)
    if record or every:
        for x, y in zip(sol.backward(got), other.backward(got)):
            assert torch.equal(x, y)
    with pytest.raises(P.RorBkError) as e:
        sol.fabgmres(b, max_outer=iters, inner_iters=2)
    assert e.value.code == P.RORBK_ERR_OOM
    out = np.zeros(3, dtype=np.int32)         # never written: the call is refused
    with pytest.raises(P.RorBkError) as e:
        binding._check(P.lib().ror_bk_sample(sol.h, 1, 0, iters, out.ctypes.data), "ror_bk_sample")
    assert e.value.code == P.RORBK_ERR_OOM
