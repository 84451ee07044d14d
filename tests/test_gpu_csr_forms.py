"""The CSR block step picks its form from two limits by themselves: more than
2048 entries in the current rows (further chunks, one after the other) and more
than 2048 in the next rows (not fetched ahead).  Blocks on either side of both,
one after another in every order, with a column that all rows share across the
chunk boundary; forward and adjoint.

Bars as for the other CSR sizes: FP64 1e-10 relative to the host, FP32 1e-4."""
import numpy as np
import pytest

import oracle as O

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2510_02156_amd as P  # noqa: E402
from tests.gpu_util import dev, host, rel  # noqa: E402

B, N = 40, 900
TOTALS = [200, 2047, 2048, 2049, 4096, 120, 5000, 4097]


def system(seed):
    rng = np.random.default_rng(seed)
    rows = []
    for total in TOTALS:
        for i in range(B):
            c = total // B + (i < total % B)
            rows.append(np.sort(np.concatenate([[0], 1 + rng.choice(N - 1, c - 1, replace=False)])))
    ptr = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int64)
    off = ptr[::B]
    assert list(np.diff(off)) == TOTALS
    return {"format": "csr", "m": len(rows), "n": N, "rowptr": ptr,
            "colidx": np.concatenate(rows).astype(np.int32), "val": rng.standard_normal(ptr[-1])}


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_csr_steps_on_either_side_of_both_limits(dtype):
    s, lam, iters = system(1), 0.1, 24
    s["val"] = host(dev(s["val"], dtype)).astype(np.float64)
    k, m = len(TOTALS), s["m"]
    rng = np.random.default_rng(2)
    b = -O.residual(s, np.zeros(m), rng.standard_normal(N))
    b = host(dev(b, dtype)).astype(np.float64)
    # every ordered pair of blocks, adjacent in the sequence of draws
    pairs = [(i, (i + d) % k) for d in range(k) for i in range(k)]
    tau = np.array([t for p in pairs for t in p], np.int32)[:3 * iters].copy()
    seen = set(zip(tau[:-1], tau[1:]))
    assert {(a > 2048, c > 2048) for a, c in ((TOTALS[i], TOTALS[j]) for i, j in seen)} == {
        (x, y) for x in (False, True) for y in (False, True)}
    I = np.stack([np.sort(rng.choice(m, B, replace=False)) if it % 3 == 0 else
                  np.arange(B) + B * (5 if it % 3 == 1 else 6) for it in range(iters)]).astype(np.int32)
    sol = P.Solver(None, B, lam, rowptr=dev(s["rowptr"], torch.int64),
                   colidx=dev(s["colidx"], torch.int32), values=dev(s["val"], dtype), shape=(m, N))
    sol.set_replay(tau, I, iters)
    print(f"csr forms {dtype}", flush=True)
    x, _ = sol.solve(dev(b, dtype), tol=0.0, max_iters=iters, replay=True, record=True)
    want = np.zeros(N)
    for it in range(iters):
        for S in [np.arange(t * B, (t + 1) * B) for t in tau[3 * it:3 * it + 3]] + [I[it]]:
            want = O.apply_block(s, S, lam, b, want)
    bar = 1e-10 if dtype == torch.float64 else 1e-4
    assert rel(host(x), want) < bar
    g = host(dev(rng.standard_normal(N), dtype)).astype(np.float64)
    gb, gx0 = sol.backward(dev(g, dtype))
    rb, rx0 = O.backward(s, B, lam, tau, I, iters, False, g)
    assert np.linalg.norm(host(gb) - rb) < bar * np.linalg.norm(rb)
    assert np.linalg.norm(host(gx0) - rx0) < bar * np.linalg.norm(g)
