"""Sizes where the tiled kernels change form: block inverses and greedy solves
around multiples of the 16-row tile, rows of every alignment with NaN in the
padding between them, the few-rows form of the residual, CSR blocks with empty
rows and a column that every row shares, adjoint runs longer than one batch of
greedy inverses.

Bars: FP64 solves and adjoints 1e-10 relative to the FP64 oracle with its
selections, stored inverses 50 cond eps (as for the other sizes); residuals
n + 8 roundings of the vector type on |A||x| + |b|; FP32 solves 1e-4.
"""
import numpy as np
import pytest

import oracle as O

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2510_02156_amd as P  # noqa: E402
from tests.gpu_util import DEV, bf16_tensor, bf16_values, dev, host, rel  # noqa: E402


def normal(m, n, seed):
    rng = np.random.default_rng(seed)
    return rng.standard_normal((m, n)), rng.standard_normal(n)


def padded(A, storage, left, right):
    """A on the GPU as a view that starts `left` elements into rows of
    left + n + right elements, NaN elsewhere; and the values it holds."""
    if storage == "bf16":
        t, v = bf16_tensor(A), bf16_values(A)
    else:
        t = dev(A, torch.float64 if storage == "f64" else torch.float32)
        v = host(t).astype(np.float64)
    buf = torch.full((A.shape[0], left + A.shape[1] + right), float("nan"), dtype=t.dtype,
                     device=DEV)
    buf[:, left:left + A.shape[1]] = t
    return buf[:, left:left + A.shape[1]], v


def ragged_csr(m, seed):
    """Square, 0 to 12 entries a row; every row that is not empty has column 0."""
    rng = np.random.default_rng(seed)
    rows = []
    for i in range(m):
        c = int(rng.integers(0, 13))
        rows.append(np.zeros(0, np.int64) if c == 0 else np.unique(
            np.concatenate([[0], rng.integers(0, m, c - 1)])))
    ptr = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int64)
    return {"format": "csr", "m": m, "n": m, "rowptr": ptr,
            "colidx": np.concatenate(rows).astype(np.int32),
            "val": rng.standard_normal(ptr[-1])}, rng.standard_normal(m)


def csr_solver(s, br, lam, dtype=torch.float64):
    return P.Solver(None, br, lam, rowptr=dev(s["rowptr"], torch.int64),
                    colidx=dev(s["colidx"], torch.int32), values=dev(s["val"], dtype),
                    shape=(s["m"], s["n"]))


@pytest.mark.parametrize("br", [1, 2, 15, 16, 17, 32, 47, 48, 49, 64, 65, 72, 73, 80, 96, 112, 128,
                                129, 144, 160])
@pytest.mark.parametrize("even", [False, True])
def test_block_inverses(br, even):
    """Blocks of br and (ragged partition) br + 1 rows; odd and even row strides."""
    m, n, lam = 4 * br + 3 if br > 3 else 7, 2 * br + (4 if even else 5), 1e-2
    A, _ = normal(m, n, br)
    print(f"inverses br={br} n={n}", flush=True)
    sol = P.Solver(dev(A), br, lam)
    off = O.partition(m, br)
    for t in (0, len(off) - 2):
        blk = A[off[t]:off[t + 1]]
        G = blk @ blk.T + lam * np.eye(len(blk))
        assert rel(sol.block_inverse(t), np.linalg.inv(G)) < 50 * np.linalg.cond(G) * 2.3e-16


@pytest.mark.parametrize("br", [1, 15, 16, 47, 49, 64, 65, 80, 81, 96, 97, 113, 128, 129, 145, 160,
                                161])
def test_greedy_solves(br):
    m, n, lam, iters = 5 * br, 401, 1e-2, 10
    A, xs = normal(m, n, 100 + br)
    b = A @ xs
    print(f"greedy br={br}", flush=True)
    ref = O.solve(A, br, lam, b, seed=6, max_iters=iters)
    sol = P.Solver(dev(A), br, lam)
    assert sol.K == br
    sol.set_replay(ref["tau"], ref["I"], iters)
    x, _ = sol.solve(dev(b), seed=0, tol=0.0, max_iters=iters, replay=True)
    assert rel(host(x), ref["x"]) < 1e-10


@pytest.mark.parametrize("storage", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("left,right", [(0, 0), (1, 0), (0, 1), (3, 2), (4, 0)])
def test_rows_of_any_alignment(storage, left, right):
    vec = torch.float64 if storage == "f64" else torch.float32
    eps = 2.0 ** -53 if storage == "f64" else 2.0 ** -24
    for n in (1, 2, 3, 5, 7, 8, 9, 63, 65, 127, 129, 511, 513, 1023, 1025, 2047, 2049, 4097):
        A, xs = normal(70, n, n)
        At, v = padded(A, storage, left, right)
        print(f"rows {storage} n={n} left={left} right={right}", flush=True)
        sol = P.Solver(At, 9, 1e-1)
        x = xs.astype(np.float64 if storage == "f64" else np.float32).astype(np.float64)
        b = (v @ x[::-1]).astype(np.float32).astype(np.float64)
        r, _, _ = sol.residual(dev(b, vec), dev(x, vec))
        bar = (n + 8) * eps * (np.abs(v) @ np.abs(x) + np.abs(b))
        assert np.all(np.abs(host(r).astype(np.float64) - (b - v @ x)) <= bar)
        if n < 63:
            continue
        ref = O.solve(v, 9, 1e-1, b, seed=4, max_iters=6)
        sol.set_replay(ref["tau"], ref["I"], 6)
        y, _ = sol.solve(dev(b, vec), seed=0, tol=0.0, max_iters=6, replay=True)
        assert rel(host(y), ref["x"]) < (1e-10 if storage == "f64" else 1e-4)


@pytest.mark.parametrize("storage,m,n", [("f64", 4096, 200), ("f64", 6144, 1100), ("f32", 8192, 200),
                                         ("f32", 6144, 1101), ("bf16", 16384, 200),
                                         ("bf16", 4096, 1101), ("bf16", 4096, 1100)])
def test_residual_rows_per_wave(storage, m, n):
    """Both sides of the line below which a wave takes one row at a time."""
    eps = 2.0 ** -53 if storage == "f64" else 2.0 ** -24
    vec = torch.float64 if storage == "f64" else torch.float32
    for mm in (m, m + 1):
        A, x = normal(mm, n, mm)
        At, v = padded(A, storage, 0, 0)
        x = host(dev(x, vec)).astype(np.float64)
        b = v[:, 0].copy()
        r, bn, _ = P.Solver(At, 40, 1e-1).residual(dev(b, vec), dev(x, vec))
        ref = b - v @ x
        assert np.all(np.abs(host(r).astype(np.float64) - ref)
                      <= (n + 8) * eps * (np.abs(v) @ np.abs(x) + np.abs(b)))
        off = O.partition(mm, 40)
        want = np.add.reduceat(host(r).astype(np.float64) ** 2, off[:-1])
        np.testing.assert_allclose(host(bn), want, rtol=1e-12 if storage == "f64" else 1e-4)


@pytest.mark.parametrize("br", [1, 2, 16, 17, 64, 65, 128, 160])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_csr_empty_rows_and_shared_column(br, dtype):
    m, lam, iters = 643, 1e-1, 12
    s, xs = ragged_csr(m, br)
    s["val"] = host(dev(s["val"], dtype)).astype(np.float64)
    b = O.residual(s, np.zeros(m), -xs)
    print(f"csr br={br} {dtype}", flush=True)
    ref = O.solve(s, br, lam, b, seed=6, max_iters=iters)
    sol = csr_solver(s, br, lam, dtype)
    sol.set_replay(ref["tau"], ref["I"], iters)
    x, _ = sol.solve(dev(b, dtype), seed=0, tol=0.0, max_iters=iters, replay=True)
    assert rel(host(x), ref["x"]) < (1e-10 if dtype == torch.float64 else 1e-4)
    t = sol.k - 1
    off = O.partition(m, br)
    L = O.block_factor(s, np.arange(off[t], off[t + 1]), lam)
    G = L @ L.T
    if dtype == torch.float64:
        assert rel(sol.block_inverse(t), np.linalg.inv(G)) < 50 * np.linalg.cond(G) * 2.3e-16


@pytest.mark.parametrize("br,iters,csr", [(1, 65, False), (20, 64, False), (20, 65, False),
                                          (65, 129, False), (120, 66, False), (33, 130, True)])
def test_adjoint_longer_than_one_batch(br, iters, csr):
    lam = 1e-1
    if csr:
        s, xs = ragged_csr(600, 3)
        sol, n, b = csr_solver(s, br, lam), 600, O.residual(s, np.zeros(600), -xs)
    else:
        s, xs = normal(610, 131, br)
        sol, n, b = P.Solver(dev(s), br, lam), 131, s @ xs
    g = np.random.default_rng(br).standard_normal(n)
    x, _ = sol.solve(dev(b), seed=9, tol=0.0, max_iters=iters, record=True)
    rec = sol.record()
    print(f"adjoint br={br} iters={iters} csr={csr}", flush=True)
    gb, gx0 = sol.backward(dev(g))
    rb, rx0 = O.backward(s, br, lam, rec["tau"], rec["I"], iters, False, g)
    # the adjoint vectors shrink with the iterations: held to the size of g
    assert np.linalg.norm(host(gb) - rb) < 1e-10 * max(np.linalg.norm(rb), 1e-3)
    assert np.linalg.norm(host(gx0) - rx0) < 1e-10 * np.linalg.norm(g)


@pytest.mark.parametrize("kind", ["chain", "steps", "big", "col", "csr"])
def test_memory_of_closed_handles(kind):
    """A handle made in the memory of one that ended with values that are not
    finite gives what the first handle gave, bit for bit; two handles at once do
    not share memory."""
    if kind == "csr":
        s, xs = ragged_csr(900, 5)
        b = dev(O.residual(s, np.zeros(900), -xs))

        def make():
            return csr_solver(s, 64, 1e-1)
    else:
        m, n, br = {"chain": (900, 200, 40), "steps": (900, 5001, 33), "big": (900, 1100, 180),
                    "col": (900, 90, 200)}[kind]
        A, xs = normal(m, n, 8)
        At, b = dev(A), dev(A @ xs)

        def make():
            return P.Solver(At, br, 1e-1)

    def run(sol, rhs):
        return sol.solve(rhs, seed=3, tol=0.0, max_iters=9)[0]

    sol = make()
    want, W = run(sol, b), sol.setup_arrays()["W"]
    for _ in range(3):
        with pytest.raises(P.RorBkError):   # A x0 overflows: not finite
            sol.solve(b, torch.full((sol.n,), 1e308, dtype=b.dtype, device=DEV), seed=3, tol=0.0,
                      max_iters=9)
        sol.close()
        sol = make()
        assert np.array_equal(sol.setup_arrays()["W"], W)
        other = make()
        assert torch.equal(run(other, b), want) and torch.equal(run(sol, b), want)
        other.close()
    sol.close()
