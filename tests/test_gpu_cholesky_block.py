"""The 64 x 64 diagonal block of the factorisation: panels of 16 columns, their
exact fast root and its general form.

The inverse of A against numpy's in FP64.  Both factorisations are backward stable:
||dX|| <= c n 2^-53 cond(A) ||X|| with a modest c, taken as 16 for the two together.
Where a large diagonal leaves the off-diagonal part below rounding, the entries
(1 / sqrt(A_ii))^2 have to be those of correctly rounded operations.
"""
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def say(msg):
    print(f"[gpu] {msg}", flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def cpm():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2203_15461_amd import cpm as C
    C.lib()
    return C


def inverse(cpm, n, extra):
    rng = np.random.default_rng(n)
    nx = int(np.ceil(np.sqrt(n)))
    g = np.stack(np.meshgrid(np.arange(nx), np.arange(nx), indexing="ij"), -1).reshape(-1, 2)[:n]
    R = np.column_stack([3.0 * g + rng.uniform(-0.2, 0.2, (n, 2)), np.where(np.arange(n) % 2, 20.0, 0.0)])
    ctx = cpm.Context(cpm.Params(max(3.0 * nx, 12.0), max(3.0 * nx, 12.0), 20.0))
    ctx.set_electrolyte(np.array([1.0, -1.0]))
    ctx.build_elastance(torch.as_tensor(R, device="cuda"),
                        torch.as_tensor((np.arange(n) % 2).astype(np.int32), device="cuda"), 2,
                        torch.as_tensor(extra, device="cuda"))
    ctx.invert(cpm.STORE_F64)
    A, X = (torch.empty((n, n), dtype=torch.float64, device="cuda") for _ in range(2))
    ctx.copy_matrix(0, A)
    ctx.copy_matrix(1, X)
    ctx.synchronize()
    ctx.close()
    return A.cpu().numpy(), X.cpu().numpy()


# one block with padding, a full block, ragged and several blocks
@pytest.mark.parametrize("n", [2, 15, 17, 63, 64, 65, 200, 577])
def test_inverse_against_numpy(cpm, n):
    say(f"inverse of n {n}")
    A, X = inverse(cpm, n, np.random.default_rng(1).uniform(0.0, 1.0, n))
    ref = np.linalg.inv(A)
    err = np.abs(X - ref).max() / np.abs(ref).max()
    tol = 16 * n * 2.0**-53 * np.linalg.cond(A)
    say(f"  {err:.2e} of {tol:.2e}")
    assert err < tol


# roots of all ones (below 2^82 by one unit), pivots beyond the fast root's range,
# and both among ordinary large ones in one panel
@pytest.mark.parametrize("kind", ["ones", "huge", "mixed"])
def test_roots_are_correctly_rounded(cpm, kind):
    n = 80
    say(f"pivots {kind}")
    extra = np.full(n, np.nextafter(2.0**82, 0.0))
    if kind == "huge":
        extra = 2.0**410 * np.linspace(1.0, 3.9, n)
    elif kind == "mixed":
        extra[::3] = 2.0**80 * np.linspace(1.0, 3.9, n)[::3]
        extra[5::16] = 2.0**401
    A, X = inverse(cpm, n, extra)
    r = 1.0 / np.sqrt(np.diag(A))
    assert np.array_equal(np.diag(X), r * r)
