"""The split FP64 product of batched solves: K parts of 128 x 128 tiles over one
workgroup per CU, joined in order of K.

q = S (b - mean b) + d per vector, against the same product by numpy in FP64 with
the context's own S and d.  A sum of K products in any order is within K 2^-53 of
the sum of their magnitudes, here for both sides and once more for the removal of
the rounding in the total charge: 8 K 2^-53 of the largest such sum.
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


# (electrode atoms, batches): padded sizes 1024 (whole tiles), 1088 and 1472 (half
# tiles); rows of 64 (unsplit and split), 192 (a half-filled tile), 256, the largest
# split product (K = 1088: 30 x 17 tiles of 64) and one just above it; more runs
# than slabs per tile and fewer
@pytest.mark.parametrize("case", [(1020, (60, 256, 200)), (1088, (190, 1920, 1921)), (1450, (64, 130, 700))],
                         ids=str)
def test_batched_solve_against_numpy(cpm, case):
    n, batches = case
    rng = np.random.default_rng(n)
    per = n // 2
    nx = int(np.ceil(np.sqrt(per)))
    g = np.stack(np.meshgrid(np.arange(nx), np.arange(nx), indexing="ij"), -1).reshape(-1, 2)[:per]
    R = np.column_stack([np.tile(2.5 * g, (2, 1)), np.repeat([0.0, 30.0], per)])
    R[:, :2] += rng.uniform(-0.2, 0.2, (n, 2))
    eid = (R[:, 2] > 15.0).astype(np.int32)
    ctx = cpm.Context(cpm.Params(2.5 * nx, 2.5 * nx, 30.0))
    ctx.set_electrolyte(np.array([1.0, -1.0]))
    ctx.build_elastance(torch.as_tensor(R, device="cuda"), torch.as_tensor(eid, device="cuda"), 2)
    ctx.invert(cpm.STORE_F64)
    ctx.set_potential(np.array([-0.5, 0.5]))
    S = torch.empty((n, n), dtype=torch.float64, device="cuda")
    d = torch.empty(n, dtype=torch.float64, device="cuda")
    ctx.copy_matrix(2, S)
    ctx.copy_vector(1, d)
    ctx.synchronize()
    S, d = S.cpu().numpy(), d.cpu().numpy()
    for batch in batches:
        say(f"n {n} batch {batch}")
        b = rng.normal(0.0, 1.0, (batch, n))
        q = torch.empty((batch, n), dtype=torch.float64, device="cuda")
        ctx.solve_charges(torch.as_tensor(b, device="cuda"), cpm.SOLVE_F64, q)
        again = torch.empty_like(q)
        ctx.solve_charges(torch.as_tensor(b, device="cuda"), cpm.SOLVE_F64, again)
        ctx.synchronize()
        x = b - b.mean(axis=1, keepdims=True)
        ref = x @ S.T + d
        scale = (np.abs(x) @ np.abs(S.T) + np.abs(d)).max()
        err = np.abs(q.cpu().numpy() - ref).max() / scale
        say(f"  {err:.2e}")
        assert err < 8 * n * 2.0**-53
        assert torch.equal(q, again)
    ctx.close()
