"""Solves of one to three vectors in one launch: centring, product, projection and
totals, the last by whichever workgroup ends last.

q = S (b - mean b) + d and Q_e = sum over the electrode, against numpy in FP64 with
the context's own S and d: within 8 n 2^-53 of the largest sum of magnitudes (two
sums in any order, the means and the removal of the total charge).  With the FP32
copy of S, and b rounded to FP32 on both sides, 2^-24 of that sum more.  Q_e sums up
to n such charges.
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


# atoms (padded to 64, 1024, 1088, 2048, the largest, and one past it), electrodes
@pytest.mark.parametrize("case", [(40, 2), (1000, 6), (1030, 1), (2040, 5), (4090, 2), (4100, 2)], ids=str)
def test_few_vectors_against_numpy(cpm, case):
    n, n_e = case
    rng = np.random.default_rng(n)
    nx = int(np.ceil(np.sqrt(n / n_e)))
    g = np.stack(np.meshgrid(np.arange(nx), np.arange(nx), indexing="ij"), -1).reshape(-1, 2)
    R = np.concatenate([np.column_stack([2.5 * g, np.full(len(g), 4.0 * e)]) for e in range(n_e)])
    eid = np.repeat(np.arange(n_e), len(g))
    keep = np.sort(rng.permutation(len(R))[:n])
    R, eid = R[keep], eid[keep].astype(np.int32)
    R[:, :2] += rng.uniform(-0.2, 0.2, (n, 2))
    L = max(2.5 * nx, 12.0)
    ctx = cpm.Context(cpm.Params(L, L, 4.0 * n_e + 20.0))
    ctx.set_electrolyte(np.array([1.0, -1.0]))
    ctx.build_elastance(torch.as_tensor(R, device="cuda"), torch.as_tensor(eid, device="cuda"), n_e)
    ctx.invert(cpm.STORE_F64 | cpm.STORE_F32)
    ctx.set_potential(np.linspace(-0.5, 0.5, n_e))
    S = torch.empty((n, n), dtype=torch.float64, device="cuda")
    d = torch.empty(n, dtype=torch.float64, device="cuda")
    ctx.copy_matrix(2, S)
    ctx.copy_vector(1, d)
    ctx.synchronize()
    S, d = S.cpu().numpy(), d.cpu().numpy()
    onehot = np.eye(n_e)[eid]
    for mode, u in ((cpm.SOLVE_F64, 0.0), (cpm.SOLVE_F32, 2.0**-24)):
        for batch, dtype in ((1, np.float64), (3, np.float64), (2, np.float32), (1, np.float64)):
            say(f"n {n} n_e {n_e} mode {mode} batch {batch} {np.dtype(dtype).name}")
            b = rng.normal(0.0, 1.0, (batch, n)).astype(dtype)
            q = torch.empty((batch, n), dtype=torch.float64, device="cuda")
            Q = torch.empty((batch, n_e), dtype=torch.float64, device="cuda")
            bd = torch.as_tensor(b, device="cuda")
            ctx.solve_charges(bd, mode, q, Q)
            ctx.synchronize()
            first = q.cpu().numpy()
            x = b.astype(np.float64)
            x -= x.mean(axis=1, keepdims=True)
            ref = x @ S.T + d
            tol = (8 * n * 2.0**-53 + u) * (np.abs(x) @ np.abs(S.T) + np.abs(d)).max()
            err = np.abs(first - ref).max()
            errQ = np.abs(Q.cpu().numpy() - first @ onehot).max()
            say(f"  {err / tol:.2e} of the bound, totals {errQ:.1e}")
            assert err < tol
            assert errQ < n * tol
            ctx.solve_charges(bd, mode, q)             # without totals; the counters start anew
            ctx.synchronize()
            assert np.array_equal(q.cpu().numpy(), first)
    ctx.close()
