"""Vector kernels of the conjugate gradients: rows in batches of four per wave, block
totals in batches of four per wave (64 blocks).

Grids of one workgroup (many batches of rows, the last one partial), few, and more
than 64 (a second batch of totals), with the operator and the dense A, with and
without the preconditioner, against the direct FP64 solve on the same b: both are
solutions to 1e-13 of a system with condition number below 1e3.
"""
import sys

import numpy as np
import pytest

from paper_2203_15461_amd import inputs as I

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


@pytest.mark.parametrize("matrix_free", [True, False])
@pytest.mark.parametrize("blocks", [1, 5, 65])
@pytest.mark.parametrize("precond", ["0", "2"])
def test_cg_grids_match_direct_solve(cpm, monkeypatch, matrix_free, blocks, precond):
    monkeypatch.setenv("CPM_CG_BLOCKS", str(blocks))
    monkeypatch.setenv("CPM_CG_PRECOND", precond)
    w = I.scaled_graphite_capacitor(1152)
    say(f"n = {w.n}, {blocks} blocks, operator {matrix_free}, preconditioner {precond}")
    xyz = torch.as_tensor(np.stack([I.snapshot(w, s) for s in range(3)]), dtype=torch.float64,
                          device="cuda").contiguous()
    direct = cpm.setup(w)
    b = torch.empty((3, w.n), dtype=torch.float64, device="cuda")
    direct.potential_vector(xyz, b)
    q0, q1 = torch.empty_like(b), torch.empty_like(b)
    direct.solve_charges(b, 0, q0)
    ctx = cpm.setup(w, matrix_free=matrix_free)
    ctx.solve_cg(b, q1, tol=1e-13)
    ctx.synchronize()
    direct.synchronize()
    a, c = q0.cpu().numpy(), q1.cpu().numpy()
    assert np.abs(a - c).max() <= 1e-10 * np.abs(a).max()
    assert np.abs(c.sum(axis=1)).max() <= 1e-12
    direct.close()
    ctx.close()
