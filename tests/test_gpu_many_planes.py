"""A of planar electrodes: the planes' products are launched up to 16 planes at a time.

Against the oracle, every entry within 1e-12 of the largest: sums of at most 1e5
terms of either sign at 2^-53, in other orders.
"""
import sys

import numpy as np
import pytest

from oracle import cpm_oracle as O

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


# planes and atoms on each: one plane, a full group, one more, two groups and one;
# atoms in random order (columns up to the last atom), planes of unequal size
@pytest.mark.parametrize("case", [(1, 30), (16, 5), (17, 5), (33, 3), (3, 70)], ids=str)
def test_elastance_against_oracle(cpm, case):
    planes, per = case
    rng = np.random.default_rng(planes)
    L, h = 14.0, 3.0 * planes + 6.0
    counts = rng.integers(max(1, per - 2), per + 3, planes)
    z = np.repeat(3.0 * np.arange(planes), counts)
    n = len(z)
    R = np.column_stack([rng.uniform(0, L, n), rng.uniform(0, L, n), z])[rng.permutation(n)]
    eid = (R[:, 2] > R[:, 2].mean()).astype(np.int32)
    n_e = int(eid.max()) + 1
    say(f"{planes} planes, {n} atoms")
    ctx = cpm.Context(cpm.Params(L, L, h))
    ctx.set_electrolyte(np.array([1.0, -1.0]))
    extra = np.full(n, 40.0)                             # atoms may come close: A stays definite
    ctx.build_elastance(torch.as_tensor(R, device="cuda"), torch.as_tensor(eid, device="cuda"), n_e,
                        torch.as_tensor(extra, device="cuda"))
    ctx.invert(cpm.STORE_F64)
    A = torch.empty((n, n), dtype=torch.float64, device="cuda")
    ctx.copy_matrix(0, A)
    ctx.synchronize()
    got = A.cpu().numpy()
    ctx.close()
    ref = O.elastance(R, O.Params(L, L, 3 * h, 1.979, 0.3, 12.0, 1e-8), diag_extra=extra)
    err = np.abs(got - ref).max() / np.abs(ref).max()
    say(f"  {err:.2e}")
    assert err < 1e-12
