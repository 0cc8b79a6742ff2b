"""The planar real-space kernel in cells shorter than twice the cutoff.

Every x and y image of a charge within reach of a tile of atoms is an entry of
its own, and a block of 64 charges may be divided between workgroups (few
charges or configurations).  Cells from a third of r_c up, against the oracle
(all periodic images); FP64 b within 1e-11 of its largest entry (sums of up to
1e4 terms at 1e-16, pair polynomials at 1e-14).
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


# (Lx, Ly, atoms per plane, charges, batch): both short, one short, both just
# below and just above 2 r_c; fewer charges than parts of a block, a ragged
# block, several blocks
@pytest.mark.parametrize("case", [(4.0, 5.0, 3, 6, 1), (14.0, 60.0, 40, 63, 1), (23.9, 23.9, 70, 200, 1),
                                  (24.1, 24.1, 70, 200, 2), (30.0, 10.0, 20, 1000, 17)], ids=str)
def test_short_cells_against_oracle(cpm, case):
    Lx, Ly, per, m, batch = case
    h, rng = 22.0, np.random.default_rng(m)
    z = np.repeat([0.0, 3.0, h], per)
    R = np.column_stack([rng.uniform(0, Lx, 3 * per), rng.uniform(0, Ly, 3 * per), z])
    eid = (z > 11.0).astype(np.int32)
    r = np.column_stack([rng.uniform(-Lx, 2 * Lx, m), rng.uniform(0, Ly, m), rng.uniform(0.5, h - 0.5, m)])
    q = rng.uniform(0.2, 1.0, m)
    q -= q.mean()
    xyz = np.stack([r + rng.normal(0, 0.1, r.shape) for _ in range(batch)])
    say(f"short cell {Lx} x {Ly}, m {m}, batch {batch}")
    ctx = cpm.Context(cpm.Params(Lx, Ly, h))
    ctx.set_electrolyte(q)
    ctx.build_elastance(torch.as_tensor(R, device="cuda"), torch.as_tensor(eid, device="cuda"), 2)
    b = torch.empty((batch, len(R)), dtype=torch.float64, device="cuda")
    ctx.potential_vector(torch.as_tensor(xyz, device="cuda"), b)
    ctx.synchronize()
    assert ctx.info("rs_plane") == 1.0
    got = b.cpu().numpy()
    ctx.close()
    p = O.Params(Lx, Ly, 3 * h, 1.979, 0.3, 12.0, 1e-8)
    ref = np.stack([O.potential_vector(R, x, q, p) for x in xyz])
    err = float(np.abs(got - ref).max() / np.abs(ref).max())
    say(f"  {err:.2e}")
    assert err < 1e-11
