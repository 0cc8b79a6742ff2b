"""Planar electrodes on the general path of b (CPM_PV_FAST_MIN: batches below it take
explicit structure factors and the per-configuration projection): batches below and
above the switch against the oracle, FP64 within 1e-10 and FP32 within 5e-6 of the
largest entry.
"""
import sys

import numpy as np
import pytest

from oracle import cpm_oracle as O
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


# the switch at 2 and at 4; one context meets batches on both sides of it
@pytest.mark.parametrize("fast_min", ["2", "4"])
def test_small_batches_against_oracle(cpm, fast_min, monkeypatch):
    monkeypatch.setenv("CPM_PV_FAST_MIN", fast_min)
    w = I.small_capacitor("b")
    xyz = np.stack([I.snapshot(w, s) for s in range(5)])
    p = O.params_for(w)
    ref = np.stack([O.potential_vector(w.electrode_xyz, x, w.electrolyte_q, p) for x in xyz])
    ctx = cpm.setup(w)
    assert int(ctx.info("nlayers")) > 0
    for dtype, tol in ((torch.float64, 1e-10), (torch.float32, 5e-6)):
        for batch in (1, 3, 5, 1):
            say(f"general path below {fast_min}, batch {batch}, {dtype}")
            b = torch.full((batch, w.n), float("nan"), dtype=dtype, device="cuda")
            ctx.potential_vector(torch.as_tensor(xyz[:batch].copy(), device="cuda"), b)
            ctx.synchronize()
            err = np.abs(b.double().cpu().numpy() - ref[:batch]).max() / np.abs(ref[:batch]).max()
            say(f"  {err:.2e}")
            assert err < tol
    ctx.close()
