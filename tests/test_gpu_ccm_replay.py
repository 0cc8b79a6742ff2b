"""A captured step of constrained charges after new inversions of the same elastance
(also asynchronous): replays read the new inverse and give the same bits; the first
replay against the oracle at 1e-10.
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


@pytest.mark.parametrize("batch", [2, 6])
def test_replay_after_inverting_the_same_elastance(cpm, batch):
    w = I.small_capacitor("a")
    s = torch.cuda.Stream()
    ctx = cpm.setup(w, stream=s)
    mode, Q = cpm.SOLVE_F64 | cpm.SOLVE_CCM, [0.75, -0.75]
    ctx.set_charge(Q)
    x = torch.as_tensor(np.stack([I.snapshot(w, k) for k in range(batch)]), device="cuda")
    b, q = (torch.empty((batch, w.n), dtype=torch.float64, device="cuda") for _ in range(2))
    torch.cuda.synchronize()
    ctx.capture_step(x, b, mode, q)
    ctx.replay_step()
    ctx.synchronize()
    first = q.clone()
    p = O.params_for(w)
    Ainv = O.capacitance(O.elastance(w.electrode_xyz, p)).Ainv
    bo = O.potential_vector(w.electrode_xyz, I.snapshot(w, 0), w.electrolyte_q, p)
    qo, _ = O.constrained_charges(Ainv, w.electrode_id, 2, bo, np.array(Q))
    assert np.abs(first[0].cpu().numpy() - qo).max() < 1e-10 * np.abs(qo).max()
    for again in range(3):
        ctx.invert(cpm.STORE_F64 | (cpm.INVERT_ASYNC if again == 1 else 0))
        ctx.set_potential(w.v_electrode)
        ctx.set_charge(Q)
        ctx.synchronize()
        q.fill_(float("nan"))
        torch.cuda.synchronize()
        ctx.replay_step()
        ctx.synchronize()
        say(f"batch {batch}, inversion {again + 2}: {float((q - first).abs().max()):.2e}")
        assert torch.equal(q, first)
    ctx.close()
