"""Captures beside eager solves that need no larger buffers: a captured step stays
valid after eager solves of other kinds and of equal or smaller batches, and a caller
can capture such a solve itself.  Replays equal the eager results bit for bit.
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


def empty(*shape):
    return torch.full(shape, float("nan"), dtype=torch.float64, device="cuda")


# a size whose FP64 products of 200 vectors split (1152), and one whose do not
@pytest.mark.parametrize("n,most", [(288, 64), (1152, 256)])
def test_eager_solves_between_replays(cpm, n, most):
    w = I.small_capacitor("a") if n == 288 else I.scaled_graphite_capacitor(n)
    s = torch.cuda.Stream()
    ctx = cpm.setup(w, store=cpm.STORE_F64 | cpm.STORE_BF16X2, stream=s)
    xyz = torch.as_tensor(np.stack([I.snapshot(w, k % 3) for k in range(most)]), device="cuda")
    b, q, Qe = empty(most, w.n), empty(most, w.n), empty(most, 2)
    torch.cuda.synchronize()
    ctx.capture_step(xyz, b, cpm.SOLVE_BF16X2 | cpm.SOLVE_REFINE, q, Qe)
    ctx.replay_step()
    ctx.synchronize()
    first = q.clone()
    for batch in (1, 3, most, most - 56, 2):
        say(f"n {w.n}: eager FP64 solve of {batch}, then the replay")
        ctx.solve_charges(b[:batch].contiguous(), cpm.SOLVE_F64, empty(batch, w.n))
        ctx.synchronize()
        q.fill_(float("nan"))
        torch.cuda.synchronize()
        ctx.replay_step()
        ctx.synchronize()
        assert torch.equal(q, first)
    ctx.close()


@pytest.mark.parametrize("batch", [1, 200])
def test_first_small_solve_in_the_callers_capture(cpm, batch):
    w = I.scaled_graphite_capacitor(1152)
    s = torch.cuda.Stream()
    ctx = cpm.setup(w, store=cpm.STORE_F64 | cpm.STORE_BF16X2, stream=s)
    rng = np.random.default_rng(1)
    b = torch.as_tensor(rng.normal(0.0, 1.0, (256, w.n)), device="cuda")
    q, ref = empty(batch, w.n), empty(batch, w.n)
    ctx.solve_charges(b, cpm.SOLVE_BF16X2, empty(256, w.n))      # buffers for 256 vectors
    ctx.synchronize()
    say(f"capture of an FP64 solve of {batch} by the caller")
    g = torch.cuda.CUDAGraph()
    x = b[:batch].contiguous()
    with torch.cuda.graph(g, stream=s):
        ctx.solve_charges(x, cpm.SOLVE_F64, q)
    for _ in range(3):
        x.copy_(torch.as_tensor(rng.normal(0.0, 1.0, (batch, w.n))))
        torch.cuda.synchronize()
        ctx.solve_charges(x, cpm.SOLVE_F64, ref)
        ctx.synchronize()
        q.fill_(float("nan"))
        torch.cuda.synchronize()
        with torch.cuda.stream(s):
            g.replay()
        torch.cuda.synchronize()
        assert torch.equal(q, ref)
    ctx.close()
