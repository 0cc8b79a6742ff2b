"""cpm_solve_charges_noalloc runs the kernels of cpm_solve_charges: the same bits, in
every mode and on both sides of every size rule (one launch for up to three vectors,
FP64 products from four on, split for few tiles), with and without totals.
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


# 288 atoms: no split; 1200 (1216 padded): split from 200 vectors; 2880: split from 4
@pytest.mark.parametrize("n", [288, 1200, 2880])
def test_same_bits_as_solve_charges(cpm, n):
    w = {288: lambda: I.small_capacitor("a"), 2880: I.graphite_capacitor}.get(
        n, lambda: I.scaled_graphite_capacitor(n))()
    ctx = cpm.setup(w, store=cpm.STORE_F64 | cpm.STORE_F32 | cpm.STORE_BF16X2)
    ctx.set_charge([0.4, -0.4])
    rng = np.random.default_rng(n)
    every = torch.as_tensor(rng.normal(0.0, 1.0, (128, w.n)), device="cuda")
    cases = [(m, k) for m in (cpm.SOLVE_F64, cpm.SOLVE_F64 | cpm.SOLVE_CCM) for k in (1, 3, 4, 65, 128)]
    cases += [(m, k) for m in (cpm.SOLVE_F32, cpm.SOLVE_F32 | cpm.SOLVE_REFINE,
                               cpm.SOLVE_F64 | cpm.SOLVE_REFINE, cpm.SOLVE_BF16X2 | cpm.SOLVE_REFINE)
              for k in (2, 5, 70)]
    if w.n == 1200:
        every = torch.cat([every, every.flip(0)])
        cases.append((cpm.SOLVE_F64, 200))
    for mode, batch in cases:
        say(f"n {w.n} mode {mode:#x} batch {batch}")
        b = every[:batch].contiguous()
        if mode & 0xff == cpm.SOLVE_F32:
            b = b.float()
        out = [[torch.full(s, float("nan"), dtype=torch.float64, device="cuda")
                for s in ((batch, w.n), (batch, 2))] for _ in range(2)]
        ctx.solve_charges(b, mode, *out[0])
        ctx.solve_charges_noalloc(b, mode, *out[1])
        ctx.synchronize()
        assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
        ctx.solve_charges_noalloc(b, mode, out[1][0])             # without totals
        ctx.synchronize()
        assert torch.equal(out[0][0], out[1][0])
    ctx.close()
