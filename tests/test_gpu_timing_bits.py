"""Kernel timing changes no result: b and q of one to five configurations have the same
bits with timing off, on, and on for one family, and every family whose work runs is
counted, also where one launch does the work of several.
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


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["f64", "f32"])
@pytest.mark.parametrize("batch", [1, 3, 5])
def test_same_bits_with_timing(cpm, batch, dtype):
    w = I.graphite_capacitor()
    ctx = cpm.setup(w, store=cpm.STORE_F64 | cpm.STORE_F32)
    xyz = torch.as_tensor(np.stack([I.snapshot(w, s) for s in range(batch)]), device="cuda")
    mode = cpm.SOLVE_F64 if dtype == torch.float64 else cpm.SOLVE_F32
    mv = "matvec_f32" if mode else "matvec_f64" if batch < 4 else "gemm_f64"
    results = []
    for on in (False, True, "structure_factor", False):
        say(f"batch {batch} {dtype} timing {on}")
        ctx.enable_timing(on)
        b = torch.empty((batch, w.n), dtype=dtype, device="cuda")
        q = torch.empty((batch, w.n), dtype=torch.float64, device="cuda")
        Qe = torch.empty((batch, 2), dtype=torch.float64, device="cuda")
        ctx.potential_vector(xyz, b)
        ctx.solve_charges(b, mode, q, Qe)
        ctx.synchronize()
        results.append((b, q, Qe))
        if on is True:
            for fam in ("sf_tables", "structure_factor", "real_space_b", "sf_reduce", "projection",
                        "combine", "row_means", mv, "finalize"):
                ms, count = ctx.timing(fam)
                assert count == 1 and ms > 0, fam
    for r in results[1:]:
        assert all(torch.equal(x, y) for x, y in zip(r, results[0]))
    ctx.close()
