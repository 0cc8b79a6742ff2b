"""Explicit structure factors of planar electrodes (CPM_SF_ZBIN=0), the route of cells
beyond the bins' and tables' bounds: split-FP16 items of one, two and four M tiles with
their layer reduction against the oracle's stored results for 2880 atoms, and the
real-space sums over z-ordered charges against an order left by other positions.
"""
import os
import sys

import numpy as np
import pytest

from oracle import cpm_oracle as O
from paper_2203_15461_amd import inputs as I

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

GOLDEN = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden", "graphite_capacitor_2880.npz")


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


def rel(a, b):
    return float(np.max(np.abs(np.asarray(a) - b)) / np.max(np.abs(b)))


def b_of(C, w, xyz, dtype, fp32, before=None):
    ctx = C.Context(C.Params.of(w))
    ctx.set_electrolyte(w.electrolyte_q)
    ctx.build_elastance(torch.as_tensor(w.electrode_xyz, dtype=torch.float64, device="cuda").contiguous(),
                        torch.as_tensor(w.electrode_id, dtype=torch.int32, device="cuda"), 2)
    assert (int(ctx.info("sf_zbin")), int(ctx.info("sf_fp32"))) == (0, fp32)
    b = torch.full((len(xyz), w.n), float("nan"), dtype=dtype, device="cuda")
    if before is not None:
        ctx.potential_vector(torch.as_tensor(before, device="cuda"), b[:len(before)])
    ctx.potential_vector(torch.as_tensor(xyz, device="cuda"), b)
    ctx.synchronize()
    ctx.close()
    return b.double().cpu().numpy()


# a launch group of 64 and one of 40; tolerances of the paths: FP64 1e-10, FP32 5e-6
@pytest.mark.parametrize("env,dtype,fp32,tol", [
    ({"CPM_SF16_NT": "1"}, torch.float32, 2, 5e-6), ({}, torch.float32, 2, 5e-6),
    ({"CPM_SF16_NT": "4"}, torch.float32, 2, 5e-6), ({"CPM_SF_F16": "0"}, torch.float32, 1, 5e-6),
    ({}, torch.float64, 2, 1e-10)], ids=str)
def test_2880_against_golden(cpm, env, dtype, fp32, tol, monkeypatch):
    g = np.load(GOLDEN)
    w = I.graphite_capacitor()
    idx = [k % 3 for k in range(104)]
    xyz = np.stack([I.snapshot(w, int(g["snapshots"][k])) for k in idx])
    monkeypatch.setenv("CPM_SF_ZBIN", "0")
    for k, v in env.items():
        monkeypatch.setenv(k, v)
    say(f"2880 atoms, 104 configurations, explicit structure factors, {env or 'default'}, {dtype}")
    err = rel(b_of(cpm, w, xyz, dtype, fp32), g["b"][idx])
    say(f"  {err:.2e}")
    assert err < tol


def test_charge_order_of_real_space(cpm, monkeypatch):
    w = I.small_capacitor("a")
    xyz = np.stack([I.snapshot(w, s) for s in range(20)])
    upside_down = xyz[:1] * [1.0, 1.0, -1.0] + [0.0, 0.0, w.h]
    monkeypatch.setenv("CPM_SF_ZBIN", "0")
    got = []
    for least in ("1", "1000000000"):
        monkeypatch.setenv("CPM_RS_SORT_MIN", least)
        got.append(b_of(cpm, w, xyz, torch.float64, 2, upside_down))
    p = O.params_for(w)
    ref = np.array([O.potential_vector(w.electrode_xyz, r, w.electrolyte_q, p) for r in xyz[:3]])
    say(f"z-ordered charges against an aged order, 20 snapshots: {rel(got[0], got[1]):.2e}")
    assert rel(got[0][:3], ref) < 1e-10 and rel(got[1][:3], ref) < 1e-10
    assert not np.array_equal(got[0], got[1])          # the two orders did run
    assert rel(got[0], got[1]) < 1e-13
