"""Which k-space sums cpm_potential_vector takes (info key sf_zbin: 1 FP64 output, plus
2 FP32 output from charges binned in z; 0 explicit structure factors), by the switches
and by the sizes alone, and b of each route against the oracle: FP64 within 1e-10, FP32
within 5e-6 of the largest entry.
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


def check(C, params, oparams, R, eid, q, xyz, route, fp32):
    ctx = C.Context(params)
    ctx.set_electrolyte(q)
    ctx.build_elastance(torch.as_tensor(np.ascontiguousarray(R), device="cuda"),
                        torch.as_tensor(np.ascontiguousarray(eid), device="cuda"), int(eid.max()) + 1)
    assert (int(ctx.info("sf_zbin")), int(ctx.info("sf_fp32"))) == (route, fp32)
    ref = np.stack([O.potential_vector(R, x, q, oparams) for x in xyz])
    for dtype, tol in ((torch.float64, 1e-10), (torch.float32, 5e-6), (torch.float64, 1e-10)):
        b = torch.full((len(xyz), len(R)), float("nan"), dtype=dtype, device="cuda")
        ctx.potential_vector(torch.as_tensor(np.ascontiguousarray(xyz), device="cuda"), b)
        ctx.synchronize()
        err = np.abs(b.double().cpu().numpy() - ref).max() / np.abs(ref).max()
        say(f"  {dtype} {err:.2e}")
        assert err < tol
    ctx.close()


@pytest.mark.parametrize("env,route,fp32", [
    ({}, 3, 1), ({"CPM_SF_ZBIN": "0"}, 0, 2), ({"CPM_SF_F16": "0"}, 1, 1), ({"CPM_SF_FP32": "0"}, 3, 0),
    ({"CPM_SF_ZBIN": "0", "CPM_SF_F16": "0"}, 0, 1), ({"CPM_SF_ZBIN": "0", "CPM_SF16_NT": "1"}, 0, 2),
    ({"CPM_SF_ZBIN": "0", "CPM_SF16_NT": "4"}, 0, 2), ({"CPM_SF_ZBIN": "0", "CPM_SF_FP32": "0"}, 0, 0),
    ({"CPM_SF_MFMA": "0"}, 0, 0),
], ids=lambda e: "-".join(f"{k[4:]}={v}" for k, v in e.items()) if isinstance(e, dict) else str(e))
@pytest.mark.parametrize("batch", [1, 5])
def test_routes_by_switch(cpm, env, route, fp32, batch, monkeypatch):
    for k, v in env.items():
        monkeypatch.setenv(k, v)
    w = I.small_capacitor("b")
    say(f"{env or 'default'}, batch {batch}")
    xyz = np.stack([I.snapshot(w, s) for s in range(batch)])
    check(cpm, cpm.Params.of(w), O.params_for(w), w.electrode_xyz, w.electrode_id, w.electrolyte_q,
          xyz, route, fp32)


# cell heights 3 h whose z bins exceed 512 in neither, in FP32 only, and in both
@pytest.mark.parametrize("h,route", [(300.0, 3), (350.0, 1), (450.0, 0)])
@pytest.mark.parametrize("batch", [1, 9])
def test_routes_by_bins(cpm, h, route, batch):
    L, m = (9.0, 10.0), 70
    rng = np.random.default_rng(int(h))
    z = np.repeat([0.0, 0.4 * h, h], 12)
    R = np.column_stack([rng.uniform(0, L[0], 36), rng.uniform(0, L[1], 36), z])
    xyz = np.stack([np.column_stack([rng.uniform(0, L[0], m), rng.uniform(0, L[1], m),
                                     rng.uniform(2.5, h - 2.5, m)]) for _ in range(batch)])
    xyz[:, 0, 2] = 0.4 * h + 1.0                           # a charge near the middle plane
    q = rng.uniform(0.2, 1.0, m)
    q[m // 2:] *= -1.0
    q -= q.mean()
    say(f"cell height {3 * h}, batch {batch}")
    check(cpm, cpm.Params(L[0], L[1], h), O.Params(L[0], L[1], 3 * h, 1.979, 0.3, 12.0, 1e-8),
          R, (z > 0.5 * h).astype(np.int32), q, xyz, route, 1 if route & 2 else 2)


def test_other_electrodes_take_structure_factors(cpm):
    w = I.small_capacitor("a")
    rng = np.random.default_rng(7)
    R = w.electrode_xyz.copy()
    R[:, 2] += rng.uniform(-1e-3, 1e-3, len(R))
    w = w.with_(electrode_xyz=R, h=float(R[:, 2].max() - R[:, 2].min()))
    say("atoms on no common planes")
    check(cpm, cpm.Params.of(w), O.params_for(w), R, w.electrode_id, w.electrolyte_q,
          np.stack([I.snapshot(w, s) for s in range(2)]), 0, 2)
