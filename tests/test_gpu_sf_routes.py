"""Which k-space sums cpm_potential_vector takes (info key sf_zbin: charges binned in z
for one configuration with FP64 output 1, FP32 output 2, for batches of 64 4 and 8; 0
explicit structure factors), by the switches, by the bounds and by the sizes, and b of
each route against the oracle: FP64 within 1e-10, FP32 within 5e-6 of the largest entry.
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
    ({"CPM_SF_ZBIN": "2"}, 15, 1), ({"CPM_SF_ZBIN": "0"}, 0, 2),
    ({"CPM_SF_ZBIN": "2", "CPM_SF_F16": "0"}, 5, 1), ({"CPM_SF_ZBIN": "2", "CPM_SF_FP32": "0"}, 15, 0),
    ({"CPM_SF_ZBIN": "0", "CPM_SF_F16": "0"}, 0, 1), ({"CPM_SF_ZBIN": "0", "CPM_SF16_NT": "1"}, 0, 2),
    ({"CPM_SF_ZBIN": "0", "CPM_SF16_NT": "4"}, 0, 2), ({"CPM_SF_ZBIN": "0", "CPM_SF_FP32": "0"}, 0, 0),
    ({"CPM_SF_MFMA": "0"}, 0, 0), ({"CPM_SF_ZBIN": "2", "CPM_PV_FAST_MIN": "2"}, 12, 1),
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
@pytest.mark.parametrize("h,route", [(300.0, 15), (350.0, 5), (450.0, 0)])
@pytest.mark.parametrize("batch", [1, 9])
def test_routes_by_bins(cpm, h, route, batch, monkeypatch):
    monkeypatch.setenv("CPM_SF_ZBIN", "2")
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
          R, (z > 0.5 * h).astype(np.int32), q, xyz, route, 1 if route & 8 else 2)


# by cost: the standard capacitor; 1000 charges in a small cell on few and on many planes,
# dilute charges in a tall one.  Batches below and above a launch group's 64, and one in
# between, in one context, whose buffers serve both routes
@pytest.mark.parametrize("planes,L,h,m,route", [(6, 34.0, 75.0, 6128, 15), (16, 25.0, 45.0, 1000, 7),
                                                (48, 25.0, 45.0, 1000, 3), (8, 25.0, 150.0, 100, 3),
                                                (64, 30.0, 150.0, 300, 0)])
def test_routes_by_cost(cpm, planes, L, h, m, route):
    rng = np.random.default_rng(planes)
    half = planes // 2
    z = np.repeat(np.concatenate([np.linspace(0, 6, half), np.linspace(h - 6, h, half)]), 5)
    R = np.column_stack([rng.uniform(0, L, len(z)), rng.uniform(0, L, len(z)), z])
    eid = (z > 0.5 * h).astype(np.int32)
    q = np.where(np.arange(m) < m // 2, 1.0, -1.0)
    p = O.Params(L, L, 3 * h, 1.979, 0.3, 12.0, 1e-8)
    base = [np.column_stack([rng.uniform(0, L, m), rng.uniform(0, L, m), rng.uniform(9, h - 9, m)])
            for _ in range(3)]
    ref = np.stack([O.potential_vector(R, x, q, p) for x in base])
    ctx = cpm.Context(cpm.Params(L, L, h))
    ctx.set_electrolyte(q)
    ctx.build_elastance(torch.as_tensor(R, device="cuda"), torch.as_tensor(eid, device="cuda"), 2)
    say(f"{planes} planes, cell {L} x {h}, m {m}: route {int(ctx.info('sf_zbin'))}")
    assert int(ctx.info("sf_zbin")) == route
    for batch in (70, 1, 11, 64):
        idx = np.arange(batch) % 3
        x = torch.as_tensor(np.stack([base[i] for i in idx]), device="cuda")
        for dtype, tol in ((torch.float64, 1e-10), (torch.float32, 5e-6)):
            b = torch.full((batch, len(R)), float("nan"), dtype=dtype, device="cuda")
            ctx.potential_vector(x, b)
            ctx.synchronize()
            err = np.abs(b.double().cpu().numpy() - ref[idx]).max() / np.abs(ref).max()
            say(f"  batch {batch} {dtype} {err:.2e}")
            assert err < tol
    ctx.close()


@pytest.mark.parametrize("captured,between", [(64, 1), (1, 64)])
def test_captured_step_beside_the_other_route(cpm, captured, between):
    """A captured step on one route, eager calls on the other between its replays."""
    L, h, m, planes = 25.0, 45.0, 1000, 16
    rng = np.random.default_rng(4)
    z = np.repeat(np.concatenate([np.linspace(0, 6, 8), np.linspace(h - 6, h, 8)]), 5)
    R = np.column_stack([rng.uniform(0, L, len(z)), rng.uniform(0, L, len(z)), z])
    eid = (z > 0.5 * h).astype(np.int32)
    n = len(z)
    ctx = cpm.Context(cpm.Params(L, L, h), torch.cuda.Stream())
    ctx.set_electrolyte(np.where(np.arange(m) < m // 2, 1.0, -1.0))
    extra = torch.full((n,), 40.0, dtype=torch.float64, device="cuda")   # atoms may come close
    Rd, ed = torch.as_tensor(R, device="cuda"), torch.as_tensor(eid, device="cuda")
    torch.cuda.synchronize()
    ctx.build_elastance(Rd, ed, 2, extra)
    ctx.invert()
    ctx.set_potential([-0.5, 0.5])
    assert int(ctx.info("sf_zbin")) == 7            # FP32: one configuration binned, 64 explicit
    lo, hi = torch.tensor([0.0, 0.0, 9.0], device="cuda"), torch.tensor([L, L, h - 9.0], device="cuda")
    gen = torch.Generator(device="cuda").manual_seed(1)

    def positions(batch):
        return lo + (hi - lo) * torch.rand((batch, m, 3), dtype=torch.float64, device="cuda", generator=gen)

    def buffers(batch):
        return (torch.empty((batch, n), dtype=torch.float32, device="cuda"),
                torch.empty((batch, n), dtype=torch.float64, device="cuda"))

    x = positions(captured)
    (b, q), (be, qe), (bo, _) = buffers(captured), buffers(captured), buffers(between)
    # what an eager call could allocate, before the capture
    ctx.solve_charges(torch.zeros((64, n), dtype=torch.float32, device="cuda"), cpm.SOLVE_F64, buffers(64)[1])
    ctx.synchronize()
    ctx.capture_step(x, b, cpm.SOLVE_F64, q)
    for rep in range(3):
        x.copy_(positions(captured))
        other = positions(between)
        torch.cuda.synchronize()
        ctx.potential_vector(other, bo)
        ctx.replay_step()
        ctx.potential_vector(x, be)
        ctx.solve_charges(be, cpm.SOLVE_F64, qe)
        ctx.synchronize()
        say(f"captured {captured}, {between} between, replay {rep}")
        assert torch.equal(b, be) and torch.equal(q, qe)
    ctx.close()


def test_other_electrodes_take_structure_factors(cpm):
    w = I.small_capacitor("a")
    rng = np.random.default_rng(7)
    R = w.electrode_xyz.copy()
    R[:, 2] += rng.uniform(-1e-3, 1e-3, len(R))
    w = w.with_(electrode_xyz=R, h=float(R[:, 2].max() - R[:, 2].min()))
    say("atoms on no common planes")
    check(cpm, cpm.Params.of(w), O.params_for(w), R, w.electrode_id, w.electrolyte_q,
          np.stack([I.snapshot(w, s) for s in range(2)]), 0, 2)
