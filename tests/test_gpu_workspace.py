"""Without memory for the binned k-space sums (a bound on the context's workspace stands
for a full card) b takes the explicit structure factors instead of failing, and a bound
that leaves no room for those either is CPM_ENOMEM, with the context usable afterwards.
Against the oracle, FP64 within 1e-10 and FP32 within 5e-6 of the largest entry.
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


def test_no_room_for_the_binned_sums(cpm, monkeypatch):
    L, h, planes, per, m = (38.0, 40.0), 80.0, 40, 4, 200
    rng = np.random.default_rng(2)
    z = np.repeat(np.concatenate([np.linspace(0, 5, planes // 2), np.linspace(h - 5, h, planes // 2)]), per)
    R = np.column_stack([rng.uniform(0, L[0], len(z)), rng.uniform(0, L[1], len(z)), z])
    eid = (z > 0.5 * h).astype(np.int32)
    xyz = np.stack([np.column_stack([rng.uniform(0, L[0], m), rng.uniform(0, L[1], m),
                                     rng.uniform(7, h - 7, m)]) for _ in range(3)])
    q = np.where(np.arange(m) < m // 2, 1.0, -1.0)
    p = O.Params(L[0], L[1], 3 * h, 1.979, 0.3, 12.0, 1e-8)
    ref = np.stack([O.potential_vector(R, x, q, p) for x in xyz])
    monkeypatch.setenv("CPM_PV_GROUP", "4")
    monkeypatch.setenv("CPM_SF_ZBIN", "2")             # binned wherever there is room
    x = torch.as_tensor(xyz, device="cuda")
    routes, before, after = [], None, None
    for room in (None, 64, 1):                 # MiB beside what the build takes
        if room is not None:
            monkeypatch.setenv("CPM_MAX_WORKSPACE_MB", str(int(before / 2**20) + room))
        ctx = cpm.Context(cpm.Params(L[0], L[1], h))
        ctx.set_electrolyte(q)
        ctx.build_elastance(torch.as_tensor(R, device="cuda"), torch.as_tensor(eid, device="cuda"), 2)
        before = before or ctx.info("workspace")
        for dtype, tol in ((torch.float64, 1e-10), (torch.float32, 5e-6)):
            b = torch.full((3, len(R)), float("nan"), dtype=dtype, device="cuda")
            if room == 1:
                with pytest.raises(cpm.CpmError) as ei:
                    ctx.potential_vector(x, b)
                assert ei.value.status == 3                       # CPM_ENOMEM
                continue
            ctx.potential_vector(x, b)
            ctx.synchronize()
            err = np.abs(b.double().cpu().numpy() - ref).max() / np.abs(ref).max()
            say(f"room {room} MiB, {dtype}: {err:.2e}, {(ctx.info('workspace') - before) / 2**20:.0f} MiB taken")
            assert err < tol
        after = after or ctx.info("workspace")
        if room:
            assert ctx.info("workspace") <= before + room * 2**20
        routes.append(int(ctx.info("sf_zbin")))
        ctx.close()
    assert after > before + 64 * 2**20             # the binned sums take more than the second room
    assert routes[1] == 0 and routes[0] != 0
