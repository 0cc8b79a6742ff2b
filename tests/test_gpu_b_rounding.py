"""Rounding of the response coefficients of the binned sums (FP64 b).

b of two unit charges, where no sum over charges rounds, against long double: the root
mean square over atoms and 48 pairs is that of the explicit structure factors, within
the quarter by which two such samples may differ (1 / sqrt(2 48) each).  In a narrow tall
cell, where the column (0, 0) is far the largest.  Coefficients taken from values at
Chebyshev nodes have the rounding of the whole response at every order, and phases
whose rounding grows with k_z: half as much again to twice.
"""
import sys

import numpy as np
import pytest
from scipy.special import erfc

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

LD = np.longdouble
PI2 = LD(2) * np.arctan2(LD(0), LD(-1))
KE = 14.399645478425668


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


def trig(turns):
    t = turns - np.rint(turns)
    return np.cos(PI2 * t), np.sin(PI2 * t)


def b_long_double(R, x, q, L, h, alpha, eta, rcut):
    """b of one configuration in long double (slab with Lz = 3 h; erfc in FP64)."""
    Lx, Ly, Lz = LD(L[0]), LD(L[1]), LD(3 * h)
    kc = 2 * alpha * np.sqrt(np.log(1e8))
    q, x = q.astype(LD), x.astype(LD)
    n = np.arange(int(kc * 3 * h / (2 * np.pi)) + 1)
    zc, zs = trig(n[:, None] * (x[:, 2] / Lz)[None, :])
    planes, lay = np.unique(R[:, 2], return_inverse=True)
    pc, ps = trig(n[:, None] * (planes.astype(LD) / Lz)[None, :])
    R = R.astype(LD)
    phi = np.zeros(len(R), LD)
    for a in range(int(kc * L[0] / (2 * np.pi)) + 1):
        for b in range(-int(kc * L[1] / (2 * np.pi)), int(kc * L[1] / (2 * np.pi)) + 1):
            if a == 0 and b < 0:
                continue
            k2 = (PI2 * a / Lx) ** 2 + (PI2 * b / Ly) ** 2 + (PI2 * n / Lz) ** 2
            keep = (k2.astype(float) <= kc * kc) & (k2 > 0)
            if not keep.any():
                continue
            wt = np.where(keep, 4 * PI2 / (Lx * Ly * Lz) * np.exp(-k2 / (4 * LD(alpha) ** 2)) /
                          np.where(keep, k2, LD(1)), LD(0))
            if a or b:
                wt = np.where(n > 0, 2 * wt, wt)           # n and -n
            c, s = trig(a * (x[:, 0] / Lx) + b * (x[:, 1] / Ly))
            re = (wt * (zc @ (q * c))) @ pc + (wt * (zs @ (q * c))) @ ps
            im = (wt * (zc @ (q * s))) @ pc + (wt * (zs @ (q * s))) @ ps
            ec, es = trig(a * (R[:, 0] / Lx) + b * (R[:, 1] / Ly))
            phi += ec * re[lay] + (es * im[lay] if a or b else 0)
    for i, r in enumerate(R):
        for a in (-1, 0, 1):
            for b in (-1, 0, 1):
                d = np.sqrt((r[0] - x[:, 0] + a * Lx) ** 2 + (r[1] - x[:, 1] + b * Ly) ** 2 + (r[2] - x[:, 2]) ** 2)
                s = d < rcut
                e = erfc((alpha * d[s]).astype(float)) - erfc((eta * d[s]).astype(float))
                phi[i] += (q[s] * e / d[s]).sum()
    phi += 2 * PI2 / (Lx * Ly * Lz) * R[:, 2] * (q * x[:, 2]).sum()
    return -LD(KE) * phi


def test_response_rounding(cpm, monkeypatch):
    L, h, alpha, eta, rcut, pairs = (12.0, 12.5), 60.0, 0.3, 1.979, 12.0, 48
    rng = np.random.default_rng(9)
    z = np.repeat([0.0, 3.35, h - 3.35, h], 6)
    R = np.column_stack([rng.uniform(0, L[0], 24), rng.uniform(0, L[1], 24), z])
    eid = (z > 0.5 * h).astype(np.int32)
    q = np.array([1.0, -1.0])
    xyz = np.stack([np.column_stack([rng.uniform(0, L[0], 2), rng.uniform(0, L[1], 2),
                                     rng.uniform(6, h - 6, 2)]) for _ in range(pairs)])
    ref = np.stack([b_long_double(R, x, q, L, h, alpha, eta, rcut) for x in xyz])
    rms = {}
    for route in ("0", "2"):
        monkeypatch.setenv("CPM_SF_ZBIN", route)
        ctx = cpm.Context(cpm.Params(L[0], L[1], h, alpha=alpha, eta=eta, rcut=rcut))
        ctx.set_electrolyte(q)
        ctx.build_elastance(torch.as_tensor(R, device="cuda"), torch.as_tensor(eid, device="cuda"), 2)
        b = torch.empty((pairs, len(R)), dtype=torch.float64, device="cuda")
        for batch in (1, pairs):                   # narrow and wide items
            for s in range(0, pairs, batch):
                ctx.potential_vector(torch.as_tensor(xyz[s:s + batch].copy(), device="cuda"), b[s:s + batch])
            ctx.synchronize()
            rms[route, batch] = float(np.sqrt(((b.cpu().numpy() - ref) ** 2).mean()))
        ctx.close()
    for batch in (1, pairs):
        say(f"batches of {batch}: explicit {rms['0', batch]:.2e} V, binned {rms['2', batch]:.2e} V")
        assert rms["2", batch] < 1.25 * rms["0", batch]
