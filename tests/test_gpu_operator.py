"""The Gauss-Seidel operator form of a single dense solve (automatic engine, from 4 sweeps)
against the oracle, at the edges of its panels (128, 256 and 512 users), of its row tiles
and of the sweep counts after which b is formed anew (2, 8, 40)."""
import numpy as np
import pytest

from paper_1902_08653_amd import inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DT = {"c128": np.complex128, "c64": np.complex64}
# complex128: the parity bar of the other engines.  complex64: the solve runs in FP64 and
# its result is rounded once (2^-24 = 6e-8 per part at most).
TOL = {"c128": 1e-10, "c64": 1e-7}


def solve(H, y, prec, T, tol=0.0, lam=0.1, x0=None, pad=0, **kw):
    from paper_1902_08653_amd import cdm
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    B, U = H.shape
    plan = cdm.Plan(B, U, precision=prec, T_max=T, tol=tol, **kw)
    buf = np.full((U, B + pad), 1e6, DT[prec])
    buf[:, :B] = H.T
    Hd = torch.from_numpy(buf).cuda()
    yd = torch.from_numpy(y.astype(DT[prec])).cuda()
    x0d = None if x0 is None else torch.from_numpy(x0.astype(DT[prec])).cuda()
    plan.solve(Hd, yd, N0=lam, x0=x0d)
    x, info = plan.solve(Hd, yd, N0=lam, x0=x0d)      # the second solve starts from a used workspace
    torch.cuda.synchronize()
    out = x.cpu().numpy().astype(np.complex128), cdm.parse_info(info)[0], plan.describe()
    plan.close()
    return out


def relerr(a, b):
    return np.linalg.norm(a - b) / np.linalg.norm(b)


@pytest.mark.parametrize("prec,B,U,T,pad", [
    ("c128", 64, 32, 4, 0), ("c128", 257, 127, 5, 3), ("c64", 300, 128, 8, 1), ("c128", 40, 100, 9, 0),
    ("c128", 600, 129, 4, 0), ("c64", 511, 256, 8, 2), ("c128", 530, 257, 9, 1), ("c64", 1100, 512, 41, 0),
    ("c128", 1040, 513, 40, 5), ("c128", 2048, 1025, 4, 0)])
def test_fixed_sweeps(orc, prec, B, U, T, pad):
    inst = inputs.dense_uplink(B, U, 3 * B + U)
    H, y = inst.H.astype(DT[prec]), inst.y.astype(DT[prec])
    x, rec, desc = solve(H, y, prec, T, pad=pad)
    assert '"schedule": "operator"' in desc, desc
    ref = orc.local_cd(H.astype(np.complex128), y.astype(np.complex128), 0.1, T_max=T)
    assert rec["sweeps"] == T and rec["flags"] == 0
    assert relerr(x, ref["x"]) <= TOL[prec]


@pytest.mark.parametrize("B,U,tol", [(256, 128, 1e-1), (256, 128, 1e-11), (700, 300, 3e-3), (700, 300, 1e-11),
                                     (1200, 520, 1e-2), (1200, 520, 1e-10), (520, 520, 1e-11)])
def test_stop_and_warm_start(orc, B, U, tol):
    """Tolerances that are met in the first sweeps, next to a refresh and far from one, cold
    and from a warm start: the sweep count and x are the oracle's."""
    inst = inputs.dense_uplink(B, U, B + U)
    rng = np.random.default_rng(U)
    for x0 in (None, rng.standard_normal(U) + 1j * rng.standard_normal(U)):
        x, rec, desc = solve(inst.H, inst.y, "c128", 200, tol=tol, x0=x0)
        assert '"schedule": "operator"' in desc
        ref = orc.local_cd(inst.H, inst.y, 0.1, T_max=200, tol=tol, x0=x0)
        assert rec["sweeps"] == ref["sweeps"] and rec["flags"] == 0 and rec["rel_step"] <= tol
        assert relerr(x, ref["x"]) <= 1e-10


@pytest.mark.parametrize("B,U", [(400, 100), (700, 300)])
def test_inactive_columns_caps_and_nan(orc, B, U):
    inst = inputs.dense_uplink(B, U, B)
    H = inst.H.copy(order="F")
    H[:, [0, U - 1]] = 0
    x, rec, _ = solve(H, inst.y, "c128", 6, lam=0.0)
    assert rec["flags"] == 1 and x[0] == 0 and x[U - 1] == 0
    assert relerr(x, orc.local_cd(H, inst.y, 0.0, T_max=6)["x"]) <= 1e-10
    _, rec, _ = solve(inst.H, inst.y, "c128", 5, tol=1e-12)
    assert rec["sweeps"] == 5 and rec["flags"] == 4
    H[3, 5] = np.nan
    x, rec, _ = solve(H, inst.y, "c128", 5)
    assert rec["flags"] & 2 and not np.isfinite(x).all()


def test_complex64_is_closer_than_the_panel_form(orc):
    """The FP64 operator leaves a complex64 solve no further from the exact sweeps than the
    FP32 panel engine."""
    inst = inputs.dense_uplink(1000, 400, 5)
    H, y = inst.H.astype(np.complex64), inst.y.astype(np.complex64)
    ref = orc.local_cd(H.astype(np.complex128), y.astype(np.complex128), 0.1, T_max=20)["x"]
    new, _, _ = solve(H, y, "c64", 20)
    old, _, desc = solve(H, y, "c64", 20, engine="panel")
    assert '"schedule": "operator"' not in desc
    assert relerr(new, ref) <= relerr(old, ref)
