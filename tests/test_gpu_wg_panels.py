"""The per-instance engine's panels of columns against the oracle, at the edges of their
tiles: 1, 2 and 4 rows per thread, panels of 8 and 4 columns with a ragged last one, more
columns than rows, and an instance whose panel inverses do not fit the LDS (columns one by
one).  Also the fusion in the clusters' own launch, whose count has to return to zero.
Bars: those of the other engines (complex128 1e-10, complex64 1e-5)."""
import numpy as np
import pytest

from paper_1902_08653_amd import inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DT = {"c128": np.complex128, "c64": np.complex64}
TOL = {"c128": 1e-10, "c64": 1e-5}


def relerr(a, b):
    return np.linalg.norm(a - b) / np.linalg.norm(b)


def need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("prec", ["c128", "c64"])
@pytest.mark.parametrize("B,U,T", [(1, 1, 2), (63, 7, 3), (64, 8, 2), (65, 9, 3), (256, 31, 2), (257, 40, 3),
                                   (513, 25, 2), (1024, 17, 2), (1025, 30, 3), (2048, 12, 2), (30, 70, 4),
                                   (40, 3300, 1)])
def test_single_instance(orc, prec, B, U, T):
    from paper_1902_08653_amd import cdm
    need_gpu()
    inst = inputs.dense_uplink(B, U, B + U)
    H, y = inst.H.astype(DT[prec]), inst.y.astype(DT[prec])
    rng = np.random.default_rng(U)
    for x0 in (None, rng.standard_normal(U) + 1j * rng.standard_normal(U)):
        plan = cdm.Plan(B, U, precision=prec, T_max=T, engine="wg")
        x0h = None if x0 is None else x0.astype(DT[prec])
        x, info = plan.solve(torch.from_numpy(np.ascontiguousarray(H.T)).cuda(), torch.from_numpy(y).cuda(), N0=0.1,
                             x0=None if x0 is None else torch.from_numpy(x0h).cuda())
        torch.cuda.synchronize()
        rec = cdm.parse_info(info)[0]
        plan.close()
        ref = orc.local_cd(H.astype(np.complex128), y.astype(np.complex128), 0.1, T_max=T,
                           x0=None if x0 is None else x0h.astype(np.complex128))
        assert rec["sweeps"] == T and rec["flags"] == 0
        assert relerr(x.cpu().numpy(), ref["x"]) <= TOL[prec]


@pytest.mark.parametrize("prec", ["c128", "c64"])
def test_inactive_columns_and_stop(orc, prec):
    from paper_1902_08653_amd import cdm
    need_gpu()
    inst = inputs.dense_uplink(300, 43, 8)
    H, y = inst.H.astype(DT[prec]).copy(order="F"), inst.y.astype(DT[prec])
    H[:, [0, 8, 42]] = 0
    Hd, yd = torch.from_numpy(np.ascontiguousarray(H.T)).cuda(), torch.from_numpy(y).cuda()
    plan = cdm.Plan(300, 43, precision=prec, T_max=100, tol=1e-5, engine="wg")
    x, info = plan.solve(Hd, yd, N0=0.0)
    torch.cuda.synchronize()
    rec = cdm.parse_info(info)[0]
    plan.close()
    ref = orc.local_cd(H.astype(np.complex128), y.astype(np.complex128), 0.0, T_max=int(rec["sweeps"]))
    assert rec["flags"] == 1 and rec["rel_step"] <= 1e-5
    assert relerr(x.cpu().numpy(), ref["x"]) <= TOL[prec]


@pytest.mark.parametrize("Bc", [[20, 20, 20], [5, 300, 64, 1, 129]])
def test_fusion_in_the_clusters_launch_repeats(orc, Bc):
    """Repeated solves, then graph replays with eager solves between them."""
    from paper_1902_08653_amd import cdm
    need_gpu()
    B, U, C = sum(Bc), 11, len(Bc)
    inst = inputs.dense_uplink(B, U, C)
    plan = cdm.Plan(B, U, C_clusters=C, T_max=3, Bc=Bc)
    Hd, yd = torch.from_numpy(np.ascontiguousarray(inst.H.T)).cuda(), torch.from_numpy(inst.y).cuda()
    x = torch.empty(U, dtype=torch.complex128, device="cuda")
    info = torch.empty(32 * C, dtype=torch.uint8, device="cuda")
    ref = orc.uplink_cd(inst.H, inst.y, 0.1, 1.0, T_max=3, C_clusters=C, Bc=Bc)["x"]
    for _ in range(3):
        x.zero_()
        plan.solve(Hd, yd, N0=0.1, x=x, info=info)
        assert relerr(x.cpu().numpy(), ref) <= 1e-10
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        plan.solve(Hd, yd, N0=0.1, x=x, info=info)
    for _ in range(3):
        x.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert relerr(x.cpu().numpy(), ref) <= 1e-10
        plan.solve(Hd, yd, N0=0.1, x=x, info=info)
        assert relerr(x.cpu().numpy(), ref) <= 1e-10
    plan.close()
