"""The warm-start network's kernels at the edges of their tiles: inference in 64-row tiles,
input widths on both sides of 8."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mo():
    from oracle import mlp_oracle
    return mlp_oracle


def net_of(shape, seed, max_rows=512):
    from paper_1902_08653_amd import cdm
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    net = cdm.Mlp(*shape, max_rows=max_rows)
    w = (np.random.default_rng(seed).standard_normal(net.nparam) * np.sqrt(2.0 / shape[1])).astype(np.float32)
    net.set_weights(w)
    return net, w


def relerr(a, b):
    return np.linalg.norm(a - b) / np.linalg.norm(b)


@pytest.mark.parametrize("nin,hid", [(1, 256), (8, 256), (9, 512), (16, 256), (16, 512), (8, 512)])
def test_predict_rows_do_not_depend_on_their_tile(mo, nin, hid):
    """A row's result is the same bits wherever it stands and however many rows there are, and
    the whole agrees with the BF16-operand oracle (5e-4: a pre-activation summed in another
    order can round to the neighbouring BF16 value)."""
    net, w = net_of((nin, hid, hid, 2), nin + hid, max_rows=77)    # an odd max_rows: unaligned sections
    X = np.random.default_rng(1).standard_normal((200, nin)).astype(np.float32)
    Xd = torch.from_numpy(X).cuda()
    full = net.predict(Xd, torch.complex128).cpu().numpy()
    want = mo.forward(w.astype(np.float64), (nin, hid, hid, 2), X, bf16=True)["Y"]
    assert relerr(full.view(np.float64).reshape(-1, 2), want) <= 5e-4
    for a, b in ((0, 1), (0, 63), (5, 69), (3, 68), (100, 200)):
        part = net.predict(Xd[a:b].contiguous(), torch.complex64).cpu().numpy()
        assert np.array_equal(part, full[a:b].astype(np.complex64))
    net.close()


@pytest.mark.parametrize("nin,hid,rows", [(8, 512, 1), (8, 512, 65), (1, 256, 63), (16, 512, 127), (9, 256, 700),
                                          (5, 512, 64), (8, 256, 2049)])
def test_training_pass_against_the_oracle(mo, nin, hid, rows):
    """The fused training pass in 64-row tiles, whole and ragged, with one and several row
    splits of W2's gradient: the bars of the layered pass (2e-3 per parameter block against the
    BF16-operand oracle, 1e-4 on the loss), the squared errors by 256 values, and the same bits
    from a second call after another row count."""
    shape = (nin, hid, hid, 2)
    net, w = net_of(shape, rows, max_rows=rows + rows % 3)
    rng = np.random.default_rng(rows)
    X = rng.standard_normal((rows, nin)).astype(np.float32)
    T = rng.standard_normal((rows, 2)).astype(np.float32)
    Xd, Td = torch.from_numpy(X).cuda(), torch.from_numpy(T).cuda()
    g, parts = net.gradients(Xd, Td)
    net.gradients(Xd[:rows // 2 + 1].contiguous(), Td[:rows // 2 + 1].contiguous())
    g2, parts2 = net.gradients(Xd, Td)
    assert torch.equal(g, g2) and torch.equal(parts, parts2)
    want = mo.gradients(w.astype(np.float64), shape, X, T, bf16=True)
    for a, b in zip(mo.split(g.cpu().numpy().astype(np.float64), shape), mo.split(want, shape)):
        assert relerr(a, b) <= 2e-3
    Y = net.forward(Xd).cpu().numpy().astype(np.float64)
    sq = ((Y - T) ** 2).reshape(-1)
    sq = np.pad(sq, (0, -len(sq) % 256)).reshape(-1, 256).sum(1)
    assert np.allclose(parts.cpu().numpy(), sq, rtol=1e-4)
    net.close()
