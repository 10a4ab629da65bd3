"""The DNN step at the edges of its tiles: a cell's result does not depend on how many cells share
the call.

Every sum of the step (the layers' reductions, the sums over the species) runs in an order that the
row count does not change, so the first n cells of a large call and a call of these n cells give the
same bits; the large call itself is held to the oracle by the parity tests.  The counts sit at the
edges of the 16-cell output tiles, the 32-cell input tiles and the 128-row layer tiles, and of the
row counts at which the layers of these networks change their tile.  Cells outside the training
range and with non-finite input are mixed in, and the field's leading dimension exceeds n: those
cells and the columns beyond n stay as they were.
"""
import numpy as np
import pytest

from synth import dnnfile, fields, read_mech
from test_gpu_dnn import _cells, _net, _torch
from test_gpu_dnn_large import HC_MECH

pytestmark = pytest.mark.gpu

SIZES = [1, 15, 16, 17, 31, 33, 127, 129, 257, 1009, 1025, 2081, 4200]
LARGE = 12000


@pytest.fixture(scope="module")
def cases(tmp_path_factory, h2_path, h2_mech):
    import paper_2210_07094_amd as df
    _torch()
    d = tmp_path_factory.mktemp("nets")

    def mixed(f):
        f["T"][5::11] = np.nan       # non-finite
        f["T"][3::7] = 6000.0        # outside the box below
        return f

    def box(K):
        return (np.concatenate([[0.0, 0.0], np.full(K, -1e9)]), np.concatenate([[5000.0, 1e9], np.full(K, 1e9)]))

    _net(d / "h2.dfdnn", box=box(9))
    f9 = mixed(_cells(h2_mech, LARGE, seed=77))
    hc = read_mech(HC_MECH)
    f53 = fields.hydrocarbon_field(hc, n=LARGE)
    f53["Y"] = np.ascontiguousarray(f53["Y"])
    _net(d / "hc.dfdnn", K=53, hidden=(320, 480, 160), box=box(53))
    f53 = mixed(f53)
    out = {}
    for key, mech, f, net in (("h2", h2_path, f9, "h2.dfdnn"), ("hc", HC_MECH, f53, "hc.dfdnn")):
        dnn = df.DNN(d / net, df.Mechanism(mech))
        out[key] = dnn, f, {}
    return out


def _run(dnn, f, n, precision, ld=None):
    import paper_2210_07094_amd as df
    torch = _torch()
    K, ld, dev = f["Y"].shape[0], ld or n, "cuda:0"
    T = torch.tensor(f["T"][:n].copy(), device=dev)
    p = torch.tensor(f["p"][:n].copy(), device=dev)
    Yh = np.full((K, ld), -3.0)
    Yh[:, :n] = f["Y"][:, :n]
    Y = torch.tensor(Yh, device=dev)
    rr = torch.full((K, ld), -5.0, dtype=torch.float64, device=dev)
    st = torch.full((n,), -7, dtype=torch.int32, device=dev)
    dnn.step(T, p, Y, 1e-6, rr=rr, status=st, opts=df.dnn_opts(renormalise=1, fallback=0, precision=precision))
    torch.cuda.synchronize()
    return T.cpu().numpy(), Y.cpu().numpy(), rr.cpu().numpy(), st.cpu().numpy()


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("key", ["h2", "hc"])
@pytest.mark.parametrize("n", SIZES)
def test_result_does_not_depend_on_the_row_count(cases, key, precision, n):
    dnn, f, ref = cases[key]
    print(f"case: {key}, n={n}, precision={precision}", flush=True)
    if precision not in ref:
        ref[precision] = _run(dnn, f, LARGE, precision)
    To, Yo, ro, so = ref[precision]
    T, Y, rr, st = _run(dnn, f, n, precision, ld=n + 3)
    np.testing.assert_array_equal(st, so[:n])
    np.testing.assert_array_equal(T, To[:n])
    np.testing.assert_array_equal(Y[:, :n], Yo[:, :n])
    np.testing.assert_array_equal(rr[:, :n], ro[:, :n])
    assert np.all(Y[:, n:] == -3.0) and np.all(rr[:, n:] == -5.0)
    out = st != 0
    np.testing.assert_array_equal(T[out], f["T"][:n][out])
    np.testing.assert_array_equal(Y[:, :n][:, out], f["Y"][:, :n][:, out])
    nan = ~np.isfinite(f["T"][:n])
    assert np.all(st[nan] == 3) and np.all(st[~nan & (f["T"][:n] > 5000.0)] == 4)
