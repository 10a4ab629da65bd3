"""GPU checks of the chemistry step at the far ends of what it accepts: exponents far outside the range of the
exponential, and more cells than one launch has threads for.
"""
import numpy as np
import pytest

import oracle
import synth
from synth import fields, testmechs
from synth.mechfile import write_mech
from test_gpu_chem import _gpu_step, compare
from test_gpu_wave import HC_MECH

pytestmark = pytest.mark.gpu


def _far_out(path, tmp_path):
    """The mechanism with each falloff reaction's F_cent reduced to a constant in one of the usual ways (T*** -> 0 and
    T* -> infinity, T** infinite) by very small and large numbers, and reaction 0 of the plain ones switched off by its
    activation temperature."""
    m = synth.read_mech(path)
    t = np.asarray(m.reaction_type)
    m.troe[t == 2] = np.stack([m.troe[t == 2][:, 0], *np.full((3, int((t == 2).sum())), [[1e-100], [1e100], [1e100]])], 1)
    m.arrhenius[np.flatnonzero(t == 0)[0], 2] = 1e100
    out = str(tmp_path / "far.mech")
    write_mech(out, m)
    return m, out


@pytest.mark.parametrize("n, opts", [(65, {}), (65, {"mapping": 3}), (65, {"mapping": 1})])
def test_far_out_exponents(h2_path, tmp_path, n, opts):
    """Terms that such numbers switch on or off are 1 or 0, in every kernel."""
    import paper_2210_07094_amd as df
    m, path = _far_out(h2_path, tmp_path)
    gm, om = df.Mechanism(path), oracle.Mech(path)
    f = fields.ignition_cells(m, n=n, seed=7)
    f["Y"] = 0.98 * f["Y"] + 0.02 * np.random.default_rng(3).dirichlet(np.ones(9), n).T
    print(f"case: far out exponents, {opts}", flush=True)
    g = _gpu_step(gm, f, 1e-7, h=np.zeros(n), opts=df.chem_opts(**opts))
    o = om.chem_step(f["T"], f["p"], f["Y"], 1e-7, h_inout=np.zeros(n))
    assert np.all(o["status"] == 0) and np.array_equal(g["status"], o["status"])
    worst, flipped, tol_err = compare(g, o)
    assert worst <= 1e-8, worst
    assert flipped <= 2 and tol_err <= 10.0, (flipped, tol_err)


def test_far_out_exponents_hydrocarbon(tmp_path):
    import paper_2210_07094_amd as df
    m, path = _far_out(HC_MECH, tmp_path)
    gm, om = df.Mechanism(path), oracle.Mech(path)
    f = fields.hydrocarbon_field(m, n=17, seed=5)
    f["Y"] = np.ascontiguousarray(f["Y"])
    print("case: far out exponents, 53 species", flush=True)
    g = _gpu_step(gm, f, 1e-8, h=np.zeros(17))
    o = om.chem_step(f["T"], f["p"], f["Y"], 1e-8, h_inout=np.zeros(17), nthreads=8)
    assert np.all(o["status"] == 0) and np.array_equal(g["status"], o["status"])
    worst, flipped, tol_err = compare(g, o)
    assert worst <= 1e-8, worst
    assert flipped <= 1 and tol_err <= 10.0, (flipped, tol_err)


def test_far_out_exponents_adjoint(h2_path, tmp_path):
    """Gradients with 1e-100 and 1e100 are those with 1e-30 and 1e30 (the terms are 0 and 1 either way)."""
    import torch
    import paper_2210_07094_amd as df
    from test_gpu_adjoint import _taped
    m, path = _far_out(h2_path, tmp_path)
    t = np.asarray(m.reaction_type)
    m.troe[t == 2, 1:] = [1e-30, 1e30, 1e30]
    m.arrhenius[np.flatnonzero(t == 0)[0], 2] = 1e30
    near = str(tmp_path / "near.mech")
    write_mech(near, m)
    n = 9
    f = fields.ignition_cells(m, n=n, seed=7)
    gen = torch.Generator(device="cuda:0").manual_seed(1)
    Tb = torch.randn(n, dtype=torch.float64, device="cuda:0", generator=gen)
    Yb = torch.randn(9, n, dtype=torch.float64, device="cuda:0", generator=gen)
    out = []
    for q in (path, near):
        print(f"case: adjoint, {q}", flush=True)
        gm = df.Mechanism(q)
        _, p, _, tape, st, _ = _taped(gm, f, dt=2e-7, cap=1024)
        assert np.all(st.cpu().numpy() == df.CELL_OK)
        out.append([x.cpu().numpy() for x in gm.chem_adjoint(p, tape, 1024, Tb, Yb)])
    for a, b in zip(*out):
        assert np.all(np.isfinite(a))
        np.testing.assert_allclose(a, b, rtol=1e-12, atol=1e-14 * np.abs(b).max())


def _sparse_field(mech, n, at, K):
    """n cells on the device, unusable (NaN) except for those in `at`, and the same few cells alone."""
    import torch
    few = {"T": np.full(at.size, 1100.0), "p": np.full(at.size, 101325.0), "Y": np.zeros((K, at.size))}
    few["Y"][0], few["Y"][1] = 0.25, 0.75
    f = {"T": torch.full((n,), float("nan"), dtype=torch.float64, device="cuda:0"),
         "p": torch.full((n,), 101325.0, dtype=torch.float64, device="cuda:0"),
         "Y": torch.zeros(K, n, dtype=torch.float64, device="cuda:0")}
    f["T"][torch.as_tensor(at, device="cuda:0")] = 1100.0
    f["Y"][0], f["Y"][1] = 0.25, 0.75
    return few, f


@pytest.mark.parametrize("path, K, n, workspace", [
    ("iso", 2, 2**32 // 64, False),      # one wave per cell
    ("iso", 2, 2**32 // 64 + 1, False),
    ("iso", 2, 2**32 // 64 + 1, True),
    ("hc", 53, 2**32 // 512, False),     # eight waves per cell
    ("hc", 53, 2**32 // 512 + 1, False),
])
def test_more_cells_than_threads_of_a_launch(tmp_path, path, K, n, workspace):
    import torch
    import paper_2210_07094_amd as df
    if path == "iso":
        m, path = testmechs.isomerisation(kf=2e5), str(tmp_path / "iso.mech")
        write_mech(path, m)
    else:
        m, path = synth.read_mech(HC_MECH), HC_MECH
    gm = df.Mechanism(path)
    at = np.array([0, 1, n // 2, n - 2, n - 1])
    few, f = _sparse_field(m, n, at, K)
    print(f"case: {n} cells, {K} species, workspace {workspace}", flush=True)
    st = torch.full((n,), -7, dtype=torch.int32, device="cuda:0")
    gm.chem_step(f["T"], f["p"], f["Y"], 1e-8, status=st, workspace=gm.workspace(n) if workspace else None)
    torch.cuda.synchronize()
    assert torch.equal(st.bincount().cpu(), torch.tensor([at.size, *[0] * (df.CELL_NONFINITE - 1), n - at.size]))
    ref = _gpu_step(gm, few, 1e-8)
    np.testing.assert_array_equal(f["T"][torch.as_tensor(at, device="cuda:0")].cpu().numpy(), ref["T"])
    np.testing.assert_array_equal(f["Y"][:, torch.as_tensor(at, device="cuda:0")].cpu().numpy(), ref["Y"])


def test_adjoint_of_more_cells_than_threads_of_a_launch(tmp_path):
    import torch
    import paper_2210_07094_amd as df
    m, path, n = testmechs.isomerisation(kf=2e5), str(tmp_path / "iso.mech"), 2**32 // 64 + 1
    write_mech(path, m)
    gm = df.Mechanism(path)
    at = np.array([0, 1, n // 2, n - 2, n - 1])
    few, f = _sparse_field(m, n, at, 2)
    at_d = torch.as_tensor(at, device="cuda:0")
    out = []
    for T, p, Y in ((f["T"], f["p"], f["Y"]),
                    [torch.tensor(few[k], dtype=torch.float64, device="cuda:0") for k in ("T", "p", "Y")]):
        print(f"case: adjoint of {T.numel()} cells", flush=True)
        tape = gm.chem_step_taped(T, p, Y, 1e-9, max_substeps=4)
        Tb, Yb = torch.ones_like(T), torch.ones_like(Y)
        Yb[1] = 0.25
        out.append(gm.chem_adjoint(p, tape, 4, Tb, Yb))
        torch.cuda.synchronize()
    (T0, Y0, lnA, s), (rT0, rY0, rlnA, rs) = out
    assert bool((rY0 != 0).any())
    for a, b in ((T0, rT0), (Y0, rY0), (lnA, rlnA)):
        assert torch.equal(a[..., at_d], b)
        assert int((a != 0).sum()) == int((b != 0).sum())
    torch.testing.assert_close(s, rs, rtol=1e-13, atol=0.0)


def test_network_on_more_cells_than_threads_of_a_launch(tmp_path):
    """16 threads per cell in the output kernel; the network is the smallest there is (2 species, 160 wide)."""
    import torch
    import paper_2210_07094_amd as df
    from test_gpu_dnn import _net
    m, path, n = testmechs.isomerisation(kf=2e5), str(tmp_path / "iso.mech"), 2**32 // 16 + 1
    write_mech(path, m)
    _net(tmp_path / "n.dfdnn", K=2, hidden=(160,))
    gm = df.Mechanism(path)
    dnn = df.DNN(tmp_path / "n.dfdnn", gm)
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < dnn.workspace_bytes(n) + 48 * n:
        pytest.skip("not enough device memory for that many cells")
    at = np.array([0, 1, n // 2, n - 2, n - 1])
    few, f = _sparse_field(m, n, at, 2)
    print(f"case: network on {n} cells", flush=True)
    st = torch.full((n,), -7, dtype=torch.int32, device="cuda:0")
    ws = dnn.workspace(n)
    dnn.step(f["T"], f["p"], f["Y"], 1e-6, status=st, workspace=ws, opts=df.dnn_opts(fallback=0))
    torch.cuda.synchronize()
    del ws
    assert torch.equal(st.bincount().cpu(), torch.tensor([at.size, *[0] * (df.CELL_NONFINITE - 1), n - at.size]))
    r = [torch.tensor(few[k], dtype=torch.float64, device="cuda:0") for k in ("T", "p", "Y")]
    dnn.step(r[0], r[1], r[2], 1e-6, opts=df.dnn_opts(fallback=0))
    at_d = torch.as_tensor(at, device="cuda:0")
    assert torch.equal(f["T"][at_d], r[0]) and torch.equal(f["Y"][:, at_d], r[2])
    del f, st
    torch.cuda.empty_cache()
