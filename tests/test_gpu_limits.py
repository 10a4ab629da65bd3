"""GPU checks of the chemistry step at the far ends of what it accepts: exponents far outside the range of the
exponential.
"""
import numpy as np
import pytest

import oracle
import synth
from synth import fields
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
