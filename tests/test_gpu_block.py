"""GPU checks of the one-block-per-cell kernel at the edges of its layout: no third-body reaction at all, the
most that fit its eight lanes per wave (64) and one more (which takes the one-wave kernel), and reaction
counts inside and beyond its LDS; the forms of a call that reach it; and more fallback cells than blocks.

Parity bar as in test_gpu_wave (<= 1e-8 relative against the oracle where the accept/reject sequences agree).
"""
import copy

import numpy as np
import pytest

import oracle
import synth
from synth import fields
from synth.mechfile import write_mech
from test_gpu_chem import _gpu_step, compare
from test_gpu_dnn import _net
from test_gpu_wave import HC_MECH

pytestmark = pytest.mark.gpu


def _rows(m, idx):
    """The mechanism with the reactions idx (a repeated one at a quarter of its rate)."""
    m = copy.deepcopy(m)
    idx = np.asarray(idx)
    again = np.array([i in idx[:n] for n, i in enumerate(idx)])
    for f in ("reaction_type", "nu_reac", "nu_prod", "arrhenius", "efficiency", "falloff_low", "troe"):
        setattr(m, f, np.asarray(getattr(m, f))[idx].copy())
    m.arrhenius[again, 0] *= 0.25
    return m


def _mechanism(kind):
    m = synth.read_mech(HC_MECH)
    t = np.asarray(m.reaction_type)
    every, tb, plain = list(range(t.size)), list(np.flatnonzero(t == 1)), list(np.flatnonzero(t == 0))
    n3 = int((t != 0).sum())
    if kind == "no third body":
        return _rows(m, plain)
    if kind == "64 third-body":
        return _rows(m, every + tb[:64 - n3])
    if kind == "65 third-body":
        return _rows(m, every + tb[:65 - n3])
    return _rows(m, every + plain[:kind - t.size])  # a reaction count


@pytest.mark.parametrize("kind", ["no third body", "64 third-body", "65 third-body", 390, 503])
def test_mechanism_edges(tmp_path, kind):
    import paper_2210_07094_amd as df
    m = _mechanism(kind)
    path = str(tmp_path / "m.mech")
    write_mech(path, m)
    gm, om = df.Mechanism(path), oracle.Mech(path)
    f = fields.hydrocarbon_field(m, n=256, seed=5)
    idx = np.argsort(f["T"])[np.linspace(0, 255, 17).astype(int)]
    s = {"T": f["T"][idx].copy(), "p": f["p"][idx].copy(), "Y": np.ascontiguousarray(f["Y"][:, idx])}
    print(f"case: {kind}, {len(m.reaction_type)} reactions", flush=True)
    g = _gpu_step(gm, s, 1e-7, h=np.zeros(17), ld=20, rr=True)
    o = om.chem_step(s["T"], s["p"], s["Y"], 1e-7, h_inout=np.zeros(17), nthreads=8)
    assert np.array_equal(g["status"], o["status"])
    worst, flipped, tol_err = compare(g, o)
    assert worst <= 1e-8, worst
    assert flipped <= 1 and tol_err <= 10.0, (flipped, tol_err)


def test_forms_of_a_call(tmp_path):
    """A cell's bits do not depend on the launch: alone, in the field, mapping 0 or 3, from the fallback list of a
    DNN step whose box holds no cell (more cells than that launch has blocks); a sub-step limit
    ends every cell in status 1 or 0 as the oracle does."""
    import torch
    import paper_2210_07094_amd as df
    m, gm, om = synth.read_mech(HC_MECH), df.Mechanism(HC_MECH), oracle.Mech(HC_MECH)
    n = 2311
    f = fields.hydrocarbon_field(m, n=n, seed=9)
    f["Y"] = np.ascontiguousarray(f["Y"])
    print("case: field", flush=True)
    a = _gpu_step(gm, f, 1e-8, rr=True)
    print("case: mapping 3", flush=True)
    b = _gpu_step(gm, f, 1e-8, rr=True, opts=df.chem_opts(mapping=3))
    print("case: first 5 cells", flush=True)
    c = _gpu_step(gm, {"T": f["T"][:5], "p": f["p"][:5], "Y": np.ascontiguousarray(f["Y"][:, :5])}, 1e-8, rr=True)
    for k in ("T", "Y", "rr", "status"):
        np.testing.assert_array_equal(a[k], b[k])
        np.testing.assert_array_equal(a[k][..., :5], c[k])
    # the fallback list: the network's time step is 1e-6, so compare at that one on the cells it takes
    _net(tmp_path / "n.dfdnn", K=53, hidden=(160, 160), box=(np.full(55, 1e9), np.full(55, 2e9)))
    dnn = df.DNN(tmp_path / "n.dfdnn", gm)
    cold = np.argsort(f["T"])[:2200]
    s = {"T": f["T"][cold].copy(), "p": f["p"][cold].copy(), "Y": np.ascontiguousarray(f["Y"][:, cold])}
    print("case: 2,200 fallback cells", flush=True)
    ref = _gpu_step(gm, s, 1e-6)
    t = {k: torch.tensor(s[k], device="cuda:0") for k in ("T", "p", "Y")}
    st = torch.full((2200,), -7, dtype=torch.int32, device="cuda:0")
    dnn.step(t["T"], t["p"], t["Y"], 1e-6, status=st)
    torch.cuda.synchronize()
    assert np.all(st.cpu().numpy() == 4)
    np.testing.assert_array_equal(t["T"].cpu().numpy(), ref["T"])
    np.testing.assert_array_equal(t["Y"].cpu().numpy(), ref["Y"])
    print("case: a limit of 7 sub-steps", flush=True)
    s = {"T": f["T"][:9], "p": f["p"][:9], "Y": np.ascontiguousarray(f["Y"][:, :9])}
    g = _gpu_step(gm, s, 1e-6, opts=df.chem_opts(max_steps=7))
    o = om.chem_step(s["T"], s["p"], s["Y"], 1e-6, opts=oracle.default_opts(max_steps=7))
    np.testing.assert_array_equal(g["status"], o["status"])
