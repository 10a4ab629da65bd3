"""GPU checks of the schedules of the detailed-chemistry step for a mechanism that does not fit one wave per cell:
the 16-lane, 32-lane and mixed launches and the queue of 16-lane groups and cold cells per lane.

The hydrogen mechanism of the other schedule tests fits (its mappings 0, 2, 4 and 5 and its queue are one
kernel, with the same bits throughout); four falloff reactions among 24 leave no lanes for the last one's
quad.  Parity bar as in test_gpu_sched.
"""
import numpy as np
import pytest

import oracle
from synth import fields
from synth.mechfile import write_mech
from synth.mechgen import generate_h2_mechanism
from test_gpu_chem import compare
from test_gpu_sched import RTOL_PARITY, SCHEDULES, _cells, _run

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def wide(tmp_path_factory):
    """24 reactions, four of them falloff: (mechanism, GPU handle, oracle handle)."""
    import paper_2210_07094_amd as df
    m = generate_h2_mechanism(seed=20221016, n_exchange=18, n_third_body=2, n_troe=4)
    path = str(tmp_path_factory.mktemp("wide") / "wide.mech")
    write_mech(path, m)
    return m, df.Mechanism(path), oracle.Mech(path)


@pytest.mark.parametrize("label,kw", [*SCHEDULES, ("queue, 5 waves 16-lane groups", dict(schedule=2, coop_blocks=5))],
                         ids=lambda v: v if isinstance(v, str) else "")
def test_per_cell_dt_parity(wide, label, kw):
    import paper_2210_07094_amd as df
    m, gm, om = wide
    f = _cells(m)
    print(f"case: {label}", flush=True)
    g = _run(gm, f, df.chem_opts(**kw), ld=1100, rr=True)
    o = om.chem_step(f["T"], f["p"], f["Y"], f["dt"], h_inout=np.zeros(f["T"].size), want_rr=True)
    assert np.array_equal(g["status"], o["status"])
    worst, flipped, tol_err = compare(g, o)
    assert worst <= RTOL_PARITY, worst
    assert flipped <= 3 and tol_err <= 10.0, (flipped, tol_err)


def test_group_schedules_same_bits(wide):
    """16 lanes, 32 lanes (the second 16 taking half the rate constants), 32 lanes for the head of the cost
    order (512 of the 4,096 cells) and the queue's groups do the same arithmetic for a cell.  With
    five group waves, or none, the cold cells go one per lane first (rounding may differ there) and the hot ones to
    groups."""
    import paper_2210_07094_amd as df
    m, gm, _ = wide
    f = fields.hot_kernel_field_2d(m, nx=64, ny=64)
    f["dt"] = np.full(f["T"].size, 1e-6)
    print("case: 16 lanes", flush=True)
    a = _run(gm, f, df.chem_opts(schedule=1, mapping=2))
    for kw in (dict(schedule=1, mapping=4), dict(schedule=1, mapping=5), dict(schedule=1, mapping=0),
               dict(schedule=2, coop_blocks=0)):
        print(f"case: {kw}", flush=True)
        b = _run(gm, f, df.chem_opts(**kw))
        for k in ("status", "n_acc", "n_rej", "T", "Y"):
            assert np.array_equal(a[k], b[k]), (kw, k)
    hot = f["T"] > 600.0
    assert hot.sum() > 100
    for blocks in (5, -1):
        print(f"case: coop_blocks {blocks}", flush=True)
        c = _run(gm, f, df.chem_opts(schedule=2, coop_blocks=blocks))
        assert np.array_equal(a["status"], c["status"])
        for k in ("n_acc", "n_rej", "T", "Y"):
            assert np.array_equal(a[k][..., hot], c[k][..., hot]), (blocks, k)


@pytest.mark.parametrize("n", [300, 1, 513])
def test_head_and_its_rest(wide, n):
    """Fewer cells than the 32-lane head (no 16-lane block runs), and one more than it holds."""
    import paper_2210_07094_amd as df
    m, gm, _ = wide
    f = _cells(m, n=n, seed=17)
    print(f"case: head variant, {n} cells", flush=True)
    a = _run(gm, f, df.chem_opts(schedule=1, mapping=2))
    e = _run(gm, f, df.chem_opts(schedule=1, mapping=5))
    for k in ("status", "n_acc", "n_rej", "T", "Y"):
        assert np.array_equal(a[k], e[k]), k
    assert np.all(a["status"] == df.CELL_OK)


def test_autotune(wide):
    import paper_2210_07094_amd as df
    import torch
    m, gm, om = wide
    f = _cells(m, n=2048, seed=5)
    T, p, Y, dt = (torch.tensor(f[k], device="cuda:0") for k in ("T", "p", "Y", "dt"))
    print("case: autotune", flush=True)
    o = gm.autotune(T, p, Y, dt)
    assert o.schedule in (1, 2) and o.coop_blocks >= -1 and o.mapping in (0, 1, 4)
    g = _run(gm, f, o)
    ro = om.chem_step(f["T"], f["p"], f["Y"], f["dt"], h_inout=np.zeros(f["T"].size))
    worst, flipped, tol_err = compare(g, ro)
    assert worst <= RTOL_PARITY and flipped <= 3 and tol_err <= 10.0


@pytest.mark.parametrize("n", [40 * 1024, 40 * 1024 + 1])
def test_cold_cells_per_lane_of_a_mechanism_that_fits_a_wave(h2_path, h2_mech, n):
    """Where a queue call with coop_blocks leaves one wave per cell (the bits of the static launch) for 16-lane groups
    and cold cells one per lane (the parity bar against it)."""
    import paper_2210_07094_amd as df
    gm = df.Mechanism(h2_path)
    c = _cells(h2_mech, n=1001)
    c["T"][500:] = np.linspace(300.0, 490.0, 501)
    f = {k: np.resize(c[k], n) for k in ("T", "p", "dt")}
    f["Y"] = np.ascontiguousarray(c["Y"][:, np.arange(n) % 1001])
    f["dt"] = f["dt"] * 0.02
    print(f"case: {n} cells", flush=True)
    a = _run(gm, f, df.chem_opts())
    for blocks in (8, -1):
        print(f"case: coop_blocks {blocks}", flush=True)
        b = _run(gm, f, df.chem_opts(schedule=2, coop_blocks=blocks))
        assert np.array_equal(a["status"], b["status"]) and np.all(a["status"] == df.CELL_OK)
        if n <= 40 * 1024:
            for k in ("T", "Y", "n_acc", "n_rej"):
                assert np.array_equal(a[k], b[k]), k
        else:
            worst, flipped, tol_err = compare(b, a)
            assert worst <= RTOL_PARITY, worst
            assert flipped <= n // 500 and tol_err <= 10.0, (flipped, tol_err)
