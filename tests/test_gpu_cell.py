"""GPU checks of the one-wave-per-cell kernel for small mechanisms at the edges of its layout: how many
reactions and falloff reactions fit the lanes (and the first sizes that do not, which take the 16-lane
kernel), a species on both sides of a reaction, and the cell counts at which the queue's groups, fixed
first units and four-cell units begin and end, and at which a queue call leaves the kernel.

Parity bar as in test_gpu_chem (<= 1e-8 relative against the oracle where the accept/reject sequences
agree); a cell's result does not depend on who takes it, so the queue (with workspace) and the plain
launch (without) agree bit for bit.
"""
import numpy as np
import pytest

import oracle
import synth
from synth import fields
from synth.mechfile import write_mech
from synth.mechgen import generate_h2_mechanism
from test_gpu_chem import compare

pytestmark = pytest.mark.gpu


def _with_both_sides(m):
    """Reaction 0 becomes 2 H + H2 <=> 2 H2 (H2 on both sides)."""
    iH, iH2 = m.index("H"), m.index("H2")
    m.nu_reac[0], m.nu_prod[0] = 0, 0
    m.nu_reac[0, iH], m.nu_reac[0, iH2], m.nu_prod[0, iH2] = 2, 1, 2
    m.arrhenius[0] = (1e15, 0.0, 500.0)
    return m


def _step(gm, f, dt, workspace):
    import torch
    n = f["T"].size
    t = {k: torch.tensor(np.ascontiguousarray(f[k]), device="cuda:0") for k in ("T", "p", "Y")}
    st = torch.full((n,), -7, dtype=torch.int32, device="cuda:0")
    ns = torch.full((2 * n,), -7, dtype=torch.int32, device="cuda:0")
    rr = torch.full_like(t["Y"], -7.0)
    gm.chem_step(t["T"], t["p"], t["Y"], dt, rr=rr, status=st, n_steps=ns,
                 workspace=gm.workspace(n) if workspace else None)
    torch.cuda.synchronize()
    return {"T": t["T"].cpu().numpy(), "Y": t["Y"].cpu().numpy(), "rr": rr.cpu().numpy(), "status": st.cpu().numpy(),
            "n_acc": ns[:n].cpu().numpy(), "n_rej": ns[n:].cpu().numpy()}


@pytest.mark.parametrize("n_ex,n_tb,n_troe,both", [
    (1, 1, 0, False),      # two reactions
    (10, 3, 3, False),     # 16 reactions, three quads in the lower half
    (18, 3, 3, False),     # 24 reactions: the last quad in the upper half
    (18, 2, 4, False),     # one falloff reaction more: no lanes left, the 16-lane kernel
    (18, 4, 2, True),      # a species on both sides
    (18, 6, 1, False),     # 25 reactions: eight list entries per lane
    (19, 8, 1, False),     # 28 reactions: the last that leave a quad
    (19, 11, 0, False),    # 30 reactions, no falloff
    (19, 9, 2, False),     # 30 reactions with falloff: no lanes left, the 16-lane kernel
])
def test_mechanism_edges(tmp_path, n_ex, n_tb, n_troe, both):
    import paper_2210_07094_amd as df
    m = generate_h2_mechanism(seed=20221016, n_exchange=n_ex, n_third_body=n_tb, n_troe=n_troe)
    if both:
        m = _with_both_sides(m)
    path = str(tmp_path / "m.mech")
    write_mech(path, m)
    gm, om = df.Mechanism(path), oracle.Mech(path)
    f = fields.ignition_cells(m, n=65, seed=7)
    f["T"][::5] = np.linspace(400.0, 900.0, f["T"][::5].size)
    f["Y"] = 0.98 * f["Y"] + 0.02 * np.random.default_rng(3).dirichlet(np.ones(9), 65).T
    print(f"case: {n_ex}+{n_tb}+{n_troe} reactions, both sides {both}", flush=True)
    g = _step(gm, f, 1e-7, True)
    o = om.chem_step(f["T"], f["p"], f["Y"], 1e-7, h_inout=np.zeros(65))
    assert np.array_equal(g["status"], o["status"])
    worst, flipped, tol_err = compare(g, o)
    assert worst <= 1e-8, worst
    assert flipped <= 2 and tol_err <= 10.0, (flipped, tol_err)


@pytest.mark.parametrize("n", [1, 2, 7, 9, 63, 1023, 1024, 1025, 2047, 2049, 4095, 4097, 8191, 9001, 70001])
def test_queue_takes_every_cell_once(h2_path, h2_mech, n):
    import paper_2210_07094_amd as df
    gm = df.Mechanism(h2_path)
    f = fields.ignition_cells(h2_mech, n=n, seed=n)
    rng = np.random.default_rng(n)
    f["T"] = np.where(rng.random(n) < 0.7, rng.uniform(300.0, 500.0, n), f["T"])
    f["T"][n // 2] = np.nan
    print(f"case: {n} cells", flush=True)
    a, b = _step(gm, f, 2e-8, True), _step(gm, f, 2e-8, False)
    for k in a:
        assert np.array_equal(a[k], b[k], equal_nan=True), k
    assert a["status"][n // 2] == df.CELL_NONFINITE
    assert np.all(np.delete(a["status"], n // 2) == df.CELL_OK)


@pytest.mark.parametrize("n_ex,n_tb,n_troe,both", [
    (1, 1, 0, False), (10, 3, 3, False), (18, 3, 3, False), (18, 4, 2, True), (18, 6, 0, False),
    (18, 2, 4, False),     # no lanes left for the fourth falloff reaction: the 8-lane sweep
])
def test_sweep_mechanism_edges(tmp_path, n_ex, n_tb, n_troe, both):
    """Rows of the sensitivity matrix against the oracle's, the bar of test_gpu_adjoint."""
    import paper_2210_07094_amd as df
    from test_gpu_adjoint import RTOL_ROW, _full_matrix, _oracle_rows, _taped
    m = generate_h2_mechanism(seed=20221016, n_exchange=n_ex, n_third_body=n_tb, n_troe=n_troe)
    if both:
        m = _with_both_sides(m)
    path = str(tmp_path / "m.mech")
    write_mech(path, m)
    gm, om = df.Mechanism(path), oracle.Mech(path)
    f = fields.ignition_cells(m, n=3, seed=7)
    f["Y"] = 0.98 * f["Y"] + 0.02 * np.random.default_rng(3).dirichlet(np.ones(9), 3).T
    print(f"case: sweep, {n_ex}+{n_tb}+{n_troe} reactions, both sides {both}", flush=True)
    _, p, _, tape, st, ns = _taped(gm, f, dt=2e-7, cap=4096)
    ns = ns.cpu().numpy()
    assert np.all(st.cpu().numpy() == df.CELL_OK)
    G = _full_matrix(gm, p, tape, 3, cap=4096)
    matched = 0
    for i in range(3):
        S, sto, nacc, nrej = _oracle_rows(m, om, f, i, dt=2e-7)
        if (nacc, nrej) != (ns[i], ns[3 + i]):
            continue
        matched += 1
        err = np.abs(G[i] - S) / np.abs(S).max(axis=1, keepdims=True)
        assert err.max() <= RTOL_ROW, (i, err.max())
    assert matched >= 2


@pytest.mark.parametrize("n", [1024, 1025, 8704, 8705])
def test_taped_step_order(h2_path, h2_mech, n):
    """The cost order of a taped step lies in the lengths of the tape's last sub-step: a tape that is just
    long enough gives the gradients of a longer one bit for bit, and the step is the untaped one."""
    import torch
    import paper_2210_07094_amd as df
    from test_gpu_adjoint import _taped
    gm = df.Mechanism(h2_path)
    f = fields.ignition_cells(h2_mech, n=n, seed=3)
    print(f"case: taped order, {n} cells", flush=True)
    plain = _step(gm, f, 1e-7, False)
    cap = int(plain["n_acc"].max())
    gen = torch.Generator(device="cuda:0").manual_seed(1)
    Tb = torch.randn(n, dtype=torch.float64, device="cuda:0", generator=gen)
    Yb = torch.randn(9, n, dtype=torch.float64, device="cuda:0", generator=gen)
    out = []
    for c in (cap, cap + 7, cap - 1):
        T, p, Y, tape, st, ns = _taped(gm, f, dt=1e-7, cap=c)
        assert np.array_equal(T.cpu().numpy(), plain["T"]) and np.array_equal(Y.cpu().numpy(), plain["Y"])
        full = plain["n_acc"] > c
        assert np.array_equal(st.cpu().numpy(), np.where(full, df.CELL_TAPE_FULL, df.CELL_OK))
        out.append([x.cpu().numpy() for x in gm.chem_adjoint(p, tape, c, Tb, Yb)[:3]])
    ok = plain["n_acc"] <= cap - 1
    assert ok.any() and not ok.all()
    for a, b, c in zip(*out):
        assert np.array_equal(a, b)
        assert np.array_equal(a[..., ok], c[..., ok]) and np.all(c[..., ~ok] == 0)


def test_sweep_without_room_for_the_order(h2_path, h2_mech):
    """A workspace of the per-cell gradients alone (8 M n bytes, without the cell order) is accepted and gives the
    same bits; one byte less is refused."""
    import ctypes as C

    import torch
    import paper_2210_07094_amd as df
    from paper_2210_07094_amd import _lib
    from test_gpu_adjoint import _taped
    gm, n = df.Mechanism(h2_path), 70
    f = fields.ignition_cells(h2_mech, n=n, seed=4)
    print("case: sweep with a workspace of 8 M n bytes", flush=True)
    _, p, _, tape, _, _ = _taped(gm, f, dt=1e-7, cap=512)
    gen = torch.Generator(device="cuda:0").manual_seed(2)
    Tb = torch.randn(n, dtype=torch.float64, device="cuda:0", generator=gen)
    Yb = torch.randn(9, n, dtype=torch.float64, device="cuda:0", generator=gen)
    ref = gm.chem_adjoint(p, tape, 512, Tb, Yb)
    M, L = gm.n_reactions, _lib.lib()
    out = [torch.empty_like(x) for x in ref]
    ws = torch.empty(8 * M * n, dtype=torch.uint8, device="cuda:0")

    def call(size):
        q = [C.c_void_p(x.data_ptr()) for x in (p, tape, Tb, Yb, *out, ws)]
        return L.df_chem_adjoint(gm._h, n, n, q[0], q[1], tape.numel(), 512, q[2], q[3], q[4], q[5], q[6], q[7], q[8],
                                 size, C.c_void_p(torch.cuda.current_stream().cuda_stream))

    assert call(ws.numel() - 1) == _lib.DF_E_INVALID
    assert call(ws.numel()) == _lib.DF_OK
    torch.cuda.synchronize()
    for a, b in zip(ref, out):
        assert torch.equal(a, b)


@pytest.mark.parametrize("n", [352 * 1024, 352 * 1024 + 1])
def test_queue_of_many_cells(h2_path, h2_mech, n):
    """Where a queue call changes from one wave per cell (the bits of the static launch) to the 16-lane queue (the
    parity bar against it)."""
    import torch
    import paper_2210_07094_amd as df
    gm = df.Mechanism(h2_path)
    f = fields.ignition_cells(h2_mech, n=1001, seed=3)
    f = {"T": np.resize(f["T"], n), "p": np.resize(f["p"], n),
         "Y": np.ascontiguousarray(f["Y"][:, np.arange(n) % 1001])}
    print(f"case: queue, {n} cells", flush=True)
    a = _step(gm, f, 1e-8, True)
    t = {k: torch.tensor(f[k], device="cuda:0") for k in ("T", "p", "Y")}
    st = torch.full((n,), -7, dtype=torch.int32, device="cuda:0")
    ns = torch.full((2 * n,), -7, dtype=torch.int32, device="cuda:0")
    gm.chem_step(t["T"], t["p"], t["Y"], 1e-8, status=st, n_steps=ns, workspace=gm.workspace(n),
                 opts=df.chem_opts(schedule=2))
    torch.cuda.synchronize()
    b = {"T": t["T"].cpu().numpy(), "Y": t["Y"].cpu().numpy(), "status": st.cpu().numpy(),
         "n_acc": ns[:n].cpu().numpy(), "n_rej": ns[n:].cpu().numpy()}
    np.testing.assert_array_equal(a["status"], b["status"])
    if n <= 352 * 1024:
        for k in ("T", "Y", "n_acc", "n_rej"):
            np.testing.assert_array_equal(a[k], b[k])
    else:
        worst, flipped, tol_err = compare(b, a)
        assert worst <= 1e-8, worst
        assert flipped <= n // 500 and tol_err <= 10.0, (flipped, tol_err)


@pytest.mark.parametrize("n, out", [(300, 0), (300, 300), (2049, 1), (5000, 257), (5000, 4999)])
def test_fallback_list(h2_path, h2_mech, tmp_path, n, out):
    """Cells outside the training box of a DNN step reach the kernel through a list whose length is known on the
    device only: none, a few, more than the blocks of the launch, all but one; the bits of a plain step."""
    import torch
    import paper_2210_07094_amd as df
    from test_gpu_dnn import _net
    K = 9
    _net(tmp_path / "n.dfdnn", hidden=(160,), box=(np.full(K + 2, -1e300), np.r_[1e300, 2e5, np.full(K, 1e300)]))
    gm = df.Mechanism(h2_path)
    dnn = df.DNN(tmp_path / "n.dfdnn", gm)
    f = fields.ignition_cells(h2_mech, n=n, seed=n)
    pick = np.random.default_rng(out).permutation(n)[:out]
    f["p"][pick] = 3e5  # beyond the box
    print(f"case: {out} of {n} cells outside the box", flush=True)
    t = {k: torch.tensor(np.ascontiguousarray(f[k]), device="cuda:0") for k in ("T", "p", "Y")}
    st = torch.full((n,), -7, dtype=torch.int32, device="cuda:0")
    dnn.step(t["T"], t["p"], t["Y"], 1e-6, status=st)
    torch.cuda.synchronize()
    st = st.cpu().numpy()
    assert np.all(st[pick] == df.CELL_DNN_FALLBACK) and np.all(np.delete(st, pick) == df.CELL_OK)
    if out:
        ref = _step(gm, {"T": f["T"][pick], "p": f["p"][pick], "Y": np.ascontiguousarray(f["Y"][:, pick])}, 1e-6, False)
        np.testing.assert_array_equal(t["T"].cpu().numpy()[pick], ref["T"])
        np.testing.assert_array_equal(t["Y"].cpu().numpy()[:, pick], ref["Y"])
