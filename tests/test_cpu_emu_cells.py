"""The kernels with one wave or one block of eight waves per cell run on the CPU under sanitizers, against the oracle.

As test_cpu_emu.py does for the older kernels (what is emulated and how stands in cpu_emu/hip/hip_runtime.h):
df_chem_cell.hip in each form of its launch (cells claimed from an order by eight-wave blocks, shared out in LDS, through
a list whose length lies in memory, with a tape), the reverse sweep df_adjoint_cell.hip, and df_chem_block.hip.  The
device has two compute units here, so that nine cells fill its blocks' waves unevenly.  Three builds, one with the
sanitizers and two with automatic variables filled with a pattern and with zeros; the latter two also run the waves of
a block in different orders, and must agree bit for bit: a value that depends on a barrier that is not
there, or on which wave takes a cell, makes them differ.

Changes to the sources are textual: dynamic LDS is a pointer to the emulated block's area, register constraints
of empty assembler statements are dropped, the argument segment is the argument itself, the FP64 vector type is the
one that both compilers know, and a kernel attribute of the GPU compiler goes.
"""
import os
import re
import subprocess

import numpy as np
import pytest

import oracle
import synth
from oracle import sensitivity as sens
from synth import fields
from test_cpu_emu import BUILDS, CLANG, CSRC, EMU, H2, HC, ROOT, _cheapest_hc_cells, _parity

SOURCES = ["df_cell.h", "df_chem_cell.hip", "df_chem_block.hip", "df_adjoint_cell.hip"]
EDITS = [  # (pattern, replacement, occurrences in all files)
    (r"extern __shared__ double (lds|sh)\[\];", r"double *\1 = ::emu::dyn_lds<double>();", 3),
    (r'asm(?: volatile)?\("" : "\+[sv]"\([^;]*?\)\);', "", 9),
    (r"__attribute__\(\(ext_vector_type\(4\)\)\)", "__attribute__((vector_size(32)))", 1),
    (r"__attribute__\(\(amdgpu_waves_per_eu\(1, 1\)\)\)", "", 1),
    (r"typedef const __attribute__\(\(address_space\(4\)\)\) StepArgs \*ArgPtr;", "typedef const StepArgs *ArgPtr;", 1),
    (r"const auto seg = [^;]*__builtin_amdgcn_kernarg_segment_ptr\(\);", "", 1),
    (r"auto p = ArgPtr\(seg [^;]*;", "const ArgPtr p = &a;", 1),
]


@pytest.fixture(scope="module")
def exes(tmp_path_factory):
    d = tmp_path_factory.mktemp("emu_cells")
    text = {s: open(os.path.join(CSRC, s)).read() for s in SOURCES}
    for pat, rep, n in EDITS:
        found = 0
        for s in SOURCES:
            text[s], k = re.subn(pat, rep, text[s])
            found += k
        assert found == n, (pat, found)
    for s, t in text.items():
        (d / s).write_text(t)
    files = [os.path.join(CSRC, "df_mech.cpp"), *(str(d / s) for s in SOURCES[1:]), os.path.join(EMU, "emu_cells.cpp")]
    common = ["-std=c++17", "-w", "-I", str(d), "-I", EMU, "-I", os.path.join(ROOT, "include"), "-I", CSRC]
    procs, out = {}, {}
    for name, flags in BUILDS.items():
        if flags[0] == CLANG and not os.path.exists(CLANG):
            pytest.skip("clang++ of the ROCm toolchain not found")
        out[name] = str(d / f"emu_{name}")
        procs[name] = subprocess.Popen([*flags, *common, "-x", "c++", *files, "-o", out[name]], stdout=subprocess.PIPE,
                                       stderr=subprocess.STDOUT, text=True)
    for name, p in procs.items():
        log, _ = p.communicate(timeout=900)
        assert p.returncode == 0, f"{name} build failed:\n{log[-4000:]}"
    return out


def _run_all(exes, tmp, mech_path, form, K, f, dt):
    n = f["T"].size
    fin = tmp / "in.bin"
    with open(fin, "wb") as h:
        h.write(np.int64(n).tobytes())
        h.write(np.float64(dt).tobytes())
        for k in ("p", "T", "Y"):
            h.write(np.ascontiguousarray(f[k], np.float64).tobytes())
    procs = {}
    for seed, (name, exe) in enumerate(exes.items()):
        env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0:abort_on_error=0", UBSAN_OPTIONS="print_stacktrace=1",
                   EMU_SEED=str(seed))
        fout = tmp / f"out_{name}.bin"
        procs[name] = (subprocess.Popen([exe, mech_path, form, str(fin), str(fout)], stdout=subprocess.PIPE,
                                        stderr=subprocess.PIPE, text=True, env=env), fout)
    res = {}
    for name, (pr, fout) in procs.items():
        _, err = pr.communicate(timeout=120)
        assert pr.returncode == 0, f"{name} {form}: exit {pr.returncode}\n{err[-6000:]}"
        b = open(fout, "rb").read()
        at = 8 * n * (K + 1)
        res[name] = ({"T": np.frombuffer(b, np.float64, n, 0), "Y": np.frombuffer(b, np.float64, K * n, 8 * n).reshape(K, n),
                      "status": np.frombuffer(b, np.int32, n, at), "n_steps": np.frombuffer(b, np.int32, 2 * n, at + 4 * n),
                      "grad": np.frombuffer(b, np.float64, -1, at + 12 * n).reshape(-1, n)}, b)
    assert res["init_pattern"][1] == res["init_zero"][1], "results depend on uninitialised variables or on the wave order"
    return res


def _cells(n):
    mech = synth.read_mech(H2)
    f = fields.ignition_cells(mech, n=n, seed=5)
    f["T"][::2] = np.linspace(350.0, 700.0, f["T"][::2].size)
    f["Y"] = 0.98 * f["Y"] + 0.02 * np.random.default_rng(3).dirichlet(np.ones(9), n).T
    return mech, f


@pytest.mark.parametrize("form, n", [("queue", 7), ("queue", 21), ("plain", 2), ("plain", 19), ("list", 21)])
def test_one_wave_per_cell(exes, tmp_path, form, n):
    mech, f = _cells(n)
    dt = 1e-10
    res = _run_all(exes, tmp_path, H2, form, 9, f, dt)
    o = oracle.Mech(H2).chem_step(f["T"], f["p"], f["Y"], dt)
    if form == "list":  # every second cell was taken
        for k in ("T", "Y", "n_acc", "n_rej"):
            o[k] = np.array(o[k])
        o["T"][1::2], o["Y"][:, 1::2], o["n_acc"][1::2], o["n_rej"][1::2] = f["T"][1::2], f["Y"][:, 1::2], 0, 0
    for g, _ in res.values():
        _parity(g, o)


def test_tape_and_sweep(exes, tmp_path):
    mech, f = _cells(10)
    dt, om = 1e-10, oracle.Mech(H2)
    res = _run_all(exes, tmp_path, H2, "tape", 9, f, dt)
    o = om.chem_step(f["T"], f["p"], f["Y"], dt)
    for g, _ in res.values():
        _parity(g, o)
        for i in (0, 9):  # gradients with seeds of one: the sums of the sensitivity matrix's rows
            _, _, _, hs, _ = om.record(f["T"][i], f["p"][i], f["Y"][:, i], dt)
            y0 = np.concatenate([[f["T"][i]], f["Y"][:, i]])
            _, S = sens.sensitivities(sens.Kinetics(mech), oracle.rodas4_tableau(), f["p"][i], y0, hs)
            ref = S.sum(axis=0)
            assert np.abs(g["grad"][:, i] - ref).max() <= 1e-9 * np.abs(S).max()


def test_one_block_per_cell(exes, tmp_path):
    mech, om, f = _cheapest_hc_cells(2, 1e-9)
    res = _run_all(exes, tmp_path, HC, "block", 53, f, 1e-9)
    o = om.chem_step(f["T"], f["p"], f["Y"], 1e-9)
    for g, _ in res.values():
        _parity(g, o)
