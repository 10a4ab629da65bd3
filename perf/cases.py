"""The work that a user of the chemistry library has it do, as cases that can be timed and compared.

Every case is one call (or one training step, or one forward and reverse sweep) through the package's
public entry points, on inputs made on the device from a seed:

    for case in listed():
        state = prepare(case, seed=1)
        outputs = run(state)

Kinds of work, and what each stands for in a solver's program:

* ``integrate``  the FP64 detailed-chemistry step of one flow step: a sweep of 0-D reactors, a batch
  of igniting cells, a field with hot kernels in cold premixture, a field of developed flame, a mixing
  layer with a step length per cell, and the 53-species mechanism;
* ``infer``      the DNN step in place of the integrator, in bf16 or with FP8 hidden layers;
* ``train``      one Adam step of the network on a batch;
* ``adjoint``    the taped step and its reverse sweep through ``chem_step_diff``.
"""
import functools
import math
import os
import tempfile

import numpy as np
import torch

import paper_2210_07094_amd as df

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
H2_MECH = os.path.join(ROOT, "synth", "data", "h2_synth_9sp_24r.mech")
HC_MECH = os.path.join(ROOT, "synth", "data", "hc_synth_53sp_325r.mech")
H2_NET = os.path.join(ROOT, "paper_2210_07094_amd", "data", "h2_dnn_1600_800_400.dfdnn")
FLAME = os.path.join(ROOT, "synth", "data", "h2_field_snapshot_s.npz")
HC_HIDDEN = (3200, 1600, 800)

DEV = "cuda:0"
P_ATM = 101325.0
R = 8.31446261815324
DT = 1e-6           # a flow step of the solver, and the step the networks are trained for
TAPE_CAP = 1024     # accepted sub-steps per cell that the tape holds

# Mean attempted sub-steps per cell of each kind of field (accepted ones for the adjoint), and the
# FP64 operations (an FMA is two) that one of them takes at the least: right-hand sides, Jacobian,
# factorisation, solves and error test, as bench.py counts them.
ATTEMPTS = {"ignition": 105.0, "kernels": 7.0, "flame": 1.0, "mixing": 12.7, "hydrocarbon": 589.0, "adjoint": 240.0}
ATTEMPT_FLOPS = {9: 2.0 * 17393, 53: 2.0 * 339233}
SWEEP_FLOPS = 2.0 * 84397
SPECIES = {"ignition": 9, "kernels": 9, "flame": 9, "mixing": 9, "hydrocarbon": 53}


# ---- the cases ------------------------------------------------------------------------------------


def listed():
    return [
        # A sweep of 0-D reactors (an ignition-delay curve), the smallest call of the integrator: one
        # cell's chain of sub-steps and the launches around it.
        {"name": "reactors_21", "kind": "integrate", "field": "ignition", "n": 21},
        # A batch of igniting premixed cells, every one of them stiff; a ragged count.
        {"name": "ignition_1001", "kind": "integrate", "field": "ignition", "n": 1001},
        # The flow solver's field before ignition has spread: few hot kernels, most cells cold.
        {"name": "kernels_65536", "kind": "integrate", "field": "kernels", "n": 65536},
        # The same field later, a developed flame: every cell takes about one sub-step.
        {"name": "flame_65536", "kind": "integrate", "field": "flame", "n": 65536},
        # A 64^3 mixing layer with local time steps through the work queue, the uneven load of a
        # large flame.
        {"name": "mixing_262144_queue", "kind": "integrate", "field": "mixing", "n": 262144, "queue": True},
        # Hydrocarbon chemistry: 53 species, one wavefront per cell.
        {"name": "hydrocarbon_500", "kind": "integrate", "field": "hydrocarbon", "n": 500},
        # The DNN on one 0-D reactor: launches and latency only.
        {"name": "infer_1", "kind": "infer", "net": "h2", "n": 1, "fp8": False},
        # The DNN on a small ragged batch (a sub-domain of a parallel run).
        {"name": "infer_1000", "kind": "infer", "net": "h2", "n": 1000, "fp8": False},
        # The DNN on the whole field.
        {"name": "infer_65536", "kind": "infer", "net": "h2", "n": 65536, "fp8": False},
        # The large network of the 53-species mechanism with its FP8 layers.
        {"name": "infer_hc_65536_fp8", "kind": "infer", "net": "hc", "n": 65536, "fp8": True},
        # One step of training the network on the device.
        {"name": "train_8192", "kind": "train", "n": 8192},
        # Gradients of the step with respect to state and rate constants (forward and backward).
        {"name": "adjoint_4096", "kind": "adjoint", "n": 4096, "dt": 1e-5},
    ]


def _size(rng, lo, hi):
    """A size spread over the logarithm of [lo, hi], odd ones among them."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["ignition", "kernels", "flame", "mixing", "hydrocarbon", "infer", "infer", "infer_hc", "train",
                       "adjoint"])
    if kind == "ignition":
        return {"kind": "integrate", "field": "ignition", "n": _size(rng, 1, 4096)}
    if kind == "kernels":
        return {"kind": "integrate", "field": "kernels", "n": _size(rng, 4096, 65536)}
    if kind == "flame":
        return {"kind": "integrate", "field": "flame", "n": _size(rng, 1000, 65536)}
    if kind == "mixing":
        return {"kind": "integrate", "field": "mixing", "n": _size(rng, 16384, 262144),
                "queue": rng.random() < 0.5}
    if kind == "hydrocarbon":
        return {"kind": "integrate", "field": "hydrocarbon", "n": _size(rng, 16, 500)}
    if kind == "infer":
        return {"kind": "infer", "net": "h2", "n": _size(rng, 1, 65536), "fp8": rng.random() < 0.4}
    if kind == "infer_hc":
        return {"kind": "infer", "net": "hc", "n": _size(rng, 1000, 65536), "fp8": rng.random() < 0.5}
    if kind == "train":
        return {"kind": "train", "n": _size(rng, 256, 8192)}
    return {"kind": "adjoint", "n": _size(rng, 64, 4096),
            "dt": math.exp(rng.uniform(math.log(1e-6), math.log(1e-5)))}


# ---- mechanism, network and field data ------------------------------------------------------------


@functools.lru_cache(maxsize=None)
def _mech_data(path):
    """Species names, molar masses [kg/mol] and NASA-7 rows of a mechanism file."""
    with open(path) as fh:
        words = [w for line in fh if not line.startswith("#") for w in line.split()]
    K = int(words[words.index("n_species") + 1])
    names = words[words.index("species") + 1:][:K]
    mass = np.array(words[words.index("molar_mass") + 1:][:K], dtype=float) * 1e-3
    nasa = np.array(words[words.index("nasa7") + 1:][:7 * K], dtype=float).reshape(K, 7)
    return {"K": K, "names": names, "W": mass, "nasa": nasa}


@functools.lru_cache(maxsize=None)
def _mechanism(path):
    """The loaded mechanism, one handle for the whole program."""
    return df.Mechanism(path)


@functools.lru_cache(maxsize=None)
def _hc_net_path():
    """The 55-3200-1600-800-53 network with seeded weights: no trained one exists."""
    rng = np.random.default_rng(3)
    K = 53
    dims = [K + 2, *HC_HIDDEN, K]
    f = _hydrocarbon(4096, torch.Generator(device=DEV).manual_seed(5005))
    x = _features(f["T"], f["p"], f["Y"], 0.1).cpu().numpy()
    mu, sig = x.mean(axis=1), np.maximum(x.std(axis=1), 1e-6)
    lo = np.concatenate([[200.0, 0.5 * P_ATM], np.full(K, -10.5)])
    hi = np.concatenate([[3000.0, 20.0 * P_ATM], np.full(K, 0.5)])
    path = os.path.join(tempfile.mkdtemp(prefix="hc_net_"), "hc.dfdnn")
    with open(path, "wb") as fh:
        fh.write(b"DFDNN01\0")
        np.array([len(dims) - 1, *dims, K, 0], dtype="<i4").tofile(fh)
        np.array([0.1, DT, *mu, *sig, *np.zeros(K), *np.full(K, 0.02), *lo, *hi], dtype="<f8").tofile(fh)
        for l in range(len(dims) - 1):
            w = rng.standard_normal((dims[l + 1], dims[l]), dtype=np.float32) * math.sqrt(2.0 / dims[l])
            w *= 0.1 if l == len(dims) - 2 else 1.0
            torch.from_numpy(w).to(torch.bfloat16).view(torch.int16).numpy().tofile(fh)
            (0.05 * rng.standard_normal(dims[l + 1], dtype=np.float32)).tofile(fh)
    return path


@functools.lru_cache(maxsize=None)
def _net_data(path):
    """A network file's widths, normalisation and weights, as float64 on the device."""
    raw = open(path, "rb").read()
    L = int(np.frombuffer(raw, "<i4", 1, 8)[0])
    dims = [int(v) for v in np.frombuffer(raw, "<i4", L + 1, 12)]
    at, K = 12 + 4 * (L + 1), dims[-1]
    at += 8
    lam, dt = np.frombuffer(raw, "<f8", 2, at)
    at += 16
    out = {"dims": dims, "lam": float(lam)}
    for name, n in (("mu_in", K + 2), ("sig_in", K + 2), ("mu_out", K), ("sig_out", K), ("lo", K + 2), ("hi", K + 2)):
        out[name] = torch.tensor(np.frombuffer(raw, "<f8", n, at), device=DEV)
        at += 8 * n
    out["W"], out["b"] = [], []
    for l in range(L):
        n = dims[l] * dims[l + 1]
        bits = np.frombuffer(raw, "<u2", n, at).astype(np.uint32) << 16
        out["W"].append(torch.tensor(bits.view(np.float32), dtype=torch.float64, device=DEV).view(dims[l + 1], dims[l]))
        at += 2 * n
        out["b"].append(torch.tensor(np.frombuffer(raw, "<f4", dims[l + 1], at), dtype=torch.float64, device=DEV))
        at += 4 * dims[l + 1]
    return out


@functools.lru_cache(maxsize=None)
def _network(net):
    """The loaded network, one handle for the whole program."""
    return df.DNN(H2_NET, _mechanism(H2_MECH)) if net == "h2" else df.DNN(_hc_net_path(), _mechanism(HC_MECH))


@functools.lru_cache(maxsize=None)
def _flame_field():
    z = np.load(FLAME)
    return {k: torch.tensor(z[k], device=DEV) for k in ("T", "p", "Y")}


def _uniform(gen, n, lo, hi):
    return lo + (hi - lo) * torch.rand(n, dtype=torch.float64, device=DEV, generator=gen)


def _premixed(path, phi, fuel, fuel_moles, oxidiser):
    """Mass fractions [K, n] of fuel and air at equivalence ratio phi [n]."""
    m = _mech_data(path)
    moles = torch.zeros(m["K"], phi.numel(), dtype=torch.float64, device=DEV)
    moles[m["names"].index(fuel)] = fuel_moles * phi
    for name, v in oxidiser.items():
        moles[m["names"].index(name)] = v
    mass = moles * torch.tensor(m["W"], device=DEV)[:, None]
    return mass / mass.sum(0)


def _h2_air(phi):
    return _premixed(H2_MECH, phi, "H2", 2.0, {"O2": 1.0, "N2": 3.76})


def _ignition(n, gen):
    return {"T": _uniform(gen, n, 1000.0, 1600.0), "Y": _h2_air(_uniform(gen, n, 0.5, 2.0))}


def _kernels(n, gen):
    """Eight Gaussian hot kernels in cold premixture on a nearly square grid."""
    nx = int(math.ceil(math.sqrt(n)))
    cell = torch.arange(n, device=DEV)
    x, y = (cell % nx).double(), torch.div(cell, nx, rounding_mode="floor").double()
    amp, sig = _uniform(gen, 8, 900.0, 1500.0), _uniform(gen, 8, nx / 64.0, nx / 16.0)
    cx, cy = _uniform(gen, 8, 0.0, nx), _uniform(gen, 8, 0.0, nx)
    T = torch.full((n,), 300.0, dtype=torch.float64, device=DEV)
    for k in range(8):
        T += amp[k] * torch.exp(-((x - cx[k]) ** 2 + (y - cy[k]) ** 2) / (2.0 * sig[k] ** 2))
    return {"T": T.clamp(max=1800.0), "Y": _h2_air(torch.ones(n, dtype=torch.float64, device=DEV))}


def _flame(n, gen):
    """Cells of the stored developed-flame field."""
    f = _flame_field()
    at = torch.randint(f["T"].numel(), (n,), device=DEV, generator=gen)
    return {"T": f["T"][at], "p": f["p"][at], "Y": f["Y"][:, at]}


def _mixing(n, gen):
    """An H2/N2 fuel and air mixing layer, burnt around stoichiometry, with a step length per cell."""
    m = _mech_data(H2_MECH)
    W = torch.tensor(m["W"], device=DEV)
    iH2, iO2, iH2O, iN2 = (m["names"].index(s) for s in ("H2", "O2", "H2O", "N2"))

    def mass(moles):
        v = torch.zeros(m["K"], dtype=torch.float64, device=DEV)
        for i, x in moles.items():
            v[i] = x * W[i]
        return v / v.sum()

    fuel, ox = mass({iH2: 0.5, iN2: 0.5}), mass({iO2: 1.0, iN2: 3.76})
    s = float(0.5 * W[iO2] / W[iH2])
    z_st = float(ox[iO2] / (s * fuel[iH2] + ox[iO2]))
    side = max(2, round(n ** (1.0 / 3.0)))
    row = torch.div(torch.arange(n, device=DEV), side, rounding_mode="floor") % side
    Z = 0.5 * (1.0 - torch.tanh((row.double() - 0.5 * (side - 1)) / (0.1 * side)))
    Z = (Z + 0.02 * torch.randn(n, dtype=torch.float64, device=DEV, generator=gen)).clamp(0.0, 1.0)
    Yu = Z * fuel[:, None] + (1.0 - Z) * ox[:, None]
    burn = torch.minimum(Yu[iH2], Yu[iO2] / s)
    Yb = Yu.clone()
    Yb[iH2] -= burn
    Yb[iO2] -= s * burn
    Yb[iH2O] += (1.0 + s) * burn
    c = torch.exp(-((Z - z_st) / 0.1) ** 2)
    Y = ((1.0 - c) * Yu + c * Yb).clamp(min=0.0)
    T = 300.0 + 2200.0 * c + 50.0 * torch.randn(n, dtype=torch.float64, device=DEV, generator=gen)
    dt = torch.exp(_uniform(gen, n, math.log(1e-7), math.log(1e-5)))
    return {"T": T.clamp(300.0, 2500.0), "Y": Y / Y.sum(0), "dt": dt}


def _hydrocarbon(n, gen):
    """CH4/air between unburnt and burnt, every minor species present, 1 to 10 atm."""
    m = _mech_data(HC_MECH)
    T, p = _uniform(gen, n, 300.0, 2400.0), P_ATM * _uniform(gen, n, 1.0, 10.0)
    phi, c = _uniform(gen, n, 0.5, 1.5), _uniform(gen, n, 0.0, 1.0)
    Yu = _premixed(HC_MECH, phi, "CH4", 0.5, {"O2": 1.0, "N2": 3.72, "AR": 0.0446})
    W = torch.tensor(m["W"], device=DEV)[:, None]
    iF, iO, iC, iW = (m["names"].index(s) for s in ("CH4", "O2", "CO2", "H2O"))
    nb = Yu / W
    burn = torch.minimum(nb[iF], nb[iO] / 2.0)
    for i, k in ((iF, -1.0), (iO, -2.0), (iC, 1.0), (iW, 2.0)):
        nb[i] += k * burn
    Y = (1.0 - c) * Yu + c * nb * W
    minor = [k for k, s in enumerate(m["names"]) if s not in ("CH4", "O2", "CO2", "H2O", "N2", "AR")]
    u = torch.rand(len(minor), n, dtype=torch.float64, device=DEV, generator=gen)
    Y[minor] = torch.exp(math.log(1e-12) + (math.log(1e-3) - math.log(1e-12)) * u)
    return {"T": T, "p": p, "Y": Y / Y.sum(0)}


FIELDS = {"ignition": _ignition, "kernels": _kernels, "flame": _flame, "mixing": _mixing, "hydrocarbon": _hydrocarbon}


def _field(name, n, seed):
    f = FIELDS[name](n, torch.Generator(device=DEV).manual_seed(seed))
    f.setdefault("p", torch.full((n,), P_ATM, dtype=torch.float64, device=DEV))
    return {k: v.contiguous() for k, v in f.items()}


def _features(T, p, Y, lam):
    """Raw network inputs [K + 2, n]: T, p and the Box-Cox transform of the mass fractions."""
    return torch.cat([T[None], p[None], (Y.clamp(min=0.0) ** lam - 1.0) / lam])


def _batch(n, seed):
    """A training batch: z-scored states of igniting and hotter cells and z-scored increments, which
    have zero mean and unit variance by construction."""
    gen = torch.Generator(device=DEV).manual_seed(seed)
    net = _net_data(H2_NET)
    Y = _h2_air(_uniform(gen, n, 0.5, 2.0))
    x = _features(_uniform(gen, n, 900.0, 2400.0), torch.full((n,), P_ATM, dtype=torch.float64, device=DEV), Y,
                  net["lam"])
    x = ((x - net["mu_in"][:, None]) / torch.where(net["sig_in"] == 0, 1.0, net["sig_in"])[:, None]).T
    t = torch.randn(n, net["dims"][-1], device=DEV, generator=gen)
    return x.float().contiguous(), t


# ---- prepare and run ------------------------------------------------------------------------------


def _empty_outputs(n, K):
    return (torch.empty(K, n, dtype=torch.float64, device=DEV), torch.empty(n, dtype=torch.int32, device=DEV))


def prepare(case, seed):
    kind, n = case["kind"], case["n"]
    if kind == "integrate":
        mech = _mechanism(HC_MECH if case["field"] == "hydrocarbon" else H2_MECH)
        f = _field(case["field"], n, seed)
        rr, status = _empty_outputs(n, mech.n_species)
        return {"kind": kind, "mech": mech, "f": f, "T": torch.empty_like(f["T"]), "Y": torch.empty_like(f["Y"]),
                "dt": f.get("dt", DT), "rr": rr, "status": status, "workspace": mech.workspace(n),
                "opts": df.chem_opts(schedule=2) if case.get("queue") else None}
    if kind == "infer":
        dnn = _network(case["net"])
        f = _field("flame" if case["net"] == "h2" else "hydrocarbon", n, seed)
        rr, status = _empty_outputs(n, dnn.K)
        return {"kind": kind, "dnn": dnn, "f": f, "T": torch.empty_like(f["T"]), "Y": torch.empty_like(f["Y"]),
                "rr": rr, "status": status, "workspace": dnn.workspace(n),
                "opts": df.dnn_opts(precision=1) if case["fp8"] else None}
    if kind == "train":
        # a network of its own: training rewrites the handle's weights
        dnn = df.DNN(H2_NET, _mechanism(H2_MECH))
        x, t = _batch(n, seed)
        return {"kind": kind, "dnn": dnn, "trainer": df.Trainer(dnn, n), "x": x, "t": t}
    f = _field("ignition", n, seed)
    gen = torch.Generator(device=DEV).manual_seed(seed + 7919)
    mech = _mechanism(H2_MECH)
    return {"kind": kind, "mech": mech, "p": f["p"], "T0": f["T"].requires_grad_(), "Y0": f["Y"].requires_grad_(),
            "lnA": torch.zeros(mech.n_reactions, dtype=torch.float64, device=DEV, requires_grad=True),
            "dt": case["dt"],
            "T_bar": 1e-3 * torch.randn(n, dtype=torch.float64, device=DEV, generator=gen),
            "Y_bar": torch.randn(mech.n_species, n, dtype=torch.float64, device=DEV, generator=gen)}


def run(state):
    s = state
    if s["kind"] == "integrate":
        # the solver hands over its fields; the step works in place on the chemistry's copy
        s["T"].copy_(s["f"]["T"])
        s["Y"].copy_(s["f"]["Y"])
        s["mech"].chem_step(s["T"], s["f"]["p"], s["Y"], s["dt"], rr=s["rr"], status=s["status"],
                            workspace=s["workspace"], opts=s["opts"])
        return {"T": s["T"], "Y": s["Y"], "rr": s["rr"], "status": s["status"]}
    if s["kind"] == "infer":
        s["T"].copy_(s["f"]["T"])
        s["Y"].copy_(s["f"]["Y"])
        s["dnn"].step(s["T"], s["f"]["p"], s["Y"], DT, rr=s["rr"], status=s["status"], workspace=s["workspace"],
                      opts=s["opts"])
        return {"T": s["T"], "Y": s["Y"], "rr": s["rr"], "status": s["status"]}
    if s["kind"] == "train":
        loss = s["trainer"].step(s["x"], s["t"])
        layers = range(s["dnn"].n_layers)
        return {"loss": loss, "dW": [s["trainer"].get(l, "dW") for l in layers],
                "db": [s["trainer"].get(l, "db") for l in layers]}
    T, Y = df.chem_step_diff(s["mech"], s["T0"], s["Y0"], s["p"], s["dt"], lnA=s["lnA"], max_substeps=TAPE_CAP)
    T0_bar, Y0_bar, lnA_bar = torch.autograd.grad((T, Y), (s["T0"], s["Y0"], s["lnA"]), (s["T_bar"], s["Y_bar"]))
    return {"T": T.detach(), "Y": Y.detach(), "T0_bar": T0_bar, "Y0_bar": Y0_bar, "lnA_bar": lnA_bar}


# ---- what a pass cannot do without ----------------------------------------------------------------


def _net_flops(dims):
    return 2.0 * sum(a * b for a, b in zip(dims[:-1], dims[1:]))


def work(case):
    kind, n = case["kind"], case["n"]
    if kind == "integrate":
        K = SPECIES[case["field"]]
        per_cell = 8 * 3 + 8 * 3 * K + 4 + (8 if case["field"] == "mixing" else 0)
        return {"bytes": n * per_cell, "flops": n * ATTEMPTS[case["field"]] * ATTEMPT_FLOPS[K]}
    if kind == "infer":
        dims = [11, 1600, 800, 400, 9] if case["net"] == "h2" else [55, *HC_HIDDEN, 53]
        weights = sum(2 * a * b + 4 * b for a, b in zip(dims[:-1], dims[1:]))
        return {"bytes": n * (8 * 3 + 8 * 3 * dims[-1] + 4) + weights, "flops": n * _net_flops(dims)}
    if kind == "train":
        dims = [11, 1600, 800, 400, 9]
        params = sum(a * b + b for a, b in zip(dims[:-1], dims[1:]))
        # per parameter: weight and two moments read and written, the bf16 copy, the gradient out
        return {"bytes": n * 4 * (dims[0] + dims[-1]) + params * (4 * 6 + 2 + 4), "flops": 3.0 * n * _net_flops(dims)}
    # state in and out, seeds and gradients; the sub-steps grow with the step length
    steps = ATTEMPTS["adjoint"] * (case["dt"] / 1e-5) ** 0.5
    return {"bytes": n * 8 * (1 + 4 * 10), "flops": n * steps * (ATTEMPT_FLOPS[9] + SWEEP_FLOPS)}


# ---- the same in 64 bits --------------------------------------------------------------------------


def _forward64(net, x, W, b):
    a = x
    for l in range(len(W)):
        a = a @ W[l].T + b[l]
        if l < len(W) - 1:
            a = torch.nn.functional.gelu(a)
    return a


def _enthalpy(T, Y, m):
    """h [J/kg] and cp [J/kg/K] of the mixture."""
    a = torch.tensor(m["nasa"], device=DEV)
    iW = 1.0 / torch.tensor(m["W"], device=DEV)[:, None]
    t = T[None]
    cp = a[:, 0:1] + t * (a[:, 1:2] + t * (a[:, 2:3] + t * (a[:, 3:4] + t * a[:, 4:5])))
    h = a[:, 5:6] + t * (a[:, 0:1] + t * (a[:, 1:2] / 2 + t * (a[:, 2:3] / 3 + t * (a[:, 3:4] / 4 + t * a[:, 4:5] / 5))))
    return (Y * iW * R * h).sum(0), (Y * iW * R * cp).sum(0)


def exact(case, seed):
    """What run() returns, in plain torch and 64 bits.  None for the integrator and its adjoint: they
    are FP64 already, and another integration of the same equations agrees with them only to the
    step-size controller's tolerance."""
    n = case["n"]
    if case["kind"] == "infer":
        path = H2_NET if case["net"] == "h2" else _hc_net_path()
        net, m = _net_data(path), _mech_data(H2_MECH if case["net"] == "h2" else HC_MECH)
        f = _field("flame" if case["net"] == "h2" else "hydrocarbon", n, seed)
        x = _features(f["T"], f["p"], f["Y"], net["lam"])
        assert bool(((x >= net["lo"][:, None]) & (x <= net["hi"][:, None])).all()), "a cell outside the training box"
        x = (x - net["mu_in"][:, None]) / torch.where(net["sig_in"] == 0, 1.0, net["sig_in"])[:, None]
        u = torch.cat([_forward64(net, c, net["W"], net["b"]) for c in x.T.split(8192)]).T
        z = (f["Y"].clamp(min=0.0) ** net["lam"] - 1.0) / net["lam"]
        z = z + net["mu_out"][:, None] + net["sig_out"][:, None] * u
        Y = (1.0 + net["lam"] * z).clamp(min=0.0) ** (1.0 / net["lam"])
        Y = Y / Y.sum(0)
        h0, T = _enthalpy(f["T"], f["Y"], m)[0], f["T"].clone()
        for _ in range(30):
            h, cp = _enthalpy(T, Y, m)
            T = T - (h - h0) / cp
        # no value for rr: a difference of two nearly equal states over 1 us, most of it the rounding
        # of the bf16 activations
        return {"T": T, "Y": Y, "rr": None, "status": torch.zeros(n, dtype=torch.int32, device=DEV)}
    if case["kind"] == "train":
        net = _net_data(H2_NET)
        x, t = (v.double() for v in _batch(n, seed))
        W = [w.clone().requires_grad_() for w in net["W"]]
        b = [v.clone().requires_grad_() for v in net["b"]]
        loss = (_forward64(net, x, W, b) - t).square().mean()
        g = torch.autograd.grad(loss, W + b)
        return {"loss": loss.detach().reshape(1), "dW": list(g[:len(W)]), "db": list(g[len(W):])}
    return None
