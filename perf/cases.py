"""Performance cases of the lattice library.

Each case is one thing a program does with the library through its public
Python entry points: advancing a lattice (single steps up to long runs, small
to large, both storage precisions, both stencil kinds), advancing a batch of
uneven lattices, taking observables and spectra, drawing an initial state,
and a whole linearized run.  The recipes (models, boxes, masses, amplitudes)
are those of the synth module; preheating runs use the paper's own step of
0.0001/m.

Where a case advances a lattice, its field arrays are torch tensors the
caller owns, so the updated state comes back whole and without a copy: the
buffer that holds the state after a call (they alternate with the stage
passes), in the library's device layout [z][field][y][x].

exact() repeats a case in plain torch FP64: the documented random numbers,
the flows of the second-order map and their compositions, lattice sums,
discrete Fourier transforms.
"""
import math

import numpy as np
import torch

import paper_1201_5029_amd as sl
import synth

MODELS = ("preheat", "oscillon", "qball", "free")
STAGES = {2: 1, 4: 3, 6: 7, 8: 15}
EPS_INIT = 1e-3  # fluctuation amplitude of the free fields


def listed():
    return [
        # the smallest call: one step of the 32^3 parity lattice, then a look
        # at the background, as in an interactive or adaptive loop
        dict(name="step-32-f64", kind="evolve", model="preheat", n=32, nf=2, precision="f64",
             order=4, steps=1, stencil="7", tuned=False, watch=True),
        # a small lattice in a long run: a separate-universe run by itself
        dict(name="evolve-64-f64-o6", kind="evolve", model="preheat", n=64, nf=2, precision="f64",
             order=6, steps=100, stencil="7", tuned=False, watch=False),
        # the paper's oscillon run: one field, cache-resident, FP32 storage
        dict(name="evolve-128-oscillon-f32", kind="evolve", model="oscillon", n=128, nf=1,
             precision="f32", order=4, steps=50, stencil="7", tuned=False, watch=False),
        # an odd side (one site per lane, ragged tiles) with the isotropic
        # 27-point stencil
        dict(name="evolve-111-f64-27pt", kind="evolve", model="preheat", n=111, nf=2,
             precision="f64", order=2, steps=20, stencil="27", tuned=False, watch=False),
        # the headline: 256^3 two-field preheating, FP64, 6th order, with the
        # tuned pass shape a long run starts by picking
        dict(name="evolve-256-f64-o6", kind="evolve", model="preheat", n=256, nf=2,
             precision="f64", order=6, steps=4, stencil="7", tuned=True, watch=False),
        # the largest: 512^3 Q-ball in FP32 storage
        dict(name="evolve-512-qball-f32", kind="evolve", model="qball", n=512, nf=2,
             precision="f32", order=6, steps=2, stencil="7", tuned=False, watch=False),
        # the Delta-N scan as the request loop ticks it: 96 uneven runs
        dict(name="batch-96-runs-f32", kind="batch", nruns=96, precision="f32", order=4, steps=10,
             scan_seed=20120125),
        # observables between stretches of a run
        dict(name="energies-256-f64", kind="energies", model="preheat", n=256, nf=2,
             precision="f64", order=6, stencil="7"),
        # field, energy and number spectra of the headline lattice
        dict(name="spectra-256-f64", kind="spectra", model="preheat", n=256, nf=2,
             precision="f64", order=6, stencil="7", field=1, nbins=222),
        # the field spectrum of a Delta-N run (a side that is no power of two)
        dict(name="spectrum-96-f32", kind="spectrum", model="preheat", n=96, nf=2,
             precision="f32", order=4, stencil="7", field=0, nbins=84),
        # a new run's vacuum state, drawn on the device
        dict(name="init-128-f64", kind="init", model="preheat", n=128, nf=2, precision="f64",
             stencil="7"),
        # a whole linearized run: host fields in, host fields out
        dict(name="linear-96", kind="linear", model="preheat", n=96, nf=2, order=6, steps=200,
             stencil="7"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_model(rng):
    model = rng.choice(MODELS)
    nf = {"preheat": 2, "oscillon": 1, "qball": 2}.get(model) or rng.choice((1, 2, 3, 4))
    return model, nf


def draw(rng):
    kind = rng.choice(("evolve", "evolve", "evolve", "evolve", "batch", "energies", "spectra",
                       "spectrum", "init", "linear"))
    stencil = rng.choice(("7", "7", "7", "27"))
    precision = rng.choice(("f64", "f32"))
    order = rng.choice((2, 4, 6, 8))
    model, nf = _draw_model(rng)
    if kind == "evolve":
        n = _log_int(rng, 16, 400)
        # at most about half the bytes of the largest listed case
        per_step = 4 * (8 if precision == "f64" else 4) * nf * n ** 3 * STAGES[order]
        steps = max(1, min(_log_int(rng, 1, 200), int(2.5e10 / per_step)))
        return dict(kind=kind, model=model, n=n, nf=nf, precision=precision, order=order,
                    steps=steps, stencil=stencil, tuned=False, watch=rng.random() < 0.5)
    if kind == "batch":
        return dict(kind=kind, nruns=rng.randint(8, 96), precision=precision,
                    order=rng.choice((2, 4)), steps=rng.randint(1, 12),
                    scan_seed=rng.randrange(1 << 30))
    if kind == "linear":
        model, nf = rng.choice((("preheat", 2), ("oscillon", 1), ("qball", 2), ("free", 3)))
        return dict(kind=kind, model=model, n=_log_int(rng, 16, 128), nf=nf, order=order,
                    steps=_log_int(rng, 10, 400), stencil=stencil)
    n = _log_int(rng, 16, 256)
    case = dict(kind=kind, model=model, n=n, nf=nf, precision=precision, stencil=stencil)
    if kind == "init":
        return case
    case["order"] = order
    if kind in ("spectra", "spectrum"):
        case.update(field=rng.randrange(nf), nbins=rng.randint(8, int(math.sqrt(3) * n / 2) + 2))
    return case


# ---------------------------------------------------------------------------
# Models
# ---------------------------------------------------------------------------


def _recipe(case, seed):
    """The synth recipe of a case's model at its size, with the input seed."""
    model, n = case["model"], case["n"]
    if model == "preheat":
        r = synth.preheat(n=n, dt=0.0001)
    elif model == "oscillon":
        r = synth.oscillon(n=n)
    elif model == "qball":
        r = synth.qball(n=n)
    else:
        nf = case["nf"]
        r = dict(workload="free", n=n, L=32.0, nfields=nf, potential="free",
                 params=tuple(0.5 + 0.25 * i for i in range(nf)), mpl=5.0, a0=1.0,
                 phi0=tuple(1.0 - 0.1 * i for i in range(nf)),
                 pi0=tuple(0.05 * i for i in range(nf)), fluct="vacuum", amplitude=EPS_INIT,
                 dt=0.002, expand=True)
    # the lattice's stability bound holds over the whole range of sides
    r["dt"] = min(r["dt"], 0.25 * r["L"] / n)
    r["seed"] = seed
    r["precision"] = case.get("precision", "f64")
    r["stencil"] = None if case["stencil"] == "7" else case["stencil"]
    if case["kind"] == "init" and model != "oscillon":
        r["fluct"] = "vacuum"
    return r


def _scan(case, seed):
    """Recipes of a Delta-N scan: sides from {32, 64, 96}, phi0 = 1 + k 1e-5."""
    runs = synth.delta_n_scan(nruns=case["nruns"], seed=case["scan_seed"])
    for j, r in enumerate(runs):
        r.update(seed=seed * 1000 + j, dt=0.0001, precision=case["precision"])
    return runs


def _buffers(n, nf, precision):
    """The caller's field arrays: [parity][phi, pi][z][field][y][x]."""
    dtype = torch.float64 if precision == "f64" else torch.float32
    return torch.empty((2, 2, n, nf, n, n), dtype=dtype, device="cuda")


def _lattice(r, buffers=None):
    lat = sl.Lattice(r["n"], r["nfields"], r["L"], precision=r["precision"], expand=r["expand"],
                     mpl=r["mpl"], a0=r["a0"], buffers=buffers)
    lat.set_potential(r["potential"], r["params"])
    if r.get("stencil") is not None:
        lat.set_stencil(r["stencil"])
    return lat


def _draw_state(lat, r):
    lat.init_fluctuations(r["phi0"], r["pi0"], r["fluct"], r["amplitude"], r["seed"])


_TUNED = set()  # what this process has tuned: the library gives later lattices the shapes


def _host_state(case, r, seed):
    """Host fields around the homogeneous values, for the linearized run."""
    n, nf = r["n"], r["nfields"]
    amp = r["amplitude"]
    return synth.gaussian_state(n, nf, seed, phi_base=r["phi0"], phi_amp=amp, pi_base=r["pi0"],
                                pi_amp=amp)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "batch":
        runs = _scan(case, seed)
        dtype = torch.float64 if case["precision"] == "f64" else torch.float32
        per = [r["nfields"] * r["n"] ** 3 for r in runs]
        # one pool per parity, every member's phi and pi carved from it
        pool = torch.empty((2, 2 * sum(per)), dtype=dtype, device="cuda")
        item = pool.element_size()
        batch, lats, at = sl.Batch(), [], 0
        for r, count in zip(runs, per):
            base = [pool[p].data_ptr() + at * item for p in (0, 1)]
            lat = _lattice(r, [base[0], base[0] + count * item, base[1], base[1] + count * item])
            at += 2 * count
            _draw_state(lat, r)
            batch.add(lat)
            lats.append(lat)
        key = ("batch", case["precision"])
        if key not in _TUNED:
            batch.autotune()
            _TUNED.add(key)
        return dict(kind=kind, batch=batch, lats=lats, pool=pool, parity=0, dt=runs[0]["dt"],
                    case=case)
    r = _recipe(case, seed)
    if kind == "linear":
        phi, pi = _host_state(case, r, seed)
        lin = sl.Linear(r["n"], r["nfields"], r["L"], mpl=r["mpl"])
        lin.set_potential(r["potential"], r["params"])
        if r["stencil"] is not None:
            lin.set_stencil(r["stencil"])
        return dict(kind=kind, lin=lin, phi=phi, pi=pi, dt=r["dt"], case=case)
    if kind in ("evolve", "init"):
        buf = _buffers(r["n"], r["nfields"], r["precision"])
        lat = _lattice(r, [buf[0, 0].data_ptr(), buf[0, 1].data_ptr(), buf[1, 0].data_ptr(),
                           buf[1, 1].data_ptr()])
        state = dict(kind=kind, lat=lat, buf=buf, parity=0, dt=r["dt"], case=case, recipe=r)
        if kind == "evolve":
            _draw_state(lat, r)
            key = (case["model"], case["n"], case["precision"], case["stencil"])
            if case["tuned"] and key not in _TUNED:
                lat.autotune()
                _TUNED.add(key)
        return state
    # diagnostics of a run in progress (a field drift is pending)
    lat = _lattice(r)
    _draw_state(lat, r)
    lat.evolve(2, r["dt"], case["order"])
    lat.synchronize()
    return dict(kind=kind, lat=lat, case=case)


def run(state):
    case, kind = state["case"], state["kind"]
    if kind == "evolve":
        lat = state["lat"]
        lat.evolve(case["steps"], state["dt"], case["order"])
        state["parity"] ^= (case["steps"] * STAGES[case["order"]]) & 1
        cur = state["buf"][state["parity"]]
        out = {"phi": cur[0], "pi": cur[1]}
        if case["watch"]:
            out["background"] = np.array(lat.background())
        return out
    if kind == "batch":
        state["batch"].step(case["steps"], state["dt"], case["order"])
        state["batch"].synchronize()
        state["parity"] ^= (case["steps"] * STAGES[case["order"]]) & 1
        return state["pool"][state["parity"]]
    if kind == "energies":
        e = state["lat"].energies()
        # without friedmann_residual and h_total: both are the rounding that
        # a cancellation leaves
        return {"background": np.array([e[k] for k in ("eta", "a", "p_a", "hubble")]),
                "density": np.array([e[k] for k in ("rho", "pressure", "w_eos", "pot")]),
                "kin": np.array(e["kin"]), "grad": np.array(e["grad"]),
                "mean": np.array(e["mean"]), "var": np.array(e["var"])}
    if kind == "spectra":
        k, pf, pe, pn, count, m2 = state["lat"].spectra(case["field"], case["nbins"])
        return {"k": k, "pf": pf, "pe": pe, "pn": pn, "count": count, "m2eff": m2}
    if kind == "spectrum":
        k, p, count = state["lat"].spectrum(case["field"], case["nbins"])
        return {"k": k, "p": p, "count": count}
    if kind == "init":
        lat = state["lat"]
        _draw_state(lat, state["recipe"])
        return {"phi": state["buf"][0, 0], "pi": state["buf"][0, 1],
                "background": np.array(lat.background())}
    lin = state["lin"]
    lin.set_fields(state["phi"], state["pi"])
    lin.evolve(case["steps"], state["dt"], case["order"])
    phi, pi = lin.get_fields()
    eta, a, p_a, phi0, pi0 = lin.background()
    return {"phi": phi, "pi": pi, "background": np.array([eta, a, p_a] + phi0 + pi0)}


def work(case):
    kind = case["kind"]
    if kind == "batch":
        sites = sum(r["n"] ** 3 for r in _scan(case, 1))
        passes = case["steps"] * STAGES[case["order"]]
        b = 8 if case["precision"] == "f64" else 4
        return {"bytes": passes * 4 * b * 2 * sites, "flops": passes * 60 * sites}
    n, nf = case["n"], case["nf"]
    n3 = float(n) ** 3
    b = 4 if case.get("precision") == "f32" else 8
    fft = 2.5 * n3 * math.log2(n3)  # one real transform
    if kind == "evolve":
        passes = case["steps"] * STAGES[case["order"]]
        per_site = 30 if case["stencil"] == "7" else 50
        return {"bytes": passes * 4 * b * nf * n3, "flops": passes * per_site * nf * n3}
    if kind == "energies":
        return {"bytes": 2 * b * nf * n3, "flops": 40 * nf * n3}
    if kind == "spectra":  # phi of every field (m_eff^2), pi of the drift
        return {"bytes": 2 * b * nf * n3, "flops": 2 * fft + 40 * n3}
    if kind == "spectrum":
        return {"bytes": 2 * b * n3, "flops": fft + 10 * n3}
    if kind == "init":  # write phi and pi, and read them for the constraint
        return {"bytes": 4 * b * nf * n3, "flops": nf * (fft + 100 * n3)}
    # linearized run: host fields in and out, growth functions of the classes
    h = n // 2
    classes = (h + 3) * (h + 2) * (h + 1) / 6
    stages = case["steps"] * STAGES[case["order"]]
    return {"bytes": 4 * 8 * nf * n3,
            "flops": 4 * nf * fft + stages * classes * 2 * nf * 2 * (nf * nf + 3 * nf)}


# ---------------------------------------------------------------------------
# The same in plain torch FP64
# ---------------------------------------------------------------------------


def _i64(v):
    return v - (1 << 64) if v >= 1 << 63 else v


def _shr(x, s):
    return (x >> s) & ((1 << (64 - s)) - 1)


def _uniform(seed, counter):
    """(0, 1] uniforms of the counter-based SplitMix64 generator."""
    z = _i64(seed & (2 ** 64 - 1)) + (counter + 1) * _i64(0x9E3779B97F4A7C15)
    z = (z ^ _shr(z, 30)) * _i64(0xBF58476D1CE4E5B9)
    z = (z ^ _shr(z, 27)) * _i64(0x94D049BB133111EB)
    z = z ^ _shr(z, 31)
    return (_shr(z, 11).double() + 1.0) * 2.0 ** -53


def _normal(seed, field, count, idx, comp):
    base = 4 * (field * count + idx) + 2 * comp
    u1, u2 = _uniform(seed, base), _uniform(seed, base + 1)
    return torch.sqrt(-2.0 * torch.log(u1)) * torch.cos(2.0 * math.pi * u2)


_STENCIL = {"7": (-6.0, 1.0, 0.0, 0.0),
            "27": (-128.0 / 30.0, 14.0 / 30.0, 3.0 / 30.0, 1.0 / 30.0)}


def _k_eff2(n, c):
    """Minus the symbol of the stencil on the grid of modes [z][y][x]."""
    t = 2.0 * math.pi * torch.arange(n, device="cuda", dtype=torch.float64) / n
    if c[2] == 0.0 and c[3] == 0.0:
        s = 4.0 * torch.sin(0.5 * t) ** 2
        return s[:, None, None] + s[None, :, None] + s[None, None, :]
    q = torch.cos(t)
    z, y, x = q[:, None, None], q[None, :, None], q[None, None, :]
    return -(c[0] + 2 * c[1] * (z + y + x) + 4 * c[2] * (z * y + z * x + y * x) +
             8 * c[3] * z * y * x)


def _potential(r, f):
    """V and the list of dV/dphi_i at fields f (tensors or floats)."""
    p = r["params"]
    if r["potential"] == "free":
        return sum(0.5 * m * x * x for m, x in zip(p, f)), [m * x for m, x in zip(p, f)]
    if r["potential"] == "chaotic2":
        mc = p[0] + p[1] * f[1] * f[1]
        return 0.5 * f[0] * f[0] * mc, [f[0] * mc, p[1] * f[0] * f[0] * f[1]]
    if r["potential"] == "oscillon":
        x2 = f[0] * f[0]
        return (x2 * (0.5 * p[0] + x2 * (-0.25 * p[1] + x2 * p[2] / 6.0)),
                [f[0] * (p[0] + x2 * (-p[1] + x2 * p[2]))])
    u = 0.5 * (f[0] * f[0] + f[1] * f[1])
    lg = torch.log(u / p[2]) if torch.is_tensor(u) else math.log(u / p[2])
    g = p[0] * (1.0 + p[1] + p[1] * lg)
    return p[0] * u * (1.0 + p[1] * lg), [g * f[0], g * f[1]]


def _hessian(r, f):
    """d^2 V / dphi_i dphi_j."""
    p, nf = r["params"], len(f)
    H = [[0.0 * f[0] for _ in range(nf)] for _ in range(nf)]
    if r["potential"] == "free":
        for i in range(nf):
            H[i][i] = p[i] + 0.0 * f[0]
    elif r["potential"] == "chaotic2":
        H[0][0], H[1][1] = p[0] + p[1] * f[1] * f[1], p[1] * f[0] * f[0]
        H[0][1] = H[1][0] = 2.0 * p[1] * f[0] * f[1]
    elif r["potential"] == "oscillon":
        x2 = f[0] * f[0]
        H[0][0] = p[0] - 3.0 * p[1] * x2 + 5.0 * p[2] * x2 * x2
    else:
        u = 0.5 * (f[0] * f[0] + f[1] * f[1])
        lg = torch.log(u / p[2]) if torch.is_tensor(u) else math.log(u / p[2])
        for i in range(2):
            for j in range(2):
                H[i][j] = p[0] * p[1] * f[i] * f[j] / u
            H[i][i] = H[i][i] + p[0] * (1.0 + p[1] + p[1] * lg)
    return H


def _weights(order):
    if order == 2:
        return [1.0]
    if order == 4:
        c = 2.0 ** (1.0 / 3.0)
        return [1.0 / (2.0 - c), -c / (2.0 - c), 1.0 / (2.0 - c)]
    half = ([0.78451361047755726382, 0.23557321335935813368, -1.17767998417887100695]
            if order == 6 else
            [0.74167036436061295345, -0.40910082580003159400, 0.19075471029623837995,
             -0.57386247111608226666, 0.29906418130365592384, 0.33462491824529818378,
             0.31529309239676659663])
    return half + [1.0 - 2.0 * sum(half)] + half[::-1]


def _initial(r, c):
    """Field and momentum lists of a recipe's initial state ([z][y][x])."""
    n, L = r["n"], r["L"]
    n3 = n ** 3
    phi, pi = [], []
    for i in range(r["nfields"]):
        idx = torch.arange(n3, device="cuda")
        if r["fluct"] == "white":
            g = _normal(r["seed"], i, n3, idx, 0)
            f = r["amplitude"] * (g - g.mean())
        else:
            x, y, z = idx % n, (idx // n) % n, idx // (n * n)
            neg = ((n - z) % n * n + (n - y) % n) * n + (n - x) % n
            canon = torch.minimum(idx, neg)
            m2 = float(_hessian(r, [float(v) for v in r["phi0"]])[i][i])
            w2 = _k_eff2(n, c).reshape(-1) / (L / n) ** 2 + m2
            P = torch.where(w2 > 0, r["amplitude"] ** 2 / (2 * torch.sqrt(w2.clamp(min=1e-300)) * L ** 3),
                            torch.zeros_like(w2))
            P[0] = 0.0
            re, im = _normal(r["seed"], i, n3, canon, 0), _normal(r["seed"], i, n3, canon, 1)
            own = neg == idx
            s = torch.where(own, torch.sqrt(P), torch.sqrt(P / 2))
            im = torch.where(own, torch.zeros_like(im), torch.where(idx == canon, im, -im))
            F = torch.complex(s * re, s * im).reshape(n, n, n)
            f = torch.fft.ifftn(F).real * n3
        phi.append(f.reshape(n, n, n) + r["phi0"][i])
        pi.append(torch.full((n, n, n), float(r["pi0"][i]), device="cuda", dtype=torch.float64))
    return phi, pi


def _laplacian(f, c):
    out = c[0] * f
    for dz in (-1, 0, 1):
        for dy in (-1, 0, 1):
            for dx in (-1, 0, 1):
                k = abs(dz) + abs(dy) + abs(dx)
                if k and c[k] != 0.0:
                    out += c[k] * torch.roll(f, (dz, dy, dx), (0, 1, 2))
    return out


def _gradient(f, c):
    out = torch.zeros_like(f)
    for dz in (-1, 0, 1):
        for dy in (-1, 0, 1):
            for dx in (-1, 0, 1):
                k = abs(dz) + abs(dy) + abs(dx)
                if k and c[k] != 0.0:
                    out += 0.5 * c[k] * (torch.roll(f, (dz, dy, dx), (0, 1, 2)) - f) ** 2
    return out


def _evolved(r, c, steps, order):
    """The stored state after `steps` steps: fields at the last kick (the
    trailing drift `pend` still owed), momenta, FP32 storage offsets and the
    background."""
    phi, pi = _initial(r, c)
    n, dt, VL = r["n"], r["dt"], float(r["n"]) ** 3
    inv_dx2 = (n / r["L"]) ** 2
    inv6 = 1.0 / (6.0 * VL * r["mpl"] ** 2)
    nf = r["nfields"]
    off, offp = [float(v) for v in r["phi0"]], [float(v) for v in r["pi0"]]
    a, eta, pend = r["a0"], 0.0, 0.0
    S2 = sum(float((q * q).sum()) for q in pi)
    V, _ = _potential(r, phi)
    H = (S2 / (2 * a * a) - a * a * inv_dx2 / 2 * sum(float((f * _laplacian(f, c)).sum()) for f in phi)
         + a ** 4 * float(V.sum()))
    pa = -math.sqrt(12.0 * VL * r["mpl"] ** 2 * H)
    for _ in range(steps):
        for w in _weights(order):
            tau, half = w * dt, 0.5 * w * dt
            a -= pa * half * inv6
            pa += S2 / a ** 3 * half
            drift = pend + half / (a * a)
            for i in range(nf):
                phi[i] += drift * pi[i]
                off[i] += drift * offp[i]
            V, dV = _potential(r, phi)
            _, dv0 = _potential(r, off)
            S2 = S3 = 0.0
            for i in range(nf):
                D = _laplacian(phi[i], c)
                S3 += float((phi[i] * D).sum())
                pi[i] += a * a * tau * inv_dx2 * D - a ** 4 * tau * dV[i]
                offp[i] -= a ** 4 * tau * dv0[i]
                S2 += float((pi[i] * pi[i]).sum())
            pa += (a * S3 * inv_dx2 - 4.0 * a ** 3 * float(V.sum())) * tau
            pa += S2 / a ** 3 * half
            pend = half / (a * a)
            a -= pa * half * inv6
        eta += dt
    return dict(phi=phi, pi=pi, off=off, offp=offp, a=a, p_a=pa, eta=eta, pend=pend)


def _stored(r, s):
    """The caller's arrays of a state: remainders in FP32 storage."""
    split = r["precision"] == "f32"
    phi = torch.stack([f - (s["off"][i] if split else 0.0) for i, f in enumerate(s["phi"])], 1)
    pi = torch.stack([q - (s["offp"][i] if split else 0.0) for i, q in enumerate(s["pi"])], 1)
    return phi, pi


def _binned(n, nbins, L, values):
    """Shell means of mode arrays: |n| rounded half away from zero."""
    k = torch.arange(n, device="cuda")
    k = torch.where(2 * k >= n, k - n, k)
    m = (k[:, None, None] ** 2 + k[None, :, None] ** 2 + k[None, None, :] ** 2).reshape(-1)
    b = torch.floor(torch.sqrt(m.double())).long()
    b = torch.where(m > b * b + b, b + 1, b)
    ok = (m > 0) & (b < nbins)
    b, m = b[ok], m[ok]
    count = torch.bincount(b, minlength=nbins)
    div = count.clamp(min=1).double()

    def mean(v):
        return (torch.bincount(b, weights=v, minlength=nbins) / div).cpu().numpy()

    return (2.0 * math.pi / L * mean(torch.sqrt(m.double())), [mean(v.reshape(-1)[ok]) for v in values],
            count.cpu().numpy())


def _exact_linear(case, r, seed):
    n, nf, c = r["n"], r["nfields"], _STENCIL[case["stencil"]]
    phi, pi = (torch.from_numpy(v).cuda() for v in _host_state(case, r, seed))
    inv_dx2, VL = (n / r["L"]) ** 2, float(n) ** 3
    inv6 = 1.0 / (6.0 * VL * r["mpl"] ** 2)
    f, q = [float(v.mean()) for v in phi], [float(v.mean()) for v in pi]
    X = torch.stack([torch.fft.fftn(phi[i] - f[i]) for i in range(nf)])
    P = torch.stack([torch.fft.fftn(pi[i] - q[i]) for i in range(nf)])
    X[:, 0, 0, 0] = 0
    P[:, 0, 0, 0] = 0
    kk = _k_eff2(n, c) * inv_dx2
    a, eta, dt = r["a0"], 0.0, r["dt"]
    V, _ = _potential(r, f)
    pa = -math.sqrt(12.0 * VL * r["mpl"] ** 2 *
                    VL * (sum(v * v for v in q) / (2 * a * a) + a ** 4 * V))
    for _ in range(case["steps"]):
        for w in _weights(case["order"]):
            tau, half = w * dt, 0.5 * w * dt
            a -= pa * half * inv6
            pa += VL * sum(v * v for v in q) / a ** 3 * half
            cd = half / (a * a)
            f = [x + cd * y for x, y in zip(f, q)]
            V, dV = _potential(r, f)
            H = _hessian(r, f)
            for _ in range(2):
                pa -= 4.0 * a ** 3 * VL * V * half
                q = [y - a ** 4 * d * half for y, d in zip(q, dV)]
            X += cd * P
            P -= a * a * tau * kk * X
            for i in range(nf):
                for j in range(nf):
                    P[i] -= a ** 4 * tau * H[i][j] * X[j]
            X += cd * P
            pa += VL * sum(v * v for v in q) / a ** 3 * half
            f = [x + cd * y for x, y in zip(f, q)]
            a -= pa * half * inv6
        eta += dt
    out = [torch.stack([torch.fft.ifftn(Y[i]).real + z[i] for i in range(nf)]).cpu().numpy()
           for Y, z in ((X, f), (P, q))]
    return {"phi": out[0], "pi": out[1], "background": np.array([eta, a, pa] + f + q)}


def exact(case, seed):
    kind = case["kind"]
    if kind == "batch":
        parts = []
        for r in _scan(case, seed):
            s = _evolved(r, _STENCIL["7"], case["steps"], case["order"])
            phi, pi = _stored(r, s)
            parts += [phi.reshape(-1), pi.reshape(-1)]
        return torch.cat(parts)
    r = _recipe(case, seed)
    c = _STENCIL[case["stencil"]]
    n, nf = r["n"], r["nfields"]
    if kind == "linear":
        # thousands of passes over n^3 complex modes: small ones only
        if case["steps"] * STAGES[case["order"]] * n ** 3 * nf > 4e9:
            return None
        return _exact_linear(case, r, seed)
    if kind == "init":
        s = _evolved(r, c, 0, 2)
        phi, pi = _stored(r, s)
        return {"phi": phi, "pi": pi, "background": np.array([0.0, s["a"], s["p_a"]])}
    if kind == "evolve":
        s = _evolved(r, c, case["steps"], case["order"])
        phi, pi = _stored(r, s)
        out = {"phi": phi, "pi": pi}
        if case["watch"]:
            out["background"] = np.array([s["eta"], s["a"], s["p_a"]])
        return out
    s = _evolved(r, c, 2, case["order"])
    a, dx2, VL = s["a"], (r["L"] / n) ** 2, float(n) ** 3
    phi = [f + s["pend"] * q for f, q in zip(s["phi"], s["pi"])]
    if kind == "energies":
        kin = [float((q * q).mean()) / (2 * a ** 6) for q in s["pi"]]
        grad = [float(_gradient(f, c).mean()) / (2 * a * a * dx2) for f in phi]
        pot = float(_potential(r, phi)[0].mean())
        rho, pressure = sum(kin) + sum(grad) + pot, sum(kin) - sum(grad) / 3 - pot
        return {"background": np.array([s["eta"], a, s["p_a"],
                                        -s["p_a"] / (6 * VL * r["mpl"] ** 2 * a * a)]),
                "density": np.array([rho, pressure, pressure / rho, pot]),
                "kin": np.array(kin), "grad": np.array(grad),
                "mean": np.array([float(f.mean()) for f in phi]),
                "var": np.array([float(((f - f.mean()) ** 2).mean()) for f in phi])}
    i = case["field"]
    F2 = torch.fft.fftn(phi[i]).abs() ** 2 / VL ** 2
    if kind == "spectrum":
        k, (p,), count = _binned(n, case["nbins"], r["L"], [F2])
        return {"k": k, "p": p, "count": count}
    P2 = torch.fft.fftn(s["pi"][i]).abs() ** 2 / VL ** 2
    m2 = float(torch.as_tensor(_hessian(r, phi)[i][i]).mean())
    k2 = _k_eff2(n, c) / dx2
    rho = P2 / (2 * a ** 6) + (k2 / (2 * a * a) + 0.5 * m2) * F2
    w2 = k2 / (a * a) + m2
    num = torch.where(w2 > 0, rho / torch.sqrt(w2.clamp(min=1e-300)), torch.zeros_like(rho))
    k, (pf, pe, pn), count = _binned(n, case["nbins"], r["L"], [F2, rho, num])
    return {"k": k, "pf": pf, "pe": pe, "pn": pn, "count": count, "m2eff": m2}
