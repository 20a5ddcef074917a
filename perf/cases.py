"""The work whose speed and results are watched: what a program of this package
has it do, through the public entry points of paper_2307_07999_amd.

A case is a dict of plain values.  "path" names what it runs:

  event    one Glasma event: MV initial condition, particle species, coupled
           steps to tau_max, and the curves of every species (Event)
  scan     the same with the paper's twelve scan points as species and both
           field correlators, as scan.run_scan runs each of its events
  rows     solver runs turned into network rows (surrogate.solver_curves and
           surrogate.rows): how the surrogate's training data is made
  batch    uneven FP32 events stepped together (Batch), the serving pattern
  dipole   an MV draw and its dipole curves and saturation scale, the step that
           fixes g^2 mu for a wanted Q_s
  query    one curve asked of the trained network with host rows (MLP.query)
  infer    many rows through the network on the device (MLP.infer)
  train    epochs of minibatch training (MLP.train), then the new parameters

`exact` gives the results in 64 bits from the equations alone (torch and numpy,
nothing of the package): the network directly, and whole small events by
a plain lattice implementation below.
"""
import math
import os
import tempfile

import numpy as np
import torch

import paper_2307_07999_amd as gl
from paper_2307_07999_amd import scan, surrogate

HBARC = 0.1973269804
DTAU = 0.125                      # the paper's step, in lattice spacings
M_IR = 0.2
G2MU = 2.767                      # Q_s = 2 GeV at 512^2, L = 10 fm, 50 sheets
PAPER_A = 10.0 / 512              # the paper-scale lattice spacing [fm]
# charm and beauty at p_T0 in {0, 2, 5} GeV and massless jets at 10 GeV
BENCH = [(1.27, p, 0, -1.0) for p in (0.0, 2.0, 5.0)] + [(4.18, p, 0, -1.0) for p in (0.0, 2.0, 5.0)] + \
        [(0.0, 10.0, 1, -1.0)]
CHARM = [(1.27, 0.0, 0, -1.0)]
NET = dict(n_in=5, width=256, depth=3, n_out=2)     # the surrogate's network
OUT_POWERS = np.array([3.0, 2.0], np.float32)
# lattices that the MV initial condition takes (2^a 3^b)
SIZES = [16, 18, 24, 27, 32, 36, 48, 54, 64, 72, 81, 96, 108, 128, 144, 162, 192, 216, 243, 256, 288, 324, 384,
         432, 486, 512]


def listed():
    return [
        # an interactive question to the surrogate: one curve of 410 times,
        # host rows in, host values out; latency is all there is
        dict(name="query_curve", path="query", rows=410),
        # 64 curves at once, as a fit or a plot of a parameter scan asks them
        dict(name="infer_64_curves", path="infer", rows=64 * 410, noalloc=False),
        # a table over the whole domain, by the entry that allocates nothing;
        # an odd number of rows
        dict(name="infer_table", path="infer", rows=1000003, noalloc=True),
        # training at the protocol's batch size; 16 whole batches an epoch
        # and a remainder that each epoch's shuffle leaves out
        dict(name="train_2_epochs", path="train", rows=65573, batch=4096, epochs=2),
        # the 32^2 event of the parity tests: the smallest real run
        dict(name="event_32_f64", path="event", N=32, a_fm=0.125, precision=64, sheets=1, g2mu=1.0, probes="charm",
             n_per=1000, tau_max=1.0),
        # an odd lattice (3^5) with odd particle numbers
        dict(name="event_243_f64", path="event", N=243, a_fm=PAPER_A, precision=64, sheets=17, g2mu=G2MU,
             probes="bench", n_per=12347, tau_max=0.5),
        # the paper-scale event, FP64 and its FP32 twin
        dict(name="event_512_f64", path="event", N=512, a_fm=PAPER_A, precision=64, sheets=50, g2mu=G2MU,
             probes="bench", n_per=100000, tau_max=1.0),
        dict(name="event_512_f32", path="event", N=512, a_fm=PAPER_A, precision=32, sheets=50, g2mu=G2MU,
             probes="bench", n_per=100000, tau_max=1.0),
        # one event of the paper's figures: twelve species and both correlators
        dict(name="scan_512_f64", path="scan", N=512, a_fm=PAPER_A, precision=64, sheets=50, g2mu=G2MU,
             n_per=100000, tau_max=1.0),
        # training data of the surrogate: 256^2 runs of 10^4 particles
        dict(name="rows_24x256_f32", path="rows", runs=24, N=256, sheets=50, n_per=10000),
        # uneven events in one batch, 128^2 to 512^2, 10^4 to 10^6 particles
        dict(name="batch_10_f32", path="batch", events=10, n_lo=128, n_hi=512, p_lo=10000, p_hi=1000000, sheets=50,
             tau_max=1.0),
        # Q_s of one MV draw at the coarse training lattice
        dict(name="dipole_256", path="dipole", N=256, a_fm=10.0 / 256, sheets=50, g2mu=G2MU),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _size(rng, lo, hi):
    want = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return min((n for n in SIZES if lo <= n <= hi), key=lambda n: abs(math.log(n / want)))


def draw(rng):
    path = rng.choice(["query", "infer", "train", "event", "event", "event", "scan", "rows", "batch", "dipole"])
    if path == "query":
        return dict(path=path, rows=_log(rng, 1, 4100))
    if path == "infer":
        return dict(path=path, rows=_log(rng, 1, 1000000), noalloc=rng.random() < 0.5)
    if path == "train":
        batch = rng.choice([256, 500, 1024, 2000, 4096])
        return dict(path=path, rows=batch * rng.randint(1, 12) + rng.randint(0, batch - 1), batch=batch,
                    epochs=rng.randint(1, 2))
    if path in ("event", "scan"):
        N = _size(rng, 16, 512)
        a = math.exp(rng.uniform(math.log(PAPER_A), math.log(0.125 if N < 128 else 0.04)))
        c = dict(path=path, N=N, a_fm=a, precision=rng.choice([64, 64, 32]), sheets=_log(rng, 1, 50),
                 g2mu=G2MU if a < 0.04 else 1.0, n_per=_log(rng, 1, max(2, 0.38 * N * N)),
                 tau_max=rng.choice([0.3, 0.5, 1.0]))
        if path == "event":
            c["probes"] = rng.choice(["charm", "bench", "none"])
        return c
    if path == "rows":
        return dict(path=path, runs=rng.randint(1, 12), N=_size(rng, 64, 256), sheets=_log(rng, 1, 50),
                    n_per=_log(rng, 100, 10000))
    if path == "batch":
        lo = _size(rng, 32, 128)
        return dict(path=path, events=rng.randint(2, 8), n_lo=lo, n_hi=_size(rng, lo, 384), p_lo=_log(rng, 100, 10000),
                    p_hi=_log(rng, 20000, 300000), sheets=_log(rng, 1, 50), tau_max=rng.choice([0.3, 0.5, 1.0]))
    N = _size(rng, 16, 256)
    return dict(path=path, N=N, a_fm=math.exp(rng.uniform(math.log(PAPER_A), math.log(0.04))),
                sheets=_log(rng, 1, 50), g2mu=G2MU)


# ---- the cases through the package -------------------------------------------
def _steps(a_fm, tau_max):
    return max(1, int(math.ceil(tau_max / (DTAU * a_fm) - 1e-9)) - 1)


def _box(N):
    """L [fm] of the surrogate's runs: 10 fm at 256^2, and below that the
    paper's spacing (small lattices of 10 fm would not resolve Q_s)."""
    return 10.0 if N >= 256 else N * PAPER_A


def _species(case):
    if case["path"] == "scan":
        return [(m, p0, kind, tf) for _, kind, m, p0, tf in scan.scan_points()]
    return {"bench": BENCH, "charm": CHARM, "none": []}[case["probes"]]


def _batch_events(case):
    """(N, particles per species) of each event of an uneven batch"""
    g = np.random.default_rng(case["events"])
    sizes = [n for n in SIZES if case["n_lo"] <= n <= case["n_hi"]]
    # the largest lattice first: the batch always spans its range
    Ns = [case["n_hi"]] + [int(n) for n in g.choice(sizes, size=case["events"] - 1)]
    parts = np.exp(g.uniform(math.log(case["p_lo"]), math.log(case["p_hi"]), size=case["events"]))
    return [(n, max(1, int(p) // len(BENCH))) for n, p in zip(Ns, parts)]


def _parameters(seed):
    """He-uniform weights and small biases of the surrogate's network, flat:
    W_1 [out][in], ..., then b_1, ..."""
    g = np.random.default_rng(seed)
    dims = [NET["n_in"]] + [NET["width"]] * NET["depth"] + [NET["n_out"]]
    W = [g.uniform(-1, 1, (o, i)) * math.sqrt(6.0 / i) * (1.0 if o != NET["n_out"] else 0.1)
         for i, o in zip(dims[:-1], dims[1:])]
    b = [g.uniform(-0.1, 0.1, o) for o in dims[1:]]
    return np.concatenate([w.ravel() for w in W] + b).astype(np.float32)


def _inputs(rows, seed):
    """Network rows over the surrogate's domain: the features of curves of
    about 410 times each, at random parameters."""
    g = np.random.default_rng(seed)
    curves = -(-rows // 410)
    qs, pt = g.uniform(1.0, 3.0, curves), g.uniform(0.5, 10.0, curves)
    m = g.choice([0.0, 1.27, 4.18], curves)
    tf = HBARC / (2.0 * np.sqrt(m * m + pt * pt))
    t = np.sqrt(np.linspace(0.0, 0.99, 410))
    X = np.empty((curves, 410, 5), np.float32)
    for c, v in enumerate((qs, m, pt, tf)):
        X[:, :, c] = v[:, None]
    X[:, :, 4] = t
    return X.reshape(-1, 5)[:rows].copy()


def _targets(X):
    """Smooth curves of the size of kappa [GeV^2/fm] and <dp_T^2> [GeV^2]."""
    qs, m, pt, _, t = (X[:, k].astype(np.float64) for k in range(5))
    rise = np.exp(-6.0 * t) * t * (1.0 + 0.1 * np.sin(9.0 * t))
    return np.stack([qs ** 3 * 20.0 * rise * (1.0 + 0.03 * pt), qs ** 2 * (1.0 - np.exp(-4.0 * t)) / (1.0 + 0.1 * m)],
                    axis=1).astype(np.float32)


IN_LO = np.array([1.0, 0.0, 0.0, 0.0, 0.0], np.float32)
IN_HI = np.array([3.0, 4.18, 10.0, 0.2, 1.0], np.float32)
OUT_MEAN = np.array([0.7, 0.5], np.float32)
OUT_STD = np.array([0.6, 0.3], np.float32)


def _network(case, seed):
    train = case["path"] == "train"
    net = gl.MLP(**NET, max_batch=4096, max_samples=case["rows"] if train else 1, seed=1)
    net.params(set_to=_parameters(seed))
    net.set_scaling(IN_LO, IN_HI, OUT_MEAN, OUT_STD)
    net.set_output_power(0, OUT_POWERS)
    if case["path"] == "query":
        net.set_trust(IN_LO, np.array([3.0, 4.18, 10.0, 0.2, 1.0]), 1, [0.0, 1.27, 4.18], 1e-3, 2,
                      [0.0, 10.0 / 3.0, 20.0 / 3.0, 10.0], np.full((3, 3), 0.03), 0.05)
    return net


def prepare(case, seed):
    path = case["path"]
    s = dict(case=case, seed=seed)
    if path in ("query", "infer", "train"):
        s["net"] = _network(case, seed)
        X = _inputs(case["rows"], seed + 1)
        s["X"] = X if path == "query" else torch.from_numpy(X).cuda()
        if path == "train":
            s["Y"] = torch.from_numpy(_targets(X)).cuda()
        if path == "infer" and case["noalloc"]:
            s["Y"] = torch.empty((case["rows"], NET["n_out"]), dtype=torch.float32, device="cuda")
    elif path == "rows":
        s["params"] = surrogate.draw_params(case["runs"], case["runs"])     # the scan's points; events by the seed
    elif path == "batch":
        # the tuned tile is kept in a file, as a serving program keeps it
        s["events"] = _batch_events(case)
        s["folder"] = tempfile.TemporaryDirectory()
        s["tuned"] = os.path.join(s["folder"].name, "tile.json")
    return s


def _event(case, seed, static=False, lightlike=False):
    sp = _species(case)
    steps = _steps(case["a_fm"], case["tau_max"])
    ev = gl.Event(case["N"], case["N"] * case["a_fm"], DTAU, precision=case["precision"], max_steps=steps,
                  max_particles=sum(-(-case["n_per"] // 256) * 256 for _ in sp), static_correlator=static,
                  lightlike_correlator=lightlike)
    ev.init_glasma(case["g2mu"], M_IR, case["sheets"], seed)
    for k, (m, p0, kind, tf) in enumerate(sp):
        ev.add_species(m, p0, kind, case["n_per"], seed + 17 * k, tau_form_fm=tf)
    return ev, sp, steps


def run(s):
    case, seed = s["case"], s["seed"]
    path = case["path"]
    if path == "query":
        return s["net"].query(s["X"])
    if path == "infer":
        return s["net"].infer_noalloc(s["X"], s["Y"]) if case["noalloc"] else s["net"].infer(s["X"])
    if path == "train":
        losses = s["net"].train(s["X"], s["Y"], epochs=case["epochs"], batch=case["batch"], lr=1e-3, seed=seed)
        return losses, s["net"].params()
    if path == "event":
        ev, sp, steps = _event(case, seed)
        ev.run(steps)
        out = [(ev.broadening(k), ev.kappa(k) if kind == 0 else ev.qhat(k)) for k, (_, _, kind, _) in enumerate(sp)]
        # without probes the fields are the result: their energy terms
        out = out or ev.diagnostics()["energy"]
        ev.close()
        return out
    if path == "scan":
        ev, sp, steps = _event(case, seed, True, True)
        ev.static_start(ev.species_info(0)[0] * DTAU * case["a_fm"])
        ev.lightlike_start(0.0)
        ev.run(steps)
        out = ev.series()[:, :len(sp)].copy(), ev.static_broadening(), ev.lightlike_broadening()
        ev.close()
        return out
    if path == "rows":
        curves, _ = surrogate.solver_curves(s["params"], case["N"], _box(case["N"]), case["n_per"], seed,
                                            sheets=case["sheets"])
        return surrogate.rows(s["params"], curves)
    if path == "batch":
        steps = _steps(PAPER_A, case["tau_max"])
        evs = []
        for e, (n, per) in enumerate(s["events"]):
            ev = gl.Event(n, n * PAPER_A, DTAU, precision=32, max_steps=steps,
                          max_particles=len(BENCH) * (-(-per // 256) * 256))
            ev.init_glasma(G2MU, M_IR, case["sheets"], seed + 1000 * e)
            for k, (m, p0, kind, tf) in enumerate(BENCH):
                ev.add_species(m, p0, kind, per, seed + 1000 * e + 17 * k, tau_form_fm=tf)
            evs.append(ev)
        b = gl.Batch(evs)
        b.autotune(s["tuned"])
        b.run(steps)
        b.stream.synchronize()
        out = [ev.series() for ev in evs]
        b.close()
        for ev in evs:
            ev.close()
        return out
    ev = gl.Event(case["N"], case["N"] * case["a_fm"], DTAU, max_steps=1)
    ev.init_glasma(case["g2mu"], M_IR, case["sheets"], seed)
    out = ev.dipole(0, case["N"] // 2), ev.dipole(1, case["N"] // 2)
    ev.close()
    return out


def work(case):
    """Bytes: every step reads and writes the field state (56 reals per site)
    and the particle records (14 reals and the cell) once; an initial
    condition writes its state; the network reads its rows, weights and
    targets and writes its outputs.  Flops: about 5000 per site and step,
    1500 per particle and step, and per site and sheet of both nuclei the
    transforms, the exponential and the product (3000)."""
    path = case["path"]
    if path in ("query", "infer", "train"):
        dims = [5, 256, 256, 256, 2]
        nw = sum(a * b for a, b in zip(dims[:-1], dims[1:]))
        if path != "train":
            return dict(bytes=28.0 * case["rows"] + 2 * nw, flops=2.0 * nw * case["rows"])
        steps = case["rows"] // case["batch"] * case["epochs"]
        # a step reads its rows and targets, and reads and writes the weights
        # and both moments
        return dict(bytes=steps * (28.0 * case["batch"] + 24.0 * nw), flops=6.0 * nw * case["batch"] * steps)

    def event(N, ts, n, steps, sheets, extra=0):
        return dict(bytes=N * N * 56.0 * ts * (2 * steps + 1) + steps * n * 2 * (14.0 * ts + 8) + extra,
                    flops=steps * (5000.0 * N * N + 1500.0 * n) + 3000.0 * 2 * sheets * N * N)

    if path == "dipole":
        return dict(bytes=2 * 18 * 8.0 * case["N"] ** 2,
                    flops=(3000.0 * case["sheets"] + 36.0 * case["N"]) * 2 * case["N"] ** 2)
    if path == "rows":
        steps = _steps(_box(case["N"]) / case["N"], 1.0)
        parts = [event(case["N"], 4, case["n_per"], steps, case["sheets"])] * case["runs"]
    elif path == "batch":
        steps = _steps(PAPER_A, case["tau_max"])
        mean = math.exp(0.5 * (math.log(case["p_lo"]) + math.log(case["p_hi"])))
        sizes = [n for n in SIZES if case["n_lo"] <= n <= case["n_hi"]]
        n2 = sum(n * n for n in sizes) / len(sizes)
        parts = [event(case["n_hi"], 4, mean, steps, case["sheets"])] + \
                [event(math.sqrt(n2), 4, mean, steps, case["sheets"])] * (case["events"] - 1)
    else:
        steps, ts = _steps(case["a_fm"], case["tau_max"]), case["precision"] // 8
        # the correlators read and write 24 and 42 FP64 values per site and step
        extra = steps * case["N"] ** 2 * 2 * 8.0 * (24 + 42) if path == "scan" else 0
        parts = [event(case["N"], ts, case["n_per"] * len(_species(case)), steps, case["sheets"], extra)]
    return {k: sum(p[k] for p in parts) for k in ("bytes", "flops")}


# ---- 64-bit results without the package ---------------------------------------
def exact(case, seed):
    path = case["path"]
    if path in ("query", "infer"):
        Y = _forward64(_unflatten(_parameters(seed)), _inputs(case["rows"], seed + 1))
        return (Y, 0) if path == "query" else Y
    if path == "train":
        return _train64(case, seed)
    if path in ("event", "scan"):
        steps = _steps(case["a_fm"], case["tau_max"])
        n = case["n_per"] * len(_species(case))
        if case["N"] ** 2 * (steps + 4 * case["sheets"]) > 1.4e7 or n * steps > 5e7:
            return None                      # would take more than some seconds
        return _event64(case, seed)
    if path == "dipole":
        if case["N"] ** 2 * case["sheets"] > 4e6:
            return None
        a = case["a_fm"] / HBARC
        return tuple(_dipole64(_wilson64(case["N"], case["g2mu"] * a / math.sqrt(case["sheets"]), (M_IR * a) ** 2,
                                         case["sheets"], seed, nuc)) for nuc in (0, 1))
    return None                              # batches: many events, too long


DEV = "cuda" if torch.cuda.is_available() else "cpu"


def _unflatten(p):
    dims = [NET["n_in"]] + [NET["width"]] * NET["depth"] + [NET["n_out"]]
    p = torch.from_numpy(np.asarray(p, np.float64)).to(DEV)
    W, b, at = [], [], 0
    for i, o in zip(dims[:-1], dims[1:]):
        W.append(p[at:at + i * o].reshape(o, i).clone())
        at += i * o
    for o in dims[1:]:
        b.append(p[at:at + o].clone())
        at += o
    return W, b


def _scaled(X):
    lo, hi = (torch.from_numpy(v.astype(np.float64)).to(X.device) for v in (IN_LO, IN_HI))
    return 2.0 * (X - lo) / (hi - lo) - 1.0


def _layers(p, h):
    W, b = p
    acts, pre = [h], []
    for k, (w, c) in enumerate(zip(W, b)):
        pre.append(acts[-1] @ w.T + c)
        acts.append(pre[-1] * torch.sigmoid(pre[-1]) if k + 1 < len(W) else pre[-1])
    return acts, pre


def _forward64(p, X):
    out = []
    mu, sd, pw = (torch.from_numpy(v.astype(np.float64)).to(DEV) for v in (OUT_MEAN, OUT_STD, OUT_POWERS))
    for x in torch.from_numpy(X).split(65536):
        x = x.to(DEV).double()
        acts, _ = _layers(p, _scaled(x))
        out.append(((acts[-1] * sd + mu) * x[:, :1] ** pw).cpu())
    return torch.cat(out).numpy()


def _mt64(seed):
    """The 64-bit Mersenne Twister of the C++ standard (std::mt19937_64)."""
    n, full = 312, (1 << 64) - 1
    x = [seed & full]
    for i in range(1, n):
        x.append((6364136223846793005 * (x[-1] ^ (x[-1] >> 62)) + i) & full)
    while True:
        for i in range(n):
            y = (x[i] & 0xFFFFFFFF80000000) | (x[(i + 1) % n] & 0x7FFFFFFF)
            x[i] = x[(i + 156) % n] ^ (y >> 1) ^ (0xB5026F5AA96619E9 if y & 1 else 0)
        for z in x:
            z ^= (z >> 29) & 0x5555555555555555
            z ^= (z << 17) & 0x71D67FFFEDA60000
            z ^= (z << 37) & 0xFFF7EEE000000000 & full
            yield z ^ (z >> 43)


def _train64(case, seed):
    """Minibatch Adam on the standardised targets in FP64: each epoch shuffles
    all rows (Fisher-Yates from the end) and takes its whole batches."""
    X = _inputs(case["rows"], seed + 1)
    Y = torch.from_numpy(_targets(X)).to(DEV).double()
    X = torch.from_numpy(X).to(DEV).double()
    mu, sd, pw = (torch.from_numpy(v.astype(np.float64)).to(DEV) for v in (OUT_MEAN, OUT_STD, OUT_POWERS))
    Y = (Y / X[:, :1] ** pw - mu) / sd
    X = _scaled(X)
    W, b = _unflatten(_parameters(seed))
    par = W + b
    mom = [torch.zeros_like(v) for v in par]
    var = [torch.zeros_like(v) for v in par]
    n, B, t, losses, rng = case["rows"], case["batch"], 0, [], _mt64(seed)
    for _ in range(case["epochs"]):
        perm = list(range(n))
        for i in range(n - 1, 0, -1):
            j = next(rng) % (i + 1)
            perm[i], perm[j] = perm[j], perm[i]
        perm = torch.tensor(perm, device=DEV)
        total = 0.0
        for k in range(n // B):
            at = perm[k * B:(k + 1) * B]
            acts, pre = _layers((W, b), X[at])
            d = acts[-1] - Y[at]
            total += float((d * d).mean())
            d = 2.0 * d / d.numel()
            gW, gb = [None] * len(W), [None] * len(W)
            for layer in range(len(W) - 1, -1, -1):
                gW[layer], gb[layer] = d.T @ acts[layer], d.sum(0)
                if layer:
                    z = pre[layer - 1]
                    sg = torch.sigmoid(z)
                    d = (d @ W[layer]) * sg * (1.0 + z * (1.0 - sg))
            t += 1
            for p, g, m, v in zip(par, gW + gb, mom, var):
                m.mul_(0.9).add_(g, alpha=0.1)
                v.mul_(0.999).addcmul_(g, g, value=0.001)
                p.sub_(1e-3 * (m / (1 - 0.9 ** t)) / ((v / (1 - 0.999 ** t)).sqrt() + 1e-8))
        losses.append(total / (n // B))
    return np.array(losses), torch.cat([p.reshape(-1) for p in par]).cpu().numpy()


# A plain FP64 lattice: complex 3x3 matrices per site [..., 3, 3], site arrays
# [iy, ix], direction 0 along ix.
def _generators():
    T = np.zeros((8, 3, 3), np.complex128)
    for a, (i, j) in ((0, (0, 1)), (3, (0, 2)), (5, (1, 2))):
        T[a, i, j] = T[a, j, i] = 0.5
        T[a + 1, i, j], T[a + 1, j, i] = -0.5j, 0.5j
    T[2] = np.diag([0.5, -0.5, 0])
    T[7] = np.diag([1, 1, -2]) * 0.5 / math.sqrt(3.0)
    return torch.from_numpy(T).to(DEV)


def _mm(a, b):
    return (a[..., :, :, None] * b[..., None, :, :]).sum(-2)


def _dag(a):
    return a.conj().transpose(-1, -2)


def _alg(x):
    return (x.to(torch.complex128) @ _generators().reshape(8, 9)).reshape(*x.shape[:-1], 3, 3)


def _comps(X):
    """2 Re Tr(T^a X)"""
    return 2.0 * (X.transpose(-1, -2).reshape(*X.shape[:-2], 9) @ _generators().reshape(8, 9).T).real


def _proj(M):
    """2 Im Tr(T^a M)"""
    return _comps(-1j * M)


def _expi(x, halvings=7):
    A = 1j * _alg(x) / 2.0 ** halvings
    one = torch.eye(3, dtype=torch.complex128, device=A.device)
    r = one.expand(A.shape)
    for k in range(14, 0, -1):
        r = one + _mm(A, r) / k
    for _ in range(halvings):
        r = _mm(r, r)
    return r


def _sh(A, d, s):
    """A at x + s e_d"""
    return torch.roll(A, -s, dims=1 - d)


def _conj_by(U, X):
    return _mm(_mm(U, X), _dag(U))


def _philox(seed, c0, c1, c2):
    """Philox4x32-10 words for counters (c0, c1, c2, 0), int64 tensors."""
    M32 = 0xFFFFFFFF
    k0, k1 = seed & M32, (seed >> 32) & M32
    c1, c2, c3 = (torch.full_like(c0, v) if isinstance(v, int) else v for v in (c1, c2, 0))
    for _ in range(10):
        p0, p1 = c0 * 0xD2511F53, c2 * 0xCD9E8D57        # products mod 2^64
        c0, c1, c2, c3 = ((p1 >> 32) & M32) ^ c1 ^ k0, p1 & M32, ((p0 >> 32) & M32) ^ c3 ^ k1, p0 & M32
        k0, k1 = (k0 + 0x9E3779B9) & M32, (k1 + 0xBB67AE85) & M32
    return c0, c1, c2, c3


def _uniform(lo, hi):
    k = (((hi << 20) | (lo >> 12)) << 1) | 1
    return k.double() * 2.0 ** -53


def _normals(w):
    r = torch.sqrt(-2.0 * torch.log(_uniform(w[0], w[1])))
    t = 2.0 * math.pi * _uniform(w[2], w[3])
    return r * torch.cos(t), r * torch.sin(t)


def _wilson64(N, sigma, m2, sheets, seed, nucleus):
    site = torch.arange(N * N, device=DEV)
    s = 4.0 * torch.sin(math.pi * torch.arange(N, device=DEV, dtype=torch.float64) / N) ** 2
    den = s[:, None] + s[None, :] + m2
    V = torch.eye(3, dtype=torch.complex128, device=DEV).expand(N, N, 3, 3)
    for sheet in range(sheets):
        rho = [g for j in range(4) for g in _normals(_philox(seed, site, 4 * sheet + j, nucleus))]
        lam = torch.fft.ifft2(torch.fft.fft2(torch.stack(rho).reshape(8, N, N) * sigma) / den).real
        V = _mm(V, _expi(-lam.permute(1, 2, 0)))
    return V


def _dipole64(V):
    N = V.shape[0]
    return np.array([float(sum((V * _sh(V, d, r).conj()).real.sum() for d in (0, 1))) / (6.0 * N * N)
                     for r in range(N // 2 + 1)])


def _inv3(A):
    c = torch.cross(A[..., [1, 2, 0], :], A[..., [2, 0, 1], :], dim=-1)     # cofactor rows
    return c.transpose(-1, -2) / (A[..., 0, :] * c[..., 0, :]).sum(-1)[..., None, None]


def _match64(UA, UB):
    """[(UA + UB)(1 + U^dag)]_X = 0 by damped Newton, from the SU(3) projection
    of W (W^dag)^-1."""
    W = (UA + UB).reshape(-1, 3, 3)
    X = _mm(W, _inv3(_dag(W)))
    for _ in range(40):
        X = 0.5 * (X + _dag(_inv3(X)))
    det = (X[:, 0] * torch.cross(X[:, 1], X[:, 2], dim=-1)).sum(-1)
    U = X * torch.polar(torch.ones_like(det.real), -torch.angle(det) / 3.0)[:, None, None]
    one = torch.eye(3, dtype=torch.complex128, device=W.device)
    T = _generators()

    def residual(w, u):
        return _proj(_mm(w, one + _dag(u)))
    live = torch.arange(len(W), device=W.device)
    for _ in range(100):
        R = residual(W[live], U[live])
        big = R.abs().amax(-1)
        keep = big >= 1e-13
        live, R, big = live[keep], R[keep], big[keep]
        if not len(live):
            break
        WU = _mm(W[live], _dag(U[live]))
        J = torch.stack([_proj(_mm(WU, -1j * T[b])) for b in range(8)], -1)
        d = torch.linalg.solve(J.cpu(), -R.cpu()[..., None])[..., 0].to(W.device)
        step = torch.ones_like(big)
        for _ in range(40):
            new = _mm(_expi(d * step[:, None]), U[live])
            worse = residual(W[live], new).abs().amax(-1) >= big
            if not bool(worse.any()):
                break
            step = torch.where(worse, 0.5 * step, step)
        U[live] = new
    return U.reshape(UA.shape)


class _Lattice:
    """The field state at step n: U [2], E [2] (components), phi, pi."""

    def __init__(self, N, sigma, m2, sheets, seed):
        one = torch.eye(3, dtype=torch.complex128, device=DEV)
        Un = []
        for nuc in (0, 1):
            V = _wilson64(N, sigma, m2, sheets, seed, nuc)
            Un.append(torch.stack([_mm(V, _dag(_sh(V, d, 1))) for d in (0, 1)]))
        UA, UB = Un
        self.U = _match64(UA, UB)
        pi = 0.0
        for d in (0, 1):
            pi = pi + _proj(_mm(self.U[d] - one, _dag(UB[d]) - _dag(UA[d])))
            u, a, b = (_sh(v[d], d, -1) for v in (self.U, UA, UB))
            pi = pi + _proj(_mm(_dag(u) - one, b - a))
        self.pi = 0.5 * pi
        self.E = torch.zeros(2, N, N, 8, dtype=torch.float64, device=DEV)
        self.phi = DTAU * 0.5 * DTAU * self.pi
        self.n = 1

    def step(self):
        """One leapfrog step; returns the site fields at tau_n [6][N, N, 8]
        and the links and phi of tau_n."""
        U, E, pi = self.U, self.E, self.pi
        tau, th = self.n * DTAU, (self.n + 0.5) * DTAU
        ph = _alg(self.phi)
        Um = [_dag(_sh(U[d], d, -1)) for d in (0, 1)]            # U_d^dag(x - d)
        P = _mm(_mm(U[0], _sh(U[1], 0, 1)), _mm(_dag(_sh(U[0], 1, 1)), _dag(U[1])))
        C = _alg(_proj(P))
        C1, C2 = (_conj_by(Um[d], _sh(C, d, -1)) for d in (0, 1))
        fwd = [_conj_by(U[d], _sh(ph, d, 1)) for d in (0, 1)]
        bwd = [_conj_by(Um[d], _sh(ph, d, -1)) for d in (0, 1)]
        comm = [-1j / tau * (_mm(ph, fwd[d]) - _mm(fwd[d], ph)) for d in (0, 1)]
        F = torch.stack([_comps(-tau * (C - C2) + comm[0]), _comps(-tau * (C1 - C) + comm[1])])
        lap = (fwd[0] + bwd[0]) + (fwd[1] + bwd[1]) - 4.0 * ph
        En, pin = E + DTAU * F, pi + DTAU * _comps(lap) / tau
        Eb = 0.5 * (E + En)
        Es = [0.5 * (_alg(Eb[d]) + _conj_by(Um[d], _alg(_sh(Eb[d], d, -1)))) for d in (0, 1)]
        W = _dag(_mm(_sh(_sh(U[0], 0, -1), 1, -1), _sh(U[1], 1, -1)))
        B = 0.25 * (C + C1 + C2 + _conj_by(W, _sh(_sh(C, 0, -1), 1, -1)))
        fields = [_comps(Es[0]) / tau, _comps(Es[1]) / tau, 0.5 * (pi + pin), -_comps(0.5 * (fwd[1] - bwd[1])) / tau,
                  _comps(0.5 * (fwd[0] - bwd[0])) / tau, -_comps(B)]
        old = U, self.phi
        self.U = _mm(_expi(DTAU / th * En), U)
        self.E, self.pi, self.phi = En, pin, self.phi + DTAU * th * pin
        self.n += 1
        return fields, old

    def energy(self):
        tau = self.n * DTAU
        ph = _alg(self.phi)
        mag = sum(0.5 * _comps(_conj_by(self.U[d], _sh(ph, d, 1)) - ph).square().sum() for d in (0, 1))
        P = _mm(_mm(self.U[0], _sh(self.U[1], 0, 1)), _mm(_dag(_sh(self.U[0], 1, 1)), _dag(self.U[1])))
        return [float(v) for v in (0.5 * self.E.square().sum() / tau, 0.5 * tau * self.pi.square().sum(), mag / tau,
                                   2.0 * tau * (3.0 - torch.diagonal(P, dim1=-2, dim2=-1).sum(-1).real).sum())]


class _Probes:
    """Particles of all species, pushed with Wong's equations."""

    def __init__(self, N, a_gev, a_fm, species, n_per, seed):
        q0 = [r.real for r in sorted(np.roots([1.0, 0.0, -1.0, -5.0 / 18.0]), reverse=True)]
        for _ in range(3):
            q0 = [q - (q ** 3 - q - 5.0 / 18.0) / (3 * q * q - 1) for q in q0]
        # largest, then the middle and the lowest root
        Q0 = torch.diag(torch.tensor(q0, dtype=torch.complex128, device=DEV))
        i = torch.arange(n_per, device=DEV)
        cell, off, p, Q, self.mass, self.nform, self.tf = [], [], [], [], [], [], []
        for s, (m, p0, kind, tf) in enumerate(species):
            sd = seed + 17 * s
            w = _philox(sd, i, 0, 2 + s)
            xy = torch.stack([_uniform(w[0], w[1]), _uniform(w[2], w[3])]) * N
            near = torch.floor(xy + 0.5)
            cell.append(near.long() % N)
            off.append(xy - near)
            w = _philox(sd, i, 1, 2 + s)
            az = 2.0 * math.pi * _uniform(w[0], w[1]) if kind == 0 else torch.zeros(n_per, device=DEV,
                                                                                    dtype=torch.float64)
            pl = p0 * a_gev
            p.append(torch.stack([pl * torch.cos(az), pl * torch.sin(az), torch.zeros_like(az)]))
            Z = torch.stack([torch.complex(*_normals(_philox(sd, i, 2 + k, 2 + s))) for k in range(9)],
                            -1).reshape(-1, 3, 3)
            cols = []
            for c in range(3):
                v = Z[:, :, c]
                for u in cols:
                    v = v - (u.conj() * Z[:, :, c]).sum(-1, keepdim=True) * u
                cols.append(v / v.abs().square().sum(-1, keepdim=True).sqrt())
            Uh = torch.stack(cols, -1)
            Q.append(_comps(_conj_by(Uh, Q0.expand(n_per, 3, 3))))
            self.mass.append(m * a_gev)
            tf = tf if tf >= 0 else HBARC / (2.0 * math.sqrt(m * m + p0 * p0))
            self.tf.append(tf)
            self.nform.append(max(1, int(math.ceil(tf / (DTAU * a_fm)))))
        self.N, self.ns, self.n_per = N, len(species), n_per
        self.cell, self.off, self.p = (torch.stack(v, 1) for v in (cell, off, p))       # [.][species][n]
        self.Q, self.eta = torch.stack(Q), torch.zeros(len(species), n_per, device=DEV, dtype=torch.float64)
        self.p0 = self.p.clone()
        self.mass = torch.tensor(self.mass, device=DEV, dtype=torch.float64)[:, None].expand(-1, n_per)

    def step(self, n, fields, U, phi):
        """tau_n -> tau_{n+1}; returns the sums [species][4]"""
        on = [s for s in range(self.ns) if n >= self.nform[s]]
        row = np.zeros((self.ns, 4))
        if not on:
            return row
        tau, th = n * DTAU, (n + 0.5) * DTAU
        cell, off, p, Q, m = self.cell[:, on], self.off[:, on], self.p[:, on], self.Q[on], self.mass[on]
        cx, cy = cell
        e, b = (torch.stack([(Q * fields[k][cy, cx]).sum(-1) for k in r]) for r in ((0, 1, 2), (3, 4, 5)))
        pm = torch.stack([p[0], p[1], p[2] / tau]) + 0.5 * DTAU * e
        t = b * DTAU / (2.0 * torch.sqrt(m * m + pm.square().sum(0)))
        pq = pm + torch.cross(pm + torch.cross(pm, t, dim=0), 2.0 * t / (1.0 + t.square().sum(0)), dim=0)
        pl = pq + 0.5 * DTAU * e
        Peta = tau * pl[2]
        pz = Peta / th
        ptau = torch.sqrt(m * m + pl[0] ** 2 + pl[1] ** 2 + pz ** 2)
        off = off + DTAU * pl[:2] / ptau
        deta = DTAU * Peta / (th * th * ptau)
        eta = self.eta[on]
        X = _conj_by(_expi(-phi[cy, cx] * deta[..., None]), _alg(Q))
        for d in (0, 1):
            up, dn = off[d] >= 0.5, off[d] < -0.5
            back = cell.clone()
            back[d] = (back[d] - 1) % self.N
            fw, bw = U[d][cell[1], cell[0]], U[d][back[1], back[0]]
            X = torch.where(up[..., None, None], _conj_by(_dag(fw), X),
                            torch.where(dn[..., None, None], _conj_by(bw, X), X))
            off[d] += dn.double() - up.double()
            cell = cell.clone()
            cell[d] = (cell[d] + up.long() - dn.long()) % self.N
        half = eta + 0.5 * deta
        lab = torch.stack([pl[0], pl[1], ptau * torch.sinh(half) + pz * torch.cosh(half)])
        row[on, :3] = (lab ** 2 - self.p0[:, on] ** 2).sum(-1).T.cpu().numpy()
        row[on, 3] = self.n_per
        self.cell[:, on], self.off[:, on], self.Q[on], self.eta[on] = cell, off, _comps(X), eta + deta
        self.p[:, on] = torch.stack([pl[0], pl[1], Peta])
        return row


def _event64(case, seed):
    N, a_fm = case["N"], case["a_fm"]
    a_gev = a_fm / HBARC
    sp, steps = _species(case), _steps(a_fm, case["tau_max"])
    lat = _Lattice(N, case["g2mu"] * a_gev / math.sqrt(case["sheets"]), (M_IR * a_gev) ** 2, case["sheets"], seed)
    probes = _Probes(N, a_gev, a_fm, sp, case["n_per"], seed) if sp else None
    scan_case = case["path"] == "scan"
    series = np.zeros((steps, len(sp), 4))
    I = torch.zeros(2, 3, N, N, 8, dtype=torch.float64, device=DEV)
    Wl = torch.eye(3, dtype=torch.complex128, device=DEV).expand(N, N, 3, 3)
    corr = np.zeros((2, steps, 3))
    n_static = probes.nform[0] if scan_case else 0
    for k in range(steps):
        n = lat.n
        F, (U, phi) = lat.step()
        if probes:
            series[k] = probes.step(n, F, U, phi)
        if not scan_case:
            continue
        if n >= n_static:
            I[0] += DTAU * torch.stack(F[:3])
            corr[0, k] = 0.5 * I[0].square().sum((1, 2, 3)).cpu().numpy()
        at = int(math.floor((n - 1) * DTAU + 0.5))
        for i, f in enumerate((F[0], F[1] - F[5], F[2] + F[4])):
            I[1, i] += DTAU * _comps(_conj_by(Wl, _alg(_sh(f, 0, at))))
        corr[1, k] = 0.5 * I[1].square().sum((1, 2, 3)).cpu().numpy()
        if int(math.floor(n * DTAU + 0.5)) > at:
            Wl = _mm(Wl, _sh(U[0], 0, at))
    f2, dt = 1.0 / a_gev ** 2, DTAU * a_fm
    if scan_case:
        t = (np.arange(steps) + 1.5) * dt
        rows = [np.column_stack([t, corr[c] / (N * N) * f2, np.full(steps, float(N * N))]) for c in (0, 1)]
        return series, rows[0][n_static - 1:], rows[1]
    if not sp:
        return lat.energy()
    out = []
    for s, (_, _, kind, _) in enumerate(sp):
        k = np.arange(probes.nform[s] - 1, steps)
        mean = series[k, s, :3] / probes.n_per
        rate = np.diff(mean, axis=0, prepend=0.0) / DTAU * f2 / a_fm
        tau = (k + 1) * dt
        curve = np.column_stack([tau, tau - probes.tf[s], rate[:, 0] + rate[:, 1], rate[:, 2]]) if kind == 0 else \
            np.column_stack([tau, rate[:, 1], rate[:, 2]])
        out.append((np.column_stack([(k + 1.5) * dt, mean * f2, np.full(len(k), float(probes.n_per))]), curve))
    return out
