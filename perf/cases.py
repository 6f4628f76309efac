"""Workloads whose speed is tracked: what a user of this library has it do, through its public entry points.

A case is a dict of plain values; `prepare` makes what a program holds before the call (a system, a batch, device
positions), `run` is one pass of the call, `work` the bytes and operations it cannot do without, `exact` the result in
64 bits by plain numpy where there is one.  Sweeps have none: a trajectory of hard disks is chaotic, so after a few
hundred events any other order of operations leads to another, equally valid one.
"""
import math

import numpy as np
import torch

import paper_1409_6948_amd as P


# --------------------------------------------------------------------------------------------------------------------
# The listed cases
# --------------------------------------------------------------------------------------------------------------------
def listed():
    return [
        # one small periodic cell, the serial event chain: a reference run beside a parallel one
        _sweep("serial_256", 256, 0.70, 1, 20.0, warm=1),
        # the smallest walled system in use (4 x 4 cells of 16 disks, short chains): latency and launches count
        _sweep("pec_256", 256, 0.70, 4, 2.0, warm=4, sweeps=4),
        # an odd system: 10,007 disks, cells of 100 disks that do not divide them, a dilute fluid
        _sweep("pec_odd_10007", 10007, 0.55, 10, 5.0, warm=4),
        # 256^2 disks near the transition, few large cells: fewer cells than the chip has SIMDs
        _sweep("pec_65k", 65536, 0.70, 16, 20.0, warm=2),
        # one million disks, the headline workload
        _sweep("pec_1m", 1048576, 0.72, 64, 20.0, warm=2),
        # four million disks in the FP32-screened form, the largest call: every SIMD has several cells
        _sweep("pec_4m_fp32", 4194304, 0.716, 128, 30.0, warm=1, precision="fp32-screen"),
        # rejection at the cell boundary (the comparison variant), short chains
        _sweep("reject_16k", 16384, 0.70, 16, 0.2, warm=4, sweeps=4, reject=True),
        # a density scan: sixteen independent systems of 64 disks per cell advanced together
        dict(name="batch_16", kind="batch", n_sys=16, meta=0, n_min=4096, n_max=262144, ell=20.0, warm=1,
             precision="fp64"),
        # device-resident positions advanced in a program's own buffers, without allocation or host copies
        dict(name="static_16k", kind="static", n=16384, eta=0.70, cells=16, ell=10.0, warm=2, sweeps=2),
        # the order parameter between sweeps: neighbours within a cutoff, then Delaunay neighbours; the disks are
        # numbered along the lattice they started from, as in a dense run
        dict(name="psi6_1m", kind="psi6", columns=1024, eta=0.72, cells=64, mixed=False),
        dict(name="delaunay_1m", kind="delaunay", columns=1024, eta=0.72, cells=64, mixed=False),
        # the pair histogram at contact, the other pressure route, of a configuration long since mixed
        dict(name="gr_262k", kind="gr", columns=512, eta=0.70, cells=32, r_max=1.5, bins=500, mixed=True),
    ]


def _sweep(name, n, eta, cells, ell, warm, sweeps=1, precision="fp64", reject=False):
    return dict(name=name, kind="sweep", n=n, eta=eta, cells=cells, ell=ell, warm=warm, sweeps=sweeps,
                precision=precision, reject=reject)


# --------------------------------------------------------------------------------------------------------------------
# More of the same ranges
# --------------------------------------------------------------------------------------------------------------------
def _log_uniform(rng, a, b):
    return math.exp(rng.uniform(math.log(a), math.log(b)))


def _box(n, eta):
    return math.sqrt(n * math.pi / (4.0 * eta))


def _starts(n, eta):
    """Whether the start lattice of ceil(sqrt n) columns leaves the disks apart."""
    return _box(n, eta) / math.ceil(math.sqrt(n)) > 1.005


def _walled(rng, n_min, n_max, per_cell_min, per_cell_max):
    """A walled system: disks, density and an even number of cells per side of at least 3.2 diameters."""
    while True:
        n = int(_log_uniform(rng, n_min, n_max))
        eta = rng.uniform(0.30, 0.72)
        cells = max(4, 2 * int(math.sqrt(n / _log_uniform(rng, per_cell_min, per_cell_max)) / 2.0 + 0.5))
        side = _box(n, eta) / cells
        if _starts(n, eta) and 3.2 < side < 40.0:
            return n, eta, cells


def draw(rng):
    kind = rng.choice(["walled", "walled", "walled", "periodic", "reject", "batch", "static", "psi6", "delaunay", "gr"])
    if kind == "periodic":
        while True:
            n, eta = int(_log_uniform(rng, 64, 1500)), rng.uniform(0.20, 0.71)
            if _starts(n, eta):
                break
        c = _sweep("", n, eta, 1, _log_uniform(rng, 1.0, 20.0), warm=1)
    elif kind == "walled":
        n, eta, cells = _walled(rng, 256, 1.5e6, 16, 300)
        c = _sweep("", n, eta, cells, _log_uniform(rng, 0.5, 20.0), warm=2,
                   precision=rng.choice(["fp64", "fp64", "fp32-screen"]))
    elif kind == "reject":
        n, eta, cells = _walled(rng, 1024, 65536, 32, 128)
        c = _sweep("", n, eta, cells, _log_uniform(rng, 0.1, 1.0), warm=2, reject=True)
    elif kind == "batch":
        n_max = int(_log_uniform(rng, 8192, 131072))
        c = dict(kind="batch", n_sys=rng.randint(2, 16), meta=rng.randrange(1 << 30), n_min=4096, n_max=n_max,
                 ell=_log_uniform(rng, 2.0, 20.0), warm=1, precision=rng.choice(["fp64", "fp32-screen"]))
    elif kind == "static":
        n, eta, cells = _walled(rng, 1024, 131072, 32, 200)
        c = dict(kind="static", n=n, eta=eta, cells=cells, ell=_log_uniform(rng, 1.0, 20.0), warm=2,
                 sweeps=rng.randint(1, 4))
    else:
        columns = int(_log_uniform(rng, 64, 1000))
        eta = rng.uniform(0.66, 0.72)
        n = columns * _rows(columns)
        cells = max(4, 2 * int(math.sqrt(n / _log_uniform(rng, 64, 300)) / 2.0 + 0.5))
        c = dict(kind=kind, columns=columns, eta=eta, cells=cells, mixed=rng.random() < 0.5)
        if kind == "gr":
            c.update(r_max=rng.uniform(1.3, 1.9), bins=rng.randint(50, 1000))
    c.pop("name", None)
    return c


# --------------------------------------------------------------------------------------------------------------------
# What a program has in hand before the call
# --------------------------------------------------------------------------------------------------------------------
_PRECISION = {"fp64": P.EC_PREC_FP64, "fp32-screen": P.EC_PREC_FP32_SCREEN}


def _params(case, seed):
    cells = case["cells"]
    return P.make_params(case["n"], case["eta"], case["ell"], cells, seed=seed,
                         dir_mode=P.EC_DIR_XY if cells == 1 else P.EC_DIR_ISOTROPIC,
                         precision=_PRECISION[case.get("precision", "fp64")],
                         flags=P.EC_FLAG_REJECT if case.get("reject") else 0)


def _rows(columns):
    """Even number of lattice rows that makes a square box of `columns` columns nearly triangular."""
    return 2 * int(columns * 2.0 / math.sqrt(3.0) / 2.0 + 0.5)


def _crystal(case, seed):
    """A thermally disordered triangular crystal filling the box: every disk displaced within the free gap of its site,
    so no two overlap; numbered along the rows, or at random (`mixed`).  Returns x, y, L and every disk's column and
    row."""
    nx, ny = case["columns"], _rows(case["columns"])
    n = nx * ny
    L = _box(n, case["eta"])
    rng = np.random.default_rng(seed)
    site = rng.permutation(n) if case["mixed"] else np.arange(n)
    i, j = site % nx, site // nx
    ax, ay = L / nx, L / ny
    gap = min(ax, math.hypot(0.5 * ax, ay)) - 1.0
    r = 0.499 * gap * np.sqrt(rng.random(n))
    phi = 2.0 * np.pi * rng.random(n)
    x = (i + np.where(j % 2 == 0, 0.25, 0.75)) * ax + r * np.cos(phi)
    y = (j + 0.5) * ay + r * np.sin(phi)
    return np.mod(x, L), np.mod(y, L), L, i, j


def _batch_params(case, seed):
    """Sizes log-uniform, densities uniform in [0.30, 0.72], about 64 disks per cell; the sizes are the case's own,
    the seed gives the trajectories."""
    rng = np.random.default_rng(case["meta"])
    out = []
    for k in range(case["n_sys"]):
        side = 2 * int(round(math.sqrt(math.exp(rng.uniform(math.log(case["n_min"]), math.log(case["n_max"])))) / 2.0))
        n, eta = side * side, rng.uniform(0.30, 0.72)
        cells = max(4, 2 * int(round(math.sqrt(n / 64.0) / 2.0)))
        while cells > 4 and _box(n, eta) / cells <= 3.0:
            cells -= 2
        out.append(P.make_params(n, eta, case["ell"], cells, seed=seed * 1000 + k,
                                 precision=_PRECISION[case["precision"]]))
    return out


def prepare(case, seed):
    kind = case["kind"]
    if kind == "sweep":
        s = P.System(_params(case, seed))
        s.sweep(case["warm"])  # off the start lattice
        s.reset_tallies()
        return dict(kind=kind, system=s, sweeps=case["sweeps"])
    if kind == "batch":
        b = P.Batch(_batch_params(case, seed))
        b.sweep(case["warm"])
        for s in b.systems:
            s.reset_tallies()
        return dict(kind=kind, batch=b)
    if kind == "static":
        p = _params(case, seed)
        s = P.System(p)
        s.sweep(case["warm"])
        x, y = s.get_positions()
        k = case["sweeps"]
        return dict(kind=kind, p=p, x=torch.from_numpy(x).cuda(), y=torch.from_numpy(y).cuda(), done=case["warm"],
                    sweeps=k, digests=torch.zeros(k, dtype=torch.int64, device="cuda"),
                    err=torch.zeros(1, dtype=torch.int32, device="cuda"))
    x, y, _, _, _ = _crystal(case, seed)
    s = P.System(P.make_params(len(x), case["eta"], 20.0, case["cells"], seed=seed))
    s.set_positions(x, y)
    return dict(kind=kind, system=s, case=dict(case))


# --------------------------------------------------------------------------------------------------------------------
# One pass
# --------------------------------------------------------------------------------------------------------------------
def run(state):
    kind = state["kind"]
    if kind == "sweep":
        # advance, read the pressure, fetch the configuration
        s = state["system"]
        s.sweep(state["sweeps"])
        z, bp, counts = s.measure_pressure()
        x, y = s.get_positions()
        return dict(x=x, y=y, z=z, beta_p=bp, digests=s.get_digests(state["sweeps"]).view(np.int64),
                    counts=np.array(list(counts.values()), dtype=np.int64))
    if kind == "batch":
        b = state["batch"]
        b.sweep(1)
        got = [(s.measure_pressure()[0], s.get_positions(), s.get_digests(1)[0]) for s in b.systems]
        return dict(z=np.array([g[0] for g in got]), x=np.concatenate([g[1][0] for g in got]),
                    y=np.concatenate([g[1][1] for g in got]), digests=np.array([g[2] for g in got]).view(np.int64))
    if kind == "static":
        P.ec.sweep_static(state["p"], state["x"], state["y"], state["done"], state["sweeps"], state["digests"],
                       state["err"])
        state["done"] += state["sweeps"]
        return dict(x=state["x"], y=state["y"], digests=state["digests"], err=state["err"])
    s = state["system"]
    if kind == "psi6":
        psi, nb, per = s.measure_psi6(per_disk=True)
        return dict(re=psi.real, im=psi.imag, neighbours=nb, per_disk=per)
    if kind == "delaunay":
        psi, nb, per, count = s.measure_psi6_delaunay(per_disk=True)
        return dict(re=psi.real, im=psi.imag, neighbours=nb, per_disk=per, count=count)
    s.gr_reset()
    s.gr_accumulate(state["case"]["r_max"], state["case"]["bins"])
    counts, samples, overlaps = s.gr_counts()
    return dict(counts=counts.astype(np.int64), samples=samples, overlaps=overlaps)


# --------------------------------------------------------------------------------------------------------------------
# What a pass cannot do without
# --------------------------------------------------------------------------------------------------------------------
def _events(n, eta, ell):
    """Collisions of n chains of length ell: with a contact projection of pi/4 on average, Z - 1 = (pi/4) lifts / ell;
    Z from Henderson's equation of state, level above the transition."""
    z = min((1.0 + eta * eta / 8.0) / (1.0 - eta) ** 2, 10.3)
    return n * (1.0 + ell * (z - 1.0) * 4.0 / math.pi)


def work(case):
    """Sweeps: positions read and written once, and 100 operations per event (the contact tests of the eight disks
    around the moving one, 12 operations each, and the move).  Observables: positions read once, results written once;
    per disk six bonds of 25 operations (cutoff), eighteen nearby disks whose bisectors are cut with each other at 8
    operations (Delaunay), or the distances to the disks within the histogram's range."""
    kind = case["kind"]
    if kind == "sweep":
        k, n = case["sweeps"], case["n"]
        return dict(bytes=32.0 * n * k, flops=100.0 * k * _events(n, case["eta"], case["ell"]))
    if kind == "static":
        k, n = case["sweeps"], case["n"]
        return dict(bytes=32.0 * n * k, flops=100.0 * k * _events(n, case["eta"], case["ell"]))
    if kind == "batch":
        ps = _batch_params(case, 1)
        return dict(bytes=sum(32.0 * p.n_disks for p in ps),
                    flops=sum(100.0 * _events(p.n_disks, p.eta, case["ell"]) for p in ps))
    n = case["columns"] * _rows(case["columns"])
    if kind == "psi6":
        return dict(bytes=32.0 * n, flops=150.0 * n)
    if kind == "delaunay":
        return dict(bytes=36.0 * n, flops=18.0 * 18.0 * 8.0 * n)
    pairs = n * 4.0 * case["eta"] * case["r_max"] ** 2
    return dict(bytes=16.0 * n + 8.0 * case["bins"], flops=10.0 * pairs)


# --------------------------------------------------------------------------------------------------------------------
# The result in 64 bits
# --------------------------------------------------------------------------------------------------------------------
def exact(case, seed):
    """Psi of the disordered crystal, whose neighbours (within 1.4 diameters, and by Delaunay's rule) are the six sites
    around each site: the displacements are far too small to change them."""
    if case["kind"] not in ("psi6", "delaunay"):
        return None
    x, y, L, i, j = _crystal(case, seed)
    nx, ny = case["columns"], _rows(case["columns"])
    gx, gy = np.empty((ny, nx)), np.empty((ny, nx))
    gx[j, i], gy[j, i] = x, y
    row = np.arange(ny)[:, None]
    col = np.arange(nx)[None, :]
    odd = row % 2
    psi = np.zeros((ny, nx), dtype=np.complex128)
    for dr, dc in ((0, -1), (0, 1), (-1, -1), (-1, 0), (1, -1), (1, 0)):
        c = (col + dc + (odd if dr else 0)) % nx
        r = (row + dr) % ny
        r, c = np.broadcast_arrays(r, c)
        dx, dy = gx[r, c] - gx, gy[r, c] - gy
        dx -= L * np.round(dx / L)
        dy -= L * np.round(dy / L)
        psi += ((dx + 1j * dy) / np.hypot(dx, dy)) ** 6
    per = (psi / 6.0)[j, i]
    total = per.mean()
    out = dict(re=float(total.real), im=float(total.imag), neighbours=6.0, per_disk=per)
    if case["kind"] == "delaunay":
        out["count"] = None
    return out
