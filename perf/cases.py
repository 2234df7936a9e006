"""Workloads whose time matters to a user of the Reg-FLBM library, with a plain
FP64 torch form of the same update to hold their results against.

Every case goes through the package's public classes (Lattice, Batch) as the
benchmark, the physics runs and the tests of this repository use them.  A case
is a dict of plain values; listed() gives the fixed ones, draw() more of the
same ranges: boxes of 8^3 to 256^3 and 512^3, x extents that are multiples of
64 and others, the three storage types, the three collision models, with and
without noise, single steps and runs, statistics, structure factors, batches,
thermalised starts and checkpoint restarts.
"""
import math

import numpy as np
import torch

import paper_2507_08820_amd as rf

DEV = "cuda"
BYTES = {"f32": 4, "f16": 2, "bf16": 2}


def _step(name, dims, steps, out, **kw):
    c = dict(name=name, kind="step", nx=dims[0], ny=dims[1], nz=dims[2], storage="f32", model="reg", kT=1e-5,
             tau=0.6, tau_bulk=0.6, tau_ghost=1.0, steps=steps, stats_every=0, out=out)
    c.update(kw)
    return c


def listed():
    return [
        # the equipartition check on the smallest box: statistics on every
        # step, the state read back every ten
        _step("equipartition_16", (16, 16, 16), 10, "populations", kT=1e-4, tau=1.0, tau_bulk=1.0, stats_every=1),
        # small odd box with general ghost rates, an odd number of steps
        _step("odd_17x19x23_mrt", (17, 19, 23), 7, "populations", kT=1e-4, tau=0.7, tau_bulk=1.1, tau_ghost=0.9),
        # a box edge of the replica table that is no multiple of the wave width
        _step("box_96_f32", (96, 96, 96), 20, "populations"),
        # ragged box with 16-bit storage and the BGK comparator
        _step("ragged_130x50x70_bf16_bgk", (130, 50, 70), 20, "moments", storage="bf16", model="bgk", tau=0.8,
              tau_bulk=0.8),
        # the shear-wave / precision box
        _step("wave_128_f32", (128, 128, 128), 20, "moments", tau_bulk=1.0),
        # the equilibration-ratio protocol: statistics every 50 steps at 256^3
        _step("protocol_256_f32", (256, 256, 256), 50, "moments", kT=1.0 / 3000.0, tau=0.55, tau_bulk=0.55,
              stats_every=50),
        # 16-bit deviation storage with noise
        _step("precision_256_f16", (256, 256, 256), 20, "moments", storage="f16"),
        # the benchmark's workload: Taylor-Green flow, 512^3, FP32
        _step("taylor_green_512_f32", (512, 512, 512), 10, "moments"),
        # a structure-factor snapshot of all ten fields
        dict(name="structure_factor_256", kind="sk", nx=256, ny=256, nz=256, storage="f32", model="reg",
             kT=1.0 / 3000.0, tau=0.55, tau_bulk=0.55, tau_ghost=1.0, steps=2),
        # the batched workload: 64 boxes of 32^3 .. 96^3 in graphs of 20 steps
        dict(name="batch_64_f32", kind="batch", count=64, table=5, storage="f32", steps=20, graph=20, stats_every=0,
             small=0),
        # start of a run: thermalised populations from given fields, read back
        dict(name="thermal_start_192", kind="start", nx=192, ny=192, nz=192, storage="f32", model="reg", kT=1e-5,
             tau=0.6, tau_bulk=0.6, tau_ghost=1.0, steps=0),
        # checkpoint and resume at an odd step count
        dict(name="restart_128x112x96_f16", kind="restart", nx=128, ny=112, nz=96, storage="f16", model="reg",
             kT=1e-5, tau=0.6, tau_bulk=1.0, tau_ghost=1.0, steps=3),
    ]


# x extents: whole waves, or any size
_WHOLE = (64, 128, 192, 256, 320)


def _dims(rng, lo, hi):
    """A box of lo .. hi nodes (spread over the logarithm), sides 4 .. 320."""
    n = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    edge = n ** (1.0 / 3.0)
    if rng.random() < 0.45:
        fit = [w for w in _WHOLE if w <= 4 * edge] or [64]
        nx = rng.choice(fit)
    else:
        nx = int(round(min(320, max(4, edge * math.exp(rng.uniform(-0.6, 0.6))))))
    rest = math.sqrt(max(16.0, n / nx))
    ny = int(round(min(320, max(4, rest * math.exp(rng.uniform(-0.4, 0.4))))))
    nz = int(min(320, max(4, n / (nx * ny))))
    return nx, ny, nz


def draw(rng):
    kind = rng.choice(["step"] * 6 + ["sk", "batch", "start", "restart"])
    storage = rng.choice(["f32", "f32", "f16", "bf16"])
    if kind == "batch":
        return dict(kind="batch", count=rng.randint(2, 48), table=rng.randint(0, 9999), storage=storage,
                    steps=rng.randint(6, 20), graph=rng.choice([0, 2, 6]), stats_every=rng.choice([0, 0, 5]),
                    small=rng.randint(0, 1))
    lo, hi = (2 ** 10, 2 ** 24) if kind == "step" else (2 ** 12, 2 ** 23)
    nx, ny, nz = _dims(rng, lo, hi)
    kT = rng.choice([1e-4, 1e-5, 1e-6, 1.0 / 3000.0])
    tau = round(math.exp(rng.uniform(math.log(0.55), math.log(3.0))), 3)
    c = dict(kind=kind, nx=nx, ny=ny, nz=nz, storage=storage, model="reg", kT=kT, tau=tau, tau_bulk=tau,
             tau_ghost=1.0, steps=rng.randint(1, 5))
    if kind != "step":
        return c
    c["model"] = rng.choice(["reg", "reg", "reg", "bgk", "rec"])
    c["tau_ghost"] = rng.choice([1.0, 1.0, 0.8]) if c["model"] != "rec" else 0.9
    c["tau_bulk"] = rng.choice([tau, 1.0])
    if rng.random() < 0.2:
        c["kT"] = 0.0  # the deterministic method
    c["steps"] = max(1, min(50, int(rng.uniform(0.2, 1.0) * 2 ** 27 / (nx * ny * nz)), rng.randint(1, 50)))
    c["stats_every"] = rng.choice([0, 0, 0, 1, 5])
    if c["kT"] == 0.0:
        c["stats_every"] = 0  # the statistics are of the fluctuations
    c["out"] = "populations" if storage == "f32" and nx * ny * nz < 2 ** 22 else "moments"
    return c


# ---------------------------------------------------------------------------
# what a program has in hand

def _params(c, seed):
    kw = dict(storage=c["storage"], model=c["model"], kT=c["kT"], tau=c["tau"], tau_bulk=c["tau_bulk"],
              tau_ghost=c["tau_ghost"], seed=int(seed) + 1)
    if c["storage"] != "f32" and c["kT"] == 0.0:
        kw["storage_scale"] = 0.005  # deviation unit of the flow, as there is no thermal one
    return kw


def _flow(dims, seed):
    """Density (N,) and velocity (3, N) in node order: a Taylor-Green flow of
    amplitude 0.01 with phases of its own and a density wave of 0.1 %."""
    nx, ny, nz = dims
    ph = np.random.default_rng(int(seed)).uniform(0.0, 2.0 * math.pi, 4)
    ax = [2.0 * math.pi * torch.arange(n, dtype=torch.float64, device=DEV) / n + p for n, p in zip(dims, ph)]
    x, y, z = ax[0][None, None, :], ax[1][None, :, None], ax[2][:, None, None]
    u = torch.zeros((3, nz, ny, nx), dtype=torch.float64, device=DEV)
    u[0] = 0.01 * torch.sin(x) * torch.cos(y) * torch.cos(z)
    u[1] = -0.01 * torch.cos(x) * torch.sin(y) * torch.cos(z)
    rho = (1.0 + 1e-3 * torch.sin(x + ph[3]) * torch.cos(y)).expand(nz, ny, nx)
    return rho.reshape(-1).contiguous(), u.reshape(3, -1)


def _lattice(c, seed):
    dims = (c["nx"], c["ny"], c["nz"])
    return rf.Lattice(dims, **_params(c, seed)), _flow(dims, seed)


def _replicas(c, seed):
    g = np.random.default_rng(c["table"])
    edges = np.asarray((8, 12, 16, 20, 24, 31, 32)) if c["small"] else np.asarray((32, 48, 64, 96))
    n = c["count"]
    edge, tau, lk = g.choice(edges, size=n), g.uniform(0.55, 1.2, n), g.uniform(-6.0, -4.0, n)
    return [dict(dims=(int(e),) * 3, tau=float(t), kT=float(10.0 ** k), seed=int(seed) + 1000 + r, stream_id=r)
            for r, (e, t, k) in enumerate(zip(edge, tau, lk))]


def prepare(case, seed):
    c = case
    if c["kind"] == "batch":
        b = rf.Batch(_replicas(c, seed), storage=c["storage"])
        for r in range(len(b)):
            b[r].init_thermal()
        b.set_launch(256, 0, c["graph"])
        if c["stats_every"]:
            b.stats_config(c["stats_every"])
        return dict(case=c, batch=b)
    lat, (rho, u) = _lattice(c, seed)
    s = dict(case=c, lat=lat)
    if c["kind"] == "start":
        s.update(rho=rho, u=u)
        return s
    if c["kT"] > 0.0:
        lat.init_thermal(rho, u)
    else:
        lat.init_equilibrium(rho, u)
    if c["kind"] == "sk":
        lat.sk_sample()  # the run's earlier snapshots
        lat.step(c["steps"])
    elif c["kind"] == "restart":
        lat.step(c["steps"])
        s["params"] = _params(c, seed)
    elif c["stats_every"]:
        lat.stats_config(c["stats_every"])
    return s


def _numbers(stats):
    return {k: v.tolist() if isinstance(v, np.ndarray) else v for k, v in stats.items()}


def run(state):
    c = state["case"]
    if c["kind"] == "batch":
        b = state["batch"]
        b.step(c["steps"])
        return [b[r].moments() for r in range(len(b))]
    lat = state["lat"]
    if c["kind"] == "start":
        lat.init_thermal(state["rho"], state["u"])
        return lat.populations()
    if c["kind"] == "sk":
        lat.reset_sk()
        lat.sk_sample()
        spectra = {}
        for f in rf.FIELDS:
            sums, counts, samples = lat.sk(f)
            # per-shell means of single-precision transforms
            spectra[f] = (sums / np.maximum(counts, 1) / samples).astype(np.float32)
        return {"spectra": spectra, "counts": counts}
    if c["kind"] == "restart":
        to = rf.Lattice(lat.dims, **state["params"])  # the resumed program's own lattice
        to.set_populations(lat.populations())
        to.t = lat.t
        to.step(2)
        return to.moments()
    if c["stats_every"]:
        lat.reset_stats()
    lat.step(c["steps"])
    out = {"state": lat.populations() if c["out"] == "populations" else lat.moments()}
    if c["stats_every"]:
        out["stats"] = _numbers(lat.stats())
    return out


def _flops(kT):
    """FP32 operations of one node's update: the two transforms, equilibrium
    and relaxation, and with noise 12 Box-Muller pairs and 23 mode additions."""
    return 340 + (200 if kT > 0.0 else 0)


def work(case):
    c = case
    e = BYTES[c["storage"]]
    if c["kind"] == "batch":
        n = sum(int(np.prod(r["dims"])) for r in _replicas(c, 0))
        return {"bytes": n * (54 * e * c["steps"] + 27 * e + 40), "flops": n * c["steps"] * _flops(1.0)}
    n = c["nx"] * c["ny"] * c["nz"]
    if c["kind"] == "start":
        return {"bytes": n * (32 + 27 * e + 27 * (e + 8)), "flops": n * 600}
    if c["kind"] == "sk":
        return {"bytes": n * 27 * e, "flops": n * (80 + 10 * 2.5 * math.log2(n))}
    if c["kind"] == "restart":
        return {"bytes": n * (2 * 27 * (e + 8) + 2 * 54 * e + 27 * e + 40), "flops": n * 2 * _flops(c["kT"])}
    read = 27 * (e + 8) if c["out"] == "populations" else 27 * e + 40
    return {"bytes": n * (54 * e * c["steps"] + read), "flops": n * c["steps"] * _flops(c["kT"])}


# ---------------------------------------------------------------------------
# the same in FP64, in plain torch.  Populations as f[iz, iy, ix, z, y, x], i_a = c_a + 1.

_M32 = 0xFFFFFFFF
# mode degrees (x, y, z), k = 4 .. 26
_DEG = [(2, 0, 0), (0, 2, 0), (0, 0, 2), (1, 1, 0), (1, 0, 1), (0, 1, 1), (2, 1, 0), (2, 0, 1), (1, 2, 0), (1, 0, 2),
        (0, 1, 2), (0, 2, 1), (1, 1, 1), (2, 2, 0), (2, 0, 2), (0, 2, 2), (1, 1, 2), (1, 2, 1), (2, 1, 1), (2, 1, 2),
        (2, 2, 1), (1, 2, 2), (2, 2, 2)]
_BETA = (1.0, 1.0 / 3.0, 2.0 / 9.0)
_OMEGA = (1.0 / 6.0, 2.0 / 3.0, 1.0 / 6.0)
_POLY = [[1.0, 1.0, 1.0], [-1.0, 0.0, 1.0], [2.0 / 3.0, -1.0 / 3.0, 2.0 / 3.0]]  # [degree][i]


def _axes(m, f):
    """Applies the 3 x 3 matrix m along the three population axes."""
    for a in range(3):
        g = torch.empty_like(f)
        src, dst = f.unbind(a), g.unbind(a)
        for r in range(3):
            dst[r].copy_(m[r][0] * src[0])
            dst[r].add_(src[1], alpha=m[r][1]).add_(src[2], alpha=m[r][2])
        f = g
    return f


def _forward(f):
    return _axes(_POLY, f)


def _backward(m):
    return _axes([[_OMEGA[i] * _POLY[p][i] / _BETA[p] for p in range(3)] for i in range(3)], m)


def _philox(words, key, rounds=7):
    """Philox4x32 on int64 tensors or ints of 32-bit words."""
    w0, w1, w2, w3 = words
    k0, k1 = key
    for _ in range(rounds):
        p0, p2 = w0 * 0xD2511F53, w2 * 0xCD9E8D57
        w0, w1, w2, w3 = (((p2 >> 32) & _M32) ^ w1 ^ k0, p2 & _M32, ((p0 >> 32) & _M32) ^ w3 ^ k1, p0 & _M32)
        k0, k1 = (k0 + 0x9E3779B9) & _M32, (k1 + 0xBB67AE85) & _M32
    return w0, w1, w2, w3


def _normals(shape, step, calls, seed, sid):
    """6 * calls standard normals per node, one tensor at a time."""
    n = shape[0] * shape[1] * shape[2]
    node = torch.arange(n, dtype=torch.int64, device=DEV)
    zero = torch.zeros_like(node)
    for j in range(calls):
        w = _philox((node, zero + step, zero + j, zero + sid), (seed & _M32, seed >> 32))
        angle = (w[3] >> 16, w[3] & 0xFFFF, ((w[0] & 0xFF) << 8) | (w[1] & 0xFF))
        for m in range(3):
            rad = torch.sqrt(-2.0 * torch.log(1.0 - (w[m] >> 9).double() * 2.0 ** -23))
            th = angle[m].double() * (2.0 * math.pi / 65536.0)
            yield (rad * torch.cos(th)).view(shape)
            yield (rad * torch.sin(th)).view(shape)


def _equilibrium_modes(rho, u):
    """[pz][py][px] of rho u_x^px u_y^py u_z^pz."""
    pw = [[torch.ones_like(rho), v, v * v] for v in u]
    return [[[rho * pw[0][px] * pw[1][py] * pw[2][pz] for px in range(3)] for py in range(3)] for pz in range(3)]


def _initial(dims, rho, u, kT, seed, sid):
    nx, ny, nz = dims
    shape = (nz, ny, nx)
    m = torch.stack([torch.stack([torch.stack(r) for r in p]) for p in _equilibrium_modes(
        rho.view(shape), [v.view(shape) for v in u])])
    f = _backward(m)
    if kT > 0.0:
        for i, z in zip(range(27), _normals(shape, 0xFFFFFFFF, 5, seed, sid)):
            ix, iy, iz = i % 3, (i // 3) % 3, i // 9
            w = _OMEGA[ix] * _OMEGA[iy] * _OMEGA[iz]
            f[iz, iy, ix] += math.sqrt(3.0 * kT * w) * z
    return f


def _advance(f, t, p, sid=0):
    """One collision and streaming step."""
    shape = tuple(f.shape[3:])
    m = _forward(f)
    rho = m[0, 0, 0].clone()
    u = [m[0, 0, 1] / rho, m[0, 1, 0] / rho, m[1, 0, 0] / rho]
    eq = _equilibrium_modes(rho, u)
    bgk = p["model"] == "bgk"
    om_s = 1.0 / p["tau"]
    om_b = om_s if bgk else 1.0 / p["tau_bulk"]
    om_g = om_s if bgk else 1.0 / p["tau_ghost"]
    a2 = [m[d[2], d[1], d[0]] - eq[d[2]][d[1]][d[0]] for d in _DEG[:6]]
    trace = (a2[0] + a2[1] + a2[2]) / 3.0
    pw = [[torch.ones_like(rho), v, v * v] for v in u]
    pairs = ((0, 0), (1, 1), (2, 2), (0, 1), (0, 2), (1, 2))
    for k, d in enumerate(_DEG):
        px, py, pz = d
        e = eq[pz][py][px]
        if k < 3:
            m[pz, py, px] = e + (1.0 - om_s) * (a2[k] - trace) + (1.0 - om_b) * trace
        elif k < 6:
            m[pz, py, px] = e + (1.0 - om_s) * a2[k]
        elif p["model"] == "rec":
            rec = torch.zeros_like(rho)
            for q, (a, b) in enumerate(pairs):
                left = list(d)
                mult = left[a] * (left[a] - 1) // 2 if a == b else left[a] * left[b]
                if mult:
                    left[a] -= 1
                    left[b] -= 1
                    rec += mult * a2[q] * pw[0][left[0]] * pw[1][left[1]] * pw[2][left[2]]
            m[pz, py, px] = e + (1.0 - om_g) * rec
        else:
            m[pz, py, px] = e + (1.0 - om_g) * (m[pz, py, px] - e)
    if p["kT"] > 0.0:
        fdt = lambda om: math.sqrt(om * (2.0 - om))
        root = torch.sqrt(rho)
        first = []
        for k, z in zip(range(23), _normals(shape, t, 4, p["seed"], sid)):
            px, py, pz = _DEG[k]
            amp = math.sqrt(3.0 * p["kT"] * _BETA[px] * _BETA[py] * _BETA[pz])
            if k < 3:
                first.append(z)
                if k == 2:
                    mean = (first[0] + first[1] + first[2]) / 3.0
                    for q in range(3):
                        dx, dy, dz = _DEG[q]
                        m[dz, dy, dx] += amp * root * (fdt(om_s) * (first[q] - mean) + fdt(om_b) * mean)
            else:
                m[pz, py, px] += amp * fdt(om_s if k < 6 else om_g) * root * z
    f = _backward(m)
    for i in range(27):
        ix, iy, iz = i % 3, (i // 3) % 3, i // 9
        f[iz, iy, ix] = torch.roll(f[iz, iy, ix], (iz - 1, iy - 1, ix - 1), (0, 1, 2))
    return f


def _fields(f):
    """rho, j and Pi, (10, N)."""
    m = _forward(f)
    pick = [(0, 0, 0), (1, 0, 0), (0, 1, 0), (0, 0, 1)] + _DEG[:6]
    return torch.stack([m[d[2], d[1], d[0]].reshape(-1) for d in pick])


def _sums(f):
    v = _fields(f)
    d, j, pi = v[0] - 1.0, v[1:4], v[4:]
    u = j / v[0]
    return torch.cat([d.sum()[None], (d * d).sum()[None], j.sum(1), (j * j).sum(1), (u * u).sum(1), pi.sum(1),
                      (pi * pi).sum(1)])


def _shells(f):
    nz, ny, nx = f.shape[3:]
    k = [torch.fft.fftfreq(n, 1.0 / n, dtype=torch.float64, device=DEV) for n in (nz, ny, nx)]
    mod = torch.sqrt(k[0][:, None, None] ** 2 + k[1][None, :, None] ** 2 + k[2][None, None, :] ** 2)
    shell = torch.round(mod).to(torch.int64).reshape(-1)
    ns = int(round(math.sqrt((nx // 2) ** 2 + (ny // 2) ** 2 + (nz // 2) ** 2))) + 1
    counts = torch.bincount(shell, minlength=ns)
    counts[0] = 0
    spectra = {}
    for name, v in zip(rf.FIELDS, _fields(f)):
        p = torch.fft.fftn(v.view(nz, ny, nx)).abs().square().reshape(-1) / (nx * ny * nz)
        p[0] = 0.0
        s = torch.zeros(ns, dtype=torch.float64, device=DEV).index_add_(0, shell, p)
        spectra[name] = (s / counts.clamp(min=1)).cpu().numpy()
    return {"spectra": spectra, "counts": None}


def _f64(p, dims, rho, u, steps, sid=0, sums=None):
    f = _initial(dims, rho, u, p["kT"], p["seed"], sid)
    for t in range(steps):
        if sums is not None and t % sums["every"] == 0:
            sums["rows"].append(_sums(f))
        f = _advance(f, t, p, sid)
    return f


def exact(case, seed):
    c = case
    if c["kind"] == "batch":
        out, spent = [], 0
        for r in _replicas(c, seed):
            n = int(np.prod(r["dims"]))
            if len(out) >= 8:  # the first replicas stand for the rest
                out.append(None)
                continue
            p = dict(model="reg", kT=r["kT"], tau=r["tau"], tau_bulk=r["tau"], tau_ghost=1.0, seed=r["seed"])
            one = torch.ones(n, dtype=torch.float64, device=DEV)
            out.append(_fields(_f64(p, r["dims"], one, torch.zeros((3, n), dtype=torch.float64, device=DEV),
                                    c["steps"], r["stream_id"])))
        return out
    dims = (c["nx"], c["ny"], c["nz"])
    n = c["nx"] * c["ny"] * c["nz"]
    if n > 2 ** 25:
        return None
    kw = _params(c, seed)
    rho, u = _flow(dims, seed)
    if c["kind"] == "start":
        return _f64(kw, dims, rho, u, 0).reshape(27, n)
    if c["kind"] == "sk":
        return _shells(_f64(kw, dims, rho, u, c["steps"]))
    if c["kind"] == "restart":
        return _fields(_f64(kw, dims, rho, u, c["steps"] + 2))
    sums = dict(every=c["stats_every"], rows=[]) if c["stats_every"] else None
    f = _f64(kw, dims, rho, u, c["steps"], 0, sums)
    out = {"state": f.reshape(27, n) if c["out"] == "populations" else _fields(f)}
    if sums:
        v = sum(sums["rows"]).tolist()
        last = sums["rows"][-1].tolist()
        out["stats"] = dict(samples=None, nodes=None, sum_drho=v[0], sum_drho2=v[1], sum_j=v[2:5], sum_j2=v[5:8],
                            sum_u2=v[8:11], sum_pi=v[11:17], sum_pi2=v[17:23], mass_dev=last[0], momentum=last[2:5])
    return out
