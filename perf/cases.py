"""Measured workloads of the lattice library: what a preheating program has it do.

A case is a dict of plain values with a ``kind``:

* ``evolve``    one run: a segment of steps, then the diagnostics and the fields
                (whole arrays up to ``WHOLE`` site-fields, a fixed random sample
                of sites of every field beyond, where a program would not move
                gigabytes of FP64 to the host after every segment);
* ``ensemble``  many independent lattices in one pool: a few blocks of steps,
                then every member's diagnostics;
* ``start``     a new run from seeded initial conditions made on the device, up
                to the diagnostics of step 0;
* ``spectrum``  the power spectra of every field and derivative of a run.

Initial fields are a homogeneous inflaton near 1 plus Gaussian random
fluctuations with the vacuum-like spectrum the programs start from.
"""
import math

import numpy as np
import torch

from paper_0712_0813_amd import ce

KAPPA = 8.0 * math.pi * 0.342 ** 2   # 8 pi (phi_0/M_p)^2 at the end of inflation
AMP = 1e-3                           # fluctuation amplitude
WHOLE = 1 << 21                      # site-fields up to which an evolve case reads whole arrays
SAMPLE = 1 << 17                     # sites per field read otherwise
FROM_SEED = 1 << 27                  # site-fields from which the initial fields are made on the device
ON_CHIP = 128 << 20                  # bytes of state that 256 compute units can hold between steps

# A hybrid-like three-field polynomial model: quartic inflaton, two quadratic
# couplings, a trilinear and a sixth-order term, a mass.
POLY = ((0.25, (4, 0, 0)), (20.0, (2, 2, 0)), (15.0, (2, 0, 2)), (0.5, (1, 1, 1)),
        (0.02, (6, 0, 0)), (0.1, (0, 2, 0)))


def _evolve(name, dims, N, nf, dx, dt, steps, *, fp64=False, expansion=False, G1=100.0, G2=0.0, mu2=0.0,
            poly=False):
    return {"name": name, "kind": "evolve", "dims": dims, "N": N, "nf": nf, "dx": dx, "dt": dt, "steps": steps,
            "fp64": fp64, "expansion": expansion, "G1": G1, "G2": G2, "mu2": mu2, "poly": poly}


def listed():
    return [
        # the smallest run: a 1-D lattice in double precision, all launch latency
        _evolve("line_1024_fp64", 1, 1024, 2, 10 / 64, 0.01, 200, fp64=True, expansion=True),
        # an odd-sized plane with a user-defined three-field model
        _evolve("square_300_poly", 2, 300, 3, 10 / 64, 0.01, 200, poly=True),
        # the small static cube a program is first tried on
        _evolve("cube_32_static", 3, 32, 2, 10 / 32, 0.01, 500),
        # a cube no power of two, with a massive inflaton
        _evolve("cube_100_massive", 3, 100, 2, 10 / 64, 0.01, 200, mu2=0.1),
        # three fields in double precision
        _evolve("cube_64_3f_fp64", 3, 64, 3, 6 / 64, 0.01, 200, fp64=True, expansion=True, G1=30.0, G2=300.0),
        # ordinary serving jobs: a mid-sized cube and the largest plane of the mix
        _evolve("cube_128_expanding", 3, 128, 2, 10 / 64, 0.01, 300, expansion=True),
        _evolve("square_2048_expanding", 2, 2048, 2, 10 / 64, 0.01, 200, expansion=True),
        # a production cube, and the largest one, which fills tens of gigabytes
        _evolve("cube_256_expanding", 3, 256, 2, 20 / 256, 0.005, 150, expansion=True),
        _evolve("cube_1024_expanding", 3, 1024, 2, 40 / 1024, 0.005, 6, expansion=True, G1=1000.0),
        # a parameter scan: many small lattices advanced together in blocks
        {"name": "ensemble_256x64", "kind": "ensemble", "members": 256, "dims": 3, "N": 64, "nf": 2,
         "dx": 10 / 64, "dt": 0.01, "block": 50, "blocks": 2},
        # beginning a run of the production cube from a seed
        {"name": "start_256", "kind": "start", "dims": 3, "N": 256, "nf": 2, "dx": 20 / 256, "dt": 0.005,
         "fp64": False},
        # the output a run writes now and then: spectra of every field
        {"name": "spectrum_256", "kind": "spectrum", "dims": 3, "N": 256, "nf": 2, "dx": 20 / 256, "dt": 0.005,
         "fp64": False},
    ]


def _size(rng, low, high, multiple=4):
    """A lattice edge spread over the logarithm of its range."""
    n = math.exp(rng.uniform(math.log(low), math.log(high)))
    return max(low, min(high, int(round(n / multiple)) * multiple))


def draw(rng):
    kind = rng.choice(["evolve"] * 6 + ["ensemble", "start", "spectrum"])
    nf = rng.randint(1, 3)
    if kind == "evolve":
        dims = rng.choice([1, 2, 2, 3, 3, 3])
        if rng.random() < 0.5:   # powers of two, as most runs use
            N = 2 ** rng.randint({1: 6, 2: 5, 3: 4}[dims], {1: 16, 2: 12, 3: 9}[dims])
        else:
            N = _size(rng, {1: 64, 2: 32, 3: 16}[dims], {1: 65536, 2: 4096, 3: 320}[dims])
        poly = rng.random() < 0.2
        expansion = not poly and rng.random() < 0.5
        steps = int(max(10, min(300, 2e9 / (N ** dims * nf))))
        steps += rng.randint(0, 40) if steps > 60 else 0
        return {"kind": kind, "dims": dims, "N": N, "nf": 3 if poly else nf, "dx": rng.choice([10 / 64, 20 / 256]),
                "dt": rng.choice([0.01, 0.005]), "steps": steps, "fp64": rng.random() < 0.3, "expansion": expansion,
                "G1": round(10.0 ** rng.uniform(0, 3), 3), "G2": round(10.0 ** rng.uniform(0, 3), 3),
                "mu2": 0.0 if poly or expansion else rng.choice([0.0, 0.1]), "poly": poly}
    if kind == "ensemble":
        dims, N = rng.choice([(3, 32), (3, 64), (3, 128), (2, 256), (2, 512), (2, 1024)])
        members = max(2, min(256, int(rng.uniform(0.1, 1.0) * 1.3e8 / (N ** dims * nf))))
        return {"kind": kind, "members": members, "dims": dims, "N": N, "nf": nf, "dx": 10 / 64, "dt": 0.01,
                "block": rng.randint(20, 50), "blocks": 2}
    dims = rng.choice([2, 3, 3])
    N = 2 ** rng.randint(6, 11 if dims == 2 else 8)
    return {"kind": kind, "dims": dims, "N": N, "nf": nf, "dx": rng.choice([10 / 64, 20 / 256]),
            "dt": round(rng.uniform(0.004, 0.01), 4), "fp64": rng.random() < 0.3}


# ---- the model of a case ---------------------------------------------------

def _site_fields(case):
    return case["N"] ** case["dims"] * case["nf"]


def _members(case, seed):
    """(couplings G1, expansion flag, seed) of every member of an ensemble."""
    u = np.random.default_rng(seed + 3).random(case["members"])
    return [(float(10.0 ** (3.0 * u[j])), bool(j % 2), seed * 4096 + j) for j in range(case["members"])]


def _couplings(case):
    return [0.0, case.get("G1", 100.0), case.get("G2", 0.0) or 50.0]


def _m_eff2(case, G):
    if case.get("poly"):
        return [3.0 + 30 * 0.02, 40.0 + 0.2, 30.0]
    m = [3.0 + case.get("mu2", 0.0)] + [G[j] for j in (1, 2)]
    return m[:case["nf"]]


def _params(case, G=None, expansion=None):
    nf = case["nf"]
    exp = case.get("expansion", True) if expansion is None else expansion
    kw = dict(expansion=exp, kappa=KAPPA if exp else 0.0,
              precision=ce.CE_FP64 if case.get("fp64") else ce.CE_FP32)
    if case.get("poly"):
        kw.update(lam=0.0, terms=POLY)
    else:
        G = _couplings(case) if G is None else G
        kw.update(G=G[:nf], mu2=(case.get("mu2", 0.0), 0.0, 0.0))
    return (case["dims"], case["N"], nf, case["N"] * case["dx"], case["dt"]), kw


def _fields(case, seed):
    """Initial (phi, phidot): FP64 arrays on the GPU, [nf, N, ...]."""
    dims, N, nf = case["dims"], case["N"], case["nf"]
    L = N * case["dx"]
    gen = torch.Generator(device="cuda").manual_seed(seed + 17)
    k2 = torch.zeros((1,) * dims, dtype=torch.float64, device="cuda")
    for d in range(dims):
        last = d == dims - 1
        n = torch.fft.rfftfreq(N, 1.0 / N, dtype=torch.float64, device="cuda") if last else \
            torch.fft.fftfreq(N, 1.0 / N, dtype=torch.float64, device="cuda")
        shape = [1] * dims
        shape[d] = n.numel()
        k2 = k2 + (n * n).reshape(shape)
    inside = ((k2 > 0) & (k2 <= (N // 4) ** 2)).double()
    phi = torch.empty((nf,) + (N,) * dims, dtype=torch.float64, device="cuda")
    pid = torch.empty_like(phi)
    for i, m2 in enumerate(_m_eff2(case, _couplings(case))):
        omega = torch.sqrt(k2 * (2 * math.pi / L) ** 2 + m2)
        for out, sigma in ((phi, AMP / torch.sqrt(2 * omega * L ** dims)),
                           (pid, AMP * torch.sqrt(omega / 2) / math.sqrt(L ** dims))):
            w = torch.randn((N,) * dims, dtype=torch.float64, device="cuda", generator=gen)
            out[i] = torch.fft.irfftn(torch.fft.rfftn(w) * (sigma * inside), s=(N,) * dims) * N ** (dims / 2)
    phi[0] += 1.0
    return phi, pid


def _sites(case):
    n = case["N"] ** case["dims"]
    return np.random.default_rng(5).integers(0, n, min(SAMPLE, n // 64), dtype=np.int64)


def _spec(case, seed, G):
    return ce.make_init_spec(seed, _m_eff2(case, G), AMP)


# ---- what a program has, and one pass --------------------------------------

def prepare(case, seed):
    if case["kind"] == "ensemble":
        pool = ce.Pool(64 << 30)
        jobs = []
        for G1, exp, s in _members(case, seed):
            G = [0.0, G1, 50.0]
            a, kw = _params(case, G, exp)
            jobs.append(pool.admit_generated(ce.make_params(*a, **kw), _spec(case, s, G), 1 << 40))
        return {"case": case, "pool": pool, "jobs": jobs}
    a, kw = _params(case)
    if case["kind"] == "start":
        return {"case": case, "params": (a, kw), "spec": _spec(case, seed, _couplings(case)),
                "sites": _sites(case)}
    sim = ce.Simulation(*a, **kw)
    if _site_fields(case) >= FROM_SEED:
        sim.generate(_spec(case, seed, _couplings(case)))
    else:
        phi, pid = _fields(case, seed)
        sim.load(phi.cpu().numpy(), pid.cpu().numpy())
    sim.sync()
    return {"case": case, "sim": sim, "sites": _sites(case)}


_ENERGY = np.dtype([("step", "i8"), ("v", "f8", 18), ("residual", "f8"), ("nonfinite", "i4"), ("pad", "i4")])


def _numbers(e):
    """tau, a, a', hubble, kin[3], grad[3], pot, rho, mean[3], mean_sq[3] of a diagnostics record."""
    return np.frombuffer(e, _ENERGY)["v"][0]


def run(state):
    case = state["case"]
    if case["kind"] == "ensemble":
        pool = state["pool"]
        for _ in range(case["blocks"]):
            pool.run_block(case["block"])
        return np.stack([_numbers(pool.poll(j)[1]) for j in state["jobs"]])
    if case["kind"] == "start":
        a, kw = state["params"]
        with ce.Simulation(*a, **kw) as sim:
            sim.generate(state["spec"])
            return {"energy": _numbers(sim.energies()),
                    "sites": [sim.read_sites(i, state["sites"]) for i in range(case["nf"])]}
    sim = state["sim"]
    if case["kind"] == "spectrum":
        return [sim.spectrum(i) for i in range(case["nf"])]
    sim.step(case["steps"])
    out = {"energy": _numbers(sim.energies())}
    if _site_fields(case) <= WHOLE:
        out["f"], out["fdot"] = sim.read()
    else:
        out["sites"] = [sim.read_sites(i, state["sites"]) for i in range(case["nf"])]
    return out


def work(case):
    """Per site-field of one pass: the state (field and derivative) read and
    written, once for a state that fits on the chip and once per step for a
    larger one; about 30 flops a step.  Transforms: each array read once."""
    nsf = _site_fields(case) * case.get("members", 1)
    elem = 8 if case.get("fp64") else 4
    if case["kind"] == "start":
        return {"bytes": 3.0 * elem * nsf,     # both arrays written, read by the first half step's sums
                "flops": 2 * nsf * 5.0 * math.log2(case["N"] ** case["dims"])}
    if case["kind"] == "spectrum":
        return {"bytes": 2.0 * elem * nsf, "flops": 2 * nsf * 2.5 * math.log2(case["N"] ** case["dims"])}
    steps = case["steps"] if case["kind"] == "evolve" else case["block"] * case["blocks"]
    state = 2 * elem * _site_fields(case)   # one lattice: members are independent
    return {"bytes": 4.0 * elem * nsf * (1 if state <= ON_CHIP else steps), "flops": 30.0 * nsf * steps}


# ---- the same in 64 bits ---------------------------------------------------

def _lap(f, dims, inv_dx2):
    out = f * (-2.0 * dims)
    for d in range(1, dims + 1):
        out += torch.roll(f, 1, -d)
        out += torch.roll(f, -1, -d)
    return out.mul_(inv_dx2)


def _potential(case, f, G, a):
    """(V, dV/df_i) per site in the program variables; f: list of fields, a: scale factor (broadcastable)."""
    nf = len(f)
    if case.get("poly"):
        V, dV = torch.zeros_like(f[0]), [torch.zeros_like(x) for x in f]
        for coef, e in POLY:
            c = coef * a ** (4 - sum(e))
            p = [f[i] ** e[i] for i in range(nf)]
            V += c * p[0] * p[1] * p[2]
            for i in range(nf):
                if e[i]:
                    q = e[i] * f[i] ** (e[i] - 1)
                    for j in range(nf):
                        if j != i:
                            q = q * p[j]
                    dV[i] += c * q
        return V, dV
    f0s = f[0] * f[0]
    V = 0.25 * f0s * f0s
    chi2 = torch.zeros((), dtype=torch.float64, device=f[0].device)
    dV = [None] * nf
    for j in range(1, nf):
        t = G[j] * f[j] * f[j]
        chi2 = chi2 + t
        V = V + 0.5 * f0s * t
        dV[j] = G[j] * f0s * f[j]
    dV[0] = f0s * f[0] + f[0] * chi2
    if case.get("mu2", 0.0):
        m = case["mu2"] * a * a
        V = V + 0.5 * m * f0s
        dV[0] = dV[0] + m * f[0]
    return V, dV


def _leapfrog(case, phi, pid, G, expansion, steps):
    """The staggered leapfrog in FP64 over a batch of lattices: fields are lists
    of [B, N, ...] tensors, G and expansion per lattice.  Returns the
    diagnostics [B, 18], the fields at the last step and the derivatives half a
    step later."""
    dims, dt = case["dims"], case["dt"]
    inv_dx2 = 1.0 / case["dx"] ** 2
    f = list(phi)
    B = f[0].shape[0]
    axes = tuple(range(1, dims + 1))
    per = lambda v: v.reshape((B,) + (1,) * dims)   # noqa: E731
    mean = lambda x: x.mean(dim=axes)               # noqa: E731
    ex = torch.as_tensor(expansion, dtype=torch.float64, device=f[0].device)
    Gs = [per(torch.as_tensor(g, dtype=torch.float64, device=f[0].device).expand(B)) for g in G]
    one = torch.ones(B, dtype=torch.float64, device=f[0].device)
    nf = len(f)
    zero = torch.zeros_like(one)

    def record(tau, a, adot, kin, grad, pot, rho):
        pad = lambda v: v + [zero] * (3 - len(v))   # noqa: E731
        return torch.stack([one * tau, a, adot, adot / (a * a)] + pad(kin) + pad(grad) + [pot, rho]
                           + pad([mean(x) for x in f]) + pad([mean(x * x) for x in f]), dim=1)

    a = one.clone()
    lap = [_lap(x, dims, inv_dx2) for x in f]
    V, dV = _potential(case, f, Gs, per(a))
    kin = [0.5 * mean(p * p) for p in pid]
    grad = [-0.5 * mean(f[i] * lap[i]) for i in range(nf)]
    pot = mean(V)
    rho = sum(kin) + sum(grad) + pot
    ap = torch.sqrt(KAPPA * rho / 3.0) * ex
    app = (-ap * ap + KAPPA * (2.0 / 3.0 * sum(grad) + pot)) * ex
    rec = record(0.0, a, ap, kin, grad, pot, rho)
    pi = [pid[i] + per(ap) * f[i] + 0.5 * dt * (lap[i] - dV[i] + per(app) * f[i]) for i in range(nf)]
    y = ap + 0.5 * dt * app
    for n in range(1, steps + 1):
        for i in range(nf):
            f[i] = f[i] + dt * pi[i]
        a = a + dt * y * ex
        lap = [_lap(x, dims, inv_dx2) for x in f]
        V, dV = _potential(case, f, Gs, per(a))
        pot = mean(V)
        grad = [-0.5 * mean(f[i] * lap[i]) for i in range(nf)]
        S = KAPPA * (2.0 / 3.0 * sum(grad) + pot) / a
        A, Bq, C = dt / (4 * a), 1 + dt * y / (2 * a), dt * y * y / (4 * a) - y - dt * S
        x = -2 * C / (Bq + torch.sqrt(Bq * Bq - 4 * A * C)) * ex
        abar = 0.5 * (x + y)
        c = (S - abar * abar / a) / a * ex
        new = [pi[i] + dt * (lap[i] - dV[i] + per(c) * f[i]) for i in range(nf)]
        if n == steps:
            kin = [0.5 * mean((0.5 * (new[i] + pi[i]) - per(abar / a) * f[i]) ** 2) for i in range(nf)]
            rec = record(n * dt, a, abar, kin, grad, pot, sum(kin) + sum(grad) + pot)
        pi, y = new, x
    return rec, f, pi


def _umulhi(a, b):
    """High 64 bits of the unsigned product of an int64 tensor (as bits) and a Python integer."""
    mask = 0xFFFFFFFF
    a0, a1 = a & mask, (a >> 32) & mask
    b0, b1 = b & mask, b >> 32
    p00, p01, p10 = a0 * b0, a0 * b1, a1 * b0
    mid = ((p00 >> 32) & mask) + (p01 & mask) + (p10 & mask)
    return a1 * b1 + ((p01 >> 32) & mask) + ((p10 >> 32) & mask) + (mid >> 32)


def _signed(v):
    return v - (1 << 64) if v >= 1 << 63 else v


def _philox(ctr0, ctr1, seed):
    """First two words of Philox4x64-10 with key (seed, 0), counter (ctr0, ctr1, 0, 0), as int64 bits."""
    M0, M1 = 0xD2E7470EE14C6C93, 0xCA5A826395121157
    W0, W1 = 0x9E3779B97F4A7C15, 0xBB67AE8584CAA73B
    z = torch.zeros_like(ctr0)
    c = [ctr0, z + ctr1, z, z]
    k0, k1 = seed, 0
    for r in range(10):
        if r:
            k0, k1 = (k0 + W0) % (1 << 64), (k1 + W1) % (1 << 64)
        h0, l0 = _umulhi(c[0], M0), c[0] * _signed(M0)
        h1, l1 = _umulhi(c[2], M1), c[2] * _signed(M1)
        c = [h1 ^ c[1] ^ _signed(k0), l1, h0 ^ c[3] ^ _signed(k1), l0]
    return c[0], c[1]


def _generated(case, seed, G):
    """The seeded initial fields as the library's header defines them, FP64 on the GPU: [nf, N, ...] each."""
    dims, N, nf = case["dims"], case["N"], case["nf"]
    K, L = N // 4, N * case["dx"]
    r = torch.arange(-K, K + 1, dtype=torch.int64, device="cuda")
    n2 = torch.zeros((1,) * dims, dtype=torch.int64, device="cuda")
    b = torch.zeros((1,) * dims, dtype=torch.int64, device="cuda")
    for d in range(dims):
        shape = [1] * dims
        shape[d] = 2 * K + 1
        n2 = n2 + (r * r).reshape(shape)
        b = b * (2 * K + 1) + (r + K).reshape(shape)
    inside = ((n2 > 0) & (n2 <= K * K)).double()
    k2 = n2.double() * (2 * math.pi / L) ** 2
    out = []
    for kind in range(2):
        arr = torch.empty((nf,) + (N,) * dims, dtype=torch.float64, device="cuda")
        for i, m2 in enumerate(_m_eff2(case, G)):
            w0, w1 = _philox(b, 2 * i + kind, seed)
            u1 = (((w0 >> 11) & ((1 << 53) - 1)) + 1).double() * 2.0 ** -53
            u2 = ((w1 >> 11) & ((1 << 53) - 1)).double() * 2.0 ** -53
            omega = torch.sqrt(k2 + m2)
            s = AMP / torch.sqrt(2 * omega * L ** dims) if kind == 0 else AMP * torch.sqrt(omega / 2) / math.sqrt(L ** dims)
            c = torch.polar(s * inside * torch.sqrt(-2 * torch.log(u1)), 2 * math.pi * u2)
            full = torch.zeros((N,) * dims, dtype=torch.complex128, device="cuda")
            idx = (r % N)
            full[torch.meshgrid(*([idx] * dims), indexing="ij")] = c
            arr[i] = torch.fft.ifftn(full, norm="forward").real
            del full, c
        out.append(arr)
    out[0][0] += 1.0
    return out


def exact(case, seed):
    if case["kind"] == "ensemble":
        jobs = _members(case, seed)
        gens = [_generated(case, s, [0.0, G1, 50.0]) for G1, _, s in jobs]
        phi = [torch.stack([g[0][i] for g in gens]) for i in range(case["nf"])]
        pid = [torch.stack([g[1][i] for g in gens]) for i in range(case["nf"])]
        del gens
        G = [0.0, [j[0] for j in jobs], 50.0]
        rec, _, _ = _leapfrog(case, phi, pid, G, [float(j[1]) for j in jobs], case["block"] * case["blocks"])
        return rec.cpu().numpy()
    nsf = _site_fields(case)
    if nsf > 1 << 30:
        return None     # tens of gigabytes per temporary
    G = _couplings(case)
    seeded = case["kind"] == "start" or nsf >= FROM_SEED
    phi, pid = _generated(case, seed, G) if seeded else _fields(case, seed)
    steps = case.get("steps", 0)
    ex = [float(bool(case.get("expansion", True)))]
    rec, f, pi = _leapfrog(case, [x[None] for x in phi], [x[None] for x in pid], G, ex, steps)
    if case["kind"] == "spectrum":
        return [_spectrum(case, f[i][0], pi[i][0]) for i in range(case["nf"])]
    out = {"energy": rec[0].cpu().numpy()}
    f, pi = torch.stack([x[0] for x in f]), torch.stack([x[0] for x in pi])
    if case["kind"] == "evolve" and nsf <= WHOLE:
        out["f"], out["fdot"] = f.cpu().numpy(), pi.cpu().numpy()
    else:
        s = torch.from_numpy(_sites(case)).cuda()
        out["sites"] = [(f[i].reshape(-1)[s].cpu().numpy(), pi[i].reshape(-1)[s].cpu().numpy())
                        for i in range(case["nf"])]
    return out


def _spectrum(case, f, pi):
    dims, N = case["dims"], case["N"]
    n2 = torch.zeros((1,) * dims, dtype=torch.int64, device="cuda")
    r = torch.arange(N, dtype=torch.int64, device="cuda")
    r = torch.where(r < N // 2, r, r - N)
    for d in range(dims):
        shape = [1] * dims
        shape[d] = N
        n2 = n2 + (r * r).reshape(shape)
    key = torch.sqrt(n2.double()).floor().long()
    key = torch.where(key * key > n2, key - 1, key).reshape(-1)
    nb = math.isqrt(dims * (N // 2) ** 2) + 1
    out = []
    for g in (f, pi):
        power = torch.fft.fftn(g, norm="forward").abs().square().reshape(-1)
        out.append(torch.bincount(key, weights=power, minlength=nb).cpu().numpy())
    return out[0], out[1], torch.bincount(key, minlength=nb).double().cpu().numpy()

