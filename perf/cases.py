"""The library's measured work: what a program built on it has it do, through the public Python calls.

Each case is one call, or the short chain of calls that always go together, on a cubic grid:

  noalloc      collapse times through the allocation-free entry point (graph capture, tight loops)
  collapse     collapse times of a given spectrum over a list of smoothing radii
  velocity     collapse times with v_max, the input of the fragmentation
  displacement Zel'dovich, 2LPT and 3LPT displacement fields of a given spectrum
  realization  seeded field, collapse times, Zel'dovich and 2LPT: what the benchmark and a served
               request run
  halos        fragmentation of collapsed particles, its catalogue and its merger history
  redshift     collapse redshift of every grid point

Sizes, boxes, radius counts and precisions are those of the benchmark's and the serving trace's
workloads and of the parity tests; spectra are BBKS with sigma_8 = 0.8 on 1.5 to 4 Mpc/h cells.
"""

import math

import numpy as np
import torch

from paper_1305_1505_amd import binding as pin

SIGMA8, GAMMA, NS = 0.8, 0.21, 1.0
OMEGA_M = 0.25


def _case(name, kind, n, prec, n_radii, r_max, cell):
    return {"name": name, "kind": kind, "n": n, "prec": prec, "n_radii": n_radii, "r_max": r_max, "r_min": 0.75,
            "cell": cell}


def listed():
    return [
        # the smallest call: a small grid in a latency-bound loop that must not allocate
        _case("noalloc_32", "noalloc", 32, "fp32", 8, 4.0, 2.0),
        # test-size realization on the float64 path, 100 Mpc/h box
        _case("collapse_64_fp64", "collapse", 64, "fp64", 16, 20.0, 1.5625),
        # the smallest grid of the serving trace
        _case("collapse_128", "collapse", 128, "fp32", 32, 60.0, 2.0),
        # medium workload, 500 Mpc/h box
        _case("collapse_256", "collapse", 256, "fp32", 30, 60.0, 1.953125),
        # serving-trace grid whose size is not a power of two
        _case("collapse_384", "collapse", 384, "fp32", 32, 60.0, 2.0),
        # the largest workload, 3072 Mpc/h box, not a power of two
        _case("collapse_768", "collapse", 768, "fp32", 45, 60.0, 4.0),
        # the benchmark's grid on the float64 path
        _case("collapse_512_fp64", "collapse", 512, "fp64", 40, 60.0, 1.953125),
        # the benchmark's step: field, collapse times, Zel'dovich and 2LPT
        _case("realization_512", "realization", 512, "fp32", 40, 60.0, 1.953125),
        # collapse times with v_max ahead of a fragmentation
        _case("velocity_256", "velocity", 256, "fp32", 30, 60.0, 1.953125),
        # initial conditions: all three orders of the displacement
        _case("displacement_256", "displacement", 256, "fp32", 1, 1.0, 2.0),
        # halo finding on the collapsed particles at z = 0
        _case("halos_256", "halos", 256, "fp32", 30, 60.0, 1.953125),
        # collapse redshifts of a whole grid
        _case("redshift_256", "redshift", 256, "fp32", 30, 60.0, 1.953125),
    ]


# sizes drawn per kind; the most radii keep a drawn case below the largest listed one
_SIZES = {
    "noalloc": ((12, 16, 24, 32, 48, 64, 96, 128), (12, 16, 24, 32, 48, 64, 96)),
    "collapse": ((16, 24, 32, 48, 64, 96, 128, 192, 256, 384, 512, 768), (24, 48, 64, 96, 128, 192, 256, 384, 512)),
    "velocity": ((64, 96, 128, 192, 256, 384), (64, 96, 128, 192, 256)),
    "displacement": ((64, 96, 128, 192, 256, 384, 512), (64, 96, 128, 192, 256, 384)),
    "realization": ((64, 128, 192, 256, 384, 512), (64, 96, 128, 192, 256)),
    "halos": ((64, 96, 128, 192, 256), (64, 96, 128)),
    "redshift": ((64, 128, 192, 256, 384), (64, 128, 192, 256)),
}


def draw(rng):
    kind = rng.choice(["noalloc", "collapse", "collapse", "collapse", "velocity", "displacement", "realization",
                       "halos", "redshift"])
    prec = rng.choice(["fp32", "fp32", "fp64"])
    n = rng.choice(_SIZES[kind][prec == "fp64"])
    n_radii = 1 if kind == "displacement" else rng.randint(3, 45)
    r_max = min(60.0, n / 4) * rng.uniform(0.5, 1.0)
    case = _case("", kind, n, prec, n_radii, r_max, round(rng.uniform(1.5, 4.0), 3))
    del case["name"]
    return case


def _radii(case):
    if case["n_radii"] == 1:
        return [case["r_max"]]
    return [float(r) for r in np.geomspace(case["r_max"], case["r_min"], case["n_radii"])]


def _power(k):
    """BBKS P(k) without its amplitude, k in h/Mpc (numpy or torch)."""
    log1p = torch.log1p if isinstance(k, torch.Tensor) else np.log1p
    q = k / GAMMA
    t = log1p(2.34 * q) / (2.34 * q)
    t = t * (1 + 3.89 * q + (16.1 * q) ** 2 + (5.46 * q) ** 3 + (6.71 * q) ** 4) ** -0.25
    return k ** NS * t * t


def _frequencies(n):
    f = torch.fft.fftfreq(n, 1.0 / n, dtype=torch.float64, device="cuda")
    return f.view(n, 1, 1), f.view(1, n, 1), torch.arange(n // 2 + 1, dtype=torch.float64, device="cuda").view(1, 1, -1)


def _spectrum(case, seed):
    """A Gaussian half spectrum of the linear density field at z = 0, in the plan's precision."""
    n, box = case["n"], case["n"] * case["cell"]
    lnk = np.linspace(math.log(1e-5), math.log(1e2), 20001)
    k = np.exp(lnk)
    w = 3 * (np.sin(8 * k) - 8 * k * np.cos(8 * k)) / (8 * k) ** 3
    sigma2 = np.sum(k ** 3 * _power(k) * w * w) * (lnk[1] - lnk[0]) / (2 * math.pi ** 2)
    amplitude = SIGMA8 ** 2 / sigma2 * float(n) ** 6 / (2 * box ** 3)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    real = torch.float64 if case["prec"] == "fp64" else torch.float32
    modes = torch.randn((n, n, n // 2 + 1, 2), generator=gen, dtype=real, device="cuda")
    modes = torch.view_as_complex(modes)
    plane = modes[:, :, 0]      # the kz = 0 plane of a real field is its own conjugate under k -> -k
    modes[:, :, 0] = (plane + torch.roll(torch.flip(plane, (0, 1)), (1, 1), (0, 1)).conj()) / math.sqrt(2)
    fx, fy, fz = _frequencies(n)
    for x in range(n):          # by planes: no float64 temporaries of the whole grid
        kk = (2 * math.pi / box) * torch.sqrt(fx[x] ** 2 + fy[0] ** 2 + fz[0] ** 2)
        modes[x] *= torch.sqrt(amplitude * _power(kk.clamp_min(1e-30))).to(real)
    modes[0, 0, 0] = 0
    modes[:, :, n // 2] = 0
    modes[n // 2] = 0
    modes[:, n // 2] = 0
    return modes


class State:
    pass


def prepare(case, seed):
    s = State()
    s.case, s.seed = case, seed
    n, kind = case["n"], case["kind"]
    prec = pin.PIN_FP64 if case["prec"] == "fp64" else pin.PIN_FP32
    box, radii = n * case["cell"], _radii(case)
    if kind == "noalloc":
        real = torch.float64 if case["prec"] == "fp64" else torch.float32
        s.desc = pin.make_desc(n, box, radii, SIGMA8, GAMMA, NS, prec)
        s.dk = _spectrum(case, seed)
        s.F = torch.empty((n, n, n), dtype=real, device="cuda")
        s.ridx = torch.empty((n, n, n), dtype=torch.uint8, device="cuda")
        return s
    s.plan = pin.Plan(n, box, radii, sigma8=SIGMA8, gamma=GAMMA, ns=NS, prec=prec)
    if kind == "realization":
        return s
    s.dk = _spectrum(case, seed)
    if kind == "halos":
        s.F, _, s.vmax = s.plan.collapse_times_v(s.dk)
        s.dk = None
        s.capacity = n ** 3 // 8        # halos and mergers that the program's buffers can take
        cap = s.capacity
        s.ids, s.members = (torch.zeros(cap, dtype=torch.int32, device="cuda") for _ in range(2))
        s.centre, s.disp = (torch.zeros((3, cap), dtype=torch.float64, device="cuda") for _ in range(2))
        s.merger_f = torch.zeros(cap, dtype=torch.float64, device="cuda")
        s.merger = [torch.zeros(cap, dtype=torch.int32, device="cuda") for _ in range(4)]
    elif kind == "redshift":
        s.plan.set_growth(OMEGA_M)
        s.F, _ = s.plan.collapse_times(s.dk)
        s.dk = None
    return s


def run(s):
    kind = s.case["kind"]
    if kind == "noalloc":
        pin.pin_collapse_times_noalloc(s.desc, s.dk.data_ptr(), s.F.data_ptr(), s.ridx.data_ptr(),
                                       torch.cuda.current_stream().cuda_stream)
        return {"F": s.F, "ridx": s.ridx}
    plan = s.plan
    if kind == "collapse":
        F, ridx = plan.collapse_times(s.dk)
        return {"F": F, "ridx": ridx}
    if kind == "velocity":
        F, ridx, vmax = plan.collapse_times_v(s.dk)
        return {"F": F, "ridx": ridx, "vmax": vmax}
    if kind == "displacement":
        psi1, psi2 = plan.displacements(s.dk)
        return {"psi1": psi1, "psi2": psi2, "psi3": plan.lpt3_displacement(s.dk)}
    if kind == "realization":
        dk = plan.generate_field(s.seed)
        F, ridx = plan.collapse_times(dk)
        psi1, psi2 = plan.displacements(dk)
        return {"dk": dk, "F": F, "ridx": ridx, "psi1": psi1, "psi2": psi2}
    if kind == "halos":
        stream = torch.cuda.current_stream().cuda_stream
        label, sizes, count = plan.fragment(s.F, s.vmax)
        pin.pin_fragment_catalog(plan.handle, s.ids.data_ptr(), s.members.data_ptr(), s.centre.data_ptr(),
                                 s.disp.data_ptr(), s.capacity, stream)
        mergers = pin.pin_fragment_mergers(plan.handle, s.merger_f.data_ptr(), *[m.data_ptr() for m in s.merger],
                                           s.capacity, stream)
        return {"label": label, "sizes": sizes, "count": count, "ids": s.ids, "members": s.members,
                "centre": s.centre, "disp": s.disp, "mergers": mergers, "merger_f": s.merger_f, "merger": s.merger}
    return {"z": plan.collapse_redshift(s.F)}


def work(case):
    n, kind = case["n"], case["kind"]
    vol = float(n) ** 3
    rb = 8 if case["prec"] == "fp64" else 4
    spectrum = n * n * (n // 2 + 1) * 2.0 * rb
    fft = 2.5 * vol * math.log2(vol)            # one real transform of the grid
    point = 150.0                               # one point's collapse model
    radius = 6 * fft + 30.0 * vol + point * vol
    if kind in ("noalloc", "collapse"):
        return {"bytes": spectrum + vol * (rb + 1), "flops": case["n_radii"] * radius}
    if kind == "velocity":
        return {"bytes": spectrum + vol * (4 * rb + 1), "flops": case["n_radii"] * (radius + 3 * fft)}
    if kind == "displacement":
        # psi1; the tensor, its source and psi2; both tensors, five sources and psi3
        return {"bytes": spectrum + vol * 9 * rb, "flops": fft * (3 + 10 + 12 + 5 + 3) + 100.0 * vol}
    if kind == "realization":
        return {"bytes": spectrum + vol * (7 * rb + 1), "flops": case["n_radii"] * radius + 13 * fft + 100.0 * vol}
    if kind == "halos":
        return {"bytes": vol * (4 * rb + 8), "flops": 50.0 * vol}
    return {"bytes": 2 * vol * rb, "flops": 60.0 * vol}


# ---- the same results in 64 bits, by plain numpy and torch ------------------------------------

def _field(modes):
    n = modes.shape[0]
    return torch.fft.irfftn(modes, s=(n, n, n))


def _collapse_points(t6):
    """Inverse collapse times of a [6, m] array of tensors (xx, xy, xz, yy, yz, zz)."""
    xx, xy, xz, yy, yz, zz = t6
    m = np.stack([np.stack([xx, xy, xz], -1), np.stack([xy, yy, yz], -1), np.stack([xz, yz, zz], -1)], -2)
    lam = np.linalg.eigvalsh(m)
    l1, l2, l3 = lam[:, 2], lam[:, 1], lam[:, 0]
    delta, mu2, mu3 = l1 + l2 + l3, l1 * l2 + l1 * l3 + l2 * l3, l1 * l2 * l3
    a, b, c = -l1, -mu2 / 7, mu3 / 9 - 10 * delta * mu2 / 189
    # largest real root of F^3 + a F^2 + b F + c
    p, q = b / 3 - a * a / 9, c / 2 - a * b / 6 + a ** 3 / 27
    disc = q * q + p ** 3
    r = np.sqrt(np.maximum(-p, 1e-300))
    three = 2 * r * np.cos(np.arccos(np.clip(-q / r ** 3, -1, 1)) / 3)
    u = np.cbrt(-q - np.copysign(np.sqrt(np.maximum(disc, 0)), q))
    one = np.where(u != 0, u - p / np.where(u != 0, u, 1), 0)
    x = np.where(disc < 0, three, one) - a / 3
    for _ in range(3):
        d = (3 * x + 2 * a) * x + b
        x = np.where(d > 0, x - (((x + a) * x + b) * x + c) / np.where(d > 0, d, 1), x)
    root = np.maximum(x, 0)
    x3 = 2.0
    for _ in range(60):
        x3 -= (1 - x3 / 3 - x3 ** 2 / 21 - 23 * x3 ** 3 / 1701) / (-1 / 3 - 2 * x3 / 21 - 69 * x3 ** 2 / 1701)
    gain = x3 / (0.15 * (12 * math.pi) ** (2 / 3)) - 1
    dev = np.sqrt(((l1 - l2) ** 2 + (l2 - l3) ** 2 + (l3 - l1) ** 2) / 18)
    s = np.where(delta > 0, np.clip(1 - 3 * dev / np.where(delta > 0, delta, 1), 0, 1), 0)
    return root * (1 + gain * s)


def _exact_collapse(case, seed):
    n = case["n"]
    dk = _spectrum(case, seed).to(torch.complex128)
    f = _frequencies(n)
    f2 = f[0] ** 2 + f[1] ** 2 + f[2] ** 2
    base = dk / f2.clamp_min(1)
    F = np.zeros(n ** 3)
    for r in _radii(case):
        g = base * torch.exp(-0.5 * f2 * (2 * math.pi * r / n) ** 2)
        t6 = [_field(g * f[i] * f[j]).reshape(-1).cpu().numpy()
              for i, j in ((0, 0), (0, 1), (0, 2), (1, 1), (1, 2), (2, 2))]
        F = np.maximum(F, _collapse_points(np.stack(t6)))
    return torch.from_numpy(F.reshape(n, n, n))


def _exact_displacements(case, seed):
    n = case["n"]
    length = n * case["cell"] / (2 * math.pi)
    dk = _spectrum(case, seed).to(torch.complex128)
    f = _frequencies(n)
    f2 = f[0] ** 2 + f[1] ** 2 + f[2] ** 2
    inv = 1 / f2.clamp_min(1)
    inv[0, 0, 0] = 0
    inv[n // 2] = 0
    inv[:, n // 2] = 0
    inv[:, :, n // 2] = 0

    def gradient(source, scale):
        return torch.stack([_field(1j * scale * f[a] * inv * source) for a in range(3)])

    def tensor(source):
        return {(i, j): _field(f[i] * f[j] * inv * source) for i in range(3) for j in range(i, 3)}

    def entry(t, i, j):
        return t[min(i, j), max(i, j)]

    psi1 = gradient(dk, length)
    a = tensor(dk)
    mu2 = (a[0, 0] * a[1, 1] + a[0, 0] * a[2, 2] + a[1, 1] * a[2, 2] - a[0, 1] ** 2 - a[0, 2] ** 2 - a[1, 2] ** 2)
    source2 = torch.fft.rfftn(mu2)
    psi2 = gradient(source2, 3 * length / 7)
    b = tensor(source2)
    det = (a[0, 0] * (a[1, 1] * a[2, 2] - a[1, 2] ** 2) - a[0, 1] * (a[0, 1] * a[2, 2] - a[1, 2] * a[0, 2])
           + a[0, 2] * (a[0, 1] * a[1, 2] - a[1, 1] * a[0, 2]))
    product = sum(entry(a, i, j) * entry(b, i, j) for i in range(3) for j in range(3))
    mixed = 0.5 * ((a[0, 0] + a[1, 1] + a[2, 2]) * (b[0, 0] + b[1, 1] + b[2, 2]) - product)
    s = torch.fft.rfftn(det / 3 - 10 / 21 * mixed)
    curl = []
    for i in range(3):
        j, k = (i + 1) % 3, (i + 2) % 3
        ab = sum(entry(a, j, m) * entry(b, m, k) - entry(a, k, m) * entry(b, m, j) for m in range(3))
        curl.append(torch.fft.rfftn(ab / 7))
    psi3 = torch.stack([_field(1j * length * inv * (-f[i] * s + f[(i + 1) % 3] * curl[(i + 2) % 3]
                                                    - f[(i + 2) % 3] * curl[(i + 1) % 3])) for i in range(3)])
    return {"psi1": psi1, "psi2": psi2, "psi3": psi3}


def _exact_redshift(case, seed):
    """z with D(z) = 1/F, D the growing mode of flat LCDM, from the library's own F as its input."""
    s = prepare(case, seed)
    f = s.F.reshape(-1).cpu().numpy().astype(np.float64)
    shape = tuple(s.F.shape)
    s.plan.close()
    lam = (1 - OMEGA_M) / OMEGA_M
    y = np.linspace(math.log(1e-5), math.log(1e6), 400001)
    h = y[1] - y[0]
    node, weight = np.polynomial.legendre.leggauss(6)

    def integrand(ln_a):                       # d(a)/(a E)^3 per d(ln a), E^2 in units of Omega_m / a^3
        a = np.exp(ln_a)
        return a ** 2.5 / (1 + lam * a ** 3) ** 1.5

    step = sum(w * integrand(y[:-1] + 0.5 * h * (1 + t)) for t, w in zip(node, weight)) * 0.5 * h
    a0 = math.exp(y[0])
    total = np.concatenate([[0.4 * a0 ** 2.5], 0.4 * a0 ** 2.5 + np.cumsum(step)])
    hub = np.sqrt(np.exp(-3 * y) + lam)
    d = hub * total
    today = np.interp(0.0, y, np.log(d))
    d /= math.exp(today)
    dd = d * (-1.5 * np.exp(-3 * y) / hub ** 2) + hub * integrand(y) / math.exp(today)
    z = np.full(f.shape, -1.0)
    ok = (f > 0) & (1 / np.where(f > 0, f, 1) < d[-1])
    t = 1 / f[ok]
    k = np.clip(np.searchsorted(d, t) - 1, 0, len(y) - 2)
    x = (t - d[k]) / (d[k + 1] - d[k])
    for _ in range(4):
        hv = ((2 * x ** 3 - 3 * x ** 2 + 1) * d[k] + (x ** 3 - 2 * x ** 2 + x) * h * dd[k]
              + (3 * x ** 2 - 2 * x ** 3) * d[k + 1] + (x ** 3 - x ** 2) * h * dd[k + 1])
        hp = ((6 * x ** 2 - 6 * x) * (d[k] - d[k + 1]) + (3 * x ** 2 - 4 * x + 1) * h * dd[k]
              + (3 * x ** 2 - 2 * x) * h * dd[k + 1])
        x = np.clip(x - (hv - t) / hp, 0, 1)
    z[ok] = np.exp(-(y[k] + x * h)) - 1
    return torch.from_numpy(z.reshape(shape))


def exact(case, seed):
    n, kind = case["n"], case["kind"]
    if kind in ("noalloc", "collapse") and n ** 3 * case["n_radii"] <= 8_000_000:
        return {"F": _exact_collapse(case, seed), "ridx": None}
    if kind == "displacement" and n <= 256:
        return _exact_displacements(case, seed)
    if kind == "redshift" and n <= 256:
        return {"z": _exact_redshift(case, seed)}
    return None
