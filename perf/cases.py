"""Performance cases of the particle-mesh framework.

Each case is one pass through public entry points of `paper_2211_09958_amd.api`, at sizes of
this repository's workloads, tests and drivers: single layers (density, force, force VJP,
transforms, spectra, losses, initial conditions) on evolved, clustered particle sets, and whole
runs with their reverse-time adjoint.  Whole runs stop while displacements stay well inside one
mesh cell: the CIC force is only piecewise smooth, and past the first crossings of node planes two
correctly rounded runs part by more than their rounding.  The clustered states that late runs
reach are therefore handed to the single layers as inputs.

`exact` restates each case in 64-bit torch.
"""
import math
from types import SimpleNamespace

import numpy as np
import torch

from paper_2211_09958_amd import api

A_START = 1.0 / 64
HIDDEN = 64


def listed():
    return [
        # smallest force call: a notebook or unit-sized box, all latency
        dict(name="force_32p_64m", kind="force", ptcl=32, mesh=64, box=64.0, filter=False),
        # a monitor's spectrum inside a loop that must not allocate
        dict(name="power_noalloc_64m", kind="power_noalloc", mesh=64, box=128.0, n_bins=32),
        # one iteration of field-level reconstruction on a small box
        dict(name="fit_32p_64m_15s", kind="fit", ptcl=32, mesh=64, box=256.0, steps=15,
             a_stop=0.05, ckpt=0, lpt=1),
        # one run of a filter + step-scale training batch (one particle per cell)
        dict(name="train_128p_128m_8s", kind="train", ptcl=128, mesh=128, box=512.0, steps=8,
             a_stop=0.05, lpt=1, n_bins=32),
        # a fine run's particles assigned to a coarse mesh and its spectrum, as in evaluation
        dict(name="spectrum_256p_256m", kind="spectrum", ptcl=256, mesh=256, box=256.0, n_bins=128),
        # spectrum and losses of a final density, with their cotangents
        dict(name="losses_256p_256m", kind="losses", ptcl=256, mesh=256, box=256.0, n_bins=63),
        # forward and inverse transform of one mesh for analysis tools
        dict(name="fft_512m", kind="fft", mesh=512, box=512.0),
        # second-order initial conditions of a production lattice
        dict(name="ics_2lpt_256p", kind="ics", ptcl=256, mesh=256, box=256.0, lpt=2),
        # reverse step of filter training on the 4x finer mesh: sparse clustered particles
        dict(name="vjp_128p_512m_filter", kind="vjp", ptcl=128, mesh=512, box=128.0, filter=True),
        # force of the learned production run: one particle per cell, clustered
        dict(name="force_512p_512m_filter", kind="force", ptcl=512, mesh=512, box=512.0, filter=True),
        # forward + loss + adjoint at the medium geometry, 2LPT start
        dict(name="fit_256p_512m_3s", kind="fit", ptcl=256, mesh=512, box=2048.0, steps=3,
             a_stop=3.0 / 64, ckpt=0, lpt=2),
        # the headline geometry: forward + loss + checkpointed adjoint
        dict(name="fit_512p_1024m_2s", kind="fit", ptcl=512, mesh=1024, box=4096.0, steps=2,
             a_stop=3.0 / 64, ckpt=1, lpt=1),
    ]


def draw(rng):
    """Another case of the listed kinds: lattices 8..256 (512 without time steps), meshes 8..512
    at 1, 2 or 4 cells per particle spacing, arbitrary boxes, bin and step counts."""
    kind = rng.choice(["force", "force", "vjp", "vjp", "fit", "fit", "train", "spectrum", "losses",
                       "fft", "ics", "power_noalloc"])
    ptcl = 2 ** rng.randint(3, 8)
    mesh = min(512, ptcl * rng.choice([1, 2, 2, 4]))
    box = round(ptcl * rng.uniform(0.7, 2.5), 3)
    if kind == "power_noalloc":
        mesh = 2 ** rng.randint(3, 7)
        return dict(kind=kind, mesh=mesh, box=box, n_bins=rng.randint(3, mesh))
    if kind == "fft":
        return dict(kind=kind, mesh=2 ** rng.randint(4, 9), box=box)
    if kind in ("force", "vjp"):
        if kind == "force" and rng.random() < 0.15:
            ptcl, mesh, box = 512, 512, 2.0 * box
        return dict(kind=kind, ptcl=ptcl, mesh=mesh, box=box, filter=rng.random() < 0.5)
    if kind in ("spectrum", "losses"):
        return dict(kind=kind, ptcl=ptcl, mesh=mesh, box=box, n_bins=rng.randint(3, mesh // 2))
    if kind == "ics":
        return dict(kind=kind, ptcl=ptcl, mesh=ptcl, box=box, lpt=rng.choice([1, 2]))
    # whole runs: cells of 3 to 6 Mpc/h, displacements of a tenth of a cell
    cell = rng.uniform(3.0, 6.0)
    steps = rng.randint(1, 12) if ptcl <= 64 else rng.randint(1, 4)
    case = dict(kind=kind, ptcl=ptcl, mesh=mesh, box=round(mesh * cell, 3), steps=steps,
                a_stop=round(0.0125 * cell, 5), lpt=rng.choice([1, 2]))
    if kind == "fit":
        case["ckpt"] = rng.choice([0, 0, 1, 2])
    else:
        case["n_bins"] = rng.randint(3, mesh // 2)
    return case


# ----------------------------------------------------------------- inputs

def _cosmo():
    from dataclasses import make_dataclass
    names = ("omega_m", "omega_b", "h", "sigma8", "n_s", "T_cmb")
    return make_dataclass("Cosmo", names)(0.3, 0.05, 0.7, 0.8, 0.96, 2.7255)


def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _randn(g, *shape):
    return torch.randn(*shape, generator=g, device="cuda", dtype=torch.float32)


def _smooth_field(g, n, rms, box):
    """[n^3, 3] curl-free displacements with a falling spectrum, rms per axis in Mpc/h."""
    wk = torch.fft.rfftn(_randn(g, n, n, n))
    f = torch.fft.fftfreq(n, 1.0 / n, device="cuda")
    fh = torch.arange(n // 2 + 1, device="cuda", dtype=torch.float32)
    nv = (f[:, None, None], f[None, :, None], fh[None, None, :])
    n2 = nv[0] ** 2 + nv[1] ** 2 + nv[2] ** 2
    amp = wk * torch.where(n2 > 0, (n2 + 4.0) ** -1.4, torch.zeros_like(n2))
    out = torch.empty((n ** 3, 3), device="cuda", dtype=torch.float32)
    for j in range(3):
        s = torch.fft.irfftn(1j * nv[j] * amp, s=(n, n, n)).reshape(-1)
        out[:, j] = s * (rms / s.std())
    return out


def _clustered(g, n, box):
    """Displacements [n^3, 3] of an evolved state: a smooth flow of 5 Mpc/h (less in a small box),
    with three in ten 8^3 blocks of the lattice collapsed onto a halo a fifth their size."""
    disp = _smooth_field(g, n, min(5.0, 0.05 * box), box)
    b = min(8, n)
    m = n // b
    shrink = torch.where(torch.rand((m, m, m), generator=g, device="cuda") < 0.3, 0.8, 0.05)
    offs = (torch.arange(n, device="cuda") % b - 0.5 * (b - 1)) * (box / n)
    v = disp.view(m, b, m, b, m, b, 3)
    for j, sh in enumerate(((m, b, 1, 1, 1, 1), (1, 1, m, b, 1, 1), (1, 1, 1, 1, m, b))):
        v[..., j] -= shrink.view(m, 1, m, 1, m, 1) * offs.view(sh)
    # random motions inside the halos
    disp += _randn(g, n ** 3, 3) * (0.1 * box / n)
    return disp


def _weights(g):
    """Filter weights of the 2-64-64-1 network with a small output layer."""
    u = lambda n, b: (2.0 * torch.rand(n, generator=g, device="cuda") - 1.0) * b
    h = HIDDEN
    return torch.cat([u(2 * h, 2 ** -0.5), u(h, 2 ** -0.5), u(h * h, h ** -0.5), u(h, h ** -0.5),
                      u(h, 0.3 * h ** -0.5), u(1, 0.05)])


def _lognormal(g, n):
    return torch.exp(0.8 * _randn(g, n, n, n) - 0.32) - 1.0


def _inputs(case, seed):
    """The arrays of a case, from its sizes and the seed alone."""
    g = _gen(seed)
    k = case["kind"]
    x = SimpleNamespace()
    if k in ("force", "vjp", "spectrum"):
        x.disp = _clustered(g, case["ptcl"], case["box"])
        if case.get("filter"):
            x.weights = _weights(g)
            x.a = 0.6
        else:
            x.weights, x.a = None, 0.6
        if k == "vjp":
            x.v = _randn(g, case["ptcl"] ** 3, 3)
    elif k in ("power_noalloc", "fft"):
        x.dens = _lognormal(g, case["mesh"])
        if k == "fft":
            x.spec = torch.fft.rfftn(_lognormal(g, case["mesh"])).contiguous()
    elif k == "losses":
        x.dens = _lognormal(g, case["mesh"])
        x.disp = _clustered(g, case["ptcl"], case["box"])
        x.disp_t = x.disp + _randn(g, case["ptcl"] ** 3, 3) * (0.4 * case["box"] / case["mesh"])
        white = case["box"] ** 3 / case["mesh"] ** 3
        x.pk_t = white * np.linspace(0.6, 1.3, case["n_bins"])
    elif k == "ics":
        x.noise = _randn(g, *(case["ptcl"],) * 3)
    else:   # fit, train
        x.noise = _randn(g, *(case["ptcl"],) * 3)
        if k == "fit":
            x.target = 0.1 * _randn(g, *(case["mesh"],) * 3)
        else:
            x.weights = _weights(g)
            x.scales = 1.0 + 0.05 * torch.rand(3, case["steps"], generator=g, device="cuda",
                                               dtype=torch.float64).cpu().numpy()
            x.disp_t = _smooth_field(g, case["ptcl"], 0.3, case["box"])
            white = case["box"] ** 3 / case["mesh"] ** 3
            x.pk_t = 0.02 * white * np.linspace(1.4, 0.6, case["n_bins"])
    return x


def prepare(case, seed):
    s = _inputs(case, seed)
    s.case = case
    k = case["kind"]
    if k == "power_noalloc":
        return s
    cfg = api.make_config(case.get("ptcl", case["mesh"]) if k != "fft" else 8, case["mesh"],
                          case["box"], case.get("steps", 1), a_start=A_START,
                          a_stop=case.get("a_stop", 1.0), checkpoint_every=case.get("ckpt", 0),
                          filter=getattr(s, "weights", None) is not None,
                          lpt_order=case.get("lpt", 1))
    s.pm = api.PMContext(cfg, _cosmo())
    if k in ("force", "vjp") and s.weights is not None:
        s.pm.set_filter(s.weights)
    return s


# ------------------------------------------------------------------- runs

def _f32(*values):
    """Scalars formed from 32-bit fields, in the precision a training log keeps."""
    return torch.tensor(values, dtype=torch.float32)


def _spectrum(k, pk, modes):
    return {"k": k, "modes": modes, "pk": pk.astype(np.float32)}


def run(s):
    case, k = s.case, s.case["kind"]
    if k == "force":
        return s.pm.force(s.disp, s.a)
    if k == "vjp":
        return s.pm.force_vjp(s.disp, s.a, s.v)
    if k == "power_noalloc":
        return _spectrum(*api.power_spectrum_noalloc(s.dens, case["box"], case["n_bins"]))
    if k == "spectrum":
        dens = s.pm.density(s.disp)
        return {"dens": dens, **_spectrum(*s.pm.power_spectrum(dens, case["n_bins"]))}
    if k == "fft":
        return {"spec": s.pm.fft_r2c(s.dens), "real": s.pm.fft_c2r(s.spec)}
    if k == "losses":
        lp, g_dens = s.pm.loss_pk(s.dens, s.pk_t, case["n_bins"])
        ld, g_disp = s.pm.loss_disp(s.disp, s.disp_t, weight=1e-2)
        return {"loss": _f32(lp, ld), "g_dens": g_dens, "g_disp": g_disp}
    if k == "ics":
        disp, mom = s.pm.initial_conditions(s.noise)
        return {"disp": disp, "mom": mom}
    if k == "fit":
        disp, mom, dens = s.pm.forward(s.noise)
        loss, g = s.pm.loss_mse(dens, s.target)
        g_noise, g_cosmo, _ = s.pm.adjoint(g_dens=g)
        return {"disp": disp, "mom": mom, "dens": dens, "loss": _f32(loss), "g_noise": g_noise,
                "g_cosmo": _f32(*g_cosmo)}
    # train
    s.pm.set_filter(s.weights)
    s.pm.set_step_scales(s.scales)
    disp, _, dens = s.pm.forward(s.noise)
    lp, g_dens = s.pm.loss_pk(dens, s.pk_t, case["n_bins"])
    ld, g_disp = s.pm.loss_disp(disp, s.disp_t, weight=1e-2)
    g_noise, g_cosmo, g_filter = s.pm.adjoint(g_dens=g_dens, g_disp=g_disp, want_filter=True)
    g_scales = torch.as_tensor(s.pm.step_gradients(), dtype=torch.float32)
    return {"disp": disp, "dens": dens, "loss": _f32(lp, ld), "g_noise": g_noise,
            "g_cosmo": _f32(*g_cosmo), "g_filter": g_filter, "g_scales": g_scales}


# ------------------------------------------------------------------- work

def work(case):
    """Bytes: input and output of each stage that needs all of the one before (assignment, 3-D
    transform, three inverse transforms, interpolation), once each.  Flops: real 3-D transforms at
    2.5 N log2 N, 30 per CIC corner set, the filter network where there is one."""
    k, n = case["kind"], case["mesh"]
    P = case.get("ptcl", 0) ** 3
    r, c = 4.0 * n ** 3, 8.0 * n * n * (n // 2 + 1)
    fft = 2.5 * n ** 3 * math.log2(n ** 3)
    filt = case.get("filter") or k == "train"
    net = 2.0 * (2 * HIDDEN + HIDDEN * HIDDEN + HIDDEN) * 0.75 * n * n if filt else 0.0
    dens_b = 12.0 * P + r
    force_b = dens_b + (r + c) + (c + 3 * r) + 3 * r + 24.0 * P
    force_f = 4 * fft + 120.0 * P + net
    adj_b = 24.0 * P + 3 * r + 3 * (r + c) + (c + r) + r + 24.0 * P + (c if filt else 0.0)
    adj_f = 4 * fft + 240.0 * P + 3 * net
    if k == "force":
        return {"bytes": force_b, "flops": force_f}
    if k == "vjp":
        return {"bytes": force_b + 12.0 * P + adj_b, "flops": force_f + adj_f}
    if k == "power_noalloc":
        return {"bytes": r + 0.0, "flops": fft + 10.0 * n ** 3}
    if k == "spectrum":
        return {"bytes": dens_b + r, "flops": fft + 10.0 * n ** 3 + 30.0 * P}
    if k == "fft":
        return {"bytes": 2 * (r + c), "flops": 2 * fft}
    if k == "losses":
        return {"bytes": r + (r + c) + 36.0 * P, "flops": 2 * fft + 10.0 * n ** 3 + 12.0 * P}
    p = case["ptcl"]
    rp, cp = 4.0 * p ** 3, 8.0 * p * p * (p // 2 + 1)
    fp = 2.5 * p ** 3 * math.log2(p ** 3)
    ic_b = rp + cp + cp + 3 * rp + 24.0 * P
    ic_f = 4 * fp
    if case["lpt"] == 2:
        ic_b += rp + cp + 6 * (cp + rp) + 6 * rp + rp + cp + 3 * rp
        ic_f += 11 * fp
    if k == "ics":
        return {"bytes": ic_b, "flops": ic_f}
    forces = case["steps"] + 1
    b = ic_b + forces * (force_b + 12.0 * P) + dens_b + 3 * r
    f = ic_f + forces * force_f + fft
    b += forces * (force_b + adj_b + 60.0 * P) + 2 * ic_b
    f += forces * (force_f + adj_f) + 2 * ic_f
    return {"bytes": b, "flops": f}


# --------------------------------------------------------------- 64 bits

def _wave(n):
    f = torch.fft.fftfreq(n, 1.0 / n, device="cuda", dtype=torch.float64)
    fh = torch.arange(n // 2 + 1, device="cuda", dtype=torch.float64)
    return f[:, None, None], f[None, :, None], fh[None, None, :]


def _nyquist_free(nv, n):
    """Wave numbers with the Nyquist plane of their own axis zeroed."""
    return [torch.where(v.abs() == n // 2, torch.zeros_like(v), v) for v in nv]


def _n2(nv):
    return nv[0] ** 2 + nv[1] ** 2 + nv[2] ** 2


def _lattice(n, spacing):
    q = torch.arange(n, device="cuda", dtype=torch.float64) * spacing
    return torch.stack(torch.meshgrid(q, q, q, indexing="ij"), dim=-1).reshape(-1, 3)


def _corners(u, n):
    """Node index and weight of the 8 CIC corners of positions u (cells, node i at i)."""
    fl = torch.floor(u.detach())
    t = u - fl
    i = fl.long()
    for c in range(8):
        bits = (c >> 2 & 1, c >> 1 & 1, c & 1)
        idx = 0
        w = 1.0
        for ax in range(3):
            idx = idx * n + (i[:, ax] + bits[ax]) % n
            w = w * (t[:, ax] if bits[ax] else 1.0 - t[:, ax])
        yield idx, w


def _density(u, n):
    rho = torch.zeros(n ** 3, device="cuda", dtype=torch.float64)
    mass = n ** 3 / u.shape[0]
    for idx, w in _corners(u, n):
        rho = rho.index_add(0, idx, mass * w)
    return rho.view(n, n, n) - 1.0


def _filter(theta, n, a):
    h = HIDDEN
    w1, b1, w2, b2, w3, b3 = torch.split(theta, [2 * h, h, h * h, h, h, 1])
    x = 2.0 * torch.sqrt(torch.arange(3 * (n // 2) ** 2 + 1, device="cuda", dtype=torch.float64)) / n
    x = torch.stack([x, torch.full_like(x, a)], dim=1)
    z = torch.nn.functional.silu(x @ w1.view(h, 2).T + b1)
    z = torch.nn.functional.silu(z @ w2.view(h, h).T + b2)
    return 1.0 + (z @ w3) + b3


def _gradient(spec, n, length):
    """IDFT(i k_j / k^2 spec) for the three axes, k = 2 pi n / length."""
    nv = _wave(n)
    n2 = _n2(nv)
    g = torch.where(n2 > 0, 1.0 / n2.clamp(min=1.0), torch.zeros_like(n2)) * spec
    return [torch.fft.irfftn(1j * v * (length / (2 * math.pi)) * g, s=(n, n, n))
            for v in _nyquist_free(nv, n)]


def _force(u, n, length, theta=None, a=1.0):
    dk = torch.fft.rfftn(_density(u, n))
    if theta is not None:
        dk = dk * _filter(theta, n, a)[_n2(_wave(n)).long()]
    meshes = [m.reshape(-1) for m in _gradient(dk, n, length)]
    out = [0.0, 0.0, 0.0]
    for idx, w in _corners(u, n):
        for j in range(3):
            out[j] = out[j] + w * meshes[j][idx]
    return torch.stack(out, dim=1)


def _cells(disp, case):
    """Positions in cells of 32-bit displacements, at the resolution of the particle state."""
    p, n, length = case["ptcl"], case["mesh"], case["box"]
    units = (disp * np.float32(4294967296.0 / length)).double().round() / 4294967296.0
    return _lattice(p, n / p) + units * n - 0.5


def _shells(dens, length, n_bins):
    n = dens.shape[0]
    dk = torch.fft.rfftn(dens)
    r = torch.sqrt(_n2(_wave(n))).reshape(-1)
    b = torch.floor(r + 0.5).long()
    w = torch.full((n // 2 + 1,), 2.0, device="cuda", dtype=torch.float64)
    w[0] = w[-1] = 1.0
    w = w.expand(n, n, -1).reshape(-1)
    keep = (b >= 1) & (b <= n_bins)
    b, w, r = b[keep] - 1, w[keep], r[keep]
    p2 = (dk.real ** 2 + dk.imag ** 2).reshape(-1)[keep]
    zero = torch.zeros(n_bins, device="cuda", dtype=torch.float64)
    cnt = zero.index_add(0, b, w)
    pk = zero.index_add(0, b, w * p2) / cnt * (length ** 3 / float(n) ** 6)
    return zero.index_add(0, b, w * r) / cnt * (2 * math.pi / length), pk, cnt


def _exact_spectrum(dens, case):
    k, pk, cnt = _shells(dens, case["box"], case["n_bins"])
    return {"k": k.cpu().numpy(), "modes": cnt.cpu().numpy(), "pk": pk.cpu().numpy()}


def _loss_pk(dens, target, case):
    _, pk, cnt = _shells(dens, case["box"], case["n_bins"])
    t = torch.as_tensor(target, device="cuda")
    use = cnt > 0
    return ((pk[use] / t[use] - 1.0) ** 2).mean()


def _loss_disp(disp, target, case):
    d = disp - target
    d = d - case["box"] * torch.floor(d.detach() / case["box"] + 0.5)
    return 1e-2 * (d ** 2).sum(dim=1).mean() * (case["mesh"] / case["box"]) ** 2


def _growth(a, om):
    """D and D' (unnormalised) and E of flat LambdaCDM, by Gauss-Legendre in a' = a u^2."""
    x, w = np.polynomial.legendre.leggauss(96)
    u = torch.as_tensor(0.5 * (x + 1.0))
    w = torch.as_tensor(0.5 * w)
    aa = a * u * u
    integral = (w * 2.0 * a * u / (om / aa + (1.0 - om) * aa * aa) ** 1.5).sum()
    e = torch.sqrt(om / a ** 3 + (1.0 - om))
    return e * integral, -1.5 * om / (a ** 4 * e) * integral + e / (a * e) ** 3, e


def _growths(a, om):
    """D, G = a^3 E D', and the second-order D2, G2 at a."""
    d1 = _growth(1.0, om)[0]
    d, dd, e = _growth(a, om)
    d, dd = d / d1, dd / d1
    oma = om / (a ** 3 * e * e)
    d2 = -3.0 / 7.0 * d * d * oma ** (-1.0 / 143.0)
    g2 = a ** 3 * e * d2 * (2.0 * dd / d + 3.0 / 143.0 * (1.0 - oma) / a)
    return d, a ** 3 * e * dd, d2, g2


def _linear_pk(k, om, s8, cosmo):
    """Eisenstein-Hu no-wiggle spectrum at a = 1, normalised to sigma_8."""
    h, ob = cosmo.h, cosmo.omega_b
    oh, fb = om * h * h, ob / om
    sound = 44.5 * torch.log(9.83 / oh) / math.sqrt(1.0 + 10.0 * (ob * h * h) ** 0.75)
    alpha = 1.0 - 0.328 * torch.log(431.0 * oh) * fb + 0.38 * torch.log(22.3 * oh) * fb * fb

    def shape(k):
        gamma = om * h * (alpha + (1.0 - alpha) / (1.0 + (0.43 * k * h * sound) ** 4))
        q = k * (cosmo.T_cmb / 2.7) ** 2 / gamma
        l0 = torch.log(2.0 * math.e + 1.8 * q)
        t = l0 / (l0 + (14.2 + 731.0 / (1.0 + 62.5 * q)) * q * q)
        return k ** cosmo.n_s * t * t

    x = torch.linspace(math.log(1e-5), math.log(1e2), 65537, dtype=torch.float64)
    kk = torch.exp(x)
    y = 8.0 * kk
    win = torch.where(y < 1e-3, 1.0 - y * y / 10.0, 3.0 * (torch.sin(y) - y * torch.cos(y)) / y ** 3)
    f = kk ** 3 * shape(kk) * win * win
    simpson = torch.full_like(f, 2.0)
    simpson[1::2] = 4.0
    simpson[0] = simpson[-1] = 1.0
    var = (simpson * f).sum() * (x[1] - x[0]) / 3.0 / (2.0 * math.pi ** 2)
    return s8 * s8 / var * shape(k)


def _ics(noise, om, s8, case, cosmo):
    """(x_0 - q, p_0) and nothing else: Zel'dovich, or with the second-order term."""
    n, length = case["ptcl"], case["box"]
    nv = _wave(n)
    n2 = _n2(nv)
    top = int(n2.max().item())
    kk = 2 * math.pi / length * torch.sqrt(torch.arange(1, top + 1, dtype=torch.float64))
    amp = torch.sqrt(_linear_pk(kk, om, s8, cosmo) / (length / n) ** 3)
    amp = torch.cat([torch.zeros(1, dtype=torch.float64), amp]).to("cuda")
    dk = amp[n2.long()] * torch.fft.rfftn(noise)
    D, G, D2, G2 = [v.to("cuda") for v in _growths(A_START, om)]
    s = torch.stack([m.reshape(-1) for m in _gradient(dk, n, length)], dim=1)
    disp, mom = D * s, G * s
    if case["lpt"] == 2:
        inv = torch.where(n2 > 0, 1.0 / n2.clamp(min=1.0), torch.zeros_like(n2))
        free = _nyquist_free(nv, n)
        hess = lambda a, b: torch.fft.irfftn(
            (nv[a] * nv[a] if a == b else free[a] * free[b]) * inv * dk, s=(n, n, n))
        xx, yy, zz = hess(0, 0), hess(1, 1), hess(2, 2)
        src = xx * yy + xx * zz + yy * zz
        del xx, yy, zz
        for a, b in ((0, 1), (0, 2), (1, 2)):
            src = src - hess(a, b) ** 2
        s2 = -torch.stack([m.reshape(-1) for m in _gradient(torch.fft.rfftn(src), n, length)], dim=1)
        disp, mom = disp + D2 * s2, mom + G2 * s2
    return disp, mom


def _evolve(noise, om, s8, case, cosmo, theta=None, scales=None):
    n, length, N = case["mesh"], case["box"], case["steps"]
    q = _lattice(case["ptcl"], n / case["ptcl"]) - 0.5
    disp, mom = _ics(noise, om, s8, case, cosmo)
    a = [A_START + (case["a_stop"] - A_START) * i / N for i in range(N + 1)]
    g = [_growths(v, om) for v in a]
    gh = [_growths(0.5 * (a[i] + a[i + 1]), om) for i in range(N)]
    sc = scales if scales is not None else torch.ones(3, N, dtype=torch.float64)
    force = lambda d, v: _force(q + d * (n / length), n, length, theta, v)
    F = force(disp, a[0])
    for i in range(N):
        mom = mom + (sc[0, i] * (gh[i][1] - g[i][1]) / g[i][0]).to("cuda") * F
        disp = disp + (sc[1, i] * (g[i + 1][0] - g[i][0]) / gh[i][1]).to("cuda") * mom
        F = force(disp, a[i + 1])
        mom = mom + (sc[2, i] * (g[i + 1][1] - gh[i][1]) / g[i + 1][0]).to("cuda") * F
    return disp, mom, _density(q + disp * (n / length), n)


def exact(case, seed):
    k = case["kind"]
    if k in ("fit", "train") and case["ptcl"] > 256:
        return None   # minutes in 64 bits
    x = _inputs(case, seed)
    leaf = lambda v: torch.as_tensor(v).double().requires_grad_(True)
    if k in ("force", "vjp"):
        theta = None if x.weights is None else x.weights.double()
        if k == "force":
            with torch.no_grad():
                return _force(_cells(x.disp, case), case["mesh"], case["box"], theta, x.a)
        u = _cells(x.disp, case).requires_grad_(True)
        F = _force(u, case["mesh"], case["box"], theta, x.a)
        return torch.autograd.grad((F * x.v.double()).sum(), u)[0] * (case["mesh"] / case["box"])
    if k == "power_noalloc":
        return _exact_spectrum(x.dens.double(), case)
    if k == "spectrum":
        dens = _density(_cells(x.disp, case), case["mesh"])
        return {"dens": dens, **_exact_spectrum(dens, case)}
    if k == "fft":
        n = case["mesh"]
        return {"spec": torch.fft.rfftn(x.dens.double()),
                "real": torch.fft.irfftn(x.spec.to(torch.complex128), s=(n, n, n)) * float(n) ** 3}
    cosmo = _cosmo()
    if k == "losses":
        dens, disp = leaf(x.dens), leaf(x.disp)
        lp = _loss_pk(dens, x.pk_t, case)
        ld = _loss_disp(disp, x.disp_t.double(), case)
        return {"loss": torch.stack([lp, ld]).detach(), "g_dens": torch.autograd.grad(lp, dens)[0],
                "g_disp": torch.autograd.grad(ld, disp)[0]}
    om, s8 = leaf(cosmo.omega_m), leaf(cosmo.sigma8)
    if k == "ics":
        with torch.no_grad():
            disp, mom = _ics(x.noise.double(), om, s8, case, cosmo)
        return {"disp": disp, "mom": mom}
    noise = leaf(x.noise)
    if k == "fit":
        disp, mom, dens = _evolve(noise, om, s8, case, cosmo)
        loss = ((dens - x.target.double()) ** 2).mean()
        gn, go, gs = torch.autograd.grad(loss, (noise, om, s8))
        return {"disp": disp.detach(), "mom": mom.detach(), "dens": dens.detach(),
                "loss": loss.detach().reshape(1), "g_noise": gn, "g_cosmo": torch.stack([go, gs])}
    theta, scales = leaf(x.weights), leaf(x.scales)
    disp, _, dens = _evolve(noise, om, s8, case, cosmo, theta, scales)
    lp, ld = _loss_pk(dens, x.pk_t, case), _loss_disp(disp, x.disp_t.double(), case)
    gn, go, gs, gt, gsc = torch.autograd.grad(lp + ld, (noise, om, s8, theta, scales))
    return {"disp": disp.detach(), "dens": dens.detach(),
            "loss": torch.stack([lp, ld]).detach(), "g_noise": gn,
            "g_cosmo": torch.stack([go, gs]), "g_filter": gt, "g_scales": gsc}
