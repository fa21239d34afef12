"""The work that a program built on this library has it do, as cases that can be timed.

A survey program makes initial conditions (lpc_init_ic, lpc_init_ic_png), advances them (lpc_cola_step for one box,
lpc_cola_step_batched for many), measures them (lpc_power_spectrum, lpc_bispectrum), corrects coarse runs (lpc_net_apply)
and trains that correction (lpc_net_loss_grad, lpc_net_adam); lpc_pm_force is the single force evaluation that other
integrators call. Every case is one such call (the training case: the two calls of one step) on inputs made on the GPU
from a seed. Sizes are those of bench.py, synth/ and the tests, and draw() spreads over the ranges between them.

Inputs are Gaussian fields of the library's own spectrum (BBKS, sigma8) displaced by second-order perturbation theory to
the wanted time, written here in plain torch; exact() evaluates the same calls in FP64.

Two conventions of the outputs. Positions are periodic, so a coordinate at the box edge may come out at either end by
rounding: they are returned relative to their lattice site, x - q + L / 2 in [0, L). P(k), B, Q and the shell powers are
statistics of FP32 transforms that the library hands out in FP64 variables: they are returned as the FP32 values they
carry.
"""
import math

import numpy as np
import torch

from paper_1506_03737_amd import lpc

OM, H, SIGMA8, NS = 0.31, 0.68, 0.8, 0.96
N_LPT = -2.5
C_OVER_H0 = 2997.92458
DEV = "cuda"


# --- the cases -----------------------------------------------------------------------------------------------------

def listed():
    return [
        # one force evaluation of the smallest configuration: an integrator's inner call, bound by latency
        {"name": "force_small", "kind": "force", "n_side": 32, "n_mesh": 64, "box": 256.0, "deconv": 1, "a": 0.5},
        # a force on a late-time, clumped particle set of an odd count, on a mesh with no power-of-two plan, with
        # the fixed-point density as well
        {"name": "force_ragged", "kind": "force", "count": 1500007, "n_mesh": 270, "box": 432.0, "deconv": 2,
         "density": True},
        # the smallest whole run: ten steps, some 130 launches on a mesh that fits in cache
        {"name": "cola_small", "kind": "cola", "n_side": 32, "n_mesh": 64, "box": 256.0, "steps": 10},
        # the paper's recommended mesh (Nm = 3 N) at the single-box size: the late steps of a run
        {"name": "cola_single", "kind": "cola", "n_side": 256, "n_mesh": 768, "box": 1000.0, "steps": 4},
        # the largest box: 512^3 particles on the largest mesh the FFT takes
        {"name": "cola_large", "kind": "cola", "n_side": 512, "n_mesh": 1024, "box": 2000.0, "steps": 2},
        # mock production for a covariance: 48 boxes of three sizes in one batched call
        {"name": "mocks_batched", "kind": "batch", "boxes": 48, "sides": "96,128,160", "ratio": 2, "box": 300.0,
         "box_step": 300.0 / 47.0, "steps": 2},
        # initial conditions of the single box
        {"name": "ic_gaussian", "kind": "ic", "n_side": 256, "box": 1000.0, "a": 0.1},
        # initial conditions with equilateral non-Gaussianity at the size of a mock
        {"name": "ic_equilateral", "kind": "ic", "n_side": 160, "box": 600.0, "a": 0.1, "png": "equilateral",
         "f_nl": 1000.0},
        # P(k) of the single box on the evaluation mesh
        {"name": "power_spectrum", "kind": "pk", "n_side": 256, "n_mesh": 512, "box": 1000.0, "k_max": 1.0, "bins": 100},
        # the reduced bispectrum that judges the learned correction: 128^3 mesh, shells of 3 k_f, six triangles
        {"name": "bispectrum", "kind": "bispectrum", "n_side": 256, "n_mesh": 128, "box": 1000.0, "triangles":
         "0.05,0.05,0.05;0.1,0.1,0.1;0.2,0.2,0.2;0.3,0.3,0.3;0.1,0.2,0.15;0.1,0.2,0.25", "dk_kf": 3.0},
        # the learned correction of a coarse run (forward)
        {"name": "net_apply", "kind": "apply", "n_side": 256, "box": 1000.0},
        # one training step of the correction (forward, backward, Adam) on a training pair's grid
        {"name": "net_train", "kind": "train", "n_side": 128, "box": 500.0},
    ]


SMOOTH = sorted(2 ** i * 3 ** j * 5 ** k for i in range(1, 11) for j in range(7) for k in range(5)
                if 8 <= 2 ** i * 3 ** j * 5 ** k <= 1024)


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _smooth(rng, lo, hi):
    """An FFT size of [lo, hi], spread over its logarithm."""
    u = _log(rng, lo, hi)
    return min((n for n in SMOOTH if lo <= n <= hi), key=lambda n: abs(n - u))


def draw(rng):
    kind = rng.choices(["force", "cola", "batch", "ic", "pk", "bispectrum", "apply", "train"],
                       [4, 4, 2, 4, 3, 3, 2, 3])[0]
    spacing = _log(rng, 2.0, 8.0)  # mean particle separation in Mpc/h
    if kind == "force":
        nm = _smooth(rng, 32, 512)
        return {"kind": kind, "count": int(_log(rng, nm ** 3 / 27, nm ** 3)) | 1, "n_mesh": nm,
                "box": round(nm * spacing, 2), "deconv": rng.choice([0, 1, 2]), "density": rng.random() < 0.5}
    if kind == "cola":
        ratio = rng.choice([1, 2, 3])
        n = _smooth(rng, 16, {1: 320, 2: 320, 3: 240}[ratio])
        return {"kind": kind, "n_side": n, "n_mesh": ratio * n, "box": round(n * spacing, 2),
                "steps": rng.choice([2, 3, 5]), "plain": rng.random() < 0.25, "standard": rng.random() < 0.25,
                "deconv": rng.choice([0, 1, 1, 2])}
    if kind == "batch":
        sides = sorted({_smooth(rng, 32, 160) for _ in range(3)})
        return {"kind": kind, "boxes": rng.randrange(2, 13), "sides": ",".join(map(str, sides)),
                "ratio": rng.choice([1, 2, 3]), "box": round(sides[-1] * spacing, 2),
                "box_step": round(rng.uniform(0.0, 20.0), 2), "steps": 2}
    if kind == "ic":
        n = _smooth(rng, 16, 400)
        case = {"kind": kind, "n_side": n, "box": round(n * spacing, 2), "a": rng.choice([0.05, 0.1, 0.2])}
        if rng.random() < 0.4:
            case.update(png=rng.choice(["local", "equilateral", "orthogonal"]), f_nl=round(rng.uniform(-2000, 2000), 1))
        return case
    if kind == "pk":
        n, nm = _smooth(rng, 16, 256), _smooth(rng, 32, 640)
        box = round(n * spacing, 2)
        return {"kind": kind, "n_side": n, "n_mesh": nm, "box": box,
                "k_max": round(rng.uniform(0.5, 1.0) * math.pi * nm / box, 4), "bins": rng.randrange(8, 400)}
    if kind == "bispectrum":
        n, nm = _smooth(rng, 32, 256), _smooth(rng, 48, 200)
        box = round(n * spacing, 2)
        kf, tri = 2 * math.pi / box, []
        for _ in range(rng.randrange(1, 13)):
            k1, k2 = rng.uniform(4.0, nm / 4), rng.uniform(4.0, nm / 4)
            k3 = rng.uniform(max(4.0, abs(k1 - k2)), min(k1 + k2, nm / 2.5))
            tri.append(",".join("%.6f" % (k * kf) for k in (k1, k2, k3)))
        return {"kind": kind, "n_side": n, "n_mesh": nm, "box": box, "triangles": ";".join(tri),
                "dk_kf": rng.choice([2.0, 3.0])}
    n = 4 * int(_log(rng, 2, 64 if kind == "apply" else 40))
    return {"kind": kind, "n_side": n, "box": round(n * spacing, 2)}


# --- what the path cannot do without ---------------------------------------------------------------------------------

def _fft_flops(n):
    return 2.5 * n ** 3 * math.log2(n ** 3)  # one real 3-D transform


def _force_flops(n_mesh, particles):
    return 4 * _fft_flops(n_mesh) + 20.0 * n_mesh ** 3 + 150.0 * particles


NET_FLOPS = 76512.0  # per lattice site, forward


def work(case):
    kind = case["kind"]
    if kind == "force":
        n = case.get("count") or case["n_side"] ** 3
        return {"bytes": 24.0 * n + (8.0 * case["n_mesh"] ** 3 if case.get("density") else 0.0),
                "flops": _force_flops(case["n_mesh"], n)}
    if kind in ("cola", "batch"):
        boxes = [(n, nm) for n, nm, _ in _boxes(case)]
        evals = case["steps"] + 1
        # positions, momenta in and out, and the displacement fields in (not read by a plain run)
        return {"bytes": sum((48.0 if case.get("plain") else 72.0) * n ** 3 for n, _ in boxes),
                "flops": sum(evals * _force_flops(nm, n ** 3) for n, nm in boxes)}
    n = case["n_side"]
    if kind == "ic":
        # transforms: noise, Psi1 (3), second derivatives (6), source, Psi2 (3); a non-Gaussian field adds its own
        ffts = 14 + {None: 0, "local": 2, "equilateral": 5, "orthogonal": 5}[case.get("png")]
        return {"bytes": 52.0 * n ** 3, "flops": ffts * _fft_flops(n) + 150.0 * n ** 3}
    if kind == "pk":
        nm = case["n_mesh"]
        return {"bytes": 12.0 * n ** 3 + 20.0 * case["bins"], "flops": _fft_flops(nm) + 10.0 * nm ** 3 + 60.0 * n ** 3}
    if kind == "bispectrum":
        nm = case["n_mesh"]
        shells = {k for t in _triangles(case) for k in t}
        return {"bytes": 12.0 * n ** 3, "flops": (1 + 2 * len(shells)) * _fft_flops(nm) + 60.0 * n ** 3}
    if kind == "apply":
        return {"bytes": 40.0 * n ** 3, "flops": NET_FLOPS * n ** 3}
    return {"bytes": 36.0 * n ** 3 + 28.0 * 259443, "flops": 3.0 * NET_FLOPS * n ** 3}


# --- cosmology and initial fields (plain numpy and torch) --------------------------------------------------------------

_X, _W = np.polynomial.legendre.leggauss(128)


def _integral(f, lo, hi):
    x = 0.5 * (hi - lo) * _X + 0.5 * (hi + lo)
    return 0.5 * (hi - lo) * float(np.sum(_W * f(x)))


def _E(a):
    return np.sqrt(OM / a ** 3 + 1.0 - OM)


def _heath(a):
    # int_0^a da / (a E)^3 with a = s^(2/5): the integrand becomes smooth at 0
    return _integral(lambda s: 0.4 * s ** -0.6 / (s ** 0.4 * _E(s ** 0.4)) ** 3, 0.0, a ** 2.5)


def _growth(a):
    """D1, D2, dD1/da, dD2/da."""
    norm, e = _heath(1.0), float(_E(a))
    d1 = e * _heath(a) / norm
    dd1 = -1.5 * OM / (a ** 4 * e * e) * d1 + 1.0 / (a ** 3 * e * e * norm)
    om = OM / (OM + (1.0 - OM) * a ** 3)
    g = om ** (-1.0 / 143.0)
    dg = (-1.0 / 143.0) * g / om * (-3.0 * om * (1.0 - om) / a)
    return d1, -3.0 / 7.0 * d1 ** 2 * g, dd1, -3.0 / 7.0 * (2.0 * d1 * dd1 * g + d1 ** 2 * dg)


def _frame(a):
    """p = f1 Psi1 + f2 Psi2 of the LPT trajectory."""
    _, _, dd1, dd2 = _growth(a)
    return a ** 3 * float(_E(a)) * dd1, a ** 3 * float(_E(a)) * dd2


def _transfer(k):
    q = k / (OM * H)
    poly = 1.0 + 3.89 * q + (16.1 * q) ** 2 + (5.46 * q) ** 3 + (6.71 * q) ** 4
    log = torch.log1p if isinstance(k, torch.Tensor) else np.log1p
    return log(2.34 * q) / (2.34 * q) * poly ** -0.25


def _amplitude():
    """A of P = A k^ns T^2 with sigma(8 Mpc/h) = SIGMA8."""
    lnk = np.linspace(math.log(1e-7), math.log(1e3), 2000001)
    k = np.exp(lnk)
    x = 8.0 * k
    w = np.where(x < 1e-3, 1.0 - x ** 2 / 10.0, 3.0 * (np.sin(x) - x * np.cos(x)) / x ** 3)
    f = k ** (3.0 + NS) * _transfer(k) ** 2 * w ** 2
    return SIGMA8 ** 2 * 2.0 * math.pi ** 2 / float(np.sum(0.5 * (f[1:] + f[:-1])) * (lnk[1] - lnk[0]))


def _memo(f, cache={}):
    if f not in cache:
        cache[f] = f()
    return cache[f]


def _axes(n, box, dtype):
    """Wavenumbers along x, y and z of an r2c half spectrum (broadcastable) and the signed indices."""
    nf = torch.fft.fftfreq(n, 1.0 / n, device=DEV, dtype=dtype)
    nh = torch.arange(n // 2 + 1, device=DEV, dtype=dtype)
    idx = (nf[:, None, None], nf[None, :, None], nh[None, None, :])
    return [2.0 * math.pi / box * i for i in idx], idx


def _modes(n, box, dtype):
    """Axes, |k|^2 with 1 where a mode is dropped (k = 0 or a Nyquist index on some axis), and that mask."""
    ks, idx = _axes(n, box, dtype)
    k2 = ks[0] ** 2 + ks[1] ** 2 + ks[2] ** 2
    drop = (k2 == 0) | (idx[0].abs() == n // 2) | (idx[1].abs() == n // 2) | (idx[2] == n // 2)
    return ks, torch.where(drop, torch.ones_like(k2), k2), drop


def _inverse(spec, n):
    return torch.fft.irfftn(spec, s=(n, n, n))


def _lpt(dhat, n, box):
    """Psi1 and Psi2, each [3, n^3], of the linear density's half spectrum."""
    ks, k2, drop = _modes(n, box, dhat.real.dtype)
    phi = torch.where(drop, 0, dhat) / k2  # minus the Lagrangian potential phi1
    psi1 = torch.stack([_inverse(1j * k * phi, n).reshape(-1) for k in ks])
    d2 = lambda i, j: _inverse(ks[i] * ks[j] * phi, n)  # noqa: E731
    xx, yy, zz = d2(0, 0), d2(1, 1), d2(2, 2)
    src = xx * yy + xx * zz + yy * zz
    del xx, yy, zz
    for i, j in ((0, 1), (0, 2), (1, 2)):
        src -= d2(i, j) ** 2
    phi = torch.where(drop, 0, torch.fft.rfftn(src)) / k2
    return psi1, torch.stack([_inverse(-1j * k * phi, n).reshape(-1) for k in ks])


def _lattice(n, box, dtype=torch.float32):
    g = (torch.arange(n, device=DEV, dtype=torch.float64) + 0.5) * (box / n)
    return torch.stack([x.reshape(-1) for x in torch.meshgrid(g, g, g, indexing="ij")]).to(dtype)


def _particles(n, box, a, seed):
    """FP32 particles of a Gaussian field of the library's spectrum at scale factor a: pos, vel, psi1, psi2, q."""
    gen = torch.Generator(DEV).manual_seed(seed)
    noise = torch.randn((n, n, n), generator=gen, device=DEV)
    _, k2, drop = _modes(n, box, torch.float32)
    k = k2.sqrt()
    amp = (_memo(_amplitude) * k ** NS * _transfer(k) ** 2 * (n / box) ** 3).sqrt()
    psi1, psi2 = _lpt(torch.where(drop, 0, torch.fft.rfftn(noise) * amp), n, box)
    del noise, k2, drop, k, amp
    d1, d2, _, _ = _growth(a)
    f1, f2 = _frame(a)
    q = _lattice(n, box)
    pos = torch.remainder(q + d1 * psi1 + d2 * psi2, box)
    pos[pos >= box] = 0.0
    return pos, f1 * psi1 + f2 * psi2, psi1, psi2, q


def _clumps(count, box, seed):
    """A late-time distribution: 70 % of the particles in eight Gaussian clumps of width 0.01 L, the rest uniform."""
    gen = torch.Generator(DEV).manual_seed(seed)
    n_in = int(0.7 * count)
    centres = torch.rand((3, 8), generator=gen, device=DEV)
    which = torch.randint(0, 8, (n_in,), generator=gen, device=DEV)
    pos = torch.cat([centres[:, which] + 0.01 * torch.randn((3, n_in), generator=gen, device=DEV),
                     torch.rand((3, count - n_in), generator=gen, device=DEV)], dim=1)
    pos = torch.remainder(pos, 1.0) * box
    pos[pos >= box] = 0.0
    return pos.contiguous()


def _triangles(case):
    return [tuple(float(k) for k in t.split(",")) for t in case["triangles"].split(";")]


def _boxes(case):
    """(n_side, n_mesh, box) of every box of a run."""
    if case["kind"] == "cola":
        return [(case["n_side"], case["n_mesh"], case["box"])]
    sides = [int(s) for s in case["sides"].split(",")]
    return [(sides[j % len(sides)], case["ratio"] * sides[j % len(sides)], case["box"] + case["box_step"] * j)
            for j in range(case["boxes"])]


def _a_list(case):
    """The last `steps` steps of the ten-step schedule a = 0.1 + 0.09 i."""
    return [1.0 - 0.09 * (case["steps"] - i) for i in range(case["steps"])] + [1.0]


# The correction network: (kind, cin, cout) in parameter order, taps 27 (3^3) or 8 (2^3).
LAYERS = (("conv", 6, 16), ("conv", 16, 16), ("down", 16, 32), ("conv", 32, 32), ("down", 32, 64), ("conv", 64, 64),
          ("up", 64, 32), ("conv", 64, 32), ("up", 32, 16), ("conv", 32, 16), ("conv", 16, 3))


def _net_params(gen):
    """Weights uniform in +-sqrt(6 / fan-in) (a tenth of it in the last layer) and small biases, as one FP32 vector."""
    parts = []
    for i, (kind, cin, cout) in enumerate(LAYERS):
        taps = 27 if kind == "conv" else 8
        s = math.sqrt(6.0 / (taps * cin)) * (0.1 if i + 1 == len(LAYERS) else 1.0)
        parts += [(2.0 * torch.rand(cout * taps * cin, generator=gen, device=DEV) - 1.0) * s,
                  0.02 * (torch.rand(cout, generator=gen, device=DEV) - 0.5)]
    return torch.cat(parts).contiguous()


def _features(case, seed):
    """Input grid [N^3][6] of a coarse run (displacement and Psi1 in lattice units) and its residual target [N^3][3]."""
    n, box = case["n_side"], case["box"]
    pos, _, psi1, psi2, q = _particles(n, box, 1.0, seed)
    d = pos - q
    d -= box * torch.round(d / box)
    feat = torch.cat([d, psi1]).t().contiguous() * (n / box)
    gen = torch.Generator(DEV).manual_seed(seed + 1)
    target = 0.05 * (psi2.t() * (n / box)) + 0.1 * torch.randn((n ** 3, 3), generator=gen, device=DEV)
    return feat, target.contiguous()


# --- prepare and run -------------------------------------------------------------------------------------------------

def prepare(case, seed):
    kind = case["kind"]
    st = {"kind": kind, "cosmo": lpc.cosmology(OM, H, SIGMA8, NS)}
    if kind in ("cola", "batch"):
        return _prepare_run(case, seed, st)
    n, box = case.get("n_side"), case["box"]
    if kind == "force":
        st["pos"] = _clumps(case["count"], box, seed) if "count" in case else _particles(n, box, case["a"], seed)[0]
        count = st["pos"].shape[1]
        st["geom"] = lpc.geometry(n or 2, case["n_mesh"], box)
        st["step"] = lpc.stepping(deconv_power=case["deconv"])
        st["ws"] = lpc.workspace(st["geom"], lpc.LPC_OP_PM_FORCE, n_particles=count)
        st["grad"] = torch.empty((3, count), device=DEV)
        m = case["n_mesh"]
        st["density"] = torch.empty((m, m, m), dtype=torch.int64, device=DEV) if case.get("density") else None
    elif kind == "ic":
        st["geom"] = lpc.geometry(n, n, box)
        st["seed"], st["a"] = seed, case["a"]
        st["png"] = lpc.png(case["f_nl"], kind=case["png"]) if case.get("png") else None
        st["ps"] = lpc.ParticleSet.empty(n ** 3)
        st["ws"] = lpc.workspace(st["geom"], lpc.LPC_OP_INIT_IC)
        st["box"], st["shift"] = box, 0.5 * box - _lattice(n, box)
    elif kind in ("pk", "bispectrum"):
        st["pos"] = _particles(n, box, 1.0, seed)[0]
        st["geom"] = lpc.geometry(n, case["n_mesh"], box)
        st["ws"] = lpc.workspace(st["geom"], lpc.LPC_OP_POWER_SPECTRUM if kind == "pk" else lpc.LPC_OP_BISPECTRUM)
        if kind == "pk":
            st["k_max"], st["bins"] = case["k_max"], case["bins"]
        else:
            st["tri"], st["dk"] = _triangles(case), case["dk_kf"] * 2.0 * math.pi / box
    else:
        st["geom"] = lpc.geometry(n, n, box)
        st["ws"] = lpc.net_workspace(n)
        gen = torch.Generator(DEV).manual_seed(seed + 7)
        st["params0"] = _net_params(gen)
        if kind == "apply":
            pos, vel, psi1, psi2, q = _particles(n, box, 1.0, seed)
            st["pos0"], st["box"], st["shift"] = pos, box, 0.5 * box - q
            st["ps"] = lpc.ParticleSet(pos.clone(), vel, psi1, psi2,
                                       torch.arange(n ** 3, dtype=torch.int32, device=DEV))
        else:
            st["n"] = n
            st["feat"], st["target"] = _features(case, seed)
            # Adam's moments some way into the training
            st["m0"] = 1e-3 * torch.randn(st["params0"].shape, generator=gen, device=DEV)
            st["v0"] = 1e-5 * (0.1 + torch.rand(st["params0"].shape, generator=gen, device=DEV))
            for k in ("params", "m", "v"):
                st[k] = st[k + "0"].clone()
            st["grad"] = torch.empty_like(st["params0"])
    return st


def _prepare_run(case, seed, st):
    boxes, a = _boxes(case), _a_list(case)
    total = sum(n ** 3 for n, _, _ in boxes)
    flat = {k: torch.empty(3 * total, device=DEV) for k in ("pos0", "vel0", "pos", "vel", "psi1", "psi2", "shift")}
    ids, runs, at = torch.empty(total, dtype=torch.int32, device=DEV), [], 0
    for j, (n, nm, box) in enumerate(boxes):
        view = {k: v[3 * at:3 * (at + n ** 3)].view(3, n ** 3) for k, v in flat.items()}
        pos, vel, psi1, psi2, q = _particles(n, box, a[0], seed + j)
        for k, v in (("pos0", pos), ("vel0", vel), ("psi1", psi1), ("psi2", psi2), ("shift", 0.5 * box - q)):
            view[k].copy_(v)
        ids[at:at + n ** 3] = torch.arange(n ** 3, dtype=torch.int32, device=DEV)
        runs.append((lpc.geometry(n, nm, box),
                     lpc.ParticleSet(view["pos"], view["vel"], view["psi1"], view["psi2"], ids[at:at + n ** 3]),
                     view["shift"], box))
        at += n ** 3
    st.update(flat=flat, ids=ids, runs=runs, a=a, boxes=[(g, ps) for g, ps, _, _ in runs])
    st["step"] = lpc.stepping(cola=0 if case.get("plain") else 1, modified=0 if case.get("standard") else 1,
                              n_lpt=N_LPT, deconv_power=case.get("deconv", 1))
    st["ws"] = (lpc.workspace(runs[0][0], lpc.LPC_OP_COLA_STEP) if case["kind"] == "cola"
                else lpc.workspace_batched(st["boxes"]))
    st["rel"] = torch.empty(3 * total, device=DEV)
    return st


def run(st):
    kind = st["kind"]
    if kind == "force":
        lpc.lpc_pm_force(st["geom"], st["step"], st["pos"], st["grad"], st["ws"], density_out=st["density"])
        return [st["grad"]] if st["density"] is None else [st["grad"], st["density"]]
    if kind in ("cola", "batch"):
        f = st["flat"]
        f["pos"].copy_(f["pos0"])  # the run advances its particles in place: start from the kept snapshot
        f["vel"].copy_(f["vel0"])
        if kind == "cola":
            lpc.lpc_cola_step(st["runs"][0][0], st["cosmo"], st["step"], st["a"], st["runs"][0][1], st["ws"])
        else:
            lpc.lpc_cola_step_batched(st["boxes"], st["cosmo"], st["step"], st["a"], st["ws"])
        at = 0
        for _, ps, shift, box in st["runs"]:
            rel = st["rel"][at:at + 3 * ps.n].view(3, ps.n)
            torch.add(ps.pos, shift, out=rel)
            rel.remainder_(box)
            at += 3 * ps.n
        return {"pos": st["rel"], "vel": f["vel"]}
    if kind == "ic":
        ps = st["ps"]
        if st["png"] is None:
            lpc.lpc_init_ic(st["geom"], st["cosmo"], st["seed"], st["a"], ps, st["ws"])
        else:
            lpc.lpc_init_ic_png(st["geom"], st["cosmo"], st["seed"], st["a"], st["png"], ps, st["ws"])
        return {"pos": torch.add(ps.pos, st["shift"]).remainder_(st["box"]), "vel": ps.vel, "psi1": ps.psi1,
                "psi2": ps.psi2, "id": ps.id}
    if kind == "pk":
        k, p, cnt = lpc.lpc_power_spectrum(st["geom"], st["pos"], st["k_max"], st["bins"], st["ws"])
        return {"k": k, "p": p.astype(np.float32), "modes": cnt}
    if kind == "bispectrum":
        b, q, p = lpc.lpc_bispectrum(st["geom"], st["pos"], st["tri"], st["dk"], st["ws"])
        return {"b": b.astype(np.float32), "q": q.astype(np.float32), "p": p.astype(np.float32)}
    if kind == "apply":
        ps = st["ps"]
        ps.pos.copy_(st["pos0"])
        lpc.lpc_net_apply(st["geom"], st["params0"], ps, st["ws"])
        return torch.add(ps.pos, st["shift"]).remainder_(st["box"])
    for k in ("params", "m", "v"):
        st[k].copy_(st[k + "0"])
    loss = lpc.lpc_net_loss_grad(st["n"], st["params"], st["feat"], st["target"], st["grad"], st["ws"])
    lpc.lpc_net_adam(st["params"], st["m"], st["v"], st["grad"], 100, 1e-3)
    return {"loss": loss, "grad": st["grad"], "params": st["params"], "m": st["m"], "v": st["v"]}


# --- the same in FP64 ----------------------------------------------------------------------------------------------

def _cells(pos, nm, box):
    """Cell and 16-bit fraction of each coordinate (the deposit's fixed-point rule)."""
    u = torch.floor(pos.double() * (nm * 65536.0 / box)).long() % (nm << 16)
    return u >> 16, u & 0xffff


def _corners(cell, nm):
    for c in range(8):
        d = (c >> 2 & 1, c >> 1 & 1, c & 1)
        i = [(cell[a] + d[a]) % nm for a in range(3)]
        yield d, (i[0] * nm + i[1]) * nm + i[2]


def _density(pos, nm, box):
    """Fixed-point CIC counts, int64 [nm^3]; every particle adds 2^48."""
    cell, frac = _cells(pos, nm, box)
    out = torch.zeros(nm ** 3, dtype=torch.int64, device=DEV)
    for d, at in _corners(cell, nm):
        w = [frac[a] if d[a] else 65536 - frac[a] for a in range(3)]
        out.index_add_(0, at, w[0] * w[1] * w[2])
    return out


def _delta_hat(pos, nm, box):
    counts = _density(pos, nm, box)
    return torch.fft.rfftn((counts.double() * (nm ** 3 / pos.shape[1] * 2.0 ** -48) - 1.0).reshape(nm, nm, nm)), counts


def _window(nm):
    _, idx = _axes(nm, 1.0, torch.float64)
    return torch.sinc(idx[0] / nm) ** 2 * torch.sinc(idx[1] / nm) ** 2 * torch.sinc(idx[2] / nm) ** 2


def _force(pos, nm, box, deconv):
    dhat, counts = _delta_hat(pos, nm, box)
    ks, idx = _axes(nm, box, torch.float64)
    k2 = ks[0] ** 2 + ks[1] ** 2 + ks[2] ** 2
    k2[0, 0, 0] = 1.0
    dhat /= -k2
    del k2
    dhat[0, 0, 0] = 0
    if deconv:
        dhat /= _window(nm) ** deconv
    cell, frac = _cells(pos, nm, box)
    frac = frac.double() / 65536.0
    grad = torch.empty(pos.shape, dtype=torch.float64, device=DEV)
    for j in range(3):
        mesh = _inverse(1j * torch.where(idx[j].abs() == nm // 2, 0.0, ks[j]) * dhat, nm).reshape(-1)
        acc = torch.zeros(pos.shape[1], dtype=torch.float64, device=DEV)
        for d, at in _corners(cell, nm):
            w = [frac[a] if d[a] else 1.0 - frac[a] for a in range(3)]
            acc += w[0] * w[1] * w[2] * mesh[at]
        grad[j] = acc
    return grad, counts


def _run_exact(pos, vel, psi1, psi2, case, nm, box):
    a = _a_list(case)
    cola, modified, deconv = not case.get("plain"), not case.get("standard"), case.get("deconv", 1)
    x, p, psi1, psi2 = pos.double(), vel.double(), psi1.double(), psi2.double()
    if cola:
        f1, f2 = _frame(a[0])
        p = p - (f1 * psi1 + f2 * psi2)
    for i, ai in enumerate(a):
        lo = 0.5 * (a[i - 1] + ai) if i else ai
        hi = 0.5 * (ai + a[i + 1]) if i + 1 < len(a) else ai
        if modified:
            kick = (hi ** N_LPT - lo ** N_LPT) / (N_LPT * ai ** (N_LPT - 1.0) * ai ** 2 * float(_E(ai)))
        else:
            kick = _integral(lambda s: 1.0 / (s ** 2 * _E(s)), lo, hi)
        d1, d2, _, _ = _growth(ai)
        acc, _ = _force(x, nm, box, deconv)
        if cola:
            acc = acc + d1 * psi1 + (d2 - d1 * d1) * psi2
        p = p + kick * (-1.5 * OM) * acc
        if i + 1 < len(a):
            u = (lambda s: s ** N_LPT) if modified else (lambda s: 1.0)
            drift = _integral(lambda s: u(s) / (s ** 3 * _E(s)), ai, a[i + 1]) / u(0.5 * (ai + a[i + 1]))
            x = x + drift * p
            if cola:
                e1, e2, _, _ = _growth(a[i + 1])
                x = x + (e1 - d1) * psi1 + (e2 - d2) * psi2
            x = torch.remainder(x, box)
    if cola:
        f1, f2 = _frame(a[-1])
        p = p + f1 * psi1 + f2 * psi2
    return x, p


def _i64(v):
    return v - (1 << 64) if v >= 1 << 63 else v


def _white_noise(seed, n):
    """SplitMix64 in counter mode and Box-Muller, as lpc_init_ic documents."""
    def mix(c):
        z = (c + 1) * _i64(0x9E3779B97F4A7C15) + _i64(seed)
        z = (z ^ ((z >> 30) & ((1 << 34) - 1))) * _i64(0xBF58476D1CE4E5B9)
        z = (z ^ ((z >> 27) & ((1 << 37) - 1))) * _i64(0x94D049BB133111EB)
        z = z ^ ((z >> 31) & ((1 << 33) - 1))
        return (((z >> 11) & ((1 << 53) - 1)).double() + 0.5) * 2.0 ** -53

    c = torch.arange(n ** 3, dtype=torch.int64, device=DEV)
    return (torch.sqrt(-2.0 * torch.log(mix(2 * c))) * torch.cos(2.0 * math.pi * mix(2 * c + 1))).reshape(n, n, n)


PNG_TERMS = {"local": [(1.0, 0, 0, 0)],
             "equilateral": [(-3.0, 0, 0, 0), (6.0, 1, 0, -1), (-2.0, 1, 1, -2)],
             "orthogonal": [(-9.0, 0, 0, 0), (18.0, 1, 0, -1), (-8.0, 1, 1, -2)]}


def _ic_exact(case, seed):
    n, box, a = case["n_side"], case["box"], case["a"]
    amp, norm = _memo(_amplitude), (n / box) ** 3
    _, k2, drop = _modes(n, box, torch.float64)
    k = k2.sqrt()
    noise = torch.where(drop, 0, torch.fft.rfftn(_white_noise(seed, n)))
    if not case.get("png"):
        dhat = noise * (amp * k ** NS * _transfer(k) ** 2 * norm).sqrt()
    else:
        alpha0 = 2.0 / 3.0 * C_OVER_H0 ** 2 * (2.5 * OM * _heath(1.0)) / OM
        phi = noise * (amp * k ** (NS - 4.0) / alpha0 ** 2 * norm).sqrt()
        power = lambda s: k ** (s * (4.0 - NS) / 3.0)  # noqa: E731
        nl = torch.zeros_like(phi)
        for c, ea, eb, g in PNG_TERMS[case["png"]]:
            nl += c * power(g) * torch.fft.rfftn(_inverse(phi * power(ea), n) * _inverse(phi * power(eb), n))
        dhat = alpha0 * k2 * _transfer(k) * torch.where(drop, 0, phi + case["f_nl"] * nl)
    psi1, psi2 = _lpt(dhat, n, box)
    d1, d2, _, _ = _growth(a)
    f1, f2 = _frame(a)
    return {"pos": torch.remainder(0.5 * box + d1 * psi1 + d2 * psi2, box), "vel": f1 * psi1 + f2 * psi2, "psi1": psi1,
            "psi2": psi2, "id": None}


def _shell(kmag, kc, dk):
    return (kmag >= kc - 0.5 * dk) & (kmag < kc + 0.5 * dk)


def _net(params, x):
    """The correction network on x [6, D, D, D] in FP64."""
    def layer(i, x, act=True):
        kind, cin, cout = LAYERS[i]
        taps = 27 if kind == "conv" else 8
        off = sum(co * (27 if k == "conv" else 8) * ci + co for k, ci, co in LAYERS[:i])
        w = params[off:off + cout * taps * cin].view(cout, taps, cin)
        b = params[off + cout * taps * cin:off + cout * taps * cin + cout].view(cout, 1, 1, 1)
        dot = lambda t, v: (w[:, t] @ v.reshape(cin, -1)).view((cout,) + v.shape[1:])  # noqa: E731
        if kind == "conv":
            out = b
            for t in range(27):
                out = out + dot(t, torch.roll(x, (1 - t // 9, 1 - t // 3 % 3, 1 - t % 3), (1, 2, 3)))
        elif kind == "down":
            out = b
            for t in range(8):
                out = out + dot(t, x[:, t >> 2::2, t >> 1 & 1::2, t & 1::2])
        else:
            d = x.shape[1]
            out = torch.stack([dot(t, x) for t in range(8)]).view(2, 2, 2, cout, d, d, d)
            out = out.permute(3, 4, 0, 5, 1, 6, 2).reshape(cout, 2 * d, 2 * d, 2 * d) + b
        return torch.where(out > 0, out, 0.1 * out) if act else out

    s0 = layer(1, layer(0, x))
    s1 = layer(3, layer(2, s0))
    u1 = layer(6, layer(5, layer(4, s1)))
    u0 = layer(8, layer(7, torch.cat([u1, s1])))
    return layer(10, layer(9, torch.cat([u0, s0])), act=False)


def exact(case, seed):
    kind, st = case["kind"], None
    if kind == "ic":
        return _ic_exact(case, seed)
    if kind in ("cola", "batch"):
        a, xs, vs = _a_list(case), [], []
        for j, (n, nm, box) in enumerate(_boxes(case)):
            pos, vel, psi1, psi2, q = _particles(n, box, a[0], seed + j)
            x, p = _run_exact(pos, vel, psi1, psi2, case, nm, box)
            xs.append(torch.remainder(x + (0.5 * box - q.double()), box).reshape(-1))
            vs.append(p.reshape(-1))
        return {"pos": torch.cat(xs), "vel": torch.cat(vs)}
    n, box, nm = case.get("n_side"), case["box"], case.get("n_mesh")
    if kind == "force":
        pos = _clumps(case["count"], box, seed) if "count" in case else _particles(n, box, case["a"], seed)[0]
        grad, counts = _force(pos, nm, box, case["deconv"])
        return [grad, counts.reshape(nm, nm, nm)] if case.get("density") else [grad]
    if kind in ("pk", "bispectrum"):
        dhat, _ = _delta_hat(_particles(n, box, 1.0, seed)[0], nm, box)
        dhat /= _window(nm)
        idx = _axes(nm, box, torch.float64)[1]
        kmag = 2.0 * math.pi / box * torch.sqrt(idx[0] ** 2 + idx[1] ** 2 + idx[2] ** 2)
        mult = torch.where((idx[2] > 0) & (idx[2] < nm // 2), 2.0, 1.0).double().expand(kmag.shape)
        power = (dhat.real ** 2 + dhat.imag ** 2) * (box / nm ** 2) ** 3
    if kind == "pk":
        b = torch.floor(kmag / (case["k_max"] / case["bins"])).long()
        use = (kmag > 0) & (b < case["bins"])
        total = lambda v: torch.bincount(b[use], v[use], case["bins"])  # noqa: E731
        cnt = total(mult)
        return {"k": total(mult * kmag) / cnt, "p": total(mult * power) / cnt, "modes": cnt.long()}
    if kind == "bispectrum":
        dk, out = case["dk_kf"] * 2.0 * math.pi / box, {"b": [], "q": [], "p": []}
        for tri in _triangles(case):
            num, den, p = 1.0, 1.0, []
            for kc in tri:
                s = _shell(kmag, kc, dk)
                num = num * _inverse(torch.where(s, dhat, 0), nm)
                den = den * _inverse(s.to(torch.complex128), nm)
                p.append(float((mult * power)[s].sum() / mult[s].sum()))
            b = float(num.sum() / den.sum()) * (box ** 2 / nm ** 3) ** 3
            out["b"].append(b)
            out["q"].append(b / (p[0] * p[1] + p[1] * p[2] + p[2] * p[0]))
            out["p"].append(p)
        return {k: np.array(v) for k, v in out.items()}
    st = prepare(case, seed)
    p = st["params0"].double()
    if kind == "apply":
        pos = st["pos0"].double()
        q = _lattice(n, box, torch.float64)
        d = pos - q
        d -= box * torch.round(d / box)
        feat = torch.cat([d, st["ps"].psi1.double()]) * (n / box)
        x = pos + _net(p, feat.view(6, n, n, n)).reshape(3, -1) * (box / n)
        return torch.remainder(x - q + 0.5 * box, box)
    p.requires_grad_(True)
    feat = st["feat"].double().t().reshape(6, n, n, n)
    loss = ((_net(p, feat).reshape(3, -1) - st["target"].double().t()) ** 2).mean()
    loss.backward()
    g = p.grad
    m, v = 0.9 * st["m0"].double() + 0.1 * g, 0.999 * st["v0"].double() + 0.001 * g * g
    new = p.detach() - 1e-3 * (m / (1 - 0.9 ** 100)) / (torch.sqrt(v / (1 - 0.999 ** 100)) + 1e-8)
    return {"loss": float(loss), "grad": g, "params": new, "m": m, "v": v}
