"""Workloads whose speed is measured: calls of the transform plans as a user's program makes them.

Each case is one plan (truncation, grid, fields, precision form) and one call or pair of calls on
it.  `listed` holds fixed cases, from one field on a small full grid (launch latency) to the 9 km
grid with 411 fields (the benchmark workload); `draw` gives others of the same ranges.  Inputs are
made on the GPU from a seed; `exact` evaluates the same maps in plain torch float64.
"""
import math

import numpy as np
import torch

import paper_1908_06097_amd as shtx

# Calls: "step" inverse then direct transform of its grids; "inv", "dir", "inv_adj", "dir_adj"
# one transform; "grad" the inverse transform under autograd, forward and backward; "uv" wind
# images from vorticity and divergence (the plan's truncation is the winds' plus one, its fields
# are U then V).
_CALLS = ("step", "inv", "dir", "inv_adj", "dir_adj", "grad", "uv")


def _case(call, prec, trunc, grid, nlat, nlon, nfld, graph=False, name=None):
    c = {"call": call, "prec": prec, "trunc": trunc, "grid": grid, "nlat": nlat, "nlon": nlon, "nfld": nfld,
         "graph": graph}
    return {"name": name, **c} if name else c


def listed():
    return [
        # one field on a small full grid in double precision: a single analysis, launch-bound
        _case("step", "fp64", 79, "full", 160, 320, 1, name="t79_full_f1_fp64_step"),
        # a serving loop over a few small fields, each transform replayed as a captured graph
        _case("step", "fp32", 63, "octahedral", 128, 0, 5, graph=True, name="t63_o64_f5_fp32_graph_step"),
        # a handful of fields at a moderate resolution (one model state's surface fields)
        _case("step", "fp32", 255, "octahedral", 512, 0, 7, name="t255_o256_f7_fp32_step"),
        # a whole model state (3 variables on 137 levels) at the same resolution
        _case("step", "fp32", 255, "octahedral", 512, 0, 411, name="t255_o256_f411_fp32_step"),
        # an odd count of fields on a full grid, adjoint of the inverse, split bfloat16
        _case("inv_adj", "bf16x3", 213, "full", 320, 640, 37, name="t213_full_f37_bf16x3_inv_adj"),
        # training through the inverse transform: one variable on 137 levels, forward and backward
        _case("grad", "fp32", 399, "octahedral", 800, 0, 137, name="t399_o400_f137_fp32_grad"),
        # 18 km grid, synthesis and analysis of a whole state in the two split forms
        _case("inv", "bf16x3", 639, "octahedral", 1280, 0, 411, name="t639_o640_f411_bf16x3_inv"),
        _case("dir", "fp16x3", 639, "octahedral", 1280, 0, 411, name="t639_o640_f411_fp16x3_dir"),
        # winds on 137 levels from vorticity and divergence of truncation 639
        _case("uv", "fp32", 640, "octahedral", 1280, 0, 274, name="t639_o640_wind137_fp32_uv"),
        # the same grid in double precision, one variable on 137 levels
        _case("step", "fp64", 639, "octahedral", 1280, 0, 137, name="t639_o640_f137_fp64_step"),
        # three surface fields at the highest resolution: the tables are most of the bytes
        _case("inv", "fp32", 1279, "octahedral", 2560, 0, 3, name="t1279_o1280_f3_fp32_inv"),
        # 9 km grid, the benchmark workload
        _case("step", "fp32", 1279, "octahedral", 2560, 0, 411, name="t1279_o1280_f411_fp32_step"),
    ]


def draw(rng):
    def log_int(lo, hi):
        return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))

    prec = rng.choice(["fp32", "fp32", "fp32", "fp64", "bf16x3", "fp16x3"])
    call = rng.choice(["step", "step", "inv", "dir", "inv_adj", "dir_adj", "grad", "uv"])
    full = rng.random() < 0.25
    trunc = log_int(31, 639 if full or prec == "fp64" else 1279)
    nfld = log_int(1, 411)
    if call == "uv":
        nfld = 2 * max(1, nfld // 2)
    if full:
        # linear to quadratic Gaussian grids, twice as many longitudes as latitudes
        nlat = 2 * int(rng.uniform(trunc + 2, 1.5 * trunc + 2) / 2 + 0.5)
        return _case(call, prec, trunc, "full", nlat, 2 * nlat, nfld, rng.random() < 0.25)
    return _case(call, prec, trunc, "octahedral", 2 * (trunc + 1), 0, nfld, rng.random() < 0.25)


def _nlon(case):
    nl = case["nlat"] // 2
    if case["grid"] == "full":
        return np.full(nl, case["nlon"], dtype=np.int64)
    return 20 + 4 * np.arange(nl, dtype=np.int64)


def _device():
    return torch.device("cuda")


def _types(case):
    return (torch.float64, torch.complex128) if case["prec"] == "fp64" else (torch.float32, torch.complex64)


def _spectrum(trunc, nfld, gen, cdtype):
    """Random fields with the (n + 1)^-1.5 amplitudes of smooth fields; real coefficients at m = 0."""
    dev = _device()
    n = torch.cat([torch.arange(m, trunc + 1, device=dev) for m in range(trunc + 1)])
    rdtype = torch.float64 if cdtype == torch.complex128 else torch.float32
    z = torch.randn((nfld, n.numel(), 2), dtype=rdtype, device=dev, generator=gen)
    z *= ((n + 1.0) ** -1.5).to(rdtype)[None, :, None]
    z[:, : trunc + 1, 1] = 0
    return torch.view_as_complex(z)


def _grid(case, gen, rdtype):
    """Grid fields as a model holds them: a mean, a planetary wave and small scales on every ring."""
    dev, F = _device(), case["nfld"]
    north = _nlon(case)
    nlon = np.concatenate([north, north[::-1]])
    npts = int(nlon.sum())
    ring = torch.repeat_interleave(torch.arange(len(nlon), device=dev), torch.from_numpy(nlon).to(dev))
    start = torch.from_numpy(np.concatenate([[0], np.cumsum(nlon)[:-1]])).to(dev)
    n = torch.from_numpy(nlon).to(dev)[ring]
    lam = (torch.arange(npts, device=dev) - start[ring]).double() * (2 * math.pi) / n
    theta = (ring.double() + 0.5) * (math.pi / len(nlon))
    waves = torch.stack([torch.ones_like(lam), theta.cos(), theta.sin() * lam.cos(), theta.sin() * lam.sin()])
    amp = torch.randn((F, 4), dtype=torch.float64, device=dev, generator=gen)
    g = torch.randn((F, npts), dtype=rdtype, device=dev, generator=gen)
    g *= 0.3
    g.addmm_(amp.to(rdtype), waves.to(rdtype))
    return g


def _inputs(case, seed):
    gen = torch.Generator(device=_device())
    gen.manual_seed(seed)
    rdtype, cdtype = _types(case)
    call, N, F = case["call"], case["trunc"], case["nfld"]
    if call == "uv":
        return {"vor": _spectrum(N - 1, F // 2, gen, cdtype), "div": _spectrum(N - 1, F // 2, gen, cdtype)}
    got = {}
    if call in ("step", "inv", "dir_adj", "grad"):
        got["spec"] = _spectrum(N, F, gen, cdtype)
    if call in ("dir", "inv_adj", "grad"):
        got["grid"] = _grid(case, gen, rdtype)
    return got


def prepare(case, seed):
    plan = shtx.Plan(case["trunc"], case["grid"], case["nlat"], case["nfld"], case["prec"], nlon_full=case["nlon"],
                     graph=case["graph"], uv=case["call"] == "uv")
    state = {"call": case["call"], "plan": plan, "stream": None, "grid_out": None, "spec_out": None,
             **_inputs(case, seed)}
    if case["call"] == "grad":
        state["spec"].requires_grad_()
    elif case["graph"]:
        # graph replay wants a stream of its own and buffers that stay where they are
        state["stream"] = torch.cuda.Stream()
        if case["call"] in ("step", "inv", "dir_adj", "uv"):
            state["grid_out"] = torch.empty((plan.nfld, plan.npts), dtype=plan.real_dtype, device=_device())
        if case["call"] in ("step", "dir", "inv_adj"):
            state["spec_out"] = torch.empty((plan.nfld, plan.nspec), dtype=plan.complex_dtype, device=_device())
    return state


def _call(s):
    plan, call = s["plan"], s["call"]
    if call == "step":
        g = plan.inv(s["spec"], out=s["grid_out"])
        return {"grid": g, "spec": plan.dir(g, out=s["spec_out"])}
    if call == "grad":
        g = shtx.InvTrans.apply(s["spec"], plan)
        (d,) = torch.autograd.grad(g, s["spec"], s["grid"])
        return {"grid": g, "grad": d}
    if call == "uv":
        return {"grid": plan.uv(s["vor"], s["div"], out=s["grid_out"])}
    if call in ("inv", "dir_adj"):
        return {"grid": getattr(plan, call)(s["spec"], out=s["grid_out"])}
    return {"spec": getattr(plan, call)(s["grid"], out=s["spec_out"])}


def run(state):
    if state["stream"] is None:
        return _call(state)
    with torch.cuda.stream(state["stream"]):
        return _call(state)


def work(case):
    """Per leg: the table entries the method needs, the spectral array and the grid, each once; the
    even/odd-folded Legendre sums and 2.5 n log2 n for each ring's real FFT."""
    N, F, dbl = case["trunc"], case["nfld"], case["prec"] == "fp64"
    nlon = _nlon(case)
    M = np.minimum(N, (nlon - 1) // 2)
    entries = int(((M + 1) * (N + 1) - M * (M + 1) // 2).sum())
    npts, nspec, real = 2 * int(nlon.sum()), (N + 1) * (N + 2) // 2, 8 if dbl else 4
    legs = 2 if case["call"] in ("step", "grad") else 1
    fft = 2 * float((2.5 * nlon * np.log2(nlon)).sum())
    return {"bytes": legs * (entries * real + F * (nspec * 2 + npts) * real),
            "flops": legs * F * (4.0 * entries + fft)}


# ---------------------------------------------------------------------------------------------
# The same maps in float64 torch: Gauss nodes by Newton's method in extended precision, the
# three-term recurrence of the normalised functions, dense Legendre and Fourier sums.
# ---------------------------------------------------------------------------------------------

def _gauss(nlat):
    """Northern Gauss-Legendre nodes (descending) and weights."""
    ld = np.longdouble
    i = np.arange(1, nlat // 2 + 1)
    x = np.cos(np.pi * (i - 0.25) / (nlat + 0.5)).astype(ld)
    for _ in range(5):
        p0, p1 = np.ones_like(x), x.copy()
        for n in range(2, nlat + 1):
            p0, p1 = p1, ((2 * n - 1) * x * p1 - (n - 1) * p0) / ld(n)
        d = nlat * (p0 - x * p1) / (1 - x * x)
        x = x - p1 / d
    w = 2 / ((1 - x * x) * d * d)
    return x.astype(np.float64), w.astype(np.float64)


def _legendre(N, mu):
    """P[n, m, j] with mean square 1 over the sphere's latitudes, no Condon-Shortley phase."""
    dev = _device()
    x = torch.from_numpy(mu).to(dev)
    s = torch.sqrt((1 - x) * (1 + x))
    P = torch.zeros((N + 1, N + 1, len(mu)), dtype=torch.float64, device=dev)
    m = torch.arange(N + 1, dtype=torch.float64, device=dev)
    P[0, 0] = 1
    for n in range(1, N + 1):
        P[n, n] = P[n - 1, n - 1] * s * math.sqrt((2 * n + 1) / (2 * n))
        P[n, n - 1] = P[n - 1, n - 1] * x * math.sqrt(2 * n + 1)
        if n > 1:
            q = m[: n - 1]
            den = n * n - q * q
            a = torch.sqrt((4.0 * n * n - 1) / den)
            b = torch.sqrt((2 * n + 1) * (n - 1 - q) * (n - 1 + q) / ((2 * n - 3) * den))
            P[n, : n - 1] = a[:, None] * x * P[n - 1, : n - 1] - b[:, None] * P[n - 2, : n - 1]
    return P


def _waves(n, M):
    """cos and sin of 2 pi m k / n, m = 0 .. M, k = 0 .. n - 1."""
    dev = _device()
    a = torch.arange(n, dtype=torch.float64, device=dev) * (2 * math.pi / n)
    at = torch.arange(M + 1, device=dev)[:, None] * torch.arange(n, device=dev) % n
    return a.cos()[at], a.sin()[at]


def _exact_to_grid(case, P, w, a, adjoint):
    N, F = case["trunc"], a.shape[0]
    nlon = _nlon(case)
    nl = len(nlon)
    four = torch.empty((N + 1, 4 * F, nl), dtype=torch.float64, device=a.device)
    at = 0
    for m in range(N + 1):
        K = N + 1 - m
        z = a[:, at:at + K]
        at += K
        im = torch.zeros_like(z.imag) if m == 0 else z.imag
        sign = 1.0 - 2.0 * (torch.arange(K, device=a.device) % 2)
        four[m] = torch.cat([z.real, im, z.real * sign, im * sign]) @ P[m:, m]
    npts = 2 * int(nlon.sum())
    g = torch.empty((F, npts), dtype=torch.float64, device=a.device)
    start = np.concatenate([[0], np.cumsum(nlon)])
    for j in range(nl):
        n, M = int(nlon[j]), min(N, (int(nlon[j]) - 1) // 2)
        y = four[: M + 1, :, j].t().contiguous().view(2, 2, F, M + 1)  # hemisphere, re/im, field, m
        if adjoint:
            y *= w[j] / (2 * n)
        else:
            y[..., 1:] *= 2
        c, s = _waves(n, M)
        r = (y[:, 0].reshape(2 * F, -1) @ c - y[:, 1].reshape(2 * F, -1) @ s).view(2, F, n)
        at = int(start[j])
        g[:, at:at + n] = r[0]
        g[:, npts - at - n:npts - at] = r[1]
    return g


def _exact_to_spec(case, P, w, g, adjoint):
    N, F = case["trunc"], g.shape[0]
    nlon = _nlon(case)
    nl, npts = len(nlon), g.shape[1]
    four = torch.zeros((nl, 4 * F, N + 1), dtype=torch.float64, device=g.device)
    start = np.concatenate([[0], np.cumsum(nlon)])
    for j in range(nl):
        n, M = int(nlon[j]), min(N, (int(nlon[j]) - 1) // 2)
        at = int(start[j])
        c, s = _waves(n, M)
        x = torch.cat([g[:, at:at + n], g[:, npts - at - n:npts - at]])
        re, im = x @ c.t(), x @ s.t()
        y = torch.stack([re[:F] + re[F:], -im[:F] - im[F:], re[:F] - re[F:], im[F:] - im[:F]])
        if adjoint:
            y[..., 1:] *= 2
        else:
            y *= w[j] / (2 * n)
        four[j, :, : M + 1] = y.view(4 * F, M + 1)
    a = torch.empty((F, (N + 1) * (N + 2) // 2), dtype=torch.complex128, device=g.device)
    at = 0
    for m in range(N + 1):
        K = N + 1 - m
        y = four[:, :, m].t().contiguous()
        even, odd = y[: 2 * F] @ P[m::2, m].t(), y[2 * F:] @ P[m + 1::2, m].t()
        a[:, at:at + K:2] = torch.complex(even[:F], even[F:] if m else torch.zeros_like(even[F:]))
        a[:, at + 1:at + K:2] = torch.complex(odd[:F], odd[F:] if m else torch.zeros_like(odd[F:]))
        at += K
    return a


def _exact_winds(N, vor, div):
    """Spectral U = u cos(phi) and V = v cos(phi) of truncation N + 1, fields U then V."""
    F, dev = vor.shape[0], vor.device
    out = torch.zeros((2 * F, (N + 2) * (N + 3) // 2), dtype=torch.complex128, device=dev)
    at_in = at_out = 0
    for m in range(N + 2):
        K = N + 2 - m
        n = torch.arange(m, N + 3, dtype=torch.float64, device=dev)  # m .. N + 2
        eps = torch.sqrt((n * n - m * m) / (4 * n * n - 1))
        pot = torch.zeros((2, F, K + 2), dtype=torch.complex128, device=dev)  # degrees m - 1 .. N + 2
        if m <= N:
            scale = torch.where(n > 0, -1 / (n * (n + 1)), torch.zeros_like(n))[: K - 1]
            for i, x in enumerate((vor, div)):
                z = x[:, at_in:at_in + K - 1]
                pot[i, :, 1:K] = (z.real + 0j if m == 0 else z) * scale
            at_in += K - 1
        k = n[:K]
        slope = (k + 2) * eps[1:] * pot[:, :, 2:] - (k - 1) * eps[:K] * pot[:, :, :K]
        psi, chi = pot[0, :, 1:K + 1], pot[1, :, 1:K + 1]
        out[:F, at_out:at_out + K] = 1j * m * chi - slope[0]
        out[F:, at_out:at_out + K] = 1j * m * psi + slope[1]
        at_out += K
    return out


def exact(case, seed):
    x = {k: v.to(torch.complex128 if v.is_complex() else torch.float64) for k, v in _inputs(case, seed).items()}
    mu, w = _gauss(case["nlat"])
    P = _legendre(case["trunc"], mu)
    call = case["call"]
    if call == "uv":
        return {"grid": _exact_to_grid(case, P, w, _exact_winds(case["trunc"] - 1, x["vor"], x["div"]), False)}
    if call in ("inv", "dir_adj"):
        return {"grid": _exact_to_grid(case, P, w, x["spec"], call == "dir_adj")}
    if call in ("dir", "inv_adj"):
        return {"spec": _exact_to_spec(case, P, w, x["grid"], call == "inv_adj")}
    g = _exact_to_grid(case, P, w, x["spec"], False)
    if call == "grad":
        return {"grid": g, "grad": _exact_to_spec(case, P, w, x["grid"], True)}
    return {"grid": g, "spec": _exact_to_spec(case, P, w, g, False)}
