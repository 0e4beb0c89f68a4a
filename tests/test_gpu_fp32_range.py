"""Single-precision plans over the whole range of a float.

The tiled FP32 GEMM cuts its operands into bfloat16 pieces; results have to
stay those of single precision for fields of any amplitude, for rings whose
table entries are near the smallest float, and beside values that are not
finite.  Expected values come from the FP64 oracle on the rounded inputs.
"""
import numpy as np
import pytest

import synth_inputs as si
from error_metrics import grid_errors, spec_errors
from test_gpu_transforms import TOL_RMS, _dev, _np, _oracle, _say, _shtx, _torch

pytestmark = pytest.mark.gpu

SHAPES = [(128, 128), (64, 128), (128, 64)]
N, NLAT, F = 63, 128, 40  # more than 32 fields: the tiled kernel in both directions


def _plan(shape):
    shtx = _shtx()
    plan = shtx.Plan(N, "octahedral", NLAT, F, "fp32")
    plan.set_shapes(shape, shape, plan.info.fft_cap)
    return plan, plan.ring_lengths()


# Amplitudes 2^s: around the magnitude (2^-110) below which three bfloat16 pieces
# no longer hold 24 bits, down to where a field's smallest values are
# subnormal, beside ordinary fields and one near the largest float.  Rounding
# to a multiple of 2^-149 in the FFTs is below 2^-23 of a field at 2^-116.
@pytest.mark.parametrize("shape", SHAPES)
def test_amplitudes(shape):
    o = _oracle()
    plan, nlon = _plan(shape)
    _, w = o.gauss(NLAT)
    s = np.array([0, -90, -102, -106, -110, -113, -116, 100])[np.arange(F) % 8]
    amp = np.ldexp(1.0, s)[:, None]
    a = (si.spectral_fields(N, 51, range(F)) * amp).astype(np.complex64)
    y = (np.stack([si.white_noise_grid(int(nlon.sum()), 700 + f) for f in range(F)]) * amp).astype(np.float32)
    a64, y64 = a.astype(np.complex128), y.astype(np.float64)
    spec, grid = _dev(a, plan.complex_dtype), _dev(y, plan.real_dtype)
    for name, got, ref in (("inv", plan.inv(spec), o.inv(N, nlon, a64)),
                           ("dir_adj", plan.dir_adj(spec), o.dir_adj(N, nlon, a64)),
                           ("dir", plan.dir(grid), o.dir(N, nlon, y64)),
                           ("inv_adj", plan.inv_adj(grid), o.inv_adj(N, nlon, y64))):
        # in units of each field's amplitude, so that squares stay in range
        got, ref = _np(got) / amp, ref / amp
        _, er = grid_errors(got, ref, nlon, w) if name in ("inv", "dir_adj") else spec_errors(got, ref, N)
        worst = {int(k): float(er[s == k].max()) for k in sorted(set(s))}
        _say(f"  {shape} {name} rms by exponent {worst}")
        assert np.isfinite(got).all() and er.max() < TOL_RMS["fp32"], (name, worst)


# Amplitudes around the one from which the scaled sums of a tile leave a float's
# range, in steps fine enough for tiles in which only the difference of the two
# parities' sums does.
@pytest.mark.parametrize("shape", SHAPES)
def test_largest_sums(shape):
    shtx, o = _shtx(), _oracle()
    n, nlat, nf = 15, 32, 20
    plan = shtx.Plan(n, "octahedral", nlat, nf, "fp32")
    plan.set_shapes(shape, shape, plan.info.fft_cap)
    nlon = plan.ring_lengths()
    _, w = o.gauss(nlat)
    base = si.spectral_fields(n, 55, range(nf))
    for k in range(8 * 104, 8 * 114):
        amp = 2.0 ** (k / 8)
        a = (base * amp).astype(np.complex64)
        _, er = grid_errors(_np(plan.inv(_dev(a, plan.complex_dtype))) / amp,
                            o.inv(n, nlon, a.astype(np.complex128)) / amp, nlon, w)
        assert er.max() < TOL_RMS["fp32"], (shape, k / 8, er.max())


# A mean near the largest float: the adjoint of the direct transform scales it
# down, and forms nothing larger on the way.
@pytest.mark.parametrize("grid,nlat,nl", [("octahedral", 64, 0), ("full", 64, 122)])
@pytest.mark.parametrize("nf", [1, F])
def test_adjoint_of_largest_mean(grid, nlat, nl, nf):
    shtx, o = _shtx(), _oracle()
    n = 31
    plan = shtx.Plan(n, grid, nlat, nf, "fp32", nlon_full=nl)
    nlon = plan.ring_lengths()
    a = np.zeros((nf, plan.nspec), np.complex64)
    a[:, 0] = 3e38
    got = _np(plan.dir_adj(_dev(a, plan.complex_dtype))).astype(np.float64)
    ref = o.dir_adj(n, nlon, a.astype(np.complex128))
    assert np.abs(got - ref).max() < 1e-5 * np.abs(ref).max()


# Wavenumbers whose table entries are near the smallest float on the rings away
# from the equator, with inputs of 2^30 that bring the results back into range:
# entry by entry, on the rings of a field of those wavenumbers, and in the
# coefficients of a field on one such ring.  An entry above 2^-126 has 24 bits,
# and so has every result compared.
@pytest.mark.parametrize("shape", SHAPES)
def test_small_table_entries(shape):
    shtx, o = _shtx(), _oracle()
    n, nlat, nl, m0, big = 95, 144, 288, 84, 2.0 ** 30
    plan = shtx.Plan(n, "full", nlat, F, "fp32", nlon_full=nl)
    plan.set_shapes(shape, shape, plan.info.fft_cap)
    nlon = plan.ring_lengths()
    mu, _ = plan.nodes()
    tab, want = plan.legendre(m0), o.legendre(n, m0, mu[:nlat // 2])
    held = np.abs(want) > 2.0 ** -126
    err = np.abs(tab - want)[held] / np.abs(want)[held]
    assert (np.abs(want[held]) < 2.0 ** -116).any() and err.max() < 2.0 ** -23, err.max()
    rows = np.abs(want).max(axis=1)
    small = (rows > 2.0 ** -124) & (rows < 2.0 ** -112)  # northern rings
    assert small.any()

    m, _ = si.spec_mn(n)
    a = (si.spectral_fields(n, 53, range(F)) * (m >= m0) * big).astype(np.complex64)
    ref = o.inv(n, nlon, a.astype(np.complex128)).reshape(F, nlat, nl)[:, :nlat // 2][:, small]
    got = _np(plan.inv(_dev(a, plan.complex_dtype))).astype(np.float64).reshape(F, nlat, nl)[:, :nlat // 2][:, small]
    err = np.abs(got - ref).max(axis=2) / np.abs(ref).max(axis=2)
    _say(f"  {shape} inv {int(small.sum())} rings, worst {err.max():.2e}")
    assert err.max() < 1e-5

    y = np.zeros((F, nlat, nl))
    for i, j in enumerate(np.flatnonzero(small)):
        y[i::int(small.sum()), j] = big
    y = (y.reshape(F, -1) * np.stack([si.white_noise_grid(nlat * nl, 800 + f) for f in range(F)])).astype(np.float32)
    ref = o.inv_adj(n, nlon, y.astype(np.float64))[:, m == m0]
    got = _np(plan.inv_adj(_dev(y, plan.real_dtype))).astype(np.complex128)[:, m == m0]
    err = np.abs(got - ref).max(axis=1) / np.abs(ref).max(axis=1)
    _say(f"  {shape} inv_adj worst {err.max():.2e}")
    assert err.max() < 1e-5


# Infinities and NaN of one field reach no other one, and the sums beside them
# are those of single precision: a coefficient of wavenumber 0 makes one of
# the two samples that share a complex value infinite and the other NaN.
@pytest.mark.parametrize("shape", SHAPES)
def test_values_not_finite(shape):
    plan, nlon = _plan(shape)
    a = si.spectral_fields(N, 57, range(F)).astype(np.complex64)
    clean = _np(plan.inv(_dev(a, plan.complex_dtype)))
    b = a.copy()
    b[3, 0], b[5, 5], b[7, 700] = np.inf, -np.inf, np.nan
    g = _np(plan.inv(_dev(b, plan.complex_dtype)))
    assert not np.isfinite(g[3]).any() and not np.isfinite(g[5]).any()
    assert np.isinf(g[3]).sum() == g.shape[1] // 2 and np.isinf(g[5]).sum() == g.shape[1] // 2
    assert np.isnan(g[7]).any()
    rest = [f for f in range(F) if f not in (3, 5, 7)]
    np.testing.assert_allclose(g[rest], clean[rest], rtol=0, atol=1e-5 * np.abs(clean).max())


# Every one of the six products of pieces counts: leaving one out costs 2.4e-6 to
# 2.8e-6 RMS of a sum of random operands (numpy, K = 512, all pieces rounded to
# nearest), and FP32 transforms of this size stay below 1e-6.
TOL_SIX_PRODUCTS = 1.5e-6


@pytest.mark.parametrize("shape", SHAPES)
def test_all_products(shape):
    o = _oracle()
    for n, nf in ((N, F), (130, 65)):
        plan = _shtx().Plan(n, "octahedral", 2 * (n + 1), nf, "fp32")
        plan.set_shapes(shape, shape, plan.info.fft_cap)
        nlon = plan.ring_lengths()
        _, w = o.gauss(len(nlon))
        a = si.spectral_fields(n, 59, range(nf)).astype(np.complex64)
        y = np.stack([si.white_noise_grid(int(nlon.sum()), 900 + f) for f in range(nf)]).astype(np.float32)
        a64, y64 = a.astype(np.complex128), y.astype(np.float64)
        spec, grid = _dev(a, plan.complex_dtype), _dev(y, plan.real_dtype)
        for name in ("inv", "dir_adj"):
            _, er = grid_errors(_np(getattr(plan, name)(spec)), getattr(o, name)(n, nlon, a64), nlon, w)
            _say(f"  {shape} T{n} {name} rms {er.max():.2e}")
            assert er.max() < TOL_SIX_PRODUCTS
        for name in ("dir", "inv_adj"):
            _, er = spec_errors(_np(getattr(plan, name)(grid)), getattr(o, name)(n, nlon, y64), n)
            _say(f"  {shape} T{n} {name} rms {er.max():.2e}")
            assert er.max() < TOL_SIX_PRODUCTS


def _nearest_bf16(x):
    u = x.view(np.uint32).astype(np.uint64)
    u = (u + 0x7FFF + ((u >> 16) & 1)) & 0xFFFF0000
    return u.astype(np.uint32).view(np.float32)


# The products left out stay below 2^-24 of a product, which takes pieces rounded
# to nearest: a leading piece cut instead leaves out up to 2^-23.  One
# coefficient a_1^0 in each field makes every value of F_0 one product; its
# pieces, cut, are as large as pieces get.  The part of the results' error
# that goes with what cutting leaves out (the slope of a regression on it, 1
# for cut pieces; its standard error from roundings to 2^-24 is 0.03).
@pytest.mark.parametrize("shape", SHAPES)
def test_products_left_out(shape):
    torch, o = _torch(), _oracle()
    n, nlat, nl = 31, 256, 512
    plan = _shtx().Plan(n, "full", nlat, F, "fp32", nlon_full=nl)
    plan.set_shapes(shape, shape, plan.info.fft_cap)
    mu, _ = plan.nodes()
    p = o.legendre(n, 0, mu[:nlat // 2])[:, 1].astype(np.float32)  # P_1^0 on the northern rings

    def pieces(x, first):
        h = first(x)
        m = _nearest_bf16(x - h)
        return [v.astype(np.float64) for v in (h, m, x - h - m)]

    x = (1 + 2.0 ** -7 - 2.0 ** -23 * (1 + np.arange(F))).astype(np.float32)
    a = np.zeros((F, plan.nspec), np.complex64)
    a[:, 1] = x
    got = _np(plan.inv(torch.from_numpy(a).cuda())).astype(np.float64).reshape(F, nlat, nl)[:, :nlat // 2, 0]
    exact = p.astype(np.float64)[None] * x.astype(np.float64)[:, None]
    tab, cut = pieces(p, _nearest_bf16), pieces(x, lambda v: (v.view(np.uint32) & 0xFFFF0000).view(np.float32))
    left = sum(tab[i][None] * cut[j][:, None] for i in range(3) for j in range(3 - i)) / exact - 1
    slope = ((got / exact - 1) * left).sum() / (left * left).sum()
    _say(f"  {shape} slope {slope:.3f}, error rms {np.sqrt(((got / exact - 1) ** 2).mean()):.2e}")
    assert abs(slope) < 0.5
