"""Long integrations pixel by pixel: scenes whose images span many decades.

Without receiver noise an image has pixels far below its peak.  There the
direct kernels are off by little more than the pixel's own rounding (they sum
squares), and XX and YY are never negative; both hold for the covariance form
too, whose image is a signed transform.

Bound, derived from float64 arithmetic: with U the largest value a pixel can
take (all antennas in phase at every sample, each with its kernel's sum of
weights), a pixel of a P or PQ plane is a sum of at most 81 A^2 + 4096 terms
whose magnitudes add up to at most U, in an order that is mostly pairwise:
2^-53 per rounding and a few hundred roundings in a chain give 3e-14 U; 1e-13 U
is asked for.  (One part in 1e13 of U is 5e-6 of a pixel 70 dB below the peak
of a point source; float32 sums leave 5e-9 U.)
"""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

BOUND = 1e-13


def _imager(inp, **kw):
    from paper_1904_11422_amd import Imager
    im = Imager(inp.grid_n, inp.n_chan, inp.n_pol, inp.n_ant, inp.kernel_support,
                inp.kernel_sigma_cells, inp.cell_wavelengths, **kw)
    im.set_antennas(inp.xy_m, inp.freq_hz)
    return im


def _dev(inp):
    import torch
    return (torch.from_numpy(np.ascontiguousarray(inp.efield)).cuda(),
            torch.from_numpy(np.ascontiguousarray(inp.gains)).cuda())


def _channel(inp, c):
    return synth.Inputs(inp.grid_n, 1, inp.n_pol, inp.n_ant, inp.kernel_support, inp.kernel_sigma_cells,
                        inp.cell_wavelengths, inp.xy_m, inp.freq_hz[c:c + 1], inp.gains[c:c + 1],
                        np.ascontiguousarray(inp.efield[:, c:c + 1]))


def _largest(sub):
    """U of the planes of one channel: [n_prod]."""
    X, Y = oracle.moff.antenna_cells(sub.xy_m, sub.freq_hz, sub.grid_n, sub.cell_wavelengths)
    _, _, w = oracle.moff.kernel_taps(X, Y, sub.grid_n)
    e = np.abs(oracle.moff.unpack_ci4(sub.efield[:, 0])) * np.abs(sub.gains[0]) * w[0].sum(1)   # [T, P, A]
    s = e.sum(2)
    pairs = [(0, 0)] if sub.n_pol == 1 else [(0, 0), (0, 1), (1, 0), (1, 1)]
    return np.array([(s[:, p] * s[:, q]).sum() for p, q in pairs])


def _coherent(inp, seed, same=None):
    """Every antenna receives the same sample (a point source at the zenith).
    `same`: only these two receive anything; they stand on grid points eight
    cells apart, with one kernel, so that their fringe has exact nulls on pixels."""
    rng = np.random.default_rng(seed)
    s = synth.random_bytes(rng, (inp.n_time, inp.n_chan, inp.n_pol, 1))
    ef = np.repeat(s, inp.n_ant, axis=3)
    if same is not None:
        off = np.ones(inp.n_ant, bool)
        off[list(same)] = False
        ef[..., off] = 0
        inp.freq_hz[:] = inp.freq_hz.max()
        cell_m = synth.C0 / inp.freq_hz[0] * inp.cell_wavelengths
        inp.xy_m[same[0]] = (-4 * cell_m, 0)
        inp.xy_m[same[1]] = (4 * cell_m, 0)
    inp.efield[...] = ef
    inp.gains[...] = 1
    return inp


def _least(got, P):
    """Least power of all channels, over the largest."""
    planes = got[:, [0] if P == 1 else [0, 3]].real
    return float(planes.min()), float(planes.max())


@pytest.mark.parametrize("seed,A,C,P,T,fill", [
    (931, 256, 40, 2, 1000, 0.45),
    (932, 200, 40, 1, 1250, 0.45),
    (933, 200, 40, 2, 1250, 0.66),    # wide block: its row 32 rides in row 0's imaginary part
    (934, 152, 40, 1, 1250, 0.66),
    (935, 300, 40, 2, 1250, 0.48),    # more than 256 antennas
])
def test_dark_pixels_of_a_point_source(seed, A, C, P, T, fill):
    inp = _coherent(synth.random_problem(seed, 64, A, C, P, T, fill=fill), seed)
    im = _imager(inp)
    ef, g = _dev(inp)
    got = im.accumulate(ef, g).cpu().numpy()
    assert im.last_kernel_name() == "cov_fold_kernel"
    worst = 0.0
    for c in (0, C - 1):
        sub = _channel(inp, c)
        ref = oracle.image_from(sub)[0]
        off = np.abs(got[c] - ref).max(axis=(1, 2)) / _largest(sub)
        dark = ref[0].real < 1e-5 * ref[0].real.max()
        rel = np.abs(got[c, 0] - ref[0])[dark] / ref[0].real[dark]
        print(f"  A={A} P={P} channel {c}: off by {off.max():.2e} U; {dark.sum()} pixels 50 dB down, "
              f"median {np.median(rel):.1e}, worst {rel.max():.1e}", flush=True)
        assert dark.sum() > 20
        worst = max(worst, off.max())
    low, high = _least(got, P)
    print(f"  least power {low:.2e} of {high:.2e}", flush=True)
    assert low >= 0
    assert worst <= BOUND, f"{worst:.2e}"


@pytest.mark.parametrize("seed,P,fill", [(936, 2, 0.45), (937, 1, 0.45), (938, 2, 0.66)])
def test_power_is_never_negative_where_two_antennas_cancel(seed, P, fill):
    """Two antennas with the same samples: fringes with exact nulls.  XX and YY
    stay non-negative, and |XY|^2 <= XX YY up to the arithmetic's rounding."""
    inp = _coherent(synth.random_problem(seed, 64, 60, 40, P, 1250, fill=fill), seed, same=(7, 31))
    im = _imager(inp)
    ef, g = _dev(inp)
    got = im.accumulate(ef, g).cpu().numpy()
    assert im.last_kernel_name() == "cov_fold_kernel"
    low, high = _least(got, P)
    print(f"  least power {low:.2e} of {high:.2e}", flush=True)
    assert low >= 0
    if P == 2:
        U = _largest(_channel(inp, 0))
        xy = np.abs(got[0, 1])
        over = xy - np.sqrt(got[0, 0].real * got[0, 3].real) * (1 + 1e-6)
        assert float(over.max()) <= BOUND * U[1]


def test_noise_free_integration_adds_up_to_non_negative_power():
    """Two calls adding up (reset = 0): each call's power is non-negative."""
    inp = _coherent(synth.random_problem(939, 64, 60, 40, 2, 1250, fill=0.45), 939, same=(3, 40))
    im = _imager(inp)
    ef, g = _dev(inp)
    img = im.accumulate(ef, g)
    first = img.cpu().numpy().copy()
    im.accumulate(ef, g, image=img, reset=False)
    got = img.cpu().numpy()
    assert bool((got == 2 * first).all())
    assert _least(got, 2)[0] >= 0


def test_non_finite_gains_stay_visible():
    """A NaN gain of one antenna reaches every pixel of the planes it is in
    (the sign rule must not turn NaN into zero), and none of the others."""
    inp = synth.random_problem(940, 64, 60, 40, 2, 1250, fill=0.45)
    im = _imager(inp)
    ef, g = _dev(inp)
    g[3, 0, 5] = float("nan")
    got = im.accumulate(ef, g).cpu().numpy()
    assert im.last_kernel_name() == "cov_fold_kernel"
    assert bool(np.isnan(got[3, 0].real).all() and np.isnan(got[3, 1]).all())
    assert bool(np.isfinite(got[3, 3]).all() and np.isfinite(np.delete(got, 3, axis=0)).all())


@pytest.mark.parametrize("scale", [1e-21, 1e16])
def test_gains_of_any_scale(scale):
    """Gains of very small or large magnitude: their products leave float32's
    range or its normal numbers long before the power does."""
    import torch
    inp = synth.random_problem(941, 64, 128, 40, 2, 1250, fill=0.45)
    im = _imager(inp)
    ef, g = _dev(inp)
    want = im.accumulate(ef, g).cpu().numpy()
    got = im.accumulate(ef, g * torch.tensor(scale, dtype=torch.float32, device="cuda")).cpu().numpy()
    assert im.last_kernel_name() == "cov_fold_kernel"
    err = oracle.rel_errors(got / scale ** 2, want).max()
    print(f"  scale {scale:.0e}: {err:.2e}", flush=True)
    assert err <= 1e-5


@pytest.mark.parametrize("seed,A,P,fill", [(942, 256, 2, 0.45), (943, 200, 1, 0.45), (944, 200, 2, 0.66), (945, 300, 2, 0.48)])
def test_gradient_of_dark_pixels(seed, A, P, fill):
    """A loss that looks at one pixel far below the peak: the sum over antennas
    cancels as deeply as the field does there.  Float64 up to the gradient's own
    rounding to float32 (6e-8 of an element): 2e-7 of its norm."""
    import torch
    from test_covar_shapes_gpu import _gradient
    inp = _coherent(synth.random_problem(seed, 64, A, 40, P, 900, fill=fill), seed)
    im = _imager(inp)
    ef, g = _dev(inp)
    sub = _channel(inp, 0)
    power = oracle.image_from(sub)[0, 0].real
    order = np.argsort(power.ravel())
    for rank in (0, 40, 400, 4095):
        gam = np.zeros(im.image_shape(), np.complex128)
        gam.reshape(40, -1, 4096)[:, :, order[rank]] = 1
        got = im.backward(ef, g, torch.from_numpy(gam).cuda()).cpu().numpy()
        assert im.last_form() == "covariance"
        want = _gradient(sub, gam[0])
        err = np.linalg.norm(got[:1] - want) / np.linalg.norm(want)
        print(f"  A={A} P={P} pixel at {power.ravel()[order[rank]] / power.max():.1e} of the peak: {err:.1e}", flush=True)
        assert err <= 2e-7
