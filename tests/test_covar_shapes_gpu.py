"""The covariance form at the shapes where its launches change: time splits,
passes over the channels, tiles and shares at the ends of their ranges.

References in float64 from the antennas' covariances (integers, exact), by
which an integration of any length costs the same: image_fx's sum over pairs,
and the gain gradient's.  Both are checked against the per-sample oracle below,
on the CPU.  Bars: those of the float32 routes (images 1e-5 relative L2 per
plane, gradients 1e-4).
"""
import numpy as np
import pytest

import oracle
import synth

TOL_FP32 = 1e-5
TOL_GRAD = 1e-4


def _channel(inp, c):
    return synth.Inputs(inp.grid_n, 1, inp.n_pol, inp.n_ant, inp.kernel_support, inp.kernel_sigma_cells,
                        inp.cell_wavelengths, inp.xy_m, inp.freq_hz[c:c + 1], inp.gains[c:c + 1],
                        np.ascontiguousarray(inp.efield[:, c:c + 1]))


def _parts(sub):
    """Beta [A, N^2], V[p][q] = sum_t e_p conj(e_q) [A, A] and gains [P, A] of one channel."""
    B = oracle.aperture_response(sub.xy_m, sub.freq_hz, sub.grid_n)[0].reshape(sub.n_ant, -1)
    e = oracle.unpack_ci4(sub.efield[:, 0])
    V = [[e[:, p].T @ np.conj(e[:, q]) for q in range(sub.n_pol)] for p in range(sub.n_pol)]
    return B, V, sub.gains[0].astype(np.complex128)


def _image(sub):
    B, V, g = _parts(sub)
    pairs = [(0, 0)] if sub.n_pol == 1 else [(0, 0), (0, 1), (1, 0), (1, 1)]
    N = sub.grid_n
    out = [np.einsum("ak,ak->k", B, (g[p][:, None] * V[p][q] * np.conj(g[q])) @ np.conj(B)) for p, q in pairs]
    return np.fft.fftshift(np.array(out).reshape(1, -1, N, N), axes=(-2, -1))


def _gradient(sub, grad_image):
    """oracle.grad_gains of one channel, its sum over time taken first."""
    B, V, g = _parts(sub)
    P, N = sub.n_pol, sub.grid_n
    G = np.fft.ifftshift(grad_image.astype(np.complex128), axes=(-2, -1)).reshape(-1, N * N)
    h = [[2 * G[0].real]]
    if P == 2:
        Q = G[1] + np.conj(G[2])
        h = [[2 * G[0].real, Q], [np.conj(Q), 2 * G[3].real]]
    out = np.zeros((P, sub.n_ant), np.complex128)
    for p in range(P):
        for q in range(P):
            # sum_t F_q conj(e_pa) = sum_b b_b g_qb conj(V_pq[a, b])
            out[p] += np.einsum("ak,k,ak->a", np.conj(B), h[p][q], (np.conj(V[p][q]) * g[q]) @ B)
    return out[None]


@pytest.mark.parametrize("P", [1, 2])
def test_references_match_the_per_sample_oracle(P):
    sub = synth.random_problem(960, 64, 9, 1, P, 30, fill=0.45)
    want = oracle.image_from(sub)
    assert oracle.rel_errors(_image(sub), want).max() < 1e-12
    rng = np.random.default_rng(960)
    gam = rng.normal(size=want.shape) + 1j * rng.normal(size=want.shape)
    ref = oracle.grad_gains(sub.xy_m, sub.freq_hz, sub.gains, sub.efield, 64, gam)
    assert np.linalg.norm(_gradient(sub, gam[0]) - ref) < 1e-12 * np.linalg.norm(ref)


def _imager(inp, **kw):
    from paper_1904_11422_amd import Imager
    im = Imager(inp.grid_n, inp.n_chan, inp.n_pol, inp.n_ant, inp.kernel_support,
                inp.kernel_sigma_cells, inp.cell_wavelengths, **kw)
    im.set_antennas(inp.xy_m, inp.freq_hz)
    return im


def _check(inp, channels):
    import torch
    im = _imager(inp)
    ef = torch.from_numpy(np.ascontiguousarray(inp.efield)).cuda()
    g = torch.from_numpy(np.ascontiguousarray(inp.gains)).cuda()
    print(f"  A={inp.n_ant} C={inp.n_chan} P={inp.n_pol} T={inp.n_time}", flush=True)
    got = im.accumulate(ef, g).cpu().numpy()
    assert im.last_kernel_name() == "cov_fold_kernel"
    for c in channels:
        err = oracle.rel_errors(got[c:c + 1], _image(_channel(inp, c))).max()
        assert err <= TOL_FP32, f"image, channel {c}: {err:.3e}"
    twice = torch.from_numpy(got).cuda()
    im.accumulate(ef, g, image=twice, reset=False)
    assert np.array_equal(twice.cpu().numpy(), 2 * got)
    rng = np.random.default_rng(inp.n_ant)
    gam = rng.normal(size=im.image_shape()) + 1j * rng.normal(size=im.image_shape())
    got = im.backward(ef, g, torch.from_numpy(gam).cuda()).cpu().numpy()
    assert im.last_form() == "covariance"
    for c in channels:
        want = _gradient(_channel(inp, c), gam[c])
        err = np.linalg.norm(got[c:c + 1] - want) / np.linalg.norm(want)
        assert err <= TOL_GRAD, f"gradient, channel {c}: {err:.3e}"


@pytest.mark.gpu
@pytest.mark.parametrize("seed,A,C,P,T,fill", [
    (961, 20, 4, 2, 40_001, 0.45),     # two splits at least: one exact partial sum holds 32768 samples
    (962, 24, 4, 2, 65_537, 0.66),     # three, wide block
    (963, 260, 2, 2, 32_769, 0.48),    # more than 256 antennas; the second split a single sample longer
    (964, 24, 4, 1, 131_072, 0.45),    # four, the longest call of the form
])
def test_time_splits(seed, A, C, P, T, fill):
    _check(synth.random_problem(seed, 64, A, C, P, T, fill=fill), [0, C - 1])


@pytest.mark.gpu
@pytest.mark.parametrize("seed,A,C,P,T,fill", [
    (965, 512, 67, 2, 800, 0.48),      # V of 61 channels fits (45 with the gradient's planes): two ragged passes
    (966, 500, 50, 2, 1000, 0.70),     # wide block; the gradient in two passes
])
def test_passes_over_the_channels(seed, A, C, P, T, fill):
    """More channels than the workspace holds: the passes reuse it, channels on
    both sides of every seam."""
    _check(synth.random_problem(seed, 64, A, C, P, T, fill=fill), [0, C // 2 - 1, C // 2, C // 2 + 1, C - 1])


@pytest.mark.gpu
@pytest.mark.parametrize("seed,A,C,P,T,fill", [
    (967, 512, 6, 1, 3000, 0.48),      # eight tiles of a, one share of b per workgroup
    (968, 300, 20, 1, 900, 0.66),      # wide block, more than 256 antennas, one polarisation
    (969, 4, 60, 2, 600, 0.66),        # ranges of a few antennas, several channels per workgroup
    (970, 3, 200, 1, 500, 0.45),
    (971, 101, 3, 2, 9000, 0.45),      # few channels: a channel's antennas over many workgroups
    (972, 120, 30, 2, 700, 0.2),       # crowded cells: the fold's longest program
])
def test_edges_of_antennas_and_channels(seed, A, C, P, T, fill):
    _check(synth.random_problem(seed, 64, A, C, P, T, fill=fill), [0, C // 2, C - 1])


@pytest.mark.gpu
def test_cells_of_more_antennas_than_a_program_holds_stay_direct():
    import torch
    inp = synth.random_problem(973, 64, 200, 30, 2, 600, fill=0.12, min_sep_cells=0.1)
    im = _imager(inp)
    got = im.accumulate(torch.from_numpy(inp.efield).cuda(), torch.from_numpy(inp.gains).cuda()).cpu().numpy()
    assert im.last_kernel_name() == "fused_image_kernel"
    assert oracle.rel_errors(got[:1], _image(_channel(inp, 0))).max() <= TOL_FP32
