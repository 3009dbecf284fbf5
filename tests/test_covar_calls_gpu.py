"""Calls whose route the covariance form joins: what a caller could rely on
before it holds on every route (errors of other code, alignment, memory)."""
import ctypes

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


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


@pytest.mark.parametrize("T", [20, 1000])      # the direct adjoint, the covariance form's
def test_gradient_ignores_an_older_error_of_the_thread(T):
    """An error that other code's failed HIP call left with the thread (here a
    device ordinal that does not exist) is not the gradient's."""
    import torch
    inp = synth.random_problem(951, 64, 60, 24, 2, T, fill=0.45)
    im = _imager(inp)
    ef, g = _dev(inp)
    rng = np.random.default_rng(951)
    gam = torch.from_numpy(rng.normal(size=im.image_shape()) + 0j).cuda()
    want = im.backward(ef, g, gam)
    torch.cuda.synchronize()
    out = torch.empty_like(want)
    ptr = [ctypes.c_void_p(t.data_ptr()) for t in (ef, g, gam, out)]
    assert im.L.hipSetDevice(1234) != 0
    st = im.L.epic_image_backward(im._ctx, ptr[0], T, ptr[1], ptr[2], ptr[3])
    message = im.L.epic_last_error(im._ctx)
    im.L.hipGetLastError()
    torch.cuda.synchronize()
    assert st == 0, message
    assert torch.equal(out, want)


@pytest.mark.parametrize("seed,A,C,P,T", [(952, 256, 16, 2, 1250), (955, 64, 24, 1, 700), (956, 90, 20, 2, 500)])
def test_samples_give_the_same_bits_at_any_address(seed, A, C, P, T):
    """The same samples one byte further on: the same form, the same bits."""
    import torch
    inp = synth.random_problem(seed, 64, A, C, P, T, fill=0.45)
    im = _imager(inp)
    ef, g = _dev(inp)
    rng = np.random.default_rng(seed)
    gam = torch.from_numpy(rng.normal(size=im.image_shape()) + 0j).cuda()
    want = im.accumulate(ef, g)
    assert im.last_kernel_name() == "cov_fold_kernel"
    grad = im.backward(ef, g, gam)
    buf = torch.empty(ef.numel() + 4, dtype=torch.uint8, device="cuda")
    for shift in (1, 2, 3):
        odd = buf[shift:shift + ef.numel()].view(ef.shape)
        odd.copy_(ef)
        assert torch.equal(im.accumulate(odd, g), want)
        assert im.last_kernel_name() == "cov_fold_kernel"
        assert torch.equal(im.backward(odd, g, gam), grad)


@pytest.mark.parametrize("A", [1, 2, 3, 5, 129])
def test_last_samples_of_a_buffer(A):
    """Rows of antennas that are no multiple of four, the last one at the very
    end of its buffer: the tail is read within its row."""
    import torch
    import oracle
    inp = synth.random_problem(957 + A, 64, A, 20, 1, 900, fill=0.45)
    im = _imager(inp)
    ef, g = _dev(inp)
    got = im.accumulate(ef, g).cpu().numpy()
    sub = synth.Inputs(64, 1, 1, A, 3, 0.5, 0.5, inp.xy_m, inp.freq_hz[19:], inp.gains[19:],
                       np.ascontiguousarray(inp.efield[:, 19:]))
    err = oracle.rel_errors(got[19:], oracle.image_from(sub)).max()
    print(f"  A={A}: {im.last_kernel_name()} {err:.2e}", flush=True)
    assert err <= 1e-5


def test_long_integration_of_one_channel_stays_direct():
    """One channel's covariances fill four workgroups however long it is: 94
    antennas at T = 107322 take 538 us directly and 840 by them; six channels of
    them gain."""
    import torch
    for C, route in ((1, "fused_image_kernel"), (6, "cov_fold_kernel")):
        inp = synth.random_problem(963, 64, 96, C, 1, 4, fill=0.45)
        im = _imager(inp)
        T = 100_000 // (1 if C == 1 else 4)
        ef = torch.zeros((T, C, 1, 96), dtype=torch.uint8, device="cuda")
        im.accumulate(ef, torch.from_numpy(inp.gains).cuda())
        assert im.last_kernel_name() == route


def test_workspace_goes_with_a_geometry_that_cannot_use_it():
    """The caller's own kernels, and apertures beyond the fused kernels' blocks,
    never take the covariance form: what it held (its covariances alone are
    over 200 MB at this shape) is free again, and comes back with the Gaussian."""
    import torch
    inp = synth.random_problem(954, 64, 256, 132, 2, 1, fill=0.45)
    im = _imager(inp)
    torch.cuda.synchronize()
    held = torch.cuda.mem_get_info()[0]
    im.set_antennas(inp.xy_m, inp.freq_hz, kernels=np.ones((132, 256, 3, 3), np.complex64))
    assert torch.cuda.mem_get_info()[0] - held > 200 << 20
    im.set_antennas(inp.xy_m, inp.freq_hz)
    assert abs(torch.cuda.mem_get_info()[0] - held) < 64 << 20
    few_inp = synth.random_problem(965, 64, 256, 60, 2, 1, fill=0.45)         # fewer channels hold less
    few = _imager(few_inp)
    without = torch.cuda.mem_get_info()[0]
    few.set_antennas(few_inp.xy_m, few_inp.freq_hz, kernels=np.ones((60, 256, 3, 3), np.complex64))
    assert torch.cuda.mem_get_info()[0] - without < 240 << 20
    few.close()
