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
