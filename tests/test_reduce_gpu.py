"""The fused reductions on both sides of the line between 4 and 16 sub-lanes
(33 to 64 parts per channel; blocks of 64 pixels that fill the chip or not)."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,P,C,T", [(32, 2, 9, 45), (64, 2, 15, 40), (64, 2, 16, 40), (64, 1, 16, 34),
                                     (128, 1, 3, 40), (128, 1, 4, 40), (128, 2, 4, 34)])
def test_reduction_of_33_to_64_parts(N, P, C, T):
    import torch
    from paper_1904_11422_amd import Imager
    inp = synth.random_problem(970 + N + C, N, 24, C, P, T, fill=0.4)
    im = Imager(N, C, P, 24)
    im.set_antennas(inp.xy_m, inp.freq_hz)
    got = im.accumulate(torch.from_numpy(np.ascontiguousarray(inp.efield)).cuda(),
                        torch.from_numpy(inp.gains).cuda()).cpu().numpy()
    for c in (0, C - 1):
        sub = synth.Inputs(N, 1, P, 24, 3, 0.5, 0.5, inp.xy_m, inp.freq_hz[c:c + 1], inp.gains[c:c + 1],
                           np.ascontiguousarray(inp.efield[:, c:c + 1]))
        assert oracle.rel_errors(got[c:c + 1], oracle.image_from(sub)).max() <= 1e-5
