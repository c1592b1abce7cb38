"""Range-Doppler transforms over every line length, against numpy's FP64 FFT."""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("pairs, chirps, samples", [
    (1, 1, 1), (3, 2, 1), (2, 1, 4), (3, 4, 2), (5, 8, 16), (2, 16, 8), (1, 32, 64), (7, 64, 32), (3, 128, 4),
    (2, 256, 128), (1, 512, 512), (13, 4, 1024), (1, 1024, 256), (1, 2048, 8), (2, 8, 2048), (1, 4096, 2),
    (1, 2, 4096), (33, 16, 16)])
def test_range_doppler_line_lengths(pairs, chirps, samples):
    import torch
    from paper_2305_14176_amd import raymeta
    rng = np.random.default_rng(pairs * 7 + chirps + samples)
    x = (rng.standard_normal((pairs, chirps, samples)) + 1j * rng.standard_normal((pairs, chirps, samples)))
    x = x.astype(np.complex64)
    ref = np.fft.fft2(x.astype(np.complex128), axes=(-2, -1))
    s = torch.from_numpy(x).cuda()
    got = raymeta.range_doppler(s).cpu().numpy()
    # a float32 transform of n points rounds each value a few times per factor of 8
    tol = 2.0 ** -24 * (2.0 + 2.0 * math.log2(chirps * samples))
    assert np.linalg.norm(got - ref) <= tol * np.linalg.norm(ref)
    raymeta.range_doppler(s, out=s)          # in place: the same values
    assert np.array_equal(s.cpu().numpy(), got)
