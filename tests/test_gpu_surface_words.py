"""Surface distances where the last pass gives each wavefront 8, 16, 32 or 64 words of the packed
masks, the last wavefronts fewer, against the oracle: sparse surfaces and noise."""

import numpy as np
import pytest

import test_gpu_masks as M

pytestmark = pytest.mark.gpu


# words: 16383 (8 each), 36855 (16), 73720 (32), 138240 (64)
@pytest.mark.parametrize("shape", [(43, 127, 95), (65, 63, 260), (97, 95, 230), (96, 160, 264)])
@pytest.mark.parametrize("noise", [False, True])
def test_words_per_wavefront(shape, noise):
    M.say(f"surface words {shape} noise={noise}")
    rng = np.random.default_rng(41)
    if noise:
        A, B = rng.random(shape) > 0.5, rng.random(shape) > 0.7
    else:
        z, y, x = np.meshgrid(*(np.linspace(-1, 1, n) for n in shape), indexing="ij")
        r = z * z + y * y + x * x
        A, B = r < 0.5, r + 0.1 * x < 0.3
    M._check_distances(A, B, 0.05)
