"""The row kernel's list of kept elements: every register layout of the row (elements per lane), with the kept elements spread
evenly, crowded into one place (one lane then lists all of its elements), and equal to each other; byte-exact against the oracle."""
import numpy as np
import pytest

from paper_2511_11608_amd import synth
from tests.test_gpu_parity import B28, check, check_atkf

pytestmark = pytest.mark.gpu

LENGTHS = {"f32": [255, 256, 512, 768, 1024, 1280, 2048, 4096], "bf16": [1024, 2048, 2047, 4096]}


@pytest.mark.parametrize("dtype,N", [(d, n) for d in LENGTHS for n in LENGTHS[d]])
def test_where_the_kept_elements_lie(oracle, dtype, N):
    rng = np.random.default_rng(N)
    x = rng.standard_normal((8, N)).astype(np.float32)
    n = max(1, N // 10)
    for r, at in enumerate((0, N // 3, N - n)):
        x[r, at:at + n] *= np.float32(100)
    x[3] = np.abs(x[3])
    x[4, ::11] = -50.0                                # equal keys: the lower indices stay
    x[5] = 0.25
    x[7, ::9] = np.where(np.arange(0, N, 9) % 2, 60.0, -60.0)     # the cut among equal keys of both classes
    x[6, n // 2:] = 0.0
    if dtype == "bf16":
        x = synth.f32_to_bf16_bits(x)
    check(oracle, x, dtype, 0.1, 4, B28, 1e-3)
    check_atkf(oracle, x, dtype, 0.1, 0.3, 4, 3, B28, 1e-3)
