"""Rows whose values are equal, or take few values: the row kernel's exact cut and its selection of block boundaries among many equal or
nearly equal members of one bin, in both classes; byte-exact against the oracle."""
import numpy as np
import pytest

from paper_2511_11608_amd import synth
from tests.test_gpu_parity import B28, check, check_atkf

pytestmark = pytest.mark.gpu


def rows_of(N, dtype):
    rng = np.random.default_rng(N)
    x = rng.standard_normal((12, N)).astype(np.float32)
    x[0] = 1.5                                        # one value, one class
    x[1] = np.where(np.arange(N) % 3, 1.5, -1.5)      # one value, both classes
    x[2] = np.round(x[2] * 2) / 2                     # few values, zeros among them
    x[3] = np.round(x[3] * 4) / 4 * np.float32(1e-20)
    x[4] = -2.0                                       # the negative class alone
    x[4, N // 2:] = -1.0
    x[5] = np.float32(1.0) + (rng.integers(0, 3, N) * 2.0 ** -7).astype(np.float32)       # neighbouring keys (bf16)
    x[6] = np.float32(1.0) + (rng.integers(0, 70, N) * 2.0 ** -23).astype(np.float32)     # ... (fp32): many keys of one bin
    x[6, ::2] *= -1
    x[7] = 0.0
    x[7, 5] = 3.0e38                                  # one value far above all others, which are equal
    x[7, 9:] = 1.0e-30
    x[8] = x[8] * np.exp2(rng.integers(-30, 30, N)).astype(np.float32)
    x[8, N // 3:] = np.float32(2.0 ** -40)            # the cut among equal values more than 16 octaves down
    x[9] = x[8][::-1]
    x[9, ::2] *= -1
    x[10] = np.where(rng.random(N) < 0.5, x[10], np.float32(0.75))
    return synth.f32_to_bf16_bits(x) if dtype == "bf16" else x


@pytest.mark.parametrize("dtype,N,keep,M", [("f32", 255, 0.1, 4), ("f32", 768, 0.15, 8), ("f32", 1280, 0.25, 16), ("f32", 2047, 0.3, 8), ("f32", 4096, 0.1, 8), ("f32", 4096, 0.4, 16),
                                            ("bf16", 1000, 0.1, 8), ("bf16", 2048, 0.2, 3), ("bf16", 4096, 0.1, 8), ("bf16", 4096, 0.4, 16), ("f32", 4096, 0.25, 1)])
def test_few_values(oracle, dtype, N, keep, M):
    x = rows_of(N, dtype)
    check(oracle, x, dtype, keep, M, B28, 1e-3)
    check(oracle, x[:1].copy(), dtype, keep, M, B28, 1e-3)
    for lam in (0.1, 0.6):
        check_atkf(oracle, x, dtype, keep, lam, M, max(1, M // 2), B28, 1e-3)


@pytest.mark.parametrize("lam", [0.1, 0.6])
def test_few_values_asymmetric_long(oracle, lam):
    check_atkf(oracle, rows_of(8192, "bf16"), "bf16", 0.1, lam, 8, 8, B28, 1e-3)


@pytest.mark.parametrize("N,keep,M", [(2560, 0.25, 16), (4096, 0.25, 32), (4096, 0.3, 16), (1280, 0.25, 16)])
def test_full_bins_of_fp32_rows(oracle, N, keep, M):
    """Up to 32 members in a boundary's bin, some of them with equal keys."""
    rng = np.random.default_rng(N + M)
    x = rng.standard_normal((24, N)).astype(np.float32)
    x[:, ::97] *= 8
    x[4:, ::331] *= np.float32(1e4)                   # wide bins
    x[8:] = synth.bf16_bits_to_f32(synth.f32_to_bf16_bits(x[8:]))
    x[16:, ::3] = np.abs(x[16:, ::3])
    check(oracle, x, "f32", keep, M, B28, 1e-3)
