"""The row kernel's list of kept elements: every register layout of the row (elements per lane), with the kept elements spread
evenly, crowded into one place (one lane then lists all of its elements), and equal to each other; byte-exact against the oracle."""
import numpy as np
import pytest

from paper_2511_11608_amd import synth
from tests.test_gpu_parity import B28, check, check_atkf, check_ds

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
    x[1, ::40] *= np.float32(2.0) ** 50              # the cut lies many octaves below the largest values
    if dtype == "bf16":
        x = synth.f32_to_bf16_bits(x)
    check(oracle, x, dtype, 0.1, 4, B28, 1e-3)
    check_atkf(oracle, x, dtype, 0.1, 0.3, 4, 3, B28, 1e-3)


# one row, one finishing launch, one launch for offsets and copy with 1, 2 and 4 rows a wavefront, scan and copy
@pytest.mark.parametrize("dtype,rows,N", [("f32", 1, 300), ("bf16", 1, 4096), ("f32", 257, 64), ("bf16", 4095, 70), ("f32", 4097, 64),
                                          ("bf16", 8191, 64), ("f32", 8193, 64), ("f32", 32768, 32), ("bf16", 32769, 33), ("f32", 260, 4096)])
def test_where_the_rows_go(oracle, dtype, rows, N):
    rng = np.random.default_rng(rows)
    x = rng.standard_normal((rows, N)).astype(np.float32) * rng.uniform(0.01, 30, (rows, 1)).astype(np.float32)
    x[:: 7] = 0.0                                     # rows without a word among the others
    x[3 % rows] = 1.5
    if dtype == "bf16":
        x = synth.f32_to_bf16_bits(x)
    check(oracle, x, dtype, 0.3 if N > 300 else 0.4, 2, B28, 1e-3)


@pytest.mark.parametrize("rows,N,keep", [(256, 5120, 0.1), (257, 5120, 0.1), (300, 8192, 0.05), (300, 4104, 0.14), (260, 8192, 0.07)])
def test_rows_of_two_lengths_of_list(oracle, rows, N, keep):
    """bf16 rows of 4097 to 8192 elements: one wavefront or one workgroup per row, by batch and list."""
    x = np.random.default_rng(N + rows).standard_normal((rows, N)).astype(np.float32)
    x[:, ::900] *= np.float32(40)
    x[1] = 0.5
    check(oracle, synth.f32_to_bf16_bits(x), "bf16", keep, 8, B28, 1e-3)


@pytest.mark.parametrize("dtype,N,keep", [("f32", 300, 0.3), ("f32", 4096, 0.25), ("f32", 4096, 0.3), ("bf16", 1024, 0.2), ("bf16", 4096, 0.1)])
def test_few_and_many_bitwidths(oracle, dtype, N, keep):
    """A block's lanes are dealt to candidate bitwidths and slices: sets of one, two, three and all sixteen, classes with few and many blocks."""
    x = np.random.default_rng(N).standard_normal((6, N)).astype(np.float32)
    x[0] = np.abs(x[0])                               # one class alone
    x[1, ::5] *= np.float32(30)
    x[2] = -np.abs(x[2])
    if dtype == "bf16":
        x = synth.f32_to_bf16_bits(x)
    for bits in (1 << 4, 1 << 4 | 1 << 8, 1 << 2 | 1 << 5 | 1 << 9, 0x1FFFE):
        for Mp, Mn in ((1, 1), (1, 8), (4, 4), (3, 1), (16, 16), (2, 29)):
            check_atkf(oracle, x, dtype, keep, 0.0, Mp, Mn, bits, 1e-3)
        for M in (2, 4, 16):
            check_ds(oracle, x, dtype, keep, M, bits, 0.3)
