"""Long-row stages at the edges of their tiles, tables and launch rules, byte-exact against the oracle."""
import numpy as np
import pytest

from paper_2511_11608_amd import synth
from tests.test_gpu_parity import B28, check, check_csr, check_ds, check_ladder

pytestmark = pytest.mark.gpu


def features(dtype, rows, N, seed, kind="normal"):
    rng = np.random.default_rng(seed)
    x = rng.standard_normal((rows, N)).astype(np.float32)
    if kind == "relu":
        x = np.abs(x) * (rng.random((rows, N)) < 0.5)
    elif kind == "sparse":                              # fewer non-zeros than kept elements, over thirty octaves
        x = x * (rng.random((rows, N)) < 0.03) * np.exp2(rng.uniform(-15, 15, (rows, N)))
    elif kind == "ties":                                # a few dozen distinct values
        x = np.round(x * 8) / 8
    elif kind == "outliers":
        x[:, :: N // 7] *= 3000
    elif kind == "patches":                             # constant stretches: one key fills whole tiles
        x = np.repeat(x[:, : (N + 999) // 1000], 1000, axis=1)[:, :N] + (rng.random((rows, N)) < 0.2)
    x = x.astype(np.float32)
    return synth.f32_to_bf16_bits(x) if dtype == "bf16" else x


@pytest.mark.parametrize("dtype,rows,N", [("f32", 3, 16388), ("f32", 2, 32768), ("f32", 1, 81919), ("f32", 2, 81921), ("bf16", 2, 65544), ("bf16", 3, 40961),
                                          ("f32", 40, 65536), ("f32", 41, 65533), ("f32", 300, 16640), ("bf16", 270, 33001)])
def test_tiles_and_batches(oracle, dtype, rows, N):
    check(oracle, features(dtype, rows, N, N), dtype, 0.12, 8, B28, 1e-3, use_header=bool(rows & 1))


@pytest.mark.parametrize("dtype,rows,N,keep,M", [("f32", 257, 20480, 0.05, 8), ("bf16", 257, 33001, 0.05, 8), ("bf16", 300, 8192, 0.25, 8),
                                                 ("f32", 258, 4100, 0.1, 40), ("bf16", 258, 8193, 0.1, 40), ("f32", 257, 16388, 0.9, 1),
                                                 ("f32", 260, 16640, 0.0005, 16), ("f32", 257, 70001, 0.4, 2)])
def test_large_batches(oracle, dtype, rows, N, keep, M):
    """More than 256 rows: the stages with 1024 fine bins; rows of equal values are left to the generic kernel."""
    x = features(dtype, rows, N, N)
    for i, kind in enumerate(("sparse", "ties", "patches", "relu")):       # a few rows of every structure
        x[7 + i::41] = features(dtype, rows, N, i, kind)[7 + i::41]
    x[3] = 0
    check(oracle, x, dtype, keep, M, B28, 1e-3)
    check_ds(oracle, x[:, : N - 3].copy(), dtype, keep, M, (1 << 2) | (1 << 5) | (1 << 12), 0.3)


@pytest.mark.parametrize("dtype,shift", [("f32", 0), ("f32", 1), ("bf16", 0), ("bf16", 7)])
def test_longest_rows(oracle, dtype, shift):
    """2^23 elements: 512 tiles, wherever the row starts in its first 16 bytes."""
    import torch
    from paper_2511_11608_amd import binding
    from paper_2511_11608_amd.devmem import to_device
    N = 1 << 23
    x = features(dtype, 1, N, 23)
    s_ref, m_ref = oracle.encode(x, dtype, 0.01, 8, B28, 1e-3)
    xd = to_device(x, dtype)
    big = torch.zeros(N + 16, dtype=xd.dtype, device="cuda")
    view = big[shift:shift + N].view(1, N)
    view.copy_(xd)
    sb, meta, ws = binding.alloc_buffers(view, 0.01, 8, B28)
    ws.fill_(0xA5)
    binding.slicer_encode(view, 0.01, 8, B28, 1e-3, sb, meta, ws)
    words = binding.slicer_stream_words(meta)
    assert np.array_equal(meta.cpu().numpy(), m_ref)
    assert np.array_equal(sb[:words].cpu().numpy().view(np.uint32), s_ref)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("kind", ["relu", "sparse", "ties", "outliers", "patches"])
def test_value_structures(oracle, dtype, kind):
    x = features(dtype, 3, 50_000, 11, kind)
    for keep, M in ((0.05, 4), (0.2, 16), (0.6, 31), (0.2, 33), (0.3, 64), (1.0, 5)):
        check(oracle, x, dtype, keep, M, B28, 1e-3)
    check_ds(oracle, x, dtype, 0.2, 16, (1 << 2) | (1 << 5) | (1 << 12), 0.3)
    check_ladder(oracle, x, dtype, 0.2, [8, 7, 6, 5, 4, 3, 2, 2])


@pytest.mark.parametrize("dtype,inst,n_rows,n_cols", [("f32", 2, 1, 60_000), ("f32", 2, 60_000, 1), ("f32", 3, 197, 301), ("bf16", 2, 128, 513), ("f32", 260, 40, 512)])
def test_csr_blocks(oracle, dtype, inst, n_rows, n_cols):
    for kind in ("normal", "sparse"):
        check_csr(oracle, features(dtype, inst, n_rows * n_cols, 5, kind), dtype, n_rows, n_cols, 0.1, 8, B28, 1e-3)


@pytest.mark.parametrize("inst,n_rows,n_cols,M,keep", [(2, 40_000, 1, 1, 0.3), (3, 9_000, 7, 1, 0.2), (2, 1, 50_000, 16, 0.3), (2, 7, 9_001, 16, 0.3),
                                                       (1, 2_049, 33, 2, 0.5)])
def test_csr_pointers_searched_and_walked(oracle, inst, n_rows, n_cols, M, keep):
    """Windows that hold a part of a block's row pointers, blocks with far more entries than pointers, and the reverse."""
    for kind in ("relu", "normal", "patches"):
        check_csr(oracle, features("f32", inst, n_rows * n_cols, 6, kind), "f32", n_rows, n_cols, keep, M, B28, 1e-3)


@pytest.mark.parametrize("dtype,shift", [("f32", 3), ("bf16", 5)])
def test_csr_of_long_rows_through_the_flat_stream(oracle, dtype, shift):
    """The stages write CSR themselves only for aligned tensors and pointers of eight bits and more."""
    import torch
    from paper_2511_11608_amd import binding
    from paper_2511_11608_amd.devmem import to_device
    n_rows, n_cols = 120, 400
    x = features(dtype, 2, n_rows * n_cols, 8)
    for keep in (0.0, 0.5 / (n_rows * n_cols), 100.5 / (n_rows * n_cols), 127.5 / (n_rows * n_cols), 128.5 / (n_rows * n_cols)):    # k = 0, 0, 100, 127, 128
        check_csr(oracle, x, dtype, n_rows, n_cols, keep, 4, B28, 1e-3)
    s_ref, m_ref = oracle.encode_csr(x, dtype, n_rows, n_cols, 0.1, 8, B28, 1e-3, n_threads=8)
    xd = to_device(x, dtype)
    view = torch.zeros(x.size + 16, dtype=xd.dtype, device="cuda")[shift:shift + x.size].view(x.shape)
    view.copy_(xd)
    sb, meta, ws = binding.alloc_buffers_csr(view, n_rows, n_cols, 0.1, 8, B28)
    ws.fill_(0xA5)
    binding.slicer_encode_csr(view, n_rows, n_cols, 0.1, 8, B28, 1e-3, sb, meta, ws)
    words = binding.slicer_stream_words(meta)
    assert np.array_equal(meta.cpu().numpy(), m_ref)
    assert np.array_equal(sb[:words].cpu().numpy().view(np.uint32), s_ref)


@pytest.mark.parametrize("dtype,rows,N,keep,M", [("f32", 3, 40_000, 0.8, 8), ("f32", 40, 65_549, 0.3, 8), ("bf16", 3, 40_001, 0.8, 8), ("bf16", 40, 65_549, 0.2, 8),
                                                 ("bf16", 90, 30_002, 0.5, 3), ("f32", 130, 17_000, 0.2, 16), ("f32", 2, 140_000, 0.5, 64), ("f32", 1, 600_000, 0.03, 4),
                                                 ("f32", 4, 401_000, 0.1, 8), ("bf16", 1, 1_700_003, 0.05, 4), ("f32", 16, 400_001, 0.05, 4), ("bf16", 130, 50_001, 0.7, 4), ("f32", 130, 50_002, 0.6, 64),
                                                 ("f32", 130, 50_000, 1.0, 5), ("bf16", 260, 30_000, 1.0, 2), ("f32", 260, 30_001, 0.5, 3)])
def test_dense_tiles_and_shared_rows(oracle, dtype, rows, N, keep, M):
    """Wavefronts with more entries than their room (640) beside emptier ones, in lists that are sparse, dense or the whole row; one to eight workgroups for a row's order statistics; tiles that are no
    power of two; rows of odd length whose words hold halves of two rows; the larger room for a row's bin members."""
    x = features(dtype, rows, N, N)
    x[:, N // 3: N // 2] = 0                            # some tiles hold nothing ...
    x[:, N // 2: N // 2 + 3000] = features(dtype, rows, 3000, 1)
    for i in range(rows):                               # ... and some hold only entries
        lo = (i * 997) % (N - 6000)
        big = np.abs(features("f32", 1, 5000, i)[0]) + 4
        x[i, lo:lo + 5000] = synth.f32_to_bf16_bits(big) if dtype == "bf16" else big
    check(oracle, x, dtype, keep, M, B28, 1e-3)
