"""Rows that start or end inside a 16-byte chunk: odd lengths at the edges of the register layouts, and tensors
that do not start on a 16-byte boundary, byte-exact against the oracle."""
import numpy as np
import pytest

from paper_2511_11608_amd import synth
from tests.test_gpu_parity import B28, check, check_atkf

pytestmark = pytest.mark.gpu


def features(dtype, rows, N, seed):
    rng = np.random.default_rng(seed)
    x = rng.standard_normal((rows, N)).astype(np.float32)
    x[:, :: max(1, N // 6)] *= np.float32(30)
    x[rows // 2] = np.round(x[rows // 2] * 2) / 2        # long runs of equal keys, many zeros
    return synth.f32_to_bf16_bits(x) if dtype == "bf16" else x


LENGTHS = {"f32": [3, 255, 257, 766, 769, 1277, 1281, 2047, 4093, 4095, 8191, 16381, 16383],
           "bf16": [7, 505, 511, 1017, 1025, 2047, 3001, 4089, 4095, 6001, 8185, 8191, 16383, 32761, 32767]}


@pytest.mark.parametrize("dtype,N", [(d, n) for d in LENGTHS for n in LENGTHS[d]])
def test_lengths_around_the_layouts(oracle, dtype, N):
    rows = 19 if N < 5000 else 6
    x = features(dtype, rows, N, N)
    check(oracle, x, dtype, min(0.1, 1500 / N), 4, B28, 1e-3, use_header=bool(N & 2))
    if N <= 4096:
        check_atkf(oracle, x, dtype, 0.15, 0.2, 4, 3, B28, 1e-3)


@pytest.mark.parametrize("dtype,rows,N,shift", [("f32", 9, 768, 1), ("f32", 300, 1024, 3), ("f32", 5, 4096, 2), ("bf16", 9, 4096, 1),
                                                ("bf16", 400, 512, 5), ("bf16", 4, 8192, 7), ("bf16", 3, 1001, 3),
                                                # aligned they are the longest rows of the workgroup-per-row kernel
                                                ("f32", 6, 16384, 1), ("bf16", 3, 32768, 7)])
def test_tensors_that_start_anywhere(oracle, dtype, rows, N, shift):
    import torch
    from paper_2511_11608_amd import binding
    from paper_2511_11608_amd.devmem import to_device, to_host
    x = features(dtype, rows, N, 7 * N + shift)
    s_ref, m_ref = oracle.encode(x, dtype, 0.1, 8, B28, 1e-3, n_threads=8)
    y_ref = oracle.decode(s_ref, m_ref, n_threads=8)
    xd = to_device(x, dtype)
    sb, meta, ws = binding.alloc_buffers(xd, 0.1, 8, B28)
    ws.fill_(0x5A)
    big = torch.full((rows * N + 16,), 9e30, dtype=xd.dtype, device="cuda")     # neighbours larger than every value of a row
    view = big[shift:shift + rows * N].view(rows, N)
    view.copy_(xd)
    binding.slicer_encode(view, 0.1, 8, B28, 1e-3, sb, meta, ws)
    words = binding.slicer_stream_words(meta)
    assert np.array_equal(meta.cpu().numpy(), m_ref)
    assert np.array_equal(sb[:words].cpu().numpy().view(np.uint32), s_ref)
    big.fill_(3.0)
    binding.slicer_decode_as(sb, meta, view, 8)
    torch.cuda.synchronize()
    assert np.array_equal(to_host(view.clone()), y_ref)
    assert bool((big[:shift] == 3).all()) and bool((big[shift + rows * N:] == 3).all())     # nothing beside y is written


def test_static_scratch_serves_odd_rows_without_the_long_row_tables(oracle):
    import torch
    from paper_2511_11608_amd import binding
    from paper_2511_11608_amd.devmem import to_device
    rows, N, keep = 1322, 16399, 0.02                   # 67 MiB with the tables of the long-row stages, 8 MiB without
    assert binding.slicer_sizes(binding.SLICER_F32, rows, N, keep, 8, B28)[2] > 64 << 20
    x = features("f32", rows, N, 3)
    s_ref, m_ref = oracle.encode(x, "f32", keep, 8, B28, 1e-3, n_threads=8)
    xd = to_device(x, "f32")
    sb, meta, _ = binding.alloc_buffers(xd, keep, 8, B28)
    binding.slicer_encode_static(xd, keep, 8, B28, 1e-3, sb, meta)
    words = binding.slicer_stream_words(meta)
    torch.cuda.synchronize()
    assert np.array_equal(meta.cpu().numpy(), m_ref)
    assert np.array_equal(sb[:words].cpu().numpy().view(np.uint32), s_ref)


def test_static_scratch_serves_whole_rows_without_the_long_row_tables(oracle):
    import torch
    from paper_2511_11608_amd import binding
    from paper_2511_11608_amd.devmem import to_device
    rows, N, keep, M, bits = 1560, 4928, 0.02, 33, 0x24     # 69 MiB with the tables of the long-row stages, 4 MiB without
    x = features("f32", rows, N, 4)
    s_ref, m_ref = oracle.encode(x, "f32", keep, M, bits, 1e-3, n_threads=8)
    xd = to_device(x, "f32")
    sb, meta, _ = binding.alloc_buffers(xd, keep, M, bits)
    binding.slicer_encode_static(xd, keep, M, bits, 1e-3, sb, meta)
    words = binding.slicer_stream_words(meta)
    torch.cuda.synchronize()
    assert np.array_equal(meta.cpu().numpy(), m_ref)
    assert np.array_equal(sb[:words].cpu().numpy().view(np.uint32), s_ref)
