"""The two decoders of long instances at their edges: one block to 64 of them per class, tensor rows of one column, of a few columns (sixteen
rows a workgroup) and longer than the LDS image, output chunks that start off 16 bytes, launches below and above one workgroup per
CU; byte-exact against the oracle."""
import numpy as np
import pytest

from paper_2511_11608_amd import synth
from tests.test_gpu_parity import B28, check, check_csr

pytestmark = pytest.mark.gpu


def features(dtype, rows, N):
    rng = np.random.default_rng(N + rows)
    x = rng.standard_normal((rows, N)).astype(np.float32) * np.repeat(rng.uniform(0.1, 4, (rows, N // 50 + 1)).astype(np.float32), 50, 1)[:, :N]
    x[0, : N // 2] = np.abs(x[0, : N // 2])
    x[-1, N // 3:] = 0.0                               # one end of the row holds every entry
    return synth.f32_to_bf16_bits(x) if dtype == "bf16" else x


@pytest.mark.parametrize("dtype,rows,n_rows,n_cols,M", [("f32", 3, 512, 49, 64), ("bf16", 2, 3, 20000, 5), ("f32", 9, 40, 1, 4), ("bf16", 40, 701, 13, 16),
                                                        ("f32", 2, 1, 5000, 1), ("f32", 32, 64, 784, 16), ("bf16", 1, 9000, 3, 33)])
def test_two_dimensional(oracle, dtype, rows, n_rows, n_cols, M):
    check_csr(oracle, features(dtype, rows, n_rows * n_cols), dtype, n_rows, n_cols, 0.2, M, B28, 1e-3)


@pytest.mark.parametrize("dtype,rows,N,M", [("f32", 2, 33001, 64), ("bf16", 3, 100003, 1), ("f32", 40, 40004, 16), ("bf16", 33, 70002, 33), ("f32", 1, 4099, 64)])
def test_long_rows(oracle, dtype, rows, N, M):
    for header in (False, True):
        check(oracle, features(dtype, rows, N), dtype, 0.1, M, B28, 1e-3, use_header=header)


def test_headers_read_by_many_threads(oracle):
    """slicer_decode and slicer_stream_words learn the shape from the header: 40 threads at once, each with a stream and a shape of its own."""
    import threading
    import torch
    from paper_2511_11608_amd import binding
    from paper_2511_11608_amd.devmem import to_device, to_host
    jobs = []
    for i in range(40):
        x = features("f32", 1 + i % 3, 300 + 7 * i)
        s_ref, m_ref = oracle.encode(x, "f32", 0.2, 2, B28, 1e-3)
        xd = to_device(x, "f32")
        sb, meta, ws = binding.alloc_buffers(xd, 0.2, 2, B28)
        binding.slicer_encode(xd, 0.2, 2, B28, 1e-3, sb, meta, ws)
        jobs.append((sb, meta, torch.full_like(xd, 7.0), oracle.decode(s_ref, m_ref), len(s_ref), []))
    torch.cuda.synchronize()

    def work(sb, meta, y, y_ref, words, bad):
        st = torch.cuda.Stream()
        with torch.cuda.stream(st):
            for _ in range(20):
                if binding.slicer_stream_words(meta) != words:
                    bad.append("words")
                y.fill_(3.0)
                binding.slicer_decode(sb, meta, y)
                st.synchronize()
                if not np.array_equal(to_host(y).view(np.uint32), y_ref.view(np.uint32)):
                    bad.append("values")

    threads = [threading.Thread(target=work, args=j) for j in jobs]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not any(j[5] for j in jobs)


def one_decode(oracle):
    import torch
    from paper_2511_11608_amd import binding
    from paper_2511_11608_amd.devmem import to_device, to_host
    x = features("f32", 3, 3000)
    s_ref, m_ref = oracle.encode(x, "f32", 0.2, 2, B28, 1e-3)
    y_ref = oracle.decode(s_ref, m_ref).view(np.uint32)
    xd = to_device(x, "f32")
    sb, meta, ws = binding.alloc_buffers(xd, 0.2, 2, B28)
    binding.slicer_encode(xd, 0.2, 2, B28, 1e-3, sb, meta, ws)
    y = torch.empty_like(xd)
    torch.cuda.synchronize()

    def decode():
        binding.slicer_decode(sb, meta, y)

    def check_values():
        torch.cuda.synchronize()
        assert np.array_equal(to_host(y).view(np.uint32), y_ref)
        y.fill_(3.0)

    return decode, check_values


def test_header_behind_other_work(oracle):
    """More than a millisecond of work before the call: the header is waited for in the ordinary way; 40 times, more than there are slots."""
    import torch
    decode, check_values = one_decode(oracle)
    a = torch.zeros((4096, 4096), device="cuda")
    for _ in range(40):
        for _ in range(4):
            a = a @ a                                # some milliseconds in all
        decode()
        check_values()


def test_older_errors_cost_no_header_slot(oracle):
    """An error that an earlier, unrelated call left is reported, as a launch reports it; the header's way to the host stays the fast one."""
    import time
    from paper_2511_11608_amd import binding
    decode, check_values = one_decode(oracle)
    hip = binding.load()

    def fastest():
        best = 1.0
        for _ in range(300):
            t = time.perf_counter()
            decode()
            best = min(best, time.perf_counter() - t)
        check_values()
        return best

    before = fastest()
    for _ in range(40):
        assert hip.hipSetDevice(9999) != 0
        with pytest.raises(binding.SlicerError) as ei:
            decode()
        assert ei.value.code == -3
        hip.hipGetLastError()                        # (whoever reported it may have cleared it)
    decode()
    check_values()
    assert fastest() < 1.5 * before                  # the copy and the wait take twice as long


@pytest.mark.parametrize("dtype,rows,n_rows,n_cols,keep,M", [("f32", 2, 40000, 2, 0.1, 8), ("bf16", 3, 2048, 49, 0.1, 64), ("f32", 40, 512, 49, 0.1, 8), ("f32", 1, 100000, 3, 0.05, 16),
                                                             ("f32", 9, 9000, 1, 0.2, 2), ("f32", 12, 512, 784, 0.1, 16), ("f32", 1, 100, 7, 0.2, 4)])
def test_windows_of_row_pointers(oracle, dtype, rows, n_rows, n_cols, keep, M):
    """Encoders' windows of 128 to 1024 words of pointers, walked and searched, before and behind the windows of codes; instances of a few
    elements a tensor row for the decoder."""
    check_csr(oracle, features(dtype, rows, n_rows * n_cols), dtype, n_rows, n_cols, keep, M, B28, 1e-3)
