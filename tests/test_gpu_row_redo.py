"""Rows that the long-row stages leave to the generic encoder inside their own launch, while one to eight workgroups share the row."""
import numpy as np
import pytest

from paper_2511_11608_amd import synth
from tests.test_gpu_parity import B28, check, check_csr, check_ds

pytestmark = pytest.mark.gpu


def clipped(dtype, rows, N, keep, pos, neg, seed):
    """Some large values, `pos` places of +1.5 and `neg` of -1.5 (one fine bin, far above the cut), and continuous values of either sign
    in which the cut falls: an order statistic of the cut is read from the list before the clipped bin turns out too large."""
    rng = np.random.default_rng(seed)
    k, top = int(keep * N), 600
    assert top + pos + neg < k < N
    x = np.empty((rows, N), dtype=np.float32)
    for i in range(rows):
        v = np.concatenate([2 + rng.random(top), np.full(pos, 1.5), 0.5 * rng.random(N - top - pos - neg) + 0.25])
        v *= rng.choice([-1.0, 1.0], v.size)
        v[top:top + pos] = 1.5
        x[i] = rng.permutation(np.concatenate([v, np.full(neg, -1.5)]))
    return synth.f32_to_bf16_bits(x) if dtype == "bf16" else x


# 32, 64 and 128 rows are the most that eight, four and two workgroups a row have
@pytest.mark.parametrize("rows", [1, 4, 32, 33, 64, 65, 128, 129])
@pytest.mark.parametrize("dtype,pos,neg", [("f32", 7000, 0), ("f32", 7000, 7000), ("bf16", 0, 9000)])
def test_one_value_overflows_a_shared_row(oracle, dtype, pos, neg, rows):
    x = clipped(dtype, rows, 50_001 if rows < 32 else 40_004, 0.45, pos, neg, rows)
    if rows > 3:                                        # most rows of a batch fit
        x[1::3] = clipped(dtype, len(x[1::3]), x.shape[1], 0.45, 500, 500, 1)
    check(oracle, x, dtype, 0.45, 8, B28, 1e-3)


@pytest.mark.parametrize("pos", [508, 512, 513, 1500, 2049, 4096, 6143, 6144, 6145, 12000, 16000, 16384, 16385, 30000])
def test_around_the_room_for_members(oracle, pos):
    """Rows of many blocks and long lists have room for 16384 members, the others for 6144; bins of more than 512 members are sorted."""
    for N, keep, M in ((90_000, 0.45, 8), (140_000, 0.5, 64)):
        x = clipped("f32", 2, N, keep, pos, 300, pos)
        check(oracle, x, "f32", keep, M, B28, 1e-3)
    check_ds(oracle, x, "f32", 0.5, 64, (1 << 2) | (1 << 5) | (1 << 12), 0.3)


@pytest.mark.parametrize("dtype,rows,N,keep,M", [("f32", 1, 4_000_000, 0.6, 16), ("bf16", 2, 3_000_001, 0.7, 3), ("f32", 270, 20_000, 0.5, 2), ("bf16", 270, 30_000, 0.5, 4)])
def test_crowded_bins_of_several_keys(oracle, dtype, rows, N, keep, M):
    """Long lists have thousands of members a bin; and values of a few levels, some a last place apart, put several keys and many ties into one."""
    rng = np.random.default_rng(N)
    x = rng.standard_normal((rows, N)).astype(np.float32)
    x[:, : N // 2] = np.round(x[:, : N // 2] * 4) / 4 * (1 + rng.integers(0, 3, (rows, N // 2)) * 2.0 ** -23)
    check(oracle, synth.f32_to_bf16_bits(x) if dtype == "bf16" else x, dtype, keep, M, B28, 1e-3)


def test_csr_instances(oracle):
    check_csr(oracle, clipped("f32", 3, 200 * 300, 0.4, 3000, 4000, 5), "f32", 200, 300, 0.4, 8, B28, 1e-3)
    check_csr(oracle, clipped("f32", 3, 200 * 300, 0.4, 9000, 7000, 5), "f32", 200, 300, 0.4, 8, B28, 1e-3)


@pytest.mark.parametrize("rows", [1, 8, 40, 100])
def test_beside_other_streams(oracle, rows):
    """The row's workgroups start at different times where other work holds CUs: every one of them must have left the list before the redo."""
    import torch
    from paper_2511_11608_amd import binding
    from paper_2511_11608_amd.devmem import to_device
    x = clipped("f32", rows, 40_004, 0.45, 7000, 7000, rows)
    s_ref, m_ref = oracle.encode(x, "f32", 0.45, 8, B28, 1e-3, n_threads=8)
    xd = to_device(x, "f32")
    other = torch.randn((256, 401_408), device="cuda")
    jobs = [(xd, binding.alloc_buffers(xd, 0.45, 8, B28), torch.cuda.Stream()) for _ in range(3)]
    load = (other, binding.alloc_buffers(other, 0.2, 16, B28), torch.cuda.Stream())
    torch.cuda.synchronize()
    for _ in range(4):
        with torch.cuda.stream(load[2]):
            binding.slicer_encode(other, 0.2, 16, B28, 1e-3, *load[1])
        for xj, bufs, st in jobs:
            with torch.cuda.stream(st):
                binding.slicer_encode(xj, 0.45, 8, B28, 1e-3, *bufs)
    torch.cuda.synchronize()
    for _, (sb, meta, _), _ in jobs:
        assert np.array_equal(meta.cpu().numpy(), m_ref)
        assert np.array_equal(sb[:s_ref.size].cpu().numpy().view(np.uint32), s_ref)


def test_crowded_bins_cost_no_square():
    """16000 equal values in a bin: compared with each other they took 40 to 50 times as long as a row of continuous values, sorted some three times."""
    import torch
    from paper_2511_11608_amd import binding
    from paper_2511_11608_amd.devmem import to_device

    def best(x):
        xd = to_device(x, "f32")
        bufs = binding.alloc_buffers(xd, 0.5, 64, B28)
        times = []
        for _ in range(4):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            binding.slicer_encode(xd, 0.5, 64, B28, 1e-3, *bufs)
            b.record()
            torch.cuda.synchronize()
            times.append(a.elapsed_time(b))
        return min(times)
    plain = best(np.random.default_rng(1).standard_normal((1, 140_000)).astype(np.float32))
    crowd = best(clipped("f32", 1, 140_000, 0.5, 8000, 8000, 1))
    assert crowd < 12 * plain, (crowd, plain)
