"""Asymmetric thresholds on rows that a workgroup holds, byte-exact against the oracle."""
import numpy as np
import pytest

from paper_2511_11608_amd import synth
from tests.test_gpu_parity import B28, check_atkf

pytestmark = pytest.mark.gpu


def structures(dtype, rows, N, seed):
    """Rows of every kind in turn: plain, few distinct values, one sign, mostly negative, sparse over thirty octaves, few non-zeros, equal, zero."""
    rng = np.random.default_rng(seed)
    x = rng.standard_normal((rows, N)).astype(np.float32)
    x[1::9] = np.round(x[1::9] * 4) / 4
    x[2::9] = np.abs(x[2::9])
    x[3::9] = -np.abs(x[3::9]) + (rng.random(x[3::9].shape) < 0.02) * 3
    x[4::9] *= (rng.random(x[4::9].shape) < 0.3) * np.exp2(rng.uniform(-15, 15, x[4::9].shape))
    x[5::9] *= rng.random(x[5::9].shape) < 0.01
    x[6::9] = np.where(rng.random(x[6::9].shape) < 0.5, 1.5, -1.5)
    x[7::9, : N // 2] *= 1e-6
    x[8::9] = 0
    return synth.f32_to_bf16_bits(x) if dtype == "bf16" else x


@pytest.mark.parametrize("rows", [10, 140])
@pytest.mark.parametrize("dtype,N,keep,Mp,Mn", [("bf16", 4104, 0.1, 8, 8), ("bf16", 5001, 0.2, 3, 9), ("bf16", 8192, 0.05, 16, 16), ("bf16", 12288, 0.1, 8, 8),
                                                ("bf16", 32761, 0.02, 4, 4), ("f32", 4100, 0.25, 8, 8), ("f32", 5003, 0.1, 1, 1), ("f32", 8192, 0.15, 32, 32),
                                                ("f32", 16381, 0.05, 8, 2)])
def test_kinds_of_rows(oracle, dtype, N, keep, Mp, Mn, rows):
    x = structures(dtype, rows, N, N + rows)
    for lam in (0.1, 0.7):
        check_atkf(oracle, x, dtype, keep, lam, Mp, Mn, B28, 1e-3)
    check_atkf(oracle, x[:, : N - 1].copy(), dtype, keep, 0.3, Mp, Mn, (1 << 3) | (1 << 11), 1e-3)


@pytest.mark.parametrize("rows,N", [(4100, 4104), (4100, 6152), (300, 8192)])
def test_one_wavefront_or_one_workgroup(oracle, rows, N):
    check_atkf(oracle, structures("bf16", rows, N, 3), "bf16", 0.05, 0.2, 8, 8, B28, 1e-3)


@pytest.mark.parametrize("N,keep", [(768, 0.15), (2048, 0.1), (2060, 0.1), (4096, 0.05), (5000, 0.05), (9000, 0.03)])
@pytest.mark.parametrize("members", [1, 2, 63, 64, 65, 90])
def test_members_of_one_bin(oracle, N, keep, members):
    """fp32 rows whose selections end in a bin of the first histogram pass (65536 keys) with this many members, some of them equal."""
    rng = np.random.default_rng(N + members)
    k, rows = int(keep * N), 4
    x = np.empty((rows, N), dtype=np.float32)
    for i in range(rows):
        top = max(0, k - 1 - (i * members) // 4)
        v = np.concatenate([8 + 4 * rng.random(top), 1 + np.floor(rng.random(members) * 40) * 2.0 ** -16, 0.5 * rng.random(N - top - members)])
        x[i] = rng.permutation(v) * rng.choice([-1, 1], N)
    for lam in (0.0, 0.05, 0.5):
        check_atkf(oracle, x, "f32", keep, lam, 4, 4, B28, 1e-3)


def crowded(dtype, rows, N, seed):
    """Rows whose kept elements crowd into one fine bin or spread over more octaves than a bin's members can share a word for: fewer non-zeros than
    kept elements, clipped, of few levels, a far outlier above a crowd, denormals beside large values, one value from 250 places on."""
    rng = np.random.default_rng(seed)
    x = rng.standard_normal((rows, N)).astype(np.float32)
    x[0::7] *= rng.random(x[0::7].shape) < 0.05
    x[1::7] = np.clip(x[1::7], -1.3, 1.3)
    x[2::7] = np.round(x[2::7])
    x[3::7, N // 2] = 1e30
    x[4::7] *= (rng.random(x[4::7].shape) < 0.1) * np.exp2(rng.uniform(-140, 120, x[4::7].shape))
    for i, row in enumerate(x[5::7]):
        row[rng.permutation(N)[: 250 + 4 * (i % 4)]] = -2.5
    x[6::7] = np.where(rng.random(x[6::7].shape) < 0.1, 0.25 * np.sign(x[6::7]), x[6::7] * 1e-40)
    return synth.f32_to_bf16_bits(x) if dtype == "bf16" else x


@pytest.mark.parametrize("rows", [14, 150, 300])
@pytest.mark.parametrize("dtype,N,keep,Mp,Mn", [("bf16", 4104, 0.45, 8, 8), ("bf16", 6001, 0.3, 32, 32), ("bf16", 8192, 0.2, 8, 8), ("bf16", 12288, 0.15, 1, 3),
                                                ("f32", 4100, 0.4, 32, 32), ("f32", 8192, 0.15, 8, 8), ("f32", 16384, 0.1, 16, 2)])
def test_crowded_rows(oracle, dtype, N, keep, Mp, Mn, rows):
    x = crowded(dtype, rows, N, N + rows)
    for lam in (0.1, 0.95):
        check_atkf(oracle, x, dtype, keep, lam, Mp, Mn, B28, 1e-3)


@pytest.mark.parametrize("dtype,rows,N,keep", [("f32", 256, 8192, 0.15), ("f32", 2048, 8192, 0.15), ("bf16", 256, 8192, 0.2), ("bf16", 1024, 8192, 0.2)])
@pytest.mark.parametrize("kind", ["sparse", "clipped", "levels"])
def test_no_row_is_left_to_the_generic_kernel(dtype, rows, N, keep, kind):
    """Rows that are left over are encoded one after the other by a few workgroups, which takes 20 to 450 times as long as the batch; a row that
    stays takes at most a few times as long as one of continuous values, by the sort of its list."""
    import torch
    from paper_2511_11608_amd import binding
    x = torch.randn((rows, N), device="cuda")
    y = {"sparse": x * (torch.rand_like(x) < 0.1), "clipped": x.clamp(-1.3, 1.3), "levels": torch.round(x)}[kind]
    out = torch.bfloat16 if dtype == "bf16" else torch.float32

    def best(v):
        v = v.to(out).contiguous()
        bufs = binding.alloc_buffers_pn(v, keep, 8, 8, B28)
        times = []
        for _ in range(4):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            binding.slicer_encode_atkf(v, keep, 0.1, 8, 8, B28, 1e-3, *bufs)
            b.record()
            torch.cuda.synchronize()
            times.append(a.elapsed_time(b))
        return min(times)
    plain, crowd = best(x), best(y)
    assert crowd < 8 * plain, (crowd, plain)
