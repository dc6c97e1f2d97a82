"""GPU parity of hadamard_transform_ws against the oracle: n = 2^17 .. 2^20, and n
= 2^16 (the largest size without a workspace) through the same entry.  Which way a
call takes depends on n, m and the mode: with the few rows here 2^17 out of place
runs by workgroups that share a row, the others in two passes through the fp32
workspace; tests/test_gpu_parts.py compares the two ways.

Same criterion as the other sizes (tests/metrics.py): every intermediate is fp32,
so the result is rounded once.
"""
from __future__ import annotations

import numpy as np
import pytest

from gpu_util import compare_with_oracle, say, to_device, to_host
from metrics import bits_to_f64
from paper_2412_08832_amd import hadacore as H
from paper_2412_08832_amd import workloads as W

pytestmark = pytest.mark.gpu

DTYPES = ["fp16", "bf16"]
CODE = {"fp16": H.FP16, "bf16": H.BF16}


@pytest.fixture(scope="module", autouse=True)
def _device():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    H.library()
    yield
    torch.cuda.synchronize()


def _run_ws(bits, dtype, scale, n, inplace, out_stride=None, out_fill=0xAAAA, canary=0x5C):
    """Transform through hadamard_transform_ws; returns output bits and the workspace tail."""
    import torch
    m, in_stride = bits.shape
    x = to_device(bits, dtype)
    if inplace:
        out, out_stride = x, in_stride
    else:
        out_stride = n if out_stride is None else out_stride
        out = to_device(np.full((m, out_stride), out_fill, np.uint16), dtype)
    need = H.hadamard_transform_workspace_size(m, n)
    ws = torch.full((need + 4096,), canary, dtype=torch.uint8, device="cuda")
    H.hadamard_transform_ws(x.data_ptr(), in_stride, out.data_ptr(), out_stride, m, n, CODE[dtype],
                            scale, ws.data_ptr(), need, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    return to_host(out), ws[need:].cpu().numpy()


@pytest.mark.parametrize("inplace", [False, True], ids=["out", "inplace"])
@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("L", [16, 17, 18, 19, 20])
def test_large_sizes(oracle, L, dtype, inplace):
    n = 1 << L
    m = 5 if L <= 18 else 3
    say(f"large n={n} m={m} {dtype} inplace={inplace}")
    bits = W.random_rows(m, n, dtype, seed=4000 + L)
    s = W.default_scale(n)
    out, tail = _run_ws(bits, dtype, s, n, inplace)
    assert (tail == 0x5C).all(), "workspace written past its size"
    c = compare_with_oracle(oracle, out, bits, dtype, s, n)
    say(f"  {c}")
    assert c.ok, str(c)


@pytest.mark.parametrize("dtype", DTYPES)
def test_large_strided_rows_keep_gaps(oracle, dtype):
    n = 1 << 17
    m = 4
    bits = W.random_rows(m, n, dtype, seed=17, stride=n + 24, fill_bits=0x7FC1)
    s = W.default_scale(n)
    out, _ = _run_ws(bits, dtype, s, n, False, out_stride=n + 40, out_fill=0x5A5A)
    assert (out[:, n:] == 0x5A5A).all(), "out-of-place write touched the row gap"
    c = compare_with_oracle(oracle, out[:, :n], bits, dtype, s, n)
    assert c.ok, str(c)
    out2, _ = _run_ws(bits, dtype, s, n, True)
    assert (out2[:, n:] == 0x7FC1).all(), "in-place write touched the row gap"
    assert np.array_equal(out2[:, :n], out[:, :n])


@pytest.mark.parametrize("L", [16, 18, 20])
def test_large_special_vectors(L):
    n = 1 << L
    rows = np.zeros((3, n), np.uint16)
    rows[0, 0] = 0x3C00                       # delta -> all ones
    rows[1, :] = 0x3C00                       # ones -> n e_0
    k = n // 2 + 12345                         # a Walsh row -> n e_k
    j = np.arange(n, dtype=np.int64)
    parity = np.zeros(n, dtype=np.int64)
    v = j & k
    while v.any():
        parity ^= v & 1
        v >>= 1
    rows[2] = np.where(parity == 1, 0xBC00, 0x3C00).astype(np.uint16)
    s = 2.0 ** -(L // 2)
    out, _ = _run_ws(rows, "fp16", s, n, False)
    y = bits_to_f64(out, "fp16")
    assert np.array_equal(y[0], np.full(n, s))
    e0 = np.zeros(n)
    e0[0] = n * s
    assert np.array_equal(y[1], e0)
    ek = np.zeros(n)
    ek[k] = n * s
    assert np.array_equal(y[2], ek)


def test_large_deterministic_and_wrapper():
    import torch
    n = 1 << 18
    bits = W.random_rows(4, n, "bf16", seed=99)
    a, _ = _run_ws(bits, "bf16", W.default_scale(n), n, False)
    b, _ = _run_ws(bits, "bf16", W.default_scale(n), n, True)
    assert np.array_equal(a, b)
    x = to_device(bits, "bf16")
    y = H.transform(x)                         # allocates its own workspace
    torch.cuda.synchronize()
    assert np.array_equal(to_host(y), a)


@pytest.mark.parametrize("n", [1 << 12, 1 << 16])
def test_one_pass_sizes_through_the_workspace_entry(n):
    """n <= 2^16 through hadamard_transform_ws needs no workspace and matches the one-pass call."""
    import torch
    assert H.hadamard_transform_workspace_size(33, n) == 0
    bits = W.random_rows(33, n, "fp16", seed=5)
    x = to_device(bits, "fp16")
    out = torch.empty_like(x)
    H.hadamard_transform_ws(x.data_ptr(), n, out.data_ptr(), n, 33, n, H.FP16, W.default_scale(n),
                            0, 0, torch.cuda.current_stream().cuda_stream)
    ref = H.transform(x)
    torch.cuda.synchronize()
    assert torch.equal(out, ref)


def _split_rows(m: int, per_launch: int) -> np.ndarray:
    """Rows on both sides of every launch boundary, the first and the last."""
    edges = [r for b in range(per_launch, m, per_launch) for r in (b - 2, b - 1, b, b + 1)]
    return np.unique(np.r_[0, 1, edges, m - 2, m - 1])


def test_rows_beyond_one_launch_are_split(oracle):
    """bf16 n = 128 in place with m = 2^26 + 1000 rows (16 GiB): more rows than one
    launch takes (2^33 elements per launch), so the call is two launches; rows on
    both sides of the boundary match the oracle.  The input is a 4096-row seeded
    block repeated, so every row's input is known on the host."""
    import torch
    n, per_launch = 128, 1 << 26
    m = per_launch + 1000
    block = W.random_rows(4096, n, "bf16", seed=128)
    reps = (m + 4095) // 4096
    say(f"split: bf16 n={n} m={m} in place ({m * n * 2 / 2**30:.1f} GiB)")
    x = to_device(block, "bf16").repeat(reps, 1)
    s = W.default_scale(n)
    H.hadamard_transform(x.data_ptr(), x.data_ptr(), m, n, H.BF16, s,
                         torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    rows = _split_rows(m, per_launch)
    got = to_host(x[torch.from_numpy(rows).cuda()])
    c = compare_with_oracle(oracle, got, block[rows % 4096], "bf16", s, n)
    say(f"  {c}")
    assert c.ok, str(c)
    # rows past m are untouched: the repeated block continues unchanged
    tail = to_host(x[m:])
    assert np.array_equal(tail, block[m % 4096: m % 4096 + tail.shape[0]])
    del x
    torch.cuda.empty_cache()


def test_quantized_rows_beyond_one_launch_are_split(oracle):
    """The same split for the fused FP8 output (codes and scales offset per launch)."""
    import torch
    from fp8_compare import compare_fp8
    n, per_launch = 128, 1 << 26
    m = per_launch + 1000
    block = W.random_rows(4096, n, "fp16", seed=129)
    say(f"split fp8: fp16 n={n} m={m}")
    x = to_device(block, "fp16").repeat((m + 4095) // 4096, 1)
    codes = torch.empty((m, n), dtype=torch.uint8, device="cuda")
    scales = torch.full((m,), -1.0, dtype=torch.float32, device="cuda")
    s = W.default_scale(n)
    H.hadamard_transform_fp8(x.data_ptr(), n, codes.data_ptr(), n, scales.data_ptr(), m, n,
                             H.FP16, s, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    rows = _split_rows(m, per_launch)
    idx = torch.from_numpy(rows).cuda()
    c = compare_fp8(oracle, codes[idx].cpu().numpy(), scales[idx].cpu().numpy(),
                    block[rows % 4096], "fp16", s, n)
    say(f"  {c}")
    assert c.ok, str(c)
    del x, codes, scales
    torch.cuda.empty_cache()


def test_large_rows_beyond_one_launch_are_split(oracle):
    """bf16 n = 2^17 in place with 2^16 + 16 rows (16 GiB): two launches of workgroups
    that share rows, the second with its arrive words and deferred parts behind the
    first one's in the workspace.  The input is an 8-row seeded block repeated: every
    row has its block row's bits, and the oracle checks the block."""
    import torch
    n, per_launch = 1 << 17, 1 << 16
    m = per_launch + 16
    block = W.random_rows(8, n, "bf16", seed=1717)
    s = W.default_scale(n)
    say(f"split: bf16 n={n} m={m} in place ({m * n * 2 / 2**30:.1f} GiB)")
    b = to_device(block, "bf16")
    ref = H.transform(b)
    c = compare_with_oracle(oracle, to_host(ref), block, "bf16", s, n)
    assert c.ok, str(c)
    x = b.repeat(m // 8 + 1, 1)        # eight rows past m
    need = H.hadamard_transform_workspace_size(m, n)
    ws = torch.empty(need + 4096, dtype=torch.uint8, device="cuda")
    ws[need - 4096:] = 0x5C
    H.hadamard_transform_ws(x.data_ptr(), n, x.data_ptr(), n, m, n, H.BF16, s, ws.data_ptr(), need,
                            torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    got = x.view(torch.int16).view(-1, 8, n)
    want = ref.view(torch.int16)
    for r in range(0, m // 8, 1024):
        assert bool((got[r : min(r + 1024, m // 8)] == want).all()), f"rows from {8 * r} differ"
    assert torch.equal(got[m // 8], b.view(torch.int16)), "wrote past row m"
    # parts leave the end of the workspace alone, two passes fill it
    assert bool((ws[need - 4096:] == 0x5C).all()), "not two launches of shared rows"
    del x, ws, got
    torch.cuda.empty_cache()


@pytest.mark.parametrize("L", [17, 20])
def test_workspace_alignment_does_not_change_the_result(monkeypatch, L):
    """The two passes with a workspace on a 128-byte line and with one that is 16-byte
    aligned only: same output bits, and nothing written past the workspace."""
    monkeypatch.setenv("HADACORE_VARIANT", "passes")
    import torch
    n = 1 << L
    m = 3
    bits = W.random_rows(m, n, "bf16", seed=L)
    x = to_device(bits, "bf16")
    s = W.default_scale(n)
    need = H.hadamard_transform_workspace_size(m, n)
    outs = []
    for off in (0, 16):
        buf = torch.full((256 + need + 256,), 0x5C, dtype=torch.uint8, device="cuda")
        ws = buf[256 + off: 256 + off + need]
        out = torch.empty_like(x)
        H.hadamard_transform_ws(x.data_ptr(), n, out.data_ptr(), n, m, n, H.BF16, s, ws.data_ptr(),
                                need, torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        host = buf.cpu().numpy()
        assert (host[:256 + off] == 0x5C).all() and (host[256 + off + need:] == 0x5C).all()
        outs.append(to_host(out))
    assert np.array_equal(outs[0], outs[1])
