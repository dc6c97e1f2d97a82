"""Calls whose size picks another cache policy for their loads or stores give
the bits of the same rows in a call of another size, for every n that has several
policies, on both sides of each line of the rules, with aligned rows, rows that
share 128-byte lines and rows further apart, in both dtypes."""
from __future__ import annotations

import pytest

from paper_2412_08832_amd import hadacore as H

pytestmark = pytest.mark.gpu

# (n, total elements): every n that has ordinary loads, at each count of elements where
# some rule (16 bits out of place, quantized, in place with whole lines or rows that
# share lines) changes, one row fewer and one more
SIZES = [(1 << L, total) for L in range(4, 17)
         for total in (1 << 23, 1 << 24, 7 << 22, 1 << 25)] + [(65536, 1 << 22)]


@pytest.mark.parametrize("dtype", ["fp16", "bf16"])
@pytest.mark.parametrize("pad", [0, 8, 72])
@pytest.mark.parametrize("more", [-1, 0, 1])
@pytest.mark.parametrize("n,total", SIZES)
def test_rows_do_not_depend_on_the_size_of_the_call(n, total, more, pad, dtype):
    import torch
    m = total // n + more
    gen = torch.Generator(device="cuda").manual_seed(n)
    buf = torch.randn((m, n + pad), device="cuda", generator=gen)
    buf = buf.to({"fp16": torch.float16, "bf16": torch.bfloat16}[dtype])
    x = buf[:, :n]
    rows = [0, m // 2, m - 1]
    small = buf[rows][:, :n]           # three rows: the smallest calls' policy
    y, ref = H.transform(x), H.transform(small)
    assert torch.equal(y[rows], ref)
    for f in (H.transform_fp8, H.transform_int8):
        (c, s), (rc, rs) = f(x), f(small)
        assert torch.equal(c[rows], rc) and torch.equal(s[rows], rs)
    z = buf.clone()
    H.transform(z[:, :n], out=z[:, :n])
    assert torch.equal(z[:, :n], y) and torch.equal(z[:, n:], buf[:, n:])


@pytest.mark.parametrize("dtype", ["fp16", "bf16"])
@pytest.mark.parametrize("L,m", [(18, 9), (19, 4), (19, 5), (19, 8), (19, 9), (19, 16), (19, 17),
                                 (20, 2), (20, 3), (20, 5), (20, 8), (20, 9)])
def test_two_pass_rows_do_not_depend_on_the_size_of_the_call(monkeypatch, L, m, dtype):
    """The column pass streams for calls of 2^21 to 2^23 elements (2^22 in place): the
    bits of the same rows one at a time, below that range."""
    import torch
    monkeypatch.setenv("HADACORE_VARIANT", "passes")
    n = 1 << L
    gen = torch.Generator(device="cuda").manual_seed(L * 100 + m)
    x = torch.randn((m, n + 8), device="cuda", generator=gen)
    x = x.to({"fp16": torch.float16, "bf16": torch.bfloat16}[dtype])
    ref = torch.cat([H.transform(x[r : r + 1, :n]) for r in range(m)])
    assert torch.equal(H.transform(x[:, :n]), ref)
    z = x.clone()
    H.transform(z[:, :n], out=z[:, :n])
    assert torch.equal(z[:, :n], ref) and torch.equal(z[:, n:], x[:, n:])
