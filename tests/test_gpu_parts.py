"""n = 2^17 .. 2^19 with several workgroups per row (fwht_parts_kernel): against
the oracle, and bit for bit against the two passes, out of place and in place,
with the in-place wait and without it (every part through the workspace or
copied by the row's last workgroup).

Same criterion as the other sizes (tests/metrics.py): sums in fp32, one rounding.
"""
from __future__ import annotations

import numpy as np
import pytest

from gpu_util import compare_with_oracle, say, to_device, to_host
from paper_2412_08832_amd import hadacore as H
from paper_2412_08832_amd import workloads as W

pytestmark = pytest.mark.gpu

CODE = {"fp16": H.FP16, "bf16": H.BF16}

# (log2 n, rows): one row, groups that are not a multiple of 8, a last turn of
# groups that is not full, and both sides of lines of the dispatch (the others are
# in test_path_by_size)
SHAPES = [(17, 1), (17, 7), (17, 8), (17, 131), (17, 257), (17, 384), (18, 1), (18, 8), (18, 67),
          (18, 193), (19, 7), (19, 8), (19, 32), (19, 33), (19, 40), (19, 96)]


def _call(x, out, m, n, dtype, scale, variant, monkeypatch):
    import torch
    if variant is None:
        monkeypatch.delenv("HADACORE_VARIANT", raising=False)
    else:
        monkeypatch.setenv("HADACORE_VARIANT", variant)
    need = H.hadamard_transform_workspace_size(m, n)
    ws = torch.full((need + 512,), 0x5C, dtype=torch.uint8, device="cuda")
    H.hadamard_transform_ws(x.data_ptr(), x.stride(0), out.data_ptr(), out.stride(0), m, n,
                            CODE[dtype], scale, ws.data_ptr(), need,
                            torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert bool((ws[need:] == 0x5C).all()), "workspace written past its size"


def _bits(t):
    import torch
    return t.view(torch.int16)


@pytest.mark.parametrize("dtype", ["fp16", "bf16"])
@pytest.mark.parametrize("L,m", SHAPES)
def test_parts_match_oracle_and_two_passes(oracle, monkeypatch, L, m, dtype):
    import torch
    n = 1 << L
    scale = 1.1 * W.default_scale(n)   # no power of two at any n
    say(f"parts n=2^{L} m={m} {dtype}")
    rows = np.unique([0, m // 2, m - 1])
    at = torch.from_numpy(rows).cuda()
    bits = W.random_rows(len(rows), n, dtype, seed=L * 1000 + m)
    gen = torch.Generator(device="cuda").manual_seed(m)
    some = to_device(bits, dtype)
    x = torch.randn((m, n + 8), device="cuda", generator=gen).to(some.dtype)
    x[at, :n] = some
    x[0, n // 2] = -0.0
    bits[0, n // 2] = 0x8000
    x[-1, 5::1024] = 2.0 ** -14 / 3    # small beside the rest
    bits[-1] = to_host(x[-1:, :n].contiguous())[0]
    out = torch.empty((m, n + 16), dtype=x.dtype, device="cuda").fill_(7)
    _call(x, out, m, n, dtype, scale, "parts", monkeypatch)
    assert bool((out[:, n:] == 7).all()), "wrote past a row"
    c = compare_with_oracle(oracle, to_host(out[at, :n].contiguous()), bits, dtype, scale, n)
    say(f"  {c}")
    assert c.ok, str(c)
    two = torch.empty_like(out)
    _call(x, two, m, n, dtype, scale, "passes", monkeypatch)
    assert torch.equal(_bits(two)[:, :n], _bits(out)[:, :n]), "the two passes give other bits"
    for variant in (None, "parts", "parts-defer", "passes"):
        y = x.clone()
        _call(y, y, m, n, dtype, scale, variant, monkeypatch)
        assert torch.equal(_bits(y)[:, :n], _bits(out)[:, :n]), f"in place differs ({variant})"
        assert torch.equal(_bits(y)[:, n:], _bits(x)[:, n:]), "in place wrote past a row"


@pytest.mark.parametrize("L,m,inplace,parts", [
    (17, 1, False, True), (18, 7, False, False), (18, 8, False, True), (18, 16, False, True),
    (18, 17, False, True), (18, 192, False, True), (19, 16, False, False), (19, 17, False, False),
    (19, 40, False, False), (19, 47, False, False), (19, 48, False, True), (19, 65, False, True),
    (17, 11, True, False), (17, 12, True, True), (17, 384, True, True), (17, 1023, True, True),
    (17, 1024, True, True), (18, 15, True, False),
    (18, 16, True, True), (18, 192, True, True), (19, 96, True, False)])
def test_path_by_size(monkeypatch, L, m, inplace, parts):
    """Both sides of each line of the dispatch: which way a call takes, seen from the
    workspace (the two passes fill it; the parts leave its end alone), and the bits of
    the other way."""
    import torch
    monkeypatch.delenv("HADACORE_VARIANT", raising=False)
    n = 1 << L
    gen = torch.Generator(device="cuda").manual_seed(m)
    x = torch.randn((m, n), device="cuda", generator=gen).to(torch.bfloat16)
    ws = torch.full((H.hadamard_transform_workspace_size(m, n),), 0x5C, dtype=torch.uint8,
                    device="cuda")
    y = x.clone() if inplace else torch.empty_like(x)
    H.transform(y if inplace else x, out=y, workspace=ws)
    assert bool((ws[-4096:] == 0x5C).all()) == parts
    monkeypatch.setenv("HADACORE_VARIANT", "passes" if parts else "parts")
    assert torch.equal(_bits(y), _bits(H.transform(x)))


@pytest.mark.parametrize("polls", [1, 4, 16])
@pytest.mark.parametrize("L,m", [(17, 1031), (18, 517), (19, 259)])
def test_a_wait_that_ran_out_is_the_last_of_its_workgroup(monkeypatch, L, m, polls):
    """In place with short waits, so that stored and deferred parts mix in one call: the
    bits of the two passes, and a workgroup whose wait ran out waits for no later row.

    The arrive words that the call leaves in the workspace show it: a part's bit is set
    where its workgroup stored it in the workspace.  A workgroup that no longer waits
    stores a part itself only where it is the last of its row to arrive, so of the
    workgroups that ran out on earlier rows at most one a row has no bit.
    """
    import torch
    n, A = 1 << L, 1 << (L - 15)
    gen = torch.Generator(device="cuda").manual_seed(L)
    x = torch.randn((m, n), device="cuda", generator=gen, dtype=torch.bfloat16)
    monkeypatch.setenv("HADACORE_VARIANT", "passes")
    want = H.transform(x)
    monkeypatch.setenv("HADACORE_VARIANT", f"parts-wait-{polls}")
    ws = torch.full((H.hadamard_transform_workspace_size(m, n),), 0x5C, dtype=torch.uint8,
                    device="cuda")
    y = x.clone()
    H.transform(y, out=y, workspace=ws)
    assert torch.equal(_bits(y), _bits(want))
    # deferred parts (2 bytes an element), then a row's arrive word every 256 bytes
    words = ws.view(torch.int32)[m * n // 2:].view(-1, 64)[:m, 0].cpu().numpy()
    assert ((words & 0xFF) == A).all()
    deferred = (words[:, None] >> (8 + np.arange(A))) & 1
    say(f"  n=2^{L} m={m} polls={polls}: {deferred.mean():.3f} of the parts deferred")
    slots = 2 * torch.cuda.get_device_properties(0).multi_processor_count
    groups = slots // A
    assert m > 4 * groups, "several rows a group"
    ran_out = np.zeros((groups, A), bool)
    for r in range(m):
        waits = ran_out[r % groups] & (deferred[r] == 0)
        assert waits.sum() <= 1, f"row {r}: parts {np.flatnonzero(waits)} waited again"
        ran_out[r % groups] |= deferred[r] != 0


def test_parts_special_values(monkeypatch):
    """Infinities, NaN, overflow and an all-zero row: parts and two passes, same bits."""
    import torch
    m, n = 9, 1 << 17
    x = torch.randn((m, n), device="cuda", generator=torch.Generator(device="cuda").manual_seed(1))
    x = x.to(torch.bfloat16)
    x[0, 77] = float("inf")
    x[1, 70000] = float("-inf")
    x[1, 5] = float("inf")
    x[2, 100000] = float("nan")
    x[3] = 0
    x[4] = 3e38
    x[5] = 1e-40
    outs = []
    for variant in ("parts", "passes"):
        o = torch.empty_like(x)
        _call(x, o, m, n, "bf16", W.default_scale(n), variant, monkeypatch)
        outs.append(o)
    assert torch.equal(outs[0].isnan(), outs[1].isnan())
    assert torch.equal(outs[0].nan_to_num(1.0, 2.0, 3.0), outs[1].nan_to_num(1.0, 2.0, 3.0))


@pytest.mark.parametrize("L,m", [(17, 300), (18, 64)])
def test_in_place_calls_on_two_streams(L, m):
    """In-place calls on two streams at once: each gives the bits of the call alone."""
    import torch
    n = 1 << L
    gen = torch.Generator(device="cuda").manual_seed(3)
    xs = [torch.randn((m, n), device="cuda", generator=gen).to(torch.bfloat16) for _ in range(2)]
    refs = [H.transform(x) for x in xs]
    wss = [torch.empty(H.hadamard_transform_workspace_size(m, n), dtype=torch.uint8, device="cuda")
           for _ in xs]
    streams = [torch.cuda.Stream() for _ in xs]
    for _ in range(3):
        ys = [x.clone() for x in xs]
        torch.cuda.synchronize()
        for y, ws, s in zip(ys, wss, streams):
            H.hadamard_transform_ws(y.data_ptr(), n, y.data_ptr(), n, m, n, H.BF16,
                                    W.default_scale(n), ws.data_ptr(), ws.numel(), s.cuda_stream)
        torch.cuda.synchronize()
        for y, r in zip(ys, refs):
            assert torch.equal(y, r)


def test_in_place_call_in_a_graph():
    """The clearing launch and the waits of an in-place call, captured and replayed with
    eager work between the replays: each replay gives the eager call's bits."""
    import torch
    m, n = 40, 1 << 17
    gen = torch.Generator(device="cuda").manual_seed(5)
    x = torch.randn((m, n), device="cuda", generator=gen).to(torch.bfloat16)
    y = x.clone()
    ws = torch.empty(H.hadamard_transform_workspace_size(m, n), dtype=torch.uint8, device="cuda")

    def enqueue(stream):
        H.hadamard_transform_ws(y.data_ptr(), n, y.data_ptr(), n, m, n, H.BF16, W.default_scale(n),
                                ws.data_ptr(), ws.numel(), stream)

    enqueue(torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        with torch.cuda.graph(g, stream=side):
            enqueue(side.cuda_stream)
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    for replay in range(4):
        x.copy_(torch.randn((m, n), device="cuda", generator=gen).to(torch.bfloat16))
        ref = H.transform(x)
        y.copy_(x)
        ws.fill_(0x5C)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, ref), f"replay {replay} differs from eager"
