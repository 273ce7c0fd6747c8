"""GPU tests of the frozen input gradient's split reduction: fp32 planes over
ranges of k, summed in ascending order.  Against fp64: a result may be off by
its rounding to bf16 (2^-8 of it) and by the fp32 sums (1e-5 of the largest)."""
import sys

import pytest
import torch

import paper_2606_19528_amd as lm
from workloads import quant_weight

pytestmark = pytest.mark.gpu


def _announce(msg):
    print(f"[case] {msg}", file=sys.stderr, flush=True)


def _split_bytes(T, d_in, d_out):
    return lm.lib().frozen_linear_split_bytes(T, d_in, d_out, lm.LORA_BF16)


def _check(dx, dy, W):
    ref = dy.double() @ W.double()
    bound = 2.0 ** -8 * ref.abs() + 1e-5 * ref.abs().max()
    assert bool(((dx.double() - ref).abs() <= bound).all()), float(((dx.double() - ref).abs() - bound).max())


# One token and one column block, ragged tiles, 128- and 256-row tiles at
# their edge, a last range shorter than the others, few ranges and many.
SHAPES = [(1, 8, 4096), (64, 264, 5000), (128, 256, 8200), (129, 520, 9000), (257, 1032, 20008), (1024, 3072, 20008)]


@pytest.mark.parametrize("T,d_in,d_out", SHAPES)
def test_frozen_dx_split(T, d_in, d_out):
    _announce(f"frozen split T={T} {d_out}->{d_in}")
    g = torch.Generator().manual_seed(T + d_out)
    dy = torch.randn(T, d_out, generator=g).bfloat16().cuda()
    W = (torch.randn(d_out, d_in, generator=g) * 0.02).bfloat16().cuda()
    n = _split_bytes(T, d_in, d_out)
    assert n >= 2 * T * d_in * 4
    ws = torch.full((n + 256,), 0xFF, dtype=torch.uint8, device="cuda")  # NaN planes unless written
    dx = lm.frozen_linear_bwd_dx(dy, W, torch.empty(T, d_in, dtype=torch.bfloat16, device="cuda"), ws=ws[:n])
    assert not bool((ws[: T * d_in * 4] == 0xFF).all())  # (the first plane is written: it split)
    again = lm.frozen_linear_bwd_dx(dy, W, torch.empty_like(dx))
    small = lm.frozen_linear_bwd_dx(dy, W, torch.empty_like(dx), ws=ws[: n - 16])  # no room: unsplit
    torch.cuda.synchronize()
    assert torch.equal(dx, again)
    assert bool((ws[n:] == 0xFF).all())
    _check(dx, dy, W)
    _check(small, dy, W)


@pytest.mark.parametrize("bits,group", [(8, 128), (4, 64), (8, 32)])
@pytest.mark.parametrize("T,d_in,d_out", [(40, 256, 5000), (200, 768, 9000)])
def test_frozen_dx_split_quantized(T, d_in, d_out, bits, group):
    """(Groups of 32 keep the unsplit tiles.)"""
    _announce(f"frozen split T={T} {d_out}->{d_in} int{bits} group {group}")
    g = torch.Generator().manual_seed(T + d_out)
    dy = torch.randn(T, d_out, generator=g).bfloat16().cuda()
    q = quant_weight(d_out, d_in, bits, group, seed=3)
    qd = {k: (v.cuda() if hasattr(v, "cuda") else v) for k, v in q.items()}
    c = qd["codes"]
    if bits == 4:
        c = torch.stack([c & 15, c >> 4], dim=-1).reshape(d_out, d_in)
    s = qd["scale"].t().repeat_interleave(group, dim=1)
    o = qd["offset"].t().repeat_interleave(group, dim=1)
    W = torch.addcmul(o.double(), c.double(), s.double()).float().bfloat16()  # one rounding to fp32, one to bf16
    dx = lm.frozen_linear_bwd_dx_q(dy, qd, torch.empty(T, d_in, dtype=torch.bfloat16, device="cuda"))
    torch.cuda.synchronize()
    _check(dx, dy, W)


def test_frozen_split_sizes():
    assert _split_bytes(4096, 3072, 128256) == 0      # the tiles fill the chip
    assert _split_bytes(64, 256, 1024) == 0           # too short a reduction
    assert _split_bytes(1500, 2048, 2056) == 0        # the planes would cost more than the split gains
    assert lm.lib().frozen_linear_split_bytes(64, 256, 8192, lm.LORA_F32) == 0
    assert lm.lib().frozen_linear_split_bytes(64, 100, 8192, lm.LORA_BF16) == 2 ** 64 - 1


def test_no_room_for_the_optional_workspaces():
    """Where the allocator has no room, the split dx runs unsplit and the similarity
    table over row batches; a caller's workspace fixes the choice."""
    _announce("no room for the optional workspaces")
    T, d_in, d_out = 1024, 3072, 20008
    g = torch.Generator().manual_seed(5)
    dy = torch.randn(T, d_out, generator=g).bfloat16().cuda()
    W = (torch.randn(d_out, d_in, generator=g) * 0.02).bfloat16().cuda()
    E = torch.randn(16400, 64, generator=g).bfloat16().cuda()
    n = _split_bytes(T, d_in, d_out)
    split, unsplit, full = (torch.empty(T, d_in, dtype=torch.bfloat16, device="cuda") for _ in range(3))
    tables = [torch.empty(16400, 100, dtype=torch.int32, device="cuda") for _ in range(2)]
    batched = lm.lib().topk_table_workspace_bytes(16400, 64, 100)
    small = torch.empty(batched, dtype=torch.uint8, device="cuda")
    lm.frozen_linear_bwd_dx(dy, W, split, ws=torch.empty(n, dtype=torch.uint8, device="cuda"))
    lm.frozen_linear_bwd_dx(dy, W, unsplit, ws=dy.new_empty(0))
    lm.topk_table_build(E, 100, tables[0])
    torch.cuda.synchronize()
    del small
    torch.cuda.empty_cache()
    free = torch.empty(batched, dtype=torch.uint8, device="cuda")  # (room for the smaller one, given back below)
    total = torch.cuda.get_device_properties(0).total_memory
    torch.cuda.set_per_process_memory_fraction(torch.cuda.memory_reserved() / total)
    try:
        held = []  # what the allocator still has of its own
        for size in (1 << 28, 1 << 26, 1 << 24, 1 << 22, 1 << 20):
            while True:
                try:
                    held.append(torch.empty(size, dtype=torch.uint8, device="cuda"))
                except torch.cuda.OutOfMemoryError:
                    break
        lm.frozen_linear_bwd_dx(dy, W, full)
        del free
        lm.topk_table_build(E, 100, tables[1])
        torch.cuda.synchronize()
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)
    assert torch.equal(full, unsplit)
    _check(split, dy, W)
    _check(unsplit, dy, W)
    assert torch.equal(tables[0], tables[1])


@pytest.mark.parametrize("T,d_in,d_out", [(130, 1024, 4096), (218, 256, 4096), (2683, 1024, 8576)])
def test_short_reductions_stay_whole(T, d_in, d_out):
    """Where the second launch costs more than the split gains, a bf16 product leaves
    the workspace alone."""
    _announce(f"frozen whole T={T} {d_out}->{d_in}")
    g = torch.Generator().manual_seed(T)
    dy = torch.randn(T, d_out, generator=g).bfloat16().cuda()
    W = (torch.randn(d_out, d_in, generator=g) * 0.02).bfloat16().cuda()
    ws = torch.full((max(_split_bytes(T, d_in, d_out), 1 << 20),), 0xFF, dtype=torch.uint8, device="cuda")
    dx = lm.frozen_linear_bwd_dx(dy, W, torch.empty(T, d_in, dtype=torch.bfloat16, device="cuda"), ws=ws)
    torch.cuda.synchronize()
    assert bool((ws == 0xFF).all())
    _check(dx, dy, W)
