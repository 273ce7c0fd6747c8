"""GPU parity of the quantized frozen base (codes + per-group scale and offset,
dequantized inside the GEMMs) against the fp64 oracle, which dequantizes the
same codes exactly (W = s * W_q + b per group) and then runs the LoRA
definitions.  bf16 tolerance 2e-2 per output tensor."""
import sys

import numpy as np
import pytest
import torch

from gpu_helpers import TOL, compare, gpu_lora_q, oracle_lora, relerr
from workloads import lora_inputs, quant_weight, sample_rows

pytestmark = pytest.mark.gpu

import paper_2606_19528_amd as lm  # noqa: E402


def _announce(msg):
    print(f"[case] {msg}", file=sys.stderr, flush=True)


def _dequant(orc, Wq, group):
    # the library takes scales and offsets group-major, the oracle per row
    return torch.from_numpy(orc.dequant(Wq["codes"], Wq["scale"].t(), Wq["offset"].t(), Wq["bits"], group))


def _qcase(orc, T, K, N, r, bits, group, seed, recompute=False, rows=None, s=2.0):
    _announce(f"quant T={T} K={K} N={N} r={r} bits={bits} group={group} recompute={recompute}")
    inp = lora_inputs(T, K, N, r, seed=seed)
    Wq = quant_weight(N, K, bits, group, seed=seed + 1)
    gpu = gpu_lora_q(inp, Wq, s, recompute_u=recompute)
    ref = oracle_lora(orc, dict(inp, W=_dequant(orc, Wq, group)), s, rows=rows)
    return compare(gpu, ref, torch.bfloat16, rows=rows, label=f"q{bits} T={T} K={K} N={N} r={r}")


@pytest.mark.parametrize("shape", [
    (128, 256, 256, 8, 4, 128), (129, 384, 136, 16, 4, 32), (300, 1024, 520, 5, 4, 64),
    (1, 128, 8, 1, 8, 128), (257, 512, 392, 64, 8, 16), (64, 256, 128, 0, 4, 128),
    (17, 2048, 264, 32, 4, 256), (200, 640, 1032, 16, 8, 128),
])
def test_quant_small(orc, shape):
    T, K, N, r, bits, group = shape
    _qcase(orc, T, K, N, r, bits, group, seed=T + K + N + r + bits)


@pytest.mark.parametrize("bits", [4, 8])
def test_quant_recompute_u(orc, bits):
    _qcase(orc, 256, 1536, 520, 16, bits, 128, seed=61, recompute=True)


def test_quant_full_llama_q_proj(orc):
    # the headline shape: T=1024, 3072 -> 3072, r=16, INT4 groups of 128
    _qcase(orc, 1024, 3072, 3072, 16, 4, 128, seed=71, rows=sample_rows(1024), s=32.0 / 16)


def test_quant_zero_weight_isolates_lora(orc):
    # codes, scales and offsets all zero: W = 0, so y = s u B^T and dx = du A exactly
    T, K, N, r = 96, 512, 264, 16
    _announce(f"quant zero W T={T} K={K} N={N} r={r}")
    inp = lora_inputs(T, K, N, r, seed=81)
    Wq = quant_weight(N, K, 4, 128, seed=82)
    Wq = {k: (torch.zeros_like(v) if hasattr(v, "dtype") else v) for k, v in Wq.items()}
    gpu = gpu_lora_q(inp, Wq, 2.0)
    ref = oracle_lora(orc, dict(inp, W=torch.zeros(N, K, dtype=torch.float64)), 2.0)
    compare(gpu, ref, torch.bfloat16, label="quant W=0")


# Groups of 64 weights or more run the dequantizing direct-to-LDS tiles (codes,
# scales and offsets loaded into LDS, dequantized there); the tile shape is the
# bf16 path's choice for the same product.  Cases: the 256 x 192 forward with
# ragged rows and columns and the 256 x 256 dx (side items, a reduction tail);
# the 256 x 256 forward and 128 x 128 dx in INT8 with groups of 64; 128 x 128
# both ways with groups of 256; the 28-layer stack's gate shape in INT4.
@pytest.mark.parametrize("shape", [
    (4000, 3072, 3000, 16, 4, 128), (2304, 2048, 6144, 16, 8, 64), (1000, 1536, 1032, 8, 4, 256),
    (4096, 3072, 8192, 32, 4, 128),
])
def test_quant_direct_tiles(orc, shape):
    T, K, N, r, bits, group = shape
    rows = list(range(0, T, 97)) + [T - 1]
    _qcase(orc, T, K, N, r, bits, group, seed=T + N + bits, rows=rows)


# Seeded random shapes: INT4 and INT8, groups of 16 to 256 (register-staged
# below 64, direct-to-LDS from 64), ranks 0 to 64, 1 to 4300 tokens.  dA and
# dB in full, 64 sampled rows of y and dx.
def _random_qshapes(n, seed):
    g = np.random.default_rng(seed)
    out = []
    while len(out) < n:
        T = int(g.integers(1, 4300))
        group = int(g.choice([16, 32, 64, 128, 256]))
        K = group * int(g.integers(1, max(2, 6144 // group)))
        N = 8 * int(g.integers(1, 800))
        r = int(g.choice([0, 1, 3, 8, 16, 32, 64]))
        bits = int(g.choice([4, 8]))
        if T * K * N <= 3e10:
            out.append((T, K, N, r, bits, group))
    return out


# The dx launch's dA / dB items as token parts (the plan's bwd_side_parts)
# beside the dequantizing tiles: two parts of 512 + 488 tokens with
# register-staged INT8 groups of 32, and the Llama k / v shape in INT4 with
# direct-to-LDS groups of 128 (sampled rows).
@pytest.mark.parametrize("shape", [(1000, 1536, 1032, 12, 8, 32), (4096, 3072, 1024, 32, 4, 128)])
def test_quant_side_items_in_token_parts(orc, shape):
    T, K, N, r, bits, group = shape
    assert lm.lora_linear_plan(T, K, N, r)["bwd_side_parts"] == 2
    _qcase(orc, T, K, N, r, bits, group, seed=T + K, rows=sample_rows(T, 64))


@pytest.mark.parametrize("shape", _random_qshapes(12, 404))
def test_quant_random_shapes(orc, shape):
    T, K, N, r, bits, group = shape
    _qcase(orc, T, K, N, r, bits, group, seed=sum(shape), rows=sample_rows(T, 64))


@pytest.mark.parametrize("shape", [(129, 256, 392, 8, 128), (64, 3072, 1000, 8, 128),
                                   (33, 1024, 136, 4, 16), (4000, 3072, 3000, 8, 128),
                                   (2048, 8192, 3000, 8, 64), (1024, 3072, 8192, 4, 128)])
def test_quant_frozen_dx(orc, shape):
    T, K, N, bits, group = shape
    _announce(f"quant frozen dx T={T} K={K} N={N} bits={bits} group={group}")
    g = torch.Generator().manual_seed(T + N)
    dy = torch.randn(T, N, generator=g).to(torch.bfloat16)
    Wq = quant_weight(N, K, bits, group, seed=N)
    dx = torch.empty(T, K, dtype=torch.bfloat16, device="cuda")
    lm.frozen_linear_bwd_dx_q(dy.cuda(), {k: (v.cuda() if hasattr(v, "cuda") else v)
                                          for k, v in Wq.items()}, dx)
    torch.cuda.synchronize()
    rows = list(range(0, T, 61)) + [T - 1] if T > 256 else list(range(T))
    ref = orc.frozen_dx(dy[rows], _dequant(orc, Wq, group))
    assert relerr(dx.cpu()[rows].double().numpy(), ref) <= TOL[torch.bfloat16]


def test_quant_deterministic(orc):
    T, K, N, r = 200, 1024, 392, 16
    inp = lora_inputs(T, K, N, r, seed=91)
    Wq = quant_weight(N, K, 4, 128, seed=92)
    a = gpu_lora_q(inp, Wq, 2.0)
    b = gpu_lora_q(inp, Wq, 2.0)
    for k in a:
        assert torch.equal(a[k], b[k]), k


# Sizes whose dx runs 256 x 128 dequantizing tiles (ragged rows and columns, a
# reduction that ends inside a stage, ranks in one and two LoRA stages), checked
# on sampled rows of y and dx, dA and dB in full.
@pytest.mark.parametrize("shape", [(1990, 3008, 264, 16, 4, 64), (2048, 3072, 520, 64, 8, 128)])
def test_quant_dx_256x128_tiles(orc, shape):
    T, K, N, r, bits, group = shape
    p = lm.lora_linear_plan(T, K, N, r)
    assert (p["bwd_tile_m"], p["bwd_tile_n"]) == (256, 128)
    _qcase(orc, T, K, N, r, bits, group, seed=T + K, rows=sample_rows(T, 64))
