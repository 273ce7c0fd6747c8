"""GPU parity of the top-k cosine-similarity table against the fp64 oracle.

The similarities are fp32 sums of bf16 products, so tokens whose exact
similarities lie within EPS of each other may come out in either order.  Per
checked row the test requires: k distinct indices, the token itself first,
the exact similarity of the c-th entry within EPS of the oracle's c-th
similarity (so the ranking agrees up to near-ties), the reported values
within EPS of the exact ones, and every token whose similarity clears the
oracle's k-th by more than EPS present (what is unique must match)."""
import sys

import numpy as np
import pytest
import torch

import paper_2606_19528_amd as lm  # noqa: E402

pytestmark = pytest.mark.gpu
EPS = 2e-5


def _announce(msg):
    print(f"[case] {msg}", file=sys.stderr, flush=True)


def _embeddings(V, D, seed):
    g = torch.Generator().manual_seed(seed)
    return (torch.randn(V, D, generator=g) * 0.02).to(torch.bfloat16)


def _check_rows(orc, W, table, values, k, rows):
    Wd = W.double().numpy()
    Ao, Co = orc.topk_table(W, k, rows=rows)
    nrm = np.linalg.norm(Wd, axis=1)
    for r, i in enumerate(rows):
        a = table[i].numpy().astype(np.int64)
        assert len(set(a.tolist())) == k and a.min() >= 0 and a.max() < W.shape[0], i
        assert a[0] == i, (i, a[:4])
        exact = (Wd[a] @ Wd[i]) / (nrm[a] * nrm[i])
        assert np.max(np.abs(exact - Co[r])) <= EPS, (i, np.max(np.abs(exact - Co[r])))
        assert np.max(np.abs(values[i].double().numpy() - exact)) <= EPS, i
        clear = Ao[r][Co[r] > Co[r][-1] + EPS]
        assert set(clear.tolist()) <= set(a.tolist()), i


@pytest.mark.parametrize("shape", [(700, 64, 16), (3000, 128, 50), (9000, 64, 200), (257, 24, 257),
                                   (2600, 32, 2048)])
def test_topk_table_full(orc, shape):
    V, D, k = shape
    _announce(f"topk V={V} D={D} k={k}")
    W = _embeddings(V, D, seed=V + D)
    table = torch.empty(V, k, dtype=torch.int32, device="cuda")
    values = torch.empty(V, k, dtype=torch.float32, device="cuda")
    lm.topk_table_build(W.cuda(), k, table, values)
    torch.cuda.synchronize()
    _check_rows(orc, W, table.cpu(), values.cpu(), k, list(range(V)))


def test_topk_table_several_row_batches(orc):
    # more rows than one batch (16384) and several column chunks; sampled rows
    V, D, k = 20000, 64, 64
    _announce(f"topk V={V} D={D} k={k} (sampled rows)")
    W = _embeddings(V, D, seed=3)
    table = torch.empty(V, k, dtype=torch.int32, device="cuda")
    values = torch.empty(V, k, dtype=torch.float32, device="cuda")
    lm.topk_table_build(W.cuda(), k, table, values)
    torch.cuda.synchronize()
    rows = sorted({0, 4095, 4096, 16383, 16384, V - 1, *range(7, V, 997)})
    _check_rows(orc, W, table.cpu(), values.cpu(), k, rows)


def test_topk_table_3b_vocabulary(orc):
    # the 3B model's output embedding shape, k = 1000; sampled rows
    V, D, k = 128256, 3072, 1000
    _announce(f"topk V={V} D={D} k={k} (sampled rows)")
    W = _embeddings(V, D, seed=5)
    table = torch.empty(V, k, dtype=torch.int32, device="cuda")
    values = torch.empty(V, k, dtype=torch.float32, device="cuda")
    lm.topk_table_build(W.cuda(), k, table, values)
    torch.cuda.synchronize()
    _check_rows(orc, W, table.cpu(), values.cpu(), k, [0, 1, 16384, 65537, V - 1])


def test_topk_table_deterministic():
    W = _embeddings(5000, 64, seed=11).cuda()
    a = lm.topk_table_build(W, 100)
    b = lm.topk_table_build(W, 100)
    torch.cuda.synchronize()
    assert torch.equal(a, b)


@pytest.mark.parametrize("V,D,k", [(4095, 64, 40), (4096, 64, 2048), (4097, 72, 40), (8500, 64, 100),
                                   (12300, 64, 64), (16400, 32, 1000)])
def test_topk_table_paired_equals_batched(orc, V, D, k):
    """From one block of 4096 rows the build runs rounds of block pairs, each
    similarity serving both rows (one whole block, a ragged second block, an
    odd number of blocks with a bye); given only the smaller workspace it runs
    row batches.  Both agree with the oracle and bitwise with each other; rows
    repeated far apart tie exactly, the smaller index first."""
    _announce(f"topk paired V={V} D={D} k={k}")
    W = _embeddings(V, D, seed=V)
    W[V - 1] = W[3]
    W[V // 2] = W[3]
    Wd = W.cuda()
    out = {}
    for name, n in (("paired", lm.lib().topk_table_workspace_bytes_paired(V, D, k)),
                    ("batched", lm.lib().topk_table_workspace_bytes(V, D, k))):
        ws = torch.empty(n, dtype=torch.uint8, device="cuda")
        table = torch.empty(V, k, dtype=torch.int32, device="cuda")
        values = torch.empty(V, k, dtype=torch.float32, device="cuda")
        lm.topk_table_build(Wd, k, table, values, ws=ws)
        torch.cuda.synchronize()
        out[name] = (table.cpu(), values.cpu())
    assert torch.equal(out["paired"][0], out["batched"][0]) and torch.equal(out["paired"][1], out["batched"][1])
    for table, values in out.values():
        for i in (3, V // 2, V - 1):
            assert table[i, :3].tolist() == [3, V // 2, V - 1]
        rows = [i for i in sorted({0, 1, 255, 256, 2047, 4094, *range(5, V, 613), V - 2}) if i not in (3, V // 2, V - 1)]
        _check_rows(orc, W, table, values, k, rows)


def test_topk_table_paired_all_equal():
    """Every similarity ties: each list overflows its threshold in every round,
    and the k smallest indices must come out."""
    V, D, k = 8300, 64, 20
    _announce("topk all rows equal")
    W = _embeddings(1, D, seed=1).repeat(V, 1).cuda()
    table = lm.topk_table_build(W, k)
    torch.cuda.synchronize()
    assert torch.equal(table.cpu(), torch.arange(k, dtype=torch.int32).repeat(V, 1))


@pytest.mark.parametrize("k", [6, 7, 64])
def test_topk_table_equal_rows_tie_for_every_query(k):
    """Equal rows in different blocks have bitwise equal similarities to every
    other token, whose norms vary over four decades, and stand in ascending order
    of their index, also where k cuts between them."""
    V, D = 12300, 64
    _announce(f"topk equal rows k={k}")
    W = _embeddings(V, D, seed=11).float()
    W *= 10.0 ** (4.0 * torch.rand(V, 1, generator=torch.Generator().manual_seed(12)) - 2.0)
    same = [7, 4099, 5000, 8191, 8193, 12299]
    centre = W[7].clone()
    near = list(range(100, 12000, 37))  # queries around the repeated row
    W[near] = centre * (0.5 + torch.rand(len(near), 1, generator=torch.Generator().manual_seed(13))) + 0.4 * W[near] / W[
        near].norm(dim=1, keepdim=True) * centre.norm()
    W[same] = centre
    W = W.to(torch.bfloat16)
    out = []
    for n in (lm.lib().topk_table_workspace_bytes_paired(V, D, k), lm.lib().topk_table_workspace_bytes(V, D, k)):
        table = torch.empty(V, k, dtype=torch.int32, device="cuda")
        values = torch.empty(V, k, dtype=torch.float32, device="cuda")
        lm.topk_table_build(W.cuda(), k, table, values, ws=torch.empty(n, dtype=torch.uint8, device="cuda"))
        torch.cuda.synchronize()
        out.append((table.cpu(), values.cpu()))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
    table, values = out[0]
    seen = 0
    for i in range(V):
        at = [(int(t), c) for c, t in enumerate(table[i].tolist()) if t in same]
        if not at:
            continue
        seen += 1
        assert [t for t, _ in at] == same[: len(at)], (i, at)
        assert len({float(values[i, c]) for _, c in at}) == 1, i
        assert len(at) == len(same) or at[-1][1] == k - 1, i  # none left out ahead of another token
    assert seen > 200  # queries that the repeated rows reach
