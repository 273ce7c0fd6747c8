"""GPU tests of the few-token kernel (up to 128 tokens, bf16): tiles of 32 rows by
64 columns, the reduction in one part or several that meet in the workspace, one
or two blocks of 32 rank columns, one to four row tiles.  Each test asserts through
lora_few_token_plan that its calls run that kernel (or, in one direction, at the
rule's edges and with the smaller workspace, the tiled ones).  Every result against the fp64 oracle
(max relative error <= 2e-2 per tensor, the bf16 bound of the other parity tests)."""
import sys

import pytest
import torch

import paper_2606_19528_amd as lm
from gpu_helpers import compare, gpu_lora, oracle_lora
from workloads import lora_inputs

pytestmark = pytest.mark.gpu
BF16 = torch.bfloat16
FLAG_WORDS = 2  # 32-bit words of a meeting's flag, the workspace's first contents


def _announce(msg):
    print(f"[case] {msg}", file=sys.stderr, flush=True)


# (T, d_in, d_out, r): tile edges in T; reductions of less than a stage, a
# ragged last stage, one part and many; ragged column tiles; ranks whose rows
# are not whole 16-byte vectors, one and two rank blocks, none; parts and row
# tiles together in either direction, one to four row tiles.
SHAPES = [(1, 8, 8, 4), (1, 3072, 3072, 16), (16, 264, 72, 8), (24, 3072, 1032, 16), (31, 72, 520, 12),
          (32, 1024, 64, 32), (63, 4096, 256, 4), (40, 2056, 3080, 0), (64, 256, 4104, 16),
          (32, 2056, 1032, 36), (20, 520, 2056, 40), (32, 1032, 264, 64), (17, 4104, 72, 64),
          (33, 776, 2056, 32), (64, 2048, 2048, 16), (50, 4104, 520, 24), (48, 520, 4104, 28),
          (65, 8200, 520, 24), (80, 1032, 4096, 12), (96, 4104, 1032, 16), (95, 520, 8200, 4),
          (100, 4104, 1024, 32), (103, 1024, 4096, 16), (120, 2056, 2056, 0), (127, 2048, 2056, 16),
          (128, 1040, 4096, 32), (128, 8200, 520, 8), (48, 264, 8200, 8)]
# More tiles than CUs: one direction runs the few-token kernel, the other the tiled
# ones (u in one sum or in partial sums of theirs; or u by the few-token kernel,
# its reduction whole or in parts, ahead of a tiled backward); neither does.
FWD_ONLY = [(100, 8200, 520, 4), (80, 8200, 1032, 12), (65, 8200, 2056, 4), (128, 8200, 520, 0)]
BWD_ONLY = [(103, 1024, 4104, 16), (128, 520, 8200, 32), (48, 1032, 8200, 8), (100, 1032, 16384, 16), (100, 520, 8200, 0)]
# The rule's edges: one token, one rank index or one weight row too many.
BEYOND = [(129, 3072, 2056, 24), (65, 3080, 136, 8), (128, 64, 64, 8), (128, 2048, 2040, 16), (33, 776, 2056, 36),
          (64, 256, 4104, 64), (100, 520, 3072, 40), (128, 2048, 3072, 64), (24, 1024, 520, 68), (24, 1024, 520, 6),
          (65, 8200, 8200, 0)]


def _taken(*shape):
    p = lm.lora_few_token_plan(*shape)
    return bool(p["fwd_taken"]), bool(p["bwd_taken"])


def test_narrow_shapes_cover_the_plans():
    for shapes, want in ((SHAPES, (True, True)), (FWD_ONLY, (True, False)), (BWD_ONLY, (False, True)),
                         (BEYOND, (False, False))):
        assert all(_taken(*s) == want for s in shapes), want
    plans = [lm.lora_few_token_plan(*s) | {"r": s[3]} for s in SHAPES]
    for d in ("fwd", "bwd"):
        parts, tiles_m = d + "_parts", d + "_tiles_m"
        for tiles in (1, 2, 3, 4):  # (row tiles) with the reduction whole and split
            assert {p[parts] > 1 for p in plans if p[tiles_m] == tiles and p["r"]} == {False, True}, (d, tiles)
        assert any(p[parts] > 1 and p["r"] > 32 for p in plans) and any(p[parts] == 1 and p["r"] > 32 for p in plans)
    assert {lm.lora_few_token_plan(*s)["fwd_parts"] > 1 for s in FWD_ONLY} == {False, True}
    parts = {lm.lora_linear_plan(*s)["fwd_u_parts"] > 1 for s in BWD_ONLY if s[3]}
    assert parts == {False, True}


ALL = SHAPES + FWD_ONLY + BWD_ONLY + BEYOND


@pytest.mark.parametrize("shape", ALL, ids=["x".join(map(str, s)) for s in ALL])
def test_narrow_parity(orc, shape):
    T, K, N, r = shape
    _announce(f"narrow T={T} K={K} N={N} r={r}")
    inp = lora_inputs(T, K, N, r, seed=sum(shape))
    s = 2.0
    got = gpu_lora(inp, s)
    if r:
        ref = oracle_lora(orc, inp, s)
        again = gpu_lora(inp, s, recompute_u=True)
        none = gpu_lora(inp, s, want_dx=False)
        for k in ("y", "dx", "u", "dA", "dB"):  # a recomputed u is bitwise the saved one
            assert torch.equal(got[k], again[k]), k
        assert torch.equal(got["dA"], none["dA"]) and torch.equal(got["dB"], none["dB"])
    else:
        x, W, dy = (inp[k].double() for k in ("x", "W", "dy"))
        ref = {"y": (x @ W.t()).numpy(), "dx": (dy @ W).numpy()}
    compare(got, ref, BF16, label=f"narrow {shape}")


@pytest.mark.parametrize("T,ranks", [(20, (4, 32, 36, 64)), (60, (4, 32)), (110, (4, 32))])
def test_narrow_zero_B_is_rank_0(T, ranks):
    """With B = 0 the output is the rank-0 forward's bitwise, at every rank."""
    K, N = 2056, 2056
    _announce(f"narrow B=0 T={T}")
    for r in ranks:
        assert _taken(T, K, N, r)[0] and _taken(T, K, N, 0)[0]
        inp = lora_inputs(T, K, N, r, seed=T)
        inp["B"].zero_()
        d = {k: v.cuda() for k, v in inp.items()}
        y, y0 = (torch.empty(T, N, dtype=BF16, device="cuda") for _ in range(2))
        lm.lora_linear_fwd(d["x"], d["W"], d["A"], d["B"], y, None, 2.0)
        lm.lora_linear_fwd(d["x"], d["W"], None, None, y0)
        torch.cuda.synchronize()
        assert torch.equal(y, y0), r


@pytest.mark.parametrize("fill", [0x00, 0xFF, "random"])
def test_narrow_workspace_contents_and_reuse(orc, fill):
    """The meetings' words start as whatever the workspace holds; one workspace
    serves calls of other sizes in between, and less of it the tiled kernels."""
    s = 2.0
    n = max(lm.lora_linear_workspace_bytes(op, T, K, N, r, lm.LORA_BF16)
            for T, K, N, r in ((24, 3072, 3072, 16), (120, 2048, 2056, 8)) for op in (lm.LORA_OP_FWD, lm.LORA_OP_BWD))
    ws = torch.empty(n, dtype=torch.uint8, device="cuda")
    if fill == "random":
        ws.copy_(torch.randint(0, 256, ws.shape, dtype=torch.uint8, device="cuda"))
    else:
        ws.fill_(fill)
    for it, (T, K, N, r) in enumerate([(24, 3072, 3072, 16), (120, 2048, 2056, 8), (24, 3072, 3072, 16)]):
        _announce(f"narrow workspace fill={fill} T={T}")
        assert _taken(T, K, N, r) == (True, True)
        inp = lora_inputs(T, K, N, r, seed=50 + it)
        d = {k: v.cuda() for k, v in inp.items()}
        o = {"y": torch.empty(T, N, dtype=BF16, device="cuda"), "u": torch.empty(T, r, device="cuda"),
             "dx": torch.empty(T, K, dtype=BF16, device="cuda"), "dA": torch.empty(r, K, device="cuda"),
             "dB": torch.empty(N, r, device="cuda")}
        lm.lora_linear_fwd(d["x"], d["W"], d["A"], d["B"], o["y"], o["u"], s, ws=ws)
        lm.lora_linear_bwd(d["x"], d["W"], d["A"], d["B"], o["u"], d["dy"], o["dx"], o["dA"], o["dB"], s, ws=ws)
        torch.cuda.synchronize()
        compare({k: v.cpu() for k, v in o.items()}, oracle_lora(orc, inp, s), BF16, label=f"fill={fill} it={it}")


@pytest.mark.parametrize("shape", [(24, 3072, 3072, 16), (48, 2056, 1032, 8), (63, 4096, 256, 4), (20, 2056, 520, 64),
                                   (96, 4104, 1032, 16)], ids=lambda s: "x".join(map(str, s)))
def test_tiled_kernels_at_few_tokens(orc, shape):
    """A workspace of the tiled kernels' size still serves a call, through them."""
    T, K, N, r = shape
    s = 2.0
    p = lm.lora_few_token_plan(T, K, N, r)
    assert p["fwd_tiled_bytes"] < p["fwd_bytes"] and p["bwd_tiled_bytes"] < p["bwd_bytes"]
    _announce(f"tiled kernels T={T} K={K} N={N} r={r}")
    inp = lora_inputs(T, K, N, r, seed=5)
    d = {k: v.cuda() for k, v in inp.items()}
    ref = oracle_lora(orc, inp, s)
    ws = torch.zeros(max(p["fwd_bytes"], p["bwd_bytes"]), dtype=torch.uint8, device="cuda")
    for saved in (True, False):
        o = {"y": torch.empty(T, N, dtype=BF16, device="cuda"), "u": torch.empty(T, r, device="cuda"),
             "dx": torch.empty(T, K, dtype=BF16, device="cuda"), "dA": torch.empty(r, K, device="cuda"),
             "dB": torch.empty(N, r, device="cuda")}
        lm.lora_linear_fwd(d["x"], d["W"], d["A"], d["B"], o["y"], o["u"], s, ws=ws[: p["fwd_tiled_bytes"]])
        lm.lora_linear_bwd(d["x"], d["W"], d["A"], d["B"], o["u"] if saved else None, d["dy"], o["dx"], o["dA"], o["dB"],
                           s, ws=ws[: p["bwd_tiled_bytes"]])
        torch.cuda.synchronize()
        assert int(ws[max(p["fwd_tiled_bytes"], p["bwd_tiled_bytes"]):].count_nonzero()) == 0
        compare({k: v.cpu() for k, v in o.items()}, ref, BF16, label=f"tiled workspace saved={saved}")


def test_narrow_graph_replay(orc):
    """Replays carry one tag: each must find the meetings' words as if new."""
    T, K, N, r = 123, 2048, 2056, 16
    s = 2.0
    assert _taken(T, K, N, r) == (True, True)
    d = {k: v.cuda() for k, v in lora_inputs(T, K, N, r, seed=60).items()}
    o = {"y": torch.empty(T, N, dtype=BF16, device="cuda"), "u": torch.empty(T, r, device="cuda"),
         "dx": torch.empty(T, K, dtype=BF16, device="cuda"), "dA": torch.empty(r, K, device="cuda"),
         "dB": torch.empty(N, r, device="cuda")}
    n = max(lm.lora_linear_workspace_bytes(op, T, K, N, r, lm.LORA_BF16) for op in (lm.LORA_OP_FWD, lm.LORA_OP_BWD))
    ws = torch.empty(n, dtype=torch.uint8, device="cuda")

    def step():
        lm.lora_linear_fwd(d["x"], d["W"], d["A"], d["B"], o["y"], o["u"], s, ws=ws)
        lm.lora_linear_bwd(d["x"], d["W"], d["A"], d["B"], None, d["dy"], o["dx"], o["dA"], o["dB"], s, ws=ws)

    step()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step()
    for it in range(4):
        _announce(f"narrow graph replay it={it}")
        inp = lora_inputs(T, K, N, r, seed=61 + it)
        for k in ("x", "W", "A", "B", "dy"):
            d[k].copy_(inp[k])
        for v in o.values():
            v.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        compare({k: v.cpu() for k, v in o.items()}, oracle_lora(orc, inp, s), BF16, label=f"replay {it}")
        step()  # eager calls between the replays
        torch.cuda.synchronize()


@pytest.mark.parametrize("shape", [(64, 2048, 2048, 16), (50, 1024, 3072, 16), (40, 2048, 11008, 16),
                                   (128, 1024, 4096, 16)], ids=lambda s: "x".join(map(str, s)))
def test_narrow_replays_with_parts_and_row_tiles(shape):
    """Replays (one tag) of a step whose tiles' parts meet and whose row tiles then
    meet over dA: each replay equals the eager call on its inputs bitwise, and
    leaves every flag down."""
    T, K, N, r = shape
    _announce(f"narrow replays T={T} K={K} N={N} r={r}")
    p = lm.lora_few_token_plan(T, K, N, r)
    assert p["bwd_taken"] and p["bwd_parts"] > 1 and p["bwd_tiles_m"] > 1
    inputs = [{k: v.cuda() for k, v in lora_inputs(T, K, N, r, seed=70 + i).items()} for i in range(3)]
    d = {k: torch.empty_like(v) for k, v in inputs[0].items()}

    def outputs():
        return {"y": torch.empty(T, N, dtype=BF16, device="cuda"), "u": torch.empty(T, r, device="cuda"),
                "dx": torch.empty(T, K, dtype=BF16, device="cuda"), "dA": torch.empty(r, K, device="cuda"),
                "dB": torch.empty(N, r, device="cuda")}

    def step(d, o, wf=None, wb=None):
        lm.lora_linear_fwd(d["x"], d["W"], d["A"], d["B"], o["y"], o["u"], 2.0, ws=wf)
        lm.lora_linear_bwd(d["x"], d["W"], d["A"], d["B"], o["u"], d["dy"], o["dx"], o["dA"], o["dB"], 2.0, ws=wb)

    want = []
    for i in inputs:
        want.append(outputs())
        step(i, want[-1])
    o = outputs()
    wf = torch.full((max(p["fwd_bytes"], p["fwd_tiled_bytes"]),), 0xFF, dtype=torch.uint8, device="cuda")
    wb = torch.full((max(p["bwd_bytes"], p["bwd_tiled_bytes"]),), 0xFF, dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step(d, o, wf, wb)
    tiles = p["bwd_tiles_m"] * p["bwd_tiles_n"]
    for it in range(30):
        for k in d:
            d[k].copy_(inputs[it % 3][k])
        for v in o.values():
            v.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        for k in o:
            assert torch.equal(o[k], want[it % 3][k]), (it, k)
        flags = wb.view(torch.int32)[: tiles * (p["bwd_parts"] + 1) * FLAG_WORDS]
        assert int(flags.count_nonzero()) == 0, it
        if p["fwd_parts"] > 1:
            flags = wf.view(torch.int32)[: p["fwd_tiles_m"] * p["fwd_tiles_n"] * p["fwd_parts"] * FLAG_WORDS]
            assert int(flags.count_nonzero()) == 0, it


@pytest.mark.parametrize("fill", ["int32", "int64", "ones", "fused call"])
@pytest.mark.parametrize("shape", [(24, 3072, 3072, 16), (64, 2048, 2048, 16)], ids=lambda s: "x".join(map(str, s)))
def test_narrow_over_data_of_other_calls(shape, fill):
    """The workspace holds what a program leaves in memory: the whole numbers that
    count its calls, ones, or the hand-over words and sums of a call of many
    tokens.  Every result is that of a clean workspace, bitwise."""
    T, K, N, r = shape
    _announce(f"narrow over {fill} T={T}")
    assert _taken(T, K, N, r) == (True, True)
    many = {k: v.cuda() for k, v in lora_inputs(640, K, N, r, seed=80).items()}
    d = {k: v.cuda() for k, v in lora_inputs(T, K, N, r, seed=81).items()}

    def run(d, ws):
        T = d["x"].shape[0]
        o = {"y": torch.empty(T, N, dtype=BF16, device="cuda"), "u": torch.empty(T, r, device="cuda"),
             "dx": torch.empty(T, K, dtype=BF16, device="cuda"), "dA": torch.empty(r, K, device="cuda"),
             "dB": torch.empty(N, r, device="cuda")}
        lm.lora_linear_fwd(d["x"], d["W"], d["A"], d["B"], o["y"], o["u"], 2.0, ws=ws)
        if fill == "fused call" and T < 640:
            run(many, ws)
        lm.lora_linear_bwd(d["x"], d["W"], d["A"], d["B"], None, d["dy"], o["dx"], o["dA"], o["dB"], 2.0, ws=ws)
        return o

    n = max(lm.lora_linear_workspace_bytes(op, t, K, N, r, lm.LORA_BF16)
            for t in (T, 640) for op in (lm.LORA_OP_FWD, lm.LORA_OP_BWD))
    n = (n + 7) // 8 * 8
    want = run(d, torch.zeros(n, dtype=torch.uint8, device="cuda"))
    ws = torch.empty(n, dtype=torch.uint8, device="cuda")
    for it in range(6):
        if fill == "int32":
            ws.view(torch.int32).copy_(torch.arange(n // 4, dtype=torch.int32))
        elif fill == "int64":
            ws.view(torch.int64).copy_(torch.arange(n // 8))
        elif fill == "ones":
            ws.view(torch.int32).fill_(1)
        else:
            run(many, ws)
        got = run(d, ws)
        torch.cuda.synchronize()
        for k in want:
            assert torch.equal(got[k], want[k]), (it, k)
