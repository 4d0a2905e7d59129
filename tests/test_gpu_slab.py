"""Wide bf16 models on many fact rows (fused_slab_bf16_kernel): hidden units in slabs of 64, second-layer sums in registers,
workgroups of an XCD kept in the same slab where the tables are large.  Against float64 on the same projected tables, with
the bound that the two roundings to bf16 allow."""
import pytest
import torch

from tests.helpers import kernel_names

pytestmark = pytest.mark.gpu

CHIP_PAIR = 65_536       # two 16-row tiles on each of 8 wavefronts of 256 compute units: the fewest rows the kernel takes

# n, dim_rows, layers, c_f, bias, stride of the projected tables (0: contiguous)
SHAPES = [
    (CHIP_PAIR, (700, 300), (128, 16), 0, False, 0),                    # one pair of tiles a wavefront, two slabs
    (CHIP_PAIR + 1, (500, 40, 9, 2_000), (256, 5), 0, True, 0),         # ragged end, rows of outputs not stored four at a time
    (131_072, (900, 50, 70), (64, 16), 0, True, 0),                     # one slab: two pairs, keys of the next batch in time
    (131_073 + 31, (900, 50, 70, 1), (64, 17), 4, False, 0),            # two tiles of outputs, fact columns
    (200_003, (3_000,), (192, 33), 0, True, 0),                         # four tiles, three slabs, one table
    (300_007, (800, 60), (200, 16), 0, True, 256),                      # last slab partly past l_1, its padding unreadable
    (150_001, (800, 60, 10), (104, 20, 3), 4, True, 128),               # three layers, fact columns
    (70_001, (100, 80), (256, 64, 16), 0, False, 0),
    (1_100_003, (10_000, 8_000, 9_000), (256, 16), 0, False, 0),        # paced, second batch shorter than the first
    (1_000_000, (14_000, 11_000, 20_000, 7), (192, 64, 1), 0, True, 0),  # paced, three slabs, three layers
    (1_000_003, (14_000, 16_000, 16_000), (192, 40), 0, False, 0),      # paced, two layers with four tiles of outputs
    (1_300_001, (14_000, 11_000, 20_000), (256, 32), 4, False, 0),      # paced, two tiles of outputs, fact columns
    (1_000_000, (14_000, 27_000), (256, 64), 0, True, 0),               # two tables with four tiles of outputs: not paced
    (2_500_000, (9_000, 9_000, 9_000, 500), (256, 16), 4, True, 0),     # paced, several batches, fact columns
    (524_288 + 31, (900, 50, 70, 1), (64, 17), 4, True, 0),             # two tiles of outputs, fact columns, one slab
    (262_145, (100, 80), (256, 64, 16), 0, True, 0),                    # three layers with four tiles of outputs
]
PACED = [s for s in SHAPES if s[0] >= 1_000_000 and s[2] != (256, 64)]
# faster in the kernels that take 16 rows at a time (by the rule's estimates): the shapes around them
ELSEWHERE = [s for s in SHAPES if s[0] in (131_073 + 31, 70_001)] + [
    (131_149, (40_000,), (128, 40, 8), 4, False, 0), (65_536, (10_000,) * 4, (96, 64, 16), 0, False, 128),
    (161_073, (10_000,) * 4, (64, 64, 1), 0, False, 64), (262_221, (10_000,) * 4, (56, 16, 1), 4, False, 64),
]


def _model(n, rows, layers, c_f, bias, ld, seed=3):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)

    def normal(shape, sigma=1.0):
        return (torch.randn(shape, generator=gen, device="cuda") * sigma).bfloat16()

    widths = [c_f + 8] + list(layers)
    W = [normal((a, b), a ** -0.5) for a, b in zip(widths, widths[1:])]
    b = [normal((c,), 0.5) for c in layers] if bias else None
    P = []
    for r in rows:
        t = torch.full((r, ld or layers[0]), float("nan"), device="cuda", dtype=torch.bfloat16)
        t[:, :layers[0]] = normal((r, layers[0]))
        P.append(t[:, :layers[0]])
    fks = [torch.randint(0, r, (n,), generator=gen, device="cuda", dtype=torch.int32) for r in rows]
    return (normal((n, c_f)) if c_f else None), fks, P, W, b


def _reference(X, fks, P, W, b):
    """(result, bound): hidden units rounded to bf16 once (8 significant bits: by 2^-8 of each at most), later activations and sums at about fp32."""
    z = 0 if b is None else b[0].double()
    if X is not None:
        z = z + X.double() @ W[0][:X.shape[1]].double()
    for p, f in zip(P, fks):
        z = z + p.double()[f.long()]
    h = z.clamp(min=0)
    err = h * 2.0 ** -8
    for i, w in enumerate(W[1:], 1):
        if i > 1:
            err = err + h.abs() * 2.0 ** -16
        y = h @ w.double() + (0 if b is None else b[i].double())
        err = err @ w.double().abs() + 1e-5 * (h.abs() @ w.double().abs() + 1)
        h = y.clamp(min=0)
    return y, err


@pytest.mark.parametrize("shape", SHAPES + ELSEWHERE[2:], ids=lambda s: "-".join(map(str, (s[0],) + s[2] + (len(s[1]), s[3]))))
def test_against_float64(shape):
    import paper_2306_08367_amd as lq
    X, fks, P, W, b = _model(*shape)
    want, err = _reference(X, fks, P, W, b)
    got = lq.lq_fused_join_predict(X, fks, P, W, b, y_dtype=torch.float32)
    assert bool(((got.double() - want).abs() <= err).all())
    # workgroups kept in step where the shape says so
    names = kernel_names(lambda: lq.lq_fused_join_predict(X, fks, P, W, b, Y=got))
    assert any("fused_slab_bf16_kernel" in name for name in names) == (shape not in ELSEWHERE), names
    assert any("slab_pace_clear_kernel" in name for name in names) == (shape in PACED), names
    # a caller with a small workspace, and bf16 outputs in a strided tensor
    plain = lq.lq_fused_join_predict(X, fks, P, W, b, y_dtype=torch.float32, ws=torch.empty(256, dtype=torch.uint8, device="cuda"))
    assert torch.equal(plain, got)
    Y = torch.full((shape[0], shape[2][-1] + 3), 7.0, device="cuda", dtype=torch.bfloat16)
    lq.lq_fused_join_predict(X, fks, P, W, b, Y=Y[:, :shape[2][-1]])
    assert torch.equal(Y[:, :shape[2][-1]], got.bfloat16()) and bool((Y[:, shape[2][-1]:] == 7).all())


def test_not_a_number_stays_with_its_fact_rows():
    import paper_2306_08367_amd as lq
    X, fks, P, W, b = _model(80_000, (500, 400), (128, 16), 0, True, 0)
    clean = lq.lq_fused_join_predict(X, fks, P, W, b)
    P[0][17, 3], P[1][33, 100] = float("inf"), float("nan")
    hit = (fks[0] == 17) | (fks[1] == 33)
    got = lq.lq_fused_join_predict(X, fks, P, W, b)
    assert torch.equal(got[~hit], clean[~hit])
    general = lq.lq_fused_join_predict(X, fks, P, W, b, flags=lq.LQ_FORCE_GENERIC)
    assert torch.equal(got[hit].isinf(), general[hit].isinf()) and torch.equal(got[hit].isnan(), general[hit].isnan())


def test_workspace_of_a_group_by_is_left_alone():
    """A paced call with the workspace that holds a group-by's side tables for LQ_REUSE_SIDE_TABLES."""
    import paper_2306_08367_amd as lq
    X, fks, P, W, b = _model(1_000_000, (12_000, 9_000, 2_000), (256, 16), 0, False, 0)
    rows, card = [12_000, 9_000, 2_000], [5, 1, 7]
    codes = [torch.arange(r, device="cuda", dtype=torch.int32) % c if c > 1 else None for r, c in zip(rows, card)]
    masks = [None, (torch.arange(9_000, device="cuda") % 3 > 0).to(torch.uint8), None]
    measure = [torch.arange(1_000_000, device="cuda", dtype=torch.int32)]
    ws = torch.zeros(max(lq.lq_groupby_workspace_bytes(rows, card, 1), 4_096), dtype=torch.uint8, device="cuda")
    want = lq.lq_masked_groupby_sum(fks, rows, masks, codes, card, None, measure, ws=ws)
    kept = ws.clone()
    call = lambda: lq.lq_fused_join_predict(X, fks, P, W, b, ws=ws)
    assert any("slab_pace_clear_kernel" in name for name in kernel_names(call))
    call()
    assert torch.equal(ws, kept)
    got = lq.lq_masked_groupby_sum(fks, rows, masks, codes, card, None, measure, ws=ws, flags=lq.LQ_REUSE_SIDE_TABLES)
    assert all(torch.equal(g, w) for g, w in zip(got, want))


def test_replays_of_a_graph():
    import paper_2306_08367_amd as lq
    X, fks, P, W, b = _model(1_000_000, (12_000, 9_000, 2_000), (256, 16), 0, False, 0)
    Y = torch.empty(1_000_000, 16, device="cuda", dtype=torch.bfloat16)
    ws = torch.empty(4_096, dtype=torch.uint8, device="cuda")
    want = lq.lq_fused_join_predict(X, fks, P, W, b)
    torch.cuda.synchronize()
    stream = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        lq.lq_fused_join_predict(X, fks, P, W, b, Y=Y, ws=ws)
    for _ in range(4):
        Y.zero_()
        ws.fill_(0xa5)               # what the counters held before does not matter
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(Y, want)
        assert torch.equal(lq.lq_fused_join_predict(X, fks, P, W, b), want)


@pytest.mark.parametrize("bias", [False, True], ids=["", "bias"])
@pytest.mark.parametrize("c_f", [0, 4])
@pytest.mark.parametrize("outputs", [16, 32, 64])
@pytest.mark.parametrize("tables", [1, 2, 3, 4])
def test_every_instance(tables, outputs, c_f, bias):
    """One kernel for each number of tables, tiles of outputs, and with and without fact columns and a first bias: two slabs, several
    rounds of rows, a ragged end."""
    import paper_2306_08367_amd as lq
    n = 500_003
    X, fks, P, W, b = _model(n, (900, 5_000, 70, 2_000)[:tables], (128, outputs), c_f, bias, 0, seed=tables)
    got = lq.lq_fused_join_predict(X, fks, P, W, b, y_dtype=torch.float32)
    instance = f"fused_slab_bf16_kernelILi{tables}ELi{outputs // 16}ELi{c_f}ELb{int(bias)}E"
    assert any(instance in name for name in kernel_names(lambda: lq.lq_fused_join_predict(X, fks, P, W, b, Y=got)))
    for first in range(0, n, 100_000):
        part = slice(first, min(first + 100_000, n))
        want, err = _reference(None if X is None else X[part], [f[part] for f in fks], P, W, b)
        assert bool(((got[part].double() - want).abs() <= err).all())
