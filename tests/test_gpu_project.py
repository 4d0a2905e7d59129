"""Projections onto a few outputs (gemm_rowsplit_kernel, gemm_skinny_kernel): one launch for all tables that a kernel serves,
sums scattered over the lanes of a row.  Against float64, with the bound of k fp32 multiply-adds.
Projections onto more than 16 outputs (gemm_split_kernel): fp32 operands in three bf16 pieces, what these cannot hold in fp32."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("outputs", [1, 2, 3, 4, 5, 8, 13])
@pytest.mark.parametrize("rows, cols", [
    ((1, 31, 33), (32, 32, 32)),                     # 8 lanes a row, rows around a wavefront's step of 32
    ((15, 17, 4_097), (64, 36, 60)),                 # 16 lanes, pieces that do not fill them
    ((7, 9), (128, 100)),                            # 32 lanes, steps of 8 rows
    ((3, 5, 70_001), (256, 132, 520)),               # 64 lanes, more pieces than lanes
    ((100, 1, 50, 257, 1_000), (8, 31, 32, 64, 300)),   # every kernel in one call
], ids=["8", "16", "32", "64", "mixed"])
def test_few_outputs(outputs, rows, cols):
    import paper_2306_08367_amd as lq
    gen = torch.Generator(device="cuda")
    gen.manual_seed(outputs)
    dims = [torch.randn(r, c, generator=gen, device="cuda") for r, c in zip(rows, cols)]
    W = torch.randn(3 + sum(cols), outputs, generator=gen, device="cuda")
    P = lq.lq_project_dims(dims, W, 3)
    at = 3
    for D, p in zip(dims, P):
        w = W[at:at + D.shape[1]].double()
        at += D.shape[1]
        bound = (D.shape[1] + 2) * 2.0 ** -24 * (D.double().abs() @ w.abs())
        assert bool(((p.double() - D.double() @ w).abs() <= bound).all())
        # a row does not depend on the table it is part of
        if D.shape[0] > 16:
            few = lq.lq_project_dims([D[5:16].contiguous()], torch.cat([W[:3], w.float()]), 3)[0]
            assert torch.equal(few, p[5:16])


def _project(D, W):
    import paper_2306_08367_amd as lq
    return lq.lq_project_dims([D], W, 0)[0][:, :W.shape[1]]


def _within_bound(got, D, W):
    # k fp32 multiply-adds; the products left out of nine are at most 2^-24 of the product, one of the two terms added to k
    bound = (D.shape[1] + 2) * 2.0 ** -24 * (D.double().abs() @ W.double().abs())
    return bool(((got.double() - D.double() @ W.double()).abs() <= bound).all())


@pytest.mark.parametrize("k", [1, 7, 16, 17, 31, 48, 100, 683])
@pytest.mark.parametrize("outputs", [17, 32, 33, 64, 65, 128, 130, 257])
def test_split_products(outputs, k):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1_000 * outputs + k)
    W = torch.randn(k, outputs, generator=gen, device="cuda")
    D = torch.randn(385, k, generator=gen, device="cuda") * torch.exp2(torch.randint(-20, 20, (385, 1), generator=gen, device="cuda").float())
    whole = _project(D, W)
    assert _within_bound(whole, D, W)
    for rows in (1, 31, 127, 128, 129, 256):                  # a row does not depend on the table it is part of
        assert torch.equal(_project(D[:rows].contiguous(), W), whole[:rows])
    assert torch.equal(_project(D[100:300].contiguous(), W), whole[100:300])


@pytest.mark.parametrize("k", [17, 64])
def test_split_products_of_large_tables(k):
    """Enough 256-row tiles for the larger instance, the last one ragged: the bits of the smaller one."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(k)
    rows, outputs = 65_536 + 77, 1_025
    D, W = torch.randn(rows, k, generator=gen, device="cuda"), torch.randn(k, outputs, generator=gen, device="cuda")
    got = _project(D, W)
    for at in (0, 30_000, rows - 1_000):
        part = D[at:at + 1_000].contiguous()
        assert torch.equal(_project(part, W), got[at:at + 1_000]) and _within_bound(got[at:at + 1_000], part, W)
    D[3, 1], D[rows - 1, 0] = float("inf"), float("nan")
    again = _project(D, W)
    assert torch.equal(again[4:-1], got[4:-1]) and bool(again[-1].isnan().all())
    assert torch.equal(again[3], torch.sign(W[1]) * float("inf"))


@pytest.mark.parametrize("outputs", [20, 64, 200])
def test_split_products_outside_the_range_of_the_pieces(outputs):
    """Infinities, NaNs, values next to the largest and below the smallest normal ones: as fp32 arithmetic gives them, and
    nothing else changes."""
    inf, nan = float("inf"), float("nan")
    gen = torch.Generator(device="cuda")
    gen.manual_seed(outputs)
    D, W = torch.randn(300, 40, generator=gen, device="cuda"), torch.randn(40, outputs, generator=gen, device="cuda")
    W[:, 3] = 0
    W[0, 3] = 0.5
    plain = _project(D, W)
    special = D.clone()
    special[5, 7], special[140, 0], special[299, 39] = inf, nan, -inf
    special[50], special[51] = 0, 0
    special[50, 0] = 3.4e38                                   # rounds to a bf16 infinity, times 0.5 in column 3
    got = _project(special, W)
    assert torch.equal(got[5, 4:], torch.sign(W[7, 4:]) * inf) and bool(got[140].isnan().all())
    assert torch.equal(got[299, 4:], torch.sign(W[39, 4:]) * -inf)
    assert bool(got[5, 3].isnan()) and bool(got[299, 3].isnan())   # inf * 0
    assert float(got[50, 3]) == float(special[50, 0] * 0.5) and bool((got[51] == 0).all())
    rest = torch.ones(300, dtype=torch.bool, device="cuda")
    rest[[5, 50, 51, 140, 299]] = False
    assert torch.equal(got[rest], plain[rest])
    w = W.clone()
    w[11, 9], w[12, 10] = inf, nan
    got = _project(D, w)
    assert torch.equal(got[:, 9], torch.sign(D[:, 11]) * inf) and bool(got[:, 10].isnan().all())
    assert torch.equal(got[:, 11:], plain[:, 11:]) and torch.equal(got[:, :9], plain[:, :9])


@pytest.mark.parametrize("scale_d, scale_w", [(-20, 0), (-100, 0), (-118, 0), (-130, 0), (-142, 0), (-75, -45), (0, -125), (-120, 60), (100, -100),
                                              (-70, -70), (-66, -72), (-120, 100), (-130, 110), (-124, 124), (116, -116), (120, -120), (124, -124)])
def test_split_products_of_small_numbers(scale_d, scale_w):
    """Down to subnormal operands and results: the bound of fp32 arithmetic, half a unit of the smallest subnormal a term besides."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(7)
    D = torch.ldexp(torch.randn(200, 30, generator=gen, device="cuda"), torch.tensor(scale_d, device="cuda"))
    W = torch.ldexp(torch.randn(30, 70, generator=gen, device="cuda"), torch.tensor(scale_w, device="cuda"))
    got = _project(D, W)
    bound = 32 * 2.0 ** -24 * (D.double().abs() @ W.double().abs()) + 30 * 2.0 ** -149
    assert bool(((got.double() - D.double() @ W.double()).abs() <= bound).all())


def test_split_products_of_a_small_and_a_large_operand_beside_others():
    """A term that its operand's pieces do not hold, in a sum that is not small."""
    D, W = torch.zeros(40, 30, device="cuda"), torch.zeros(30, 70, device="cuda")
    D[:, 0], D[:, 1] = 2.0 ** -140, 2.0 ** -25
    W[0], W[1] = 2.0 ** 120, 1
    assert bool((_project(D, W) == 2.0 ** -20 + 2.0 ** -25).all())
    assert bool((_project(W.t().contiguous(), D.t().contiguous()) == 2.0 ** -20 + 2.0 ** -25).all())


@pytest.mark.parametrize("rows,outputs", [(385, 130), (45_003, 50), (20_011, 1_030), (65_613, 1_025)])
def test_split_products_of_small_numbers_beside_others(rows, outputs):
    """Operands below 2^-100 in single rows and columns and results below 2^-30: no other row or column changes, and a row computed
    alone is the row of the table."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(rows)
    D = torch.randn(rows, 40, generator=gen, device="cuda") * 1e-10
    W = torch.randn(40, outputs, generator=gen, device="cuda") * 1e-3
    plain = _project(D, W)
    at, col = [0, 33, 130, rows - 2], [0, 37, outputs - 1]
    D[at, 3], W[5, col] = 1e-40, -1e-38
    D[200, 7], W[9, 20] = 1e25, 1e22                         # (and large ones: every result of such a pair)
    got = _project(D, W)
    same_row, same_col = torch.ones(rows, dtype=torch.bool, device="cuda"), torch.ones(outputs, dtype=torch.bool, device="cuda")
    same_row[at + [200]], same_col[col + [20]] = False, False
    assert torch.equal(got[same_row][:, same_col], plain[same_row][:, same_col])
    assert _within_bound(got, D, W)
    for first in (0, 1, 33, 129, 199, rows - 3):
        assert torch.equal(_project(D[first:first + 2].contiguous(), W), got[first:first + 2])
    assert torch.equal(_project(D[30:300].contiguous(), W), got[30:300])
    few = [c for c in (0, 20, 36, 37, outputs - 1) for _ in range(5)]
    assert torch.equal(_project(D, W[:, few].contiguous()), got[:, few])


@pytest.mark.parametrize("k", [17, 64, 320])
@pytest.mark.parametrize("kind", ["normal", "positive", "relu", "sparse", "single"])
def test_split_products_are_as_close_as_multiply_adds(kind, k):
    """Error against float64 in the 2-norm: at most that of a chain of k fp32 multiply-adds, also where most of them add zero and so round
    nothing.  A tenth more for the noise of 64,000 results and, with one product a result, for the products left out (2^-28 on average
    beside a rounding of 2^-25.2)."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(k)
    D, W = torch.randn(1_000, k, generator=gen, device="cuda"), torch.randn(k, 64, generator=gen, device="cuda")
    if kind == "positive":
        D, W = D.abs(), W.abs()
    elif kind == "relu":
        D = D.clamp(min=0)
    elif kind == "sparse":
        D = D * (torch.rand(1_000, k, generator=gen, device="cuda") < 0.05)
    elif kind == "single":
        D = D * torch.nn.functional.one_hot(torch.arange(1_000, device="cuda") % k, k)
    exact = D.double() @ W.double()
    chain = torch.zeros(1_000, 64, device="cuda")
    for q in range(k):                                        # (the sum of an fp32 number and a product of two in float64, rounded once more)
        chain = (chain.double() + D[:, q:q + 1].double() * W[q].double()).float()
    assert float((_project(D, W).double() - exact).norm()) <= 1.1 * float((chain.double() - exact).norm())


def _same(a, b):
    return torch.equal(a.isnan(), b.isnan()) and torch.equal(a.nan_to_num(nan=0.0), b.nan_to_num(nan=0.0))


# Rows and outputs at which each tile of gemm_split_kernel is the chosen one (on 256 compute units; whichever it is, the bits are the same): 128 rows x 32
# columns, x 64 (twice), x 128, and 256 x 128, this one for 64 or more columns of the table.  Rows and outputs end inside a tile, k inside a step.
TILES = [(385, 130, 23), (45_003, 50, 31), (45_003, 200, 33), (100_003, 200, 17), (100_003, 200, 83), (65_613, 1_025, 67)]


def _drawn(rows, outputs, k):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(rows + outputs + k)
    return torch.randn(rows, k, generator=gen, device="cuda"), torch.randn(k, outputs, generator=gen, device="cuda")


def _check_parts(D, W, whole, places):
    """Rows and columns computed alone are those of the whole, and within the bound where the sums are finite."""
    for at in places:
        at = max(0, min(at, D.shape[0] - 70))
        part = D[at:at + 70].contiguous()
        got = _project(part, W)
        assert _same(got, whole[at:at + 70])
        exact = part.double() @ W.double()
        error = (got.double() - exact).abs()
        bound = (D.shape[1] + 2) * 2.0 ** -24 * (part.double().abs() @ W.double().abs()) + D.shape[1] * 2.0 ** -149
        finite = exact.abs() < 2.0 ** 127
        assert bool((error[finite] <= bound[finite]).all()) and torch.equal(exact.isnan(), got.isnan())
        assert bool((got[exact.isinf()] == exact[exact.isinf()]).all())
    few = torch.arange(0, W.shape[1], max(1, W.shape[1] // 23), device="cuda")
    rows = slice(places[0], places[0] + 70)
    assert _same(_project(D[rows].contiguous(), W[:, few].contiguous()), whole[rows][:, few])


@pytest.mark.parametrize("rows,outputs,k", TILES)
def test_split_products_of_every_tile(rows, outputs, k):
    D, W = _drawn(rows, outputs, k)
    _check_parts(D, W, _project(D, W), (0, 90, 130, rows // 2, rows))


@pytest.mark.parametrize("rows,outputs,k", TILES)
def test_split_products_of_every_tile_outside_the_range_of_the_pieces(rows, outputs, k):
    D, W = _drawn(rows, outputs, k)
    W[1].clamp_(-0.9, 0.9)                                    # (3.4e38 times it stays finite, as it is in the float64 reference)
    plain = _project(D, W)
    inf, nan = float("inf"), float("nan")
    middle = rows // 2
    at = [5, 40, 131, 132, 133, middle, middle + 1, rows - 1]
    D[5, 7], D[131, 0], D[middle, k - 1], D[rows - 1, 3] = inf, nan, -inf, inf
    D[40, 1], D[132], D[133] = 3.4e38, 0, 0
    D[132, 5] = 1e-42
    D[middle + 1, 2] = inf
    D[middle + 1, 4] = -inf                                   # (both signs: NaN)
    got = _project(D, W)
    same = torch.ones(rows, dtype=torch.bool, device="cuda")
    same[at] = False
    assert torch.equal(got[same], plain[same])
    _check_parts(D, W, got, (0, 100, middle - 30, rows))
    W[11, 9], W[12, 10], W[:, 17], W[3, outputs - 1], W[:, 33] = inf, nan, 0, -inf, 1e-39
    again = _project(D, W)
    cols = torch.ones(outputs, dtype=torch.bool, device="cuda")
    cols[[9, 10, 17, 33, outputs - 1]] = False
    assert _same(again[:, cols], got[:, cols])
    _check_parts(D, W, again, (0, 100, middle - 30, rows))


@pytest.mark.parametrize("scale_d,scale_w", [(-120, 100), (116, -116), (-130, 0), (-70, -70), (0, -125)])
@pytest.mark.parametrize("rows,outputs,k", TILES)
def test_split_products_of_every_tile_of_small_numbers(rows, outputs, k, scale_d, scale_w):
    D, W = _drawn(rows, outputs, k)
    D, W = torch.ldexp(D, torch.tensor(scale_d, device="cuda")), torch.ldexp(W, torch.tensor(scale_w, device="cuda"))
    _check_parts(D, W, _project(D, W), (0, 90, rows // 2, rows))
