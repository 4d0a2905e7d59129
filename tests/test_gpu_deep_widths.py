"""Deeper models at the edges of the 16 x 16 tiles that their weights are staged in (fused_deep_kernel,
fused_deep_bf16_kernel): layer widths, fact columns and outputs around a tile, biases on some layers only, few rows.
Against float64, per element, with the tolerances of the other parity tests."""
import pytest
import torch

from tests.helpers import TOL_BF16, TOL_F32, assert_close

pytestmark = pytest.mark.gpu


def _check(n, c_f, layers, dtype, tol, rows=(7, 300, 41)):
    import paper_2306_08367_amd as lq
    gen = torch.Generator(device="cuda")
    gen.manual_seed(sum(layers) + n)
    cols = [8 * (k % 3 + 1) for k in range(len(rows))]
    normal = lambda *shape: torch.randn(*shape, generator=gen, device="cuda")
    dims = [normal(r, c).to(dtype) for r, c in zip(rows, cols)]
    fks = [torch.randint(0, r, (n,), generator=gen, device="cuda", dtype=torch.int32) for r in rows]
    X = normal(n, c_f).to(dtype) if c_f else None
    widths = [c_f + sum(cols), *layers]
    W = [(normal(a, b) * a ** -0.5).to(dtype) for a, b in zip(widths, widths[1:])]
    b = [normal(w).to(dtype) if j % 2 == len(layers) % 2 else None for j, w in enumerate(layers)]
    P = lq.lq_project_dims(dims, W[0], c_f)
    Y = lq.lq_fused_join_predict(X, fks, P, W, b)
    # the tables as they were projected (bf16 ones are rounded there): this checks the join stage
    h = sum(p.double()[f.long()] for p, f in zip(P, fks))
    if c_f:
        h = h + X.double() @ W[0][:c_f].double()
    for j, w in enumerate(W):
        h = h if j == 0 else h.clamp(min=0) @ w.double()
        h = h if b[j] is None else h + b[j].double()
    assert_close(Y, h.cpu().numpy(), tol, f"{n} rows, {c_f} fact columns, {layers}")


@pytest.mark.parametrize("c_f", [0, 1, 5, 17])
@pytest.mark.parametrize("layers", [(15, 17), (33, 16, 1), (64, 31, 2), (65, 33, 17), (130, 64, 16), (16, 15, 17, 1), (100, 49, 64, 33),
                                    # two layers of 128 x 128: the first in two column parts while the LDS holds it
                                    (100, 100, 100, 1), (65, 128, 128), (128, 113, 65, 16)])
def test_fp32(layers, c_f):
    for n in (1, 17, 200):
        _check(n, c_f, layers, torch.float32, TOL_F32)


@pytest.mark.parametrize("c_f", [0, 3])
@pytest.mark.parametrize("layers", [(8, 17), (72, 33, 1), (200, 64, 16), (256, 17, 5), (40, 31, 33, 16), (64, 129, 15)])
def test_bf16(layers, c_f):
    for n in (1, 17, 200):
        _check(n, c_f, layers, torch.bfloat16, TOL_BF16)


@pytest.mark.parametrize("c_f", [0, 5])
@pytest.mark.parametrize("tables", [1, 3, 4, 6])
@pytest.mark.parametrize("layers", [(100, 100, 100, 1), (128, 128, 128),       # two layers of 128 x 128: one workgroup a compute unit
                                    (64, 64), (200, 16)], ids=lambda l: "-".join(map(str, l)))
def test_fp32_several_steps(layers, tables, c_f):
    """More rows than one step of every wavefront of the chip takes (16,384 with one workgroup a compute unit): the keys and gathers that
    one step hands to the next, and one column part to the other; a ragged end."""
    _check(50_003 if 128 in layers or 100 in layers else 250_003, c_f, layers, torch.float32, TOL_F32, (7, 300, 41, 1_000, 5, 64)[:tables])


@pytest.mark.parametrize("layers", [(96, 96, 4), (72, 128, 16)], ids=lambda l: "-".join(map(str, l)))
def test_bf16_several_steps(layers):
    _check(150_003, 3, layers, torch.bfloat16, TOL_BF16)
