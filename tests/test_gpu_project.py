"""Projections onto a few outputs (gemm_rowsplit_kernel, gemm_skinny_kernel): one launch for all tables that a kernel serves,
sums scattered over the lanes of a row.  Against float64, with the bound of k fp32 multiply-adds."""
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
