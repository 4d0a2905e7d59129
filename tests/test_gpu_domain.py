"""GPU parity of group discovery and result ordering against the CPU oracle: bit-exact."""
import numpy as np
import pytest
import torch

from oracle import domain_oracle as D
from oracle import lq_oracle as O

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lq():
    import paper_2306_08367_amd as lq
    return lq


def _check_domain(lq, cols, max_card=65535):
    want_values, want_code = D.group_domain(cols)
    dev = [torch.from_numpy(np.ascontiguousarray(c, dtype=np.int32)).cuda() for c in cols]
    code, values, card = lq.lq_group_domain(dev, max_card=max_card)
    torch.cuda.synchronize()
    assert card == len(want_values)
    np.testing.assert_array_equal(values.cpu().numpy(), want_values)
    np.testing.assert_array_equal(code.cpu().numpy(), want_code)
    return code, values, card


@pytest.mark.parametrize("rows", [1, 2, 63, 64, 257, 5_000, 200_003])
@pytest.mark.parametrize("n_cols", [1, 2, 4])
def test_group_domain_sizes_and_column_counts(lq, rows, n_cols):
    r = np.random.default_rng(100 + rows + n_cols)
    cols = [r.integers(-4, 5, size=rows) for _ in range(n_cols)]
    _check_domain(lq, cols)


def test_group_domain_star_schema_attributes(lq):
    # the attribute columns of the SSB-shaped dimensions: a few distinct values over many rows
    r = np.random.default_rng(7)
    year = r.integers(1992, 1999, size=2_556)
    _check_domain(lq, [year])
    region, nation = r.integers(0, 5, size=1_500_000), r.integers(0, 25, size=1_500_000)
    code, values, card = _check_domain(lq, [region, nation])
    assert card == 125


def test_group_domain_extreme_values_and_many_groups(lq):
    r = np.random.default_rng(8)
    a = r.integers(-2**31, 2**31 - 1, size=60_000)
    a[:4] = [2**31 - 1, -2**31, 0, -1]
    _check_domain(lq, [a])                                         # nearly all rows distinct
    b = r.integers(0, 65_535, size=400_000)
    code, values, card = _check_domain(lq, [b])
    assert card > 60_000
    _check_domain(lq, [np.arange(65_535)[::-1].copy()])            # exactly the largest supported count


def test_group_domain_limits_and_empty(lq):
    dev = [torch.arange(70_000, dtype=torch.int32, device="cuda")]
    with pytest.raises(lq.LQError) as e:
        lq.lq_group_domain(dev)
    assert e.value.status == "LQ_ERR_UNSUPPORTED"
    with pytest.raises(lq.LQError) as e:
        lq.lq_group_domain([torch.arange(11, dtype=torch.int32, device="cuda")], max_card=10)
    assert e.value.status == "LQ_ERR_UNSUPPORTED"
    code, values, card = lq.lq_group_domain([torch.zeros(0, dtype=torch.int32, device="cuda")])
    assert card == 0 and code.numel() == 0 and values.shape[0] == 0


def _check_order(lq, card, sums, counts, keys):
    want = D.order_groups(card, np.zeros((1, len(counts)), dtype=np.int64) if sums is None else sums, counts, keys)
    s = None if sums is None else torch.from_numpy(np.ascontiguousarray(sums, dtype=np.int64)).cuda()
    c = torch.from_numpy(np.ascontiguousarray(counts, dtype=np.int64)).cuda()
    order, n_out = lq.lq_order_groups(card, s, c, keys)
    torch.cuda.synchronize()
    order = order.cpu().numpy()
    n = int(n_out.item())
    assert n == len(want)
    np.testing.assert_array_equal(order[:n], want)
    assert (order[n:] == -1).all()


@pytest.mark.parametrize("card", [[1], [2], [7, 25], [3, 4, 5], [64, 64, 2], [8192], [5, 3, 2, 2, 3]])
def test_order_groups_against_the_oracle(lq, card):
    r = np.random.default_rng(sum(card))
    G = int(np.prod(card))
    for trial in range(4):
        counts = r.integers(0, 3, size=G)
        sums = r.integers(-20, 20, size=(3, G)) * (counts > 0)         # few distinct values: many ties
        sums[2] = r.integers(-2**62, 2**62, size=G)                    # and the full int64 range
        keys = []
        for _ in range(int(r.integers(0, 5))):
            kind = int(r.integers(0, 3))
            index = int(r.integers(0, len(card))) if kind == 0 else (int(r.integers(0, 3)) if kind == 1 else 0)
            keys.append((kind, index, bool(r.integers(0, 2))))
        _check_order(lq, card, sums, counts, keys)
    _check_order(lq, card, None, np.zeros(G, dtype=np.int64), [])       # nothing populated
    _check_order(lq, card, None, np.ones(G, dtype=np.int64), [(D.KEY_COUNT, 0, True)])


def test_discovered_codes_feed_the_group_by_and_its_result_is_ordered(lq):
    # raw attribute values -> codes on the GPU -> group-by -> ORDER BY year ASC, revenue DESC
    r = np.random.default_rng(11)
    year = r.integers(1992, 1999, size=2_556).astype(np.int32)
    brand = r.integers(1000, 1040, size=20_000).astype(np.int32) * 7
    n = 300_001
    fk0, fk1 = r.integers(0, 2_556, size=n).astype(np.int32), r.integers(0, 20_000, size=n).astype(np.int32)
    fk1[r.integers(0, n, size=500)] = -1
    rev = r.integers(1, 10_000, size=n).astype(np.int32)
    (v0, c0), (v1, c1) = D.group_domain([year]), D.group_domain([brand])
    card = [len(v0), len(v1)]
    want_s, want_c = O.groupby_sum([fk0, fk1], [2_556, 20_000], [None, None],
                                   [c0.astype(np.int32), c1.astype(np.int32)], card, None, [rev])
    keys = [(D.KEY_GROUP_COLUMN, 0, False), (D.KEY_SUM, 0, True)]
    want_order = D.order_groups(card, want_s, want_c, keys)

    g = lambda a: torch.from_numpy(a).cuda()
    code0, values0, card0 = lq.lq_group_domain([g(year)])
    code1, values1, card1 = lq.lq_group_domain([g(brand)])
    assert [card0, card1] == card
    sums, counts = lq.lq_masked_groupby_sum([g(fk0), g(fk1)], [2_556, 20_000], None, [code0, code1], card, None,
                                            [g(rev)])
    order, n_out = lq.lq_order_groups(card, sums, counts, keys)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(sums.cpu().numpy(), want_s)
    np.testing.assert_array_equal(counts.cpu().numpy(), want_c)
    np.testing.assert_array_equal(order.cpu().numpy()[: int(n_out.item())], want_order)
    np.testing.assert_array_equal(values0.cpu().numpy(), v0)
    np.testing.assert_array_equal(values1.cpu().numpy(), v1)


def test_argument_errors(lq):
    c = torch.ones(6, dtype=torch.int64, device="cuda")
    with pytest.raises(lq.LQError) as e:
        lq.lq_order_groups([2, 3], None, c, [(D.KEY_SUM, 0, False)])       # no sums given
    assert e.value.status == "LQ_ERR_SHAPE"
    with pytest.raises(lq.LQError) as e:
        lq.lq_order_groups([2, 3], None, c, [(D.KEY_GROUP_COLUMN, 2, False)])
    assert e.value.status == "LQ_ERR_SHAPE"
    with pytest.raises(lq.LQError) as e:
        lq.lq_order_groups([2, 3], None, c, [(7, 0, False)])
    assert e.value.status == "LQ_ERR_SHAPE"
    with pytest.raises(lq.LQError) as e:
        lq.lq_group_domain([torch.zeros(4, dtype=torch.int32, device="cuda")] * 5)
    assert e.value.status == "LQ_ERR_SHAPE"


@pytest.mark.parametrize("G", [1, 2, 31, 32, 33, 64, 65, 127, 128, 129, 1_023, 1_024, 1_025, 8_191])
def test_order_groups_at_the_edges_of_its_tiles(lq, G):
    """32 groups per workgroup, 1,024 keys staged at a time; one workgroup up to 64 groups (128 with three or four keys); keys that
    pack into 50 bits and keys that do not."""
    r = np.random.default_rng(G)
    counts = r.integers(0, 2, size=G)
    sums = np.stack([r.integers(0, 2**33, size=G), r.integers(-2**62, 2**62, size=G)])
    for keys in ([(D.KEY_SUM, 0, True)], [(D.KEY_COUNT, 0, False), (D.KEY_SUM, 1, False)],
                 [(D.KEY_GROUP_COLUMN, 0, True), (D.KEY_SUM, 0, False), (D.KEY_COUNT, 0, True)],
                 [(D.KEY_COUNT, 0, True), (D.KEY_SUM, 1, True), (D.KEY_SUM, 0, False), (D.KEY_GROUP_COLUMN, 0, False)], []):
        _check_order(lq, [G], sums, counts, keys)
    _check_order(lq, [G], sums, np.zeros_like(counts), [(D.KEY_SUM, 0, True)])        # no group populated
    _check_order(lq, [G], sums // 2**62, counts, [(D.KEY_SUM, 1, True), (D.KEY_SUM, 0, False), (D.KEY_COUNT, 0, False)])   # ties
