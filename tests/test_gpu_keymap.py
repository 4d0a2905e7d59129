"""GPU parity of the key -> row mapping (Algorithm 1's domain generation + row-matching matrix)
against the MM-Join oracle: bit-exact, including the COO form of I and its use by the group-by."""
import numpy as np
import pytest
import torch

from oracle import lq_oracle as O
from oracle import mmjoin_oracle as MJ

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lq():
    import paper_2306_08367_amd as lq
    return lq


def _keys(seed, r, n, miss=0.05, lo=-2**31, hi=2**31 - 1):
    g = np.random.default_rng(seed)
    pool = np.unique(g.integers(lo, hi, size=int(r * 1.3) + 8, dtype=np.int64))
    g.shuffle(pool)
    key_S = pool[:r].astype(np.int32)
    extra = pool[r:]
    key_R = g.choice(key_S, size=n).astype(np.int32) if r else np.zeros(n, dtype=np.int32)
    if len(extra) and n:
        m = g.random(n) < miss
        key_R[m] = g.choice(extra, size=int(m.sum())).astype(np.int32)
    return key_S, key_R


@pytest.mark.parametrize("r,n", [(1, 1), (1, 100), (7, 1_000), (2_556, 100_003), (30_000, 200_001), (200_000, 1_000_000), (2_000, 1_200_003), (8_000, 1_100_000)])
def test_lookup_and_compaction_match_algorithm_1(lq, r, n):
    key_S, key_R = _keys(r + n, r, n)
    fk_w, rows_w, cols_w = MJ.key_to_row(key_R, key_S)
    table = lq.lq_keymap_build(torch.from_numpy(key_S).cuda(), flags=lq.LQ_CHECK_KEYS)
    fk = lq.lq_keymap_lookup(table, torch.from_numpy(key_R).cuda())
    rows, cols, nnz = lq.lq_compact_matches(fk)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(fk.cpu().numpy(), fk_w)
    m = int(nnz.item())
    assert m == len(rows_w)
    np.testing.assert_array_equal(rows[:m].cpu().numpy(), rows_w)
    np.testing.assert_array_equal(cols[:m].cpu().numpy(), cols_w)


def test_extreme_key_values_and_no_matches(lq):
    key_S = np.array([-2**31, 2**31 - 1, 0, -1, 1], dtype=np.int32)
    key_R = np.array([0, -1, 2**31 - 1, -2**31, 5, 1, 1, -7], dtype=np.int32)
    table = lq.lq_keymap_build(torch.from_numpy(key_S).cuda())
    fk = lq.lq_keymap_lookup(table, torch.from_numpy(key_R).cuda())
    assert fk.cpu().tolist() == [2, 3, 1, 0, -1, 4, 4, -1]
    none = lq.lq_keymap_lookup(table, torch.full((1000,), 77, dtype=torch.int32, device="cuda"))
    rows, cols, nnz = lq.lq_compact_matches(none)
    assert int(nnz.item()) == 0 and (none == -1).all()
    rows, cols, nnz = lq.lq_compact_matches(torch.empty(0, dtype=torch.int32, device="cuda"))
    assert int(nnz.item()) == 0


def test_duplicate_dimension_keys_are_reported(lq):
    keys = torch.tensor([5, 9, 5, 3], dtype=torch.int32, device="cuda")
    with pytest.raises(lq.LQError) as e:
        lq.lq_keymap_build(keys, flags=lq.LQ_CHECK_KEYS)
    assert e.value.status == "LQ_ERR_DUPLICATE_KEY"


def test_incremental_insert_equals_rebuild(lq):
    """Updating a cached domain: keys of new dimension rows are inserted into the existing map."""
    key_S, key_R = _keys(99, 50_000, 300_000, miss=0.2)
    full = lq.lq_keymap_build(torch.from_numpy(key_S).cuda())
    part = lq.lq_keymap_build(torch.from_numpy(key_S[:30_000]).cuda(), max_keys=50_000)
    kr = torch.from_numpy(key_R).cuda()
    before = lq.lq_keymap_lookup(part, kr)
    lq.lq_keymap_insert(part, torch.from_numpy(key_S[30_000:]).cuda(), 30_000, flags=lq.LQ_CHECK_KEYS)
    after = lq.lq_keymap_lookup(part, kr)
    want = lq.lq_keymap_lookup(full, kr)
    torch.cuda.synchronize()
    assert torch.equal(after, want)
    fk_w, _, _ = MJ.key_to_row(key_R, key_S[:30_000])
    np.testing.assert_array_equal(before.cpu().numpy(), fk_w)


def test_mapped_keys_feed_the_group_by(lq):
    """End to end on raw key values: map four key columns, then aggregate; unmatched keys drop out."""
    g = np.random.default_rng(5)
    n, rows_k, card = 200_003, (50, 400, 30), (5, 7, 1)
    keys_S, keys_R = zip(*[_keys(200 + k, r, n, miss=0.1) for k, r in enumerate(rows_k)])
    codes = [g.integers(0, c, size=r).astype(np.int32) if c > 1 else None for r, c in zip(rows_k, card)]
    masks = [None, None, (g.random(30) < 0.5).astype(np.uint8)]
    meas = g.integers(1, 1000, size=n).astype(np.int32)
    fks_w = [MJ.key_to_row(kr, ks)[0] for kr, ks in zip(keys_R, keys_S)]
    want_s, want_c = O.groupby_sum(fks_w, list(rows_k), masks, codes, list(card), None, [meas])
    fks = [lq.lq_keymap_lookup(lq.lq_keymap_build(torch.from_numpy(ks).cuda()), torch.from_numpy(kr).cuda())
           for kr, ks in zip(keys_R, keys_S)]
    dev = lambda a: None if a is None else torch.from_numpy(a).cuda()
    s, c = lq.lq_masked_groupby_sum(fks, list(rows_k), [dev(m) for m in masks], [dev(x) for x in codes],
                                    list(card), None, [dev(meas)])
    torch.cuda.synchronize()
    np.testing.assert_array_equal(s.cpu().numpy(), want_s)
    np.testing.assert_array_equal(c.cpu().numpy(), want_c)


def _is_direct(table):
    return int(table[12:16].view(torch.int32).item()) == 1


def _dense_keys(seed, r, n, base, fill=0.7, miss=0.05):
    """r distinct keys out of a window of r / fill consecutive integers starting at `base`, shuffled."""
    g = np.random.default_rng(seed)
    window = np.arange(int(r / fill) + 1, dtype=np.int64) + base
    g.shuffle(window)
    key_S = window[:r].astype(np.int32)
    key_R = g.choice(window, size=n).astype(np.int32)              # some hit the gaps: no match
    m = g.random(n) < miss
    key_R[m] = (base - 1 - g.integers(0, 1000, size=int(m.sum()))).astype(np.int32)   # and some lie outside the window
    return key_S, key_R


@pytest.mark.parametrize("r,n,base", [(1, 10, 5), (2_556, 1_300_001, 19920101), (2_000, 100_003, 1), (30_000, 1_200_000, 1),
                                      (200_000, 1_000_003, -150_000), (8_192, 1_048_576, -2**31 + 1000)])
def test_dense_key_ranges_use_the_direct_form(lq, r, n, base):
    key_S, key_R = _dense_keys(r + n, r, n, base)
    fk_w, rows_w, cols_w = MJ.key_to_row(key_R, key_S)
    table = lq.lq_keymap_build(torch.from_numpy(key_S).cuda(), flags=lq.LQ_CHECK_KEYS)
    assert _is_direct(table)
    fk = lq.lq_keymap_lookup(table, torch.from_numpy(key_R).cuda())
    torch.cuda.synchronize()
    np.testing.assert_array_equal(fk.cpu().numpy(), fk_w)
    # unaligned key columns take the one-key-per-thread path
    kr = torch.empty(n + 1, dtype=torch.int32, device="cuda")
    kr[1:] = torch.from_numpy(key_R)
    np.testing.assert_array_equal(lq.lq_keymap_lookup(table, kr[1:]).cpu().numpy(), fk_w)


def test_sparse_key_ranges_use_the_hashed_form(lq):
    key_S, key_R = _keys(17, 5_000, 1_100_000)
    table = lq.lq_keymap_build(torch.from_numpy(key_S).cuda(), flags=lq.LQ_CHECK_KEYS)
    assert not _is_direct(table)
    fk_w, _, _ = MJ.key_to_row(key_R, key_S)
    np.testing.assert_array_equal(lq.lq_keymap_lookup(table, torch.from_numpy(key_R).cuda()).cpu().numpy(), fk_w)


def test_direct_form_duplicates_and_inserts(lq):
    keys = torch.tensor([5, 9, 5, 3], dtype=torch.int32, device="cuda")
    with pytest.raises(lq.LQError) as e:
        lq.lq_keymap_build(keys, flags=lq.LQ_CHECK_KEYS)
    assert e.value.status == "LQ_ERR_DUPLICATE_KEY"
    # surrogate keys 1..r, new dimension rows appended with the next keys: inside the window
    key_S = np.arange(1, 40_001, dtype=np.int32)
    g = np.random.default_rng(3)
    key_R = g.integers(-5, 40_020, size=500_000).astype(np.int32)
    part = lq.lq_keymap_build(torch.from_numpy(key_S[:25_000]).cuda(), max_keys=40_000)
    assert _is_direct(part)
    lq.lq_keymap_insert(part, torch.from_numpy(key_S[25_000:]).cuda(), 25_000, flags=lq.LQ_CHECK_KEYS)
    fk_w, _, _ = MJ.key_to_row(key_R, key_S)
    np.testing.assert_array_equal(lq.lq_keymap_lookup(part, torch.from_numpy(key_R).cuda()).cpu().numpy(), fk_w)
    # a key far outside the window cannot be added to a direct map: reported, the map stays usable
    with pytest.raises(lq.LQError) as e:
        lq.lq_keymap_insert(part, torch.tensor([2_000_000_000], dtype=torch.int32, device="cuda"), 40_000,
                            flags=lq.LQ_CHECK_KEYS)
    assert e.value.status == "LQ_ERR_WORKSPACE"
    np.testing.assert_array_equal(lq.lq_keymap_lookup(part, torch.from_numpy(key_R).cuda()).cpu().numpy(), fk_w)


# ---------------------------------------------------------------- 64-bit keys

def _keys64(seed, r, n, dense, miss=0.1):
    g = np.random.default_rng(seed)
    if dense:
        base = int(g.choice([-2**62, -7, 0, 10**15, 2**63 - 1 - 3 * r]))
        pool = base + g.permutation(int(r * 1.4) + 1).astype(np.int64)
    else:
        pool = np.unique(g.integers(-2**63 + 1, 2**63 - 1, size=int(r * 1.4) + 8, dtype=np.int64))
        g.shuffle(pool)
    key_S = pool[:r].copy()
    extra = pool[r:]
    key_R = g.choice(key_S, size=n)
    if len(extra) and n:
        m = g.random(n) < miss
        key_R[m] = g.choice(extra, size=int(m.sum()))
    return key_S, key_R


@pytest.mark.parametrize("dense", [True, False])
@pytest.mark.parametrize("r,n", [(1, 3), (9, 1_001), (2_556, 100_003), (30_000, 400_000), (200_000, 1_000_001)])
def test_int64_keys_match_algorithm_1(lq, r, n, dense):
    key_S, key_R = _keys64(r + n + dense, r, n, dense)
    fk_w, rows_w, cols_w = MJ.key_to_row(key_R, key_S)
    table = lq.lq_keymap64_build(torch.from_numpy(key_S).cuda(), flags=lq.LQ_CHECK_KEYS)
    assert _is_direct(table) == (dense and r > 1 or (r == 1))
    fk = lq.lq_keymap64_lookup(table, torch.from_numpy(key_R).cuda())
    rows, cols, nnz = lq.lq_compact_matches(fk)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(fk.cpu().numpy(), fk_w)
    m = int(nnz.item())
    assert m == len(rows_w)
    np.testing.assert_array_equal(rows[:m].cpu().numpy(), rows_w)
    np.testing.assert_array_equal(cols[:m].cpu().numpy(), cols_w)
    # unaligned key column: one key per thread
    kr = torch.empty(n + 1, dtype=torch.int64, device="cuda")
    kr[1:] = torch.from_numpy(key_R)
    np.testing.assert_array_equal(lq.lq_keymap64_lookup(table, kr[1:]).cpu().numpy(), fk_w)


def test_int64_extremes_duplicates_inserts_and_the_reserved_key(lq):
    key_S = np.array([2**63 - 1, -2**63 + 1, 0, -1, 1, 2**40], dtype=np.int64)
    key_R = np.array([0, -1, 2**63 - 1, -2**63 + 1, 5, 1, 2**40, -2**63], dtype=np.int64)
    table = lq.lq_keymap64_build(torch.from_numpy(key_S).cuda(), flags=lq.LQ_CHECK_KEYS)
    assert lq.lq_keymap64_lookup(table, torch.from_numpy(key_R).cuda()).cpu().tolist() == [2, 3, 0, 1, -1, 4, 5, -1]
    with pytest.raises(lq.LQError) as e:
        lq.lq_keymap64_build(torch.tensor([5, 9, 5, 2**50], dtype=torch.int64, device="cuda"), flags=lq.LQ_CHECK_KEYS)
    assert e.value.status == "LQ_ERR_DUPLICATE_KEY"
    with pytest.raises(lq.LQError) as e:
        lq.lq_keymap64_build(torch.tensor([-2**63, 2**62], dtype=torch.int64, device="cuda"), flags=lq.LQ_CHECK_KEYS)
    assert e.value.status == "LQ_ERR_UNSUPPORTED"
    # incremental update of a hashed and of a direct map
    for dense in (False, True):
        ks, kr = _keys64(77 + dense, 40_000, 300_000, dense, miss=0.2)
        part = lq.lq_keymap64_build(torch.from_numpy(ks[:25_000]).cuda(), max_keys=40_000)
        try:
            lq.lq_keymap64_insert(part, torch.from_numpy(ks[25_000:]).cuda(), 25_000, flags=lq.LQ_CHECK_KEYS)
        except lq.LQError as err:                       # a direct map may have to be rebuilt for keys outside its window
            assert dense and err.status == "LQ_ERR_WORKSPACE"
            part = lq.lq_keymap64_build(torch.from_numpy(ks).cuda(), flags=lq.LQ_CHECK_KEYS)
        fk_w, _, _ = MJ.key_to_row(kr, ks)
        np.testing.assert_array_equal(lq.lq_keymap64_lookup(part, torch.from_numpy(kr).cuda()).cpu().numpy(), fk_w)


@pytest.mark.parametrize("wide", [False, True])
@pytest.mark.parametrize("dense", [False, True])
@pytest.mark.parametrize("r", [1, 500, 2_000, 4_096, 4_097, 8_192])
def test_small_maps_in_lds(lq, r, dense, wide):
    """More than 2^20 fact keys: small maps are served from LDS, hashed ones spread over more slots there (500 and 2,000 keys;
    4,096 fill 8,192 slots half, 4,097 are past the 64-bit limit, 8,192 at the 32-bit one).  Whole numbers, exact."""
    g = np.random.default_rng(r + dense)
    n = (1 << 20) + 4 * r + 3
    dt = np.int64 if wide else np.int32
    key_S = (g.permutation(r) + 17).astype(dt) if dense else (g.permutation(8 * r + 40)[:r].astype(dt) * dt(1_000_003 if wide else 101))
    key_R = g.choice(np.concatenate([key_S, key_S + dt(1)]), size=n).astype(dt)
    order = np.argsort(key_S)
    at = np.minimum(np.searchsorted(key_S[order], key_R), r - 1)
    want = np.where(key_S[order][at] == key_R, order[at], -1)
    build, lookup = (lq.lq_keymap64_build, lq.lq_keymap64_lookup) if wide else (lq.lq_keymap_build, lq.lq_keymap_lookup)
    table = build(torch.from_numpy(key_S).cuda(), flags=lq.LQ_CHECK_KEYS)
    np.testing.assert_array_equal(lookup(table, torch.from_numpy(key_R).cuda()).cpu().numpy(), want)


@pytest.mark.parametrize("wide", [False, True])
@pytest.mark.parametrize("off", [0, 1])
@pytest.mark.parametrize("r", [9, 40_000, 262_144, 262_145, 600_000])
def test_hashed_maps_in_memory(lq, r, off, wide):
    """Hashed maps that lookups read in place: 2^19 slots (262,144 keys) and from 2^20 on, where a 32-bit path takes the neighbouring
    bucket first.  Keys of one common factor and -1, present and absent; columns at 16 bytes and one element past it, more
    than 2^20 fact keys and few; half of the dimension inserted later.  Whole numbers, exact."""
    g = np.random.default_rng(r + off)
    dt = np.int64 if wide else np.int32
    step = dt(1_000_003 if wide else 101)
    pool = np.unique(np.concatenate([g.permutation(8 * r)[:2 * r].astype(dt) * step, np.array([-1, -2, step + 1], dtype=dt)]))
    g.shuffle(pool)
    key_S = np.concatenate([pool[:r - 1][pool[:r - 1] != -1], np.array([-1], dtype=dt)])
    order = np.argsort(key_S)
    dev = lambda a: torch.from_numpy(np.concatenate([np.zeros(off, dtype=a.dtype), a])).cuda()[off:]
    build, insert, lookup = ((lq.lq_keymap64_build, lq.lq_keymap64_insert, lq.lq_keymap64_lookup) if wide else
                             (lq.lq_keymap_build, lq.lq_keymap_insert, lq.lq_keymap_lookup))
    half = len(key_S) // 2
    whole, grown = build(dev(key_S), flags=lq.LQ_CHECK_KEYS), build(dev(key_S[:half]), max_keys=r)
    insert(grown, dev(key_S[half:]), half, flags=lq.LQ_CHECK_KEYS)
    for n in ((1 << 20) + 1_027, 5_003):
        key_R = g.choice(pool, size=n)
        at = np.minimum(np.searchsorted(key_S[order], key_R), len(key_S) - 1)
        want = np.where(key_S[order][at] == key_R, order[at], -1)
        for table in (whole, grown):
            fk = torch.empty(n + off, dtype=torch.int32, device="cuda")[off:]
            np.testing.assert_array_equal(lookup(table, dev(key_R), fk=fk).cpu().numpy(), want)


@pytest.mark.parametrize("wide,r,spacing", [(False, 2_000, 1_000), (False, 2_000, 5_000), (False, 100_000, 16), (False, 100_000, 1_003),
                                            (False, 400_000, 101), (True, 2_000, 5_000), (True, 4_096, 101), (True, 400_000, 8)])
def test_evenly_spaced_keys_do_not_crowd(lq, r, spacing, wide):
    """Dimension keys at one spacing: exact, and map and 3e6 lookups take at most three times what as many scattered keys take
    (they take 0.9 to 1.3 times; a hash that lays spaced keys out unevenly takes 4 to 700 times)."""
    g = np.random.default_rng(r)
    dt = np.int64 if wide else np.int32
    build, lookup = (lq.lq_keymap64_build, lq.lq_keymap64_lookup) if wide else (lq.lq_keymap_build, lq.lq_keymap_lookup)
    scattered = torch.from_numpy((g.choice(2**31 - 1, size=r, replace=False) + 1).astype(dt)).cuda()
    spaced = torch.from_numpy(((g.permutation(r) + 1) * spacing).astype(dt)).cuda()
    row = torch.from_numpy(g.integers(0, r, 3_000_000)).cuda()
    fk = torch.empty(len(row), dtype=torch.int32, device="cuda")

    def fastest(call):
        times = []
        for _ in range(7):
            begin, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            begin.record()
            for _ in range(8):
                call()
            end.record()
            end.synchronize()
            times.append(begin.elapsed_time(end))
        return min(times)

    took = []
    for keys in (scattered, spaced):
        table, probe = build(keys, flags=lq.LQ_CHECK_KEYS), keys[row]
        assert torch.equal(lookup(table, probe, fk=fk).long(), row)
        took.append((fastest(lambda: build(keys)), fastest(lambda: lookup(table, probe, fk=fk))))
    (b0, l0), (b1, l1) = took
    assert b1 < 3 * b0 and l1 < 3 * l0, took
