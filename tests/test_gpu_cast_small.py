"""The one-workgroup cast (up to 8192 pairs) at the sizes where its code
changes, against the CPU oracle, every index bit for bit: pair counts around
whole trips of its 1024 threads, digits of every width, empty bags before,
between and after the others and more bags than it has threads for, and the
tables' row offsets in and beyond its LDS."""
import numpy as np
import pytest

from tests.test_gpu_cast_layouts import check, gpu_cast, oracle_cast

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("pairs", [1, 63, 64, 65, 1023, 1024, 1025, 2049, 5120, 7169, 8191, 8192])
def test_pair_counts(pairs):
    check(f"{pairs} pairs", [100_000], [pairs], bags_per_table=max(1, pairs // 20), seed=pairs,
          bounds=[0])


@pytest.mark.parametrize("bits", [1, 3, 8, 10, 11, 12, 17, 21, 22, 23, 28])
def test_digit_widths(bits):
    check(f"{bits} bits", [2 ** bits], [3001], bags_per_table=41, seed=bits, bounds=[0])


def csr_check(table_rows, lengths, bags_per_table, seed):
    rng = np.random.default_rng(seed)
    off = np.concatenate([[0], np.cumsum(table_rows)]).astype(np.int64)
    bo = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    rows = np.repeat(np.repeat(np.asarray(table_rows), bags_per_table), lengths)
    idx = (rng.random(bo[-1]) * rows).astype(np.int32)
    ref, got = oracle_cast(off, bo, idx, bags_per_table), gpu_cast(off, bo, idx, bags_per_table, 0)
    assert got["num_unique"] == ref["num_unique"]
    for k in ("unique_rows", "seg_offsets", "casted_src", "casted_dst"):
        assert np.array_equal(got[k], ref[k][:len(got[k])]), k


@pytest.mark.parametrize("tables,bags", [(1, 40), (7, 1171), (3, 5000), (130, 63), (20_000, 1),
                                         (40_000, 3)])
def test_bags_and_tables(tables, bags):
    rng = np.random.default_rng(bags)
    lengths = np.where(rng.random(tables * bags) < min(0.5, 3000 / (tables * bags)),
                       rng.integers(1, 4, tables * bags), 0)
    lengths[:5] = lengths[-5:] = 0
    assert 0 < lengths.sum() <= 8192
    csr_check([1 + 3 * (k % 50) for k in range(tables)], lengths, bags, bags)
