"""Host integers handed to the library: arrays that go over as one copy give the same words as
numbers converted one by one."""
import numpy as np
import pytest

from paper_2406_17404_amd import binding as b


@pytest.mark.parametrize("values", [
    np.arange(-5, 1000, dtype=np.int32), np.arange(7, dtype=np.int64), np.arange(40, dtype=np.int32)[3::7],
    np.arange(40, dtype=np.int32)[::-1], np.array([2**31 - 1, -2**31], np.int64), np.array([2**32 + 5, -1], np.int64),
    np.arange(5, dtype=np.int32).astype(">i4"), np.array([1.9, -2.9]), np.array([3], np.uint8),
    np.zeros(0, np.int32), np.array([True, False]), [1, 2, 3], (4,), [], range(5), [np.int32(7), 8.7]],
    ids=lambda v: f"{type(v).__name__}-{getattr(v, 'dtype', '')}-{len(v)}")
def test_same_words(values):
    buf, n = b._host_i32(values)
    one_by_one = [int(v) for v in values]
    want = [((v + 2**31) % 2**32) - 2**31 for v in one_by_one]
    assert n == len(one_by_one) and list(buf)[:n] == want and len(buf) == max(1, n)


def test_the_copy_is_the_callees_own():
    a = np.arange(4, dtype=np.int32)
    buf, _ = b._host_i32(a)
    a[0] = 99
    assert buf[0] == 0


def test_other_one_dimensional_arrays_go_number_by_number():
    """What only looks like a numpy array (pandas' Series and Index have its ndim and dtype) is taken
    as before, and a masked array with a masked number in it is refused as before."""
    pd = pytest.importorskip("pandas")
    for values in (pd.Series([3, 1, 2]), pd.Series([3, 1, 2], index=[7, 8, 9]), pd.Index([4, 5]),
                   pd.Series(np.array([1, 2], np.int32)), np.ma.MaskedArray([1, 2, 3])):
        buf, n = b._host_i32(values)
        assert n == len(values) and list(buf) == [int(v) for v in values]
    with pytest.raises(Exception):
        b._host_i32(np.ma.MaskedArray([1, 2, 3], mask=[0, 1, 0]))
