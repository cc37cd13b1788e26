"""The binding's per-call marshalling against its ctypes form (CPU only):
every form of ids and groups that the one takes, the other takes with the same
values, and what one refuses the other refuses."""
import ctypes

import numpy as np
import pytest

import paper_1909_08029_amd as rip


def _read(addr, n):
    return list((ctypes.c_int32 * n).from_address(addr))


@pytest.mark.parametrize("ids", [[], [0], [3, 1, 2], (5, 7), range(4), np.array([2, 9]),
                                 [np.int64(4), True], [2 ** 31 - 1, -1], [2 ** 32 + 1, 2 ** 31]])
def test_ids(ids):
    want = rip._i32_array(list(ids))
    addr, keep = rip._i32_call(list(ids))
    assert _read(addr, max(1, len(ids))) == list(want)


@pytest.mark.parametrize("ids", [[1.0], ["1"], [None]])
def test_refused_ids(ids):
    for f in (rip._i32_array, rip._i32_call):
        with pytest.raises(TypeError):
            f(ids)


@pytest.mark.parametrize("groups", [
    lambda: [], lambda: [()], lambda: [(0, 1), [2, 3, 4]], lambda: [np.array([1, 5]), range(6, 9)],
    lambda: [(i for i in (3, 4)), (0,)], lambda: [(1.0, 2.0), "34"],
    lambda: [(float(i) for i in (3, 4))], lambda: [(2 ** 32 + 3,), (1,)]])
def test_groups(groups):
    off, mem = rip._csr(groups())
    o, m, keep = rip._csr_call(groups())
    assert _read(o, len(off)) == list(off)
    assert _read(m, len(mem)) == list(mem)


def test_refused_groups():
    for f in (rip._csr, rip._csr_call):
        with pytest.raises((TypeError, ValueError)):
            f([("x",)])
