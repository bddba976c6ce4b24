"""Workspace sizes of pauli_workspace_query, which runs on the host alone.  CPU only."""
import ctypes

import pytest

from paper_2410_09654_amd import _lib


@pytest.fixture(scope="module")
def query():
    L = _lib.load()

    def q(op, *sizes, n=64):
        ops = [_lib.PauliOpC(n, _lib.PAULI_C128, m, m, None, None, None) for m in sizes]
        ops = [ctypes.byref(o) for o in ops] + [None] * (3 - len(ops))
        nb, cap = ctypes.c_size_t(0), ctypes.c_int64(0)
        assert L.pauli_workspace_query(op, *ops, None, ctypes.byref(nb), ctypes.byref(cap)) == 0
        return nb.value

    return q


# H = 150 has its 14 tiles of O shared out over H, H = 15 has 140 tiles of its own; both make the
# same pairs, beside 116 rows of O_prev.  What is left is H itself and the margins of the bins
def test_shared_tiles_take_no_more_scratch(query):
    shared = query(_lib.PAULI_Q_LANCZOS, 150, 14 * 1024, 116 * 1024)
    alone = query(_lib.PAULI_Q_LANCZOS, 15, 140 * 1024, 116 * 1024)
    assert abs(shared - alone) < 1 << 16


# sizes that programs have been given for these calls still hold them
@pytest.mark.parametrize("n,sizes,nbytes", [(64, (100, 16000, 300000), 160565504),
                                            (64, (191, 1 << 20), 20348852224)])
def test_scratch_has_not_grown(query, n, sizes, nbytes):
    op = _lib.PAULI_Q_LANCZOS if len(sizes) == 3 else _lib.PAULI_Q_COMMUTATOR
    assert query(op, *sizes, n=n) <= nbytes
