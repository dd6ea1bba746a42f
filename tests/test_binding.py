"""The binding's argument structs field by field, without a GPU."""
from types import SimpleNamespace

import numpy as np
import pytest

from paper_2205_05836_amd import _lib, api


@pytest.mark.parametrize("subs", [
    [(3, [0, -1, -1], [-1, -1, 1]), (2, [1, -1], [-1, 0])], [(0, [], [])], [(1, [-1], [0]), (0, [], [])],
    [SimpleNamespace(width=2, init_cut=np.array([-1, 0]), meas_cut=(-1, -1))], []])
def test_subcircuit_structs(subs):
    s = api._Subs(subs)
    assert len(s.arr) == len(subs)
    for i, sub in enumerate(subs):
        w, ic, mc = sub if isinstance(sub, tuple) else (sub.width, sub.init_cut, sub.meas_cut)
        c = s.ptr(i)[0]
        assert c.width == w and c.init_cut[:w] == list(ic) and c.meas_cut[:w] == list(mc)
        assert s.n_out[i] == list(mc).count(-1)


def test_cut_list_longer_than_the_register_is_refused():
    with pytest.raises(IndexError):
        api._Subs([(2, [-1, -1, 0], [-1, -1])])


def test_gate_structs():
    """Matrices as nested lists, tuples, arrays of any number type, and larger
    ones (their leading 2 x 2 block), alone and mixed."""
    u = [[[0.5, 1j], [2 - 1j, -3]], ((1, 2), (3, 4)), np.eye(2, dtype=np.float32), np.arange(9).reshape(3, 3),
         np.array([[1, 1j], [1j, 1]], dtype=np.complex64)]
    for mats in (u, u[:1], u[4:], u[:3], []):
        ops = [("cz", 4, 1)]
        for i, m in enumerate(mats):
            ops += [("u", np.int64(i), m), SimpleNamespace(name="cz", qubits=(i, i + 1), matrix=None)]
        arr, n = api._gates(ops)
        assert n == len(ops)
        for g, op in zip(arr, ops):
            if isinstance(op, tuple) and op[0] == "u":
                want = [complex(op[2][r][c]) for r in range(2) for c in range(2)]
                assert (g.kind, g.q0) == (_lib.GATE_U, op[1])
                assert list(g.u) == [x for z in want for x in (z.real, z.imag)]
            else:
                q = op[1:] if isinstance(op, tuple) else op.qubits
                assert (g.kind, g.q0, g.q1) == (_lib.GATE_CZ, *q)
    assert api._gates([])[1] == 0
    with pytest.raises(ValueError):
        api._gates([("cx", 0, 1)])


class Rows:
    """Indexable as matrix[r][c], and nothing an array can be made of."""

    def __init__(self, m):
        self.m = m

    def __getitem__(self, r):
        return self.m[r]


class Columns:
    """matrix[r][c] is the element in row r and column c, the array form its
    transpose (as of a table whose columns are indexed first)."""

    def __init__(self, m):
        self.m = np.array(m)

    def __getitem__(self, r):
        return list(self.m[r])

    def __array__(self, dtype=None, copy=None):
        return self.m.T.astype(dtype)


def tensors():
    import torch
    m = torch.tensor([[0.5, 1j], [2 - 1j, -3]], dtype=torch.complex128)
    return [m, m.conj(), m.mH, m.clone().requires_grad_(), m.real, torch.eye(3)]


def test_gate_matrices_are_read_by_element():
    """Anything indexable as matrix[r][c] gives the elements that indexing
    gives, whatever an array made of it would hold or refuse."""
    m = [[0.5, 1j], [2 - 1j, -3]]
    for u in [Rows(m), Columns(m), {0: {0: 1, 1: 2}, 1: {0: 3, 1: 4}}, [["1", "2j"], ["3", "4"]],
              [list(row) for row in tensors()[3]]] + tensors():
        for ops in ([("u", 0, u)], [("u", 0, np.eye(2)), ("u", 1, u)], [("u", 0, u), ("u", 1, m)]):
            arr, n = api._gates(ops)
            for g, op in zip(arr, ops):
                want = [complex(op[2][r][c]) for r in range(2) for c in range(2)]
                assert list(g.u) == [x for z in want for x in (z.real, z.imag)]


@pytest.mark.parametrize("q,stored", [(2 ** 31 - 1, 2 ** 31 - 1), (2 ** 31, -2 ** 31), (2 ** 32, 0), (-2 ** 40 - 1, -1)])
def test_numbers_beyond_32_bits_are_left_to_the_library(q, stored):
    """Stored modulo 2^32, as a C field of a ctypes struct is, and judged by
    the entry point."""
    s = api._Subs([(2, [q, -1], [-1, q])])
    c = s.ptr(0)[0]
    assert (c.init_cut[0], c.init_cut[1], c.meas_cut[0], c.meas_cut[1]) == (stored, -1, -1, stored)
    arr, _ = api._gates([("u", q, np.eye(2)), ("cz", 0, q)])
    assert (arr[0].q0, arr[1].q1) == (stored, stored)
