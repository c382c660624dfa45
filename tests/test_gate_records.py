"""Gate and Pauli-term records in every form of number that a caller may hold
(numpy integers and arrays, tensors, numbers past 32 bits), as ctypes fields
take them one at a time (no GPU)."""
from fractions import Fraction

import numpy as np
import pytest
import torch

import paper_2503_19894_amd as cast
from circuits import Gate, PauliTerm


def _record(gates):
    a = cast.GateArray(gates)
    return [(a.arr[i].k, list(a.arr[i].qubits), a.arr[i].param_id, a.arr[i].param_coeff) for i in range(a.n)]


@pytest.mark.parametrize("to_int", [int, np.int8, np.int32, np.int64, np.uint8])
def test_pauli_terms_take_numpy_qubits(to_int):
    terms = cast.pauli_terms([PauliTerm(0.5, ((to_int(3), "X"), (to_int(1), "Y"), (to_int(5), "Z")))])
    assert (terms[0].coeff, terms[0].xmask, terms[0].zmask) == (0.5, 0b1010, 0b100010)


def test_pauli_terms_take_high_numpy_qubits():
    terms = cast.pauli_terms([PauliTerm(1.0, ((np.int64(33), "X"), (np.int64(2), "Z")))])
    assert (terms[0].xmask, terms[0].zmask) == (1 << 33, 4)


@pytest.mark.parametrize("angle", [[np.array(0.3)], np.array([0.3]), torch.tensor([0.3], dtype=torch.float64),
                                   [torch.tensor(0.3, dtype=torch.float64)]], ids=["0-d", "1-d", "tensor", "0-d tensor"])
def test_angles(angle):
    a = cast.GateArray([Gate("ry", (0,), angle), Gate("ry", (1,), angle)])
    want = cast.std_matrix("ry", (0.3,)).reshape(-1)
    for i in range(2):
        assert [a.arr[i].matrix[j] for j in range(8)] == list(want)


@pytest.mark.parametrize("coeff", [1.5, "1.5", Fraction(3, 2), np.float32(1.5), np.array(1.5), torch.tensor(1.5),
                                   torch.tensor([1.5])])
def test_coefficients(coeff):
    assert _record([Gate("ry", (2,), param=0, coeff=coeff), Gate("rz", (1,), param=1)]) == [
        (1, [2, 0, 0, 0, 0, 0], 0, 1.5), (1, [1, 0, 0, 0, 0, 0], 1, 1.0)]


@pytest.mark.parametrize("coeff", [None, 1j, "x"])
def test_coefficients_refused(coeff):
    with pytest.raises((TypeError, ValueError)):
        cast.GateArray([Gate("ry", (0,), param=0, coeff=coeff)])


def test_integers_keep_their_low_32_bits():
    assert _record([Gate("ry", (2 ** 70 + 1,), param=2 ** 40 + 5), Gate("ry", (-1,), param=np.int64(3)),
                    Gate("ry", (2.7,), param=3.9)]) == [
        (1, [1, 0, 0, 0, 0, 0], 5, 1.0), (1, [-1, 0, 0, 0, 0, 0], 3, 1.0), (1, [2, 0, 0, 0, 0, 0], 3, 1.0)]


def test_at_most_six_qubits():
    with pytest.raises(IndexError):
        cast.GateArray([Gate("unitary", tuple(range(7)), matrix=np.eye(128))])
