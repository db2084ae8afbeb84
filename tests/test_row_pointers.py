"""The pointer structures of the C ABI from tensors of rows, rows of any stride, and
sequences of row tensors (CPU only: addresses, no device work)."""

import ctypes as C

import pytest
import torch

from paper_1901_08532_amd import h6


def _words(st):
    return list((C.c_uint64 * (C.sizeof(st) // 8)).from_buffer_copy(st))


def _rows(n_rows, dtype=torch.float64):
    whole = torch.zeros((2 * n_rows, 7), dtype=dtype)
    return {"tensor": whole[:n_rows].clone(), "strided": whole[::2], "one row": torch.zeros(7, dtype=dtype).expand(n_rows, 7),
            "tuple": tuple(torch.zeros(7, dtype=dtype) for _ in range(n_rows)),
            "list": [torch.zeros(5 + k, dtype=dtype) for k in range(n_rows)]}


@pytest.mark.parametrize("form", ["tensor", "strided", "one row", "tuple", "list"])
def test_pointers(form):
    S, T, P = _rows(18)[form], _rows(2, torch.int64)[form], _rows(9)[form]
    m = torch.zeros(7, dtype=torch.float64)
    want = [S[k].data_ptr() for k in range(18)] + [m.data_ptr()] + [T[k].data_ptr() for k in range(2)]
    assert _words(h6.make_state(S, m, T)) == want
    assert _words(h6.make_state(S, m, None)) == want[:19] + [0, 0]
    assert _words(h6.make_pred(P)) == _words(h6.make_force(P)) == [P[k].data_ptr() for k in range(9)]


def test_too_few_rows():
    for rows in (torch.zeros(8, 4), [torch.zeros(4)] * 8):
        with pytest.raises(IndexError):
            h6.make_pred(rows)
