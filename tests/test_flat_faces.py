"""The flattening of a list of faces into offsets and int32 indices: every kind of entry that int() takes, and an index
beyond int32 refused whatever it is held in (a 0-dim numpy array is cast by numpy, not checked)."""
import numpy as np
import pytest
import torch

from paper_2104_08309_amd.api import _flat_faces


@pytest.mark.parametrize("entry", [3, np.int64(3), np.uint8(3), 3.7, np.float32(3.2), np.array(3), np.array(3.0),
                                   torch.tensor(3), torch.tensor([3]), "3"])
def test_entries(entry):
    off, flat = _flat_faces([[0, 1, 2, entry], [4, 5, 6]])
    assert off.dtype == np.int64 and off.tolist() == [0, 4, 7]
    assert flat.dtype == np.int32 and flat.tolist() == [0, 1, 2, 3, 4, 5, 6]


def test_containers_and_negative():
    for faces in ([(0, 1, -1), (2, 3, 4)], np.array([[0, 1, -1], [2, 3, 4]]), torch.tensor([[0, 1, -1], [2, 3, 4]]),
                  [np.array([0, 1, -1]), range(2, 5)]):
        assert _flat_faces(faces)[1].tolist() == [0, 1, -1, 2, 3, 4]
    off, flat = _flat_faces([])
    assert off.tolist() == [0] and flat.size == 0


@pytest.mark.parametrize("entry", [2 ** 31, -2 ** 31 - 1, 2 ** 70, np.int64(2 ** 33 + 1), np.array(2 ** 33 + 1),
                                   np.array(2.0 ** 33), np.uint64(2 ** 64 - 1), np.array(2 ** 64 - 1, dtype=np.uint64),
                                   torch.tensor(2 ** 33 + 1)])
def test_beyond_int32(entry):
    with pytest.raises(OverflowError):
        _flat_faces([[0, 1, 2], [3, 4, entry]])


@pytest.mark.parametrize("entry", [float("nan"), np.array(float("nan"))])
def test_not_a_number(entry):
    with pytest.raises(ValueError):
        _flat_faces([[0, 1, entry]])
