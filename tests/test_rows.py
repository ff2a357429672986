"""Row pointers of the ctypes binding against views of the same tensors."""
import pytest
import torch

from paper_2401_12724_amd import bysdf


@pytest.mark.parametrize("make", [
    lambda: torch.zeros(12, 7),
    lambda: torch.zeros(12, 0),
    lambda: torch.zeros(14, 9)[1:, 2:],
    lambda: torch.zeros(30, 5)[::2],
    lambda: torch.zeros(5).expand(12, 5),
    lambda: torch.zeros(12),
    lambda: torch.zeros(12, 3, dtype=torch.float64),
    lambda: [torch.zeros(4) for _ in range(12)],
    lambda: tuple(torch.zeros(12, 4)),
])
def test_rows_match_views(make):
    t = make()
    assert bysdf._rows(t, 12) == [t[i].data_ptr() for i in range(12)]


@pytest.mark.parametrize("make", [lambda: torch.zeros(11, 4), lambda: torch.zeros(()),
                                  lambda: [torch.zeros(4)] * 11])
def test_rows_refuses_what_views_refuse(make):
    with pytest.raises(IndexError):
        bysdf._rows(make(), 12)
