"""A missing row of a query (None in the place of a component's array) reaches
the library as NULL, which refuses it by its own error code."""
import torch

from paper_2401_12724_amd import bysdf


def test_missing_row_is_null():
    a, b = torch.zeros(4), torch.zeros(4)
    assert bysdf._rows((a, None, b), 3) == [a.data_ptr(), None, b.data_ptr()]
    q = dict(type=torch.zeros(4, dtype=torch.int32), h=a, u=a, v=a, wi=(a, a, None), wo=(None, b, b), shift=(None, a))
    s = bysdf._qsoa(q)
    assert s.wi_z is None and s.wo_x is None and s.shift0 is None
    assert s.wi_x == a.data_ptr() and s.wo_y == b.data_ptr() and s.shift1 == a.data_ptr()
