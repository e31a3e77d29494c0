"""Packing of wall data from a user's function whose calls refill one list or one tensor."""
import ctypes

import pytest
import torch

from paper_2605_26677_amd.solver import EdgeData, call_edges, pack_edges


def _field(c, e, length):
    p = c.field[e]
    return torch.tensor((ctypes.c_double * (2 * length)).from_address(p)[:], dtype=torch.float64).view(2, length)


def _at(n):
    return torch.arange(10, dtype=torch.float64).view(2, 5) + 100.0 * n


def test_a_list_that_each_call_refills():
    data = [(0.0, 0.0)] * 4

    def edges(n):
        data[2] = (n, -n)
        return data
    keep = []
    for out in (call_edges(edges, range(3, 9), keep), pack_edges(map(edges, range(3, 9)), keep, 6)):
        for i in range(6):
            assert tuple(out[i].value[2]) == (3.0 + i, -3.0 - i) and tuple(out[i].value[0]) == (0.0, 0.0)


@pytest.mark.parametrize("buffers", [1, 2, 3])
@pytest.mark.parametrize("how", ["tensor", "data", "view", "float32", "strided"])
def test_tensors_that_the_calls_refill(buffers, how):
    """One buffer or a few in turn, filled in place by any means, whole, as a view, in another
    type or layout."""
    dtype = torch.float32 if how == "float32" else torch.float64
    bufs = [torch.empty((5, 2), dtype=dtype).t() if how == "strided" else torch.empty((2, 5), dtype=dtype)
            for _ in range(buffers)]

    def edges(n):
        b = bufs[n % buffers]
        if how == "data":
            b.data.copy_(_at(n))
        else:
            b.copy_(_at(n))
        return [None, b.view(2, 5) if how == "view" else b, (1.0, n), None]
    keep = []
    out = call_edges(edges, range(12, 4, -1), keep)
    for i, n in enumerate(range(12, 4, -1)):
        assert torch.equal(_field(out[i], 1, 5), _at(n))
        assert tuple(out[i].value[2]) == (1.0, float(n)) and not out[i].field[0]


def test_fresh_tensors_are_neither_copied_nor_asked_for_twice():
    made, calls = [_at(n) for n in range(8)], []

    def edges(n):
        calls.append(n)
        return [made[n], made[n], None, None]
    keep = []
    out = call_edges(edges, range(8), keep)
    assert calls == list(range(8))
    assert [out[i].field[0] for i in range(8)] == [t.data_ptr() for t in made]


def test_edge_data_objects_keep_their_tensors():
    keep = []
    out = pack_edges(map(lambda n: EdgeData([None, _at(n).float(), (n, 2.0), None]), range(4)), keep, 4)
    for i in range(4):
        assert torch.equal(_field(out[i], 1, 5), _at(i)) and tuple(out[i].value[2]) == (float(i), 2.0)
