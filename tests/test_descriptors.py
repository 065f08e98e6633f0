"""The descriptor arrays of the C ABI as the native helper fills them and as the interpreter does (CPU tensors: only addresses,
sizes and dtypes are read)."""
import ctypes as C

import pytest
import torch

from paper_2605_26842_amd import binding as B

F, H = torch.float32, torch.bfloat16


def by_hand(kind, params, grads):
    """What the interpreter's loop makes of the same tensors."""
    out = (kind * len(params))()
    for a, w, g in zip(out, params, grads):
        a.w, a.g = w.data_ptr(), g.data_ptr()
        a.w_dtype, a.g_dtype = B._dtype_code(w.dtype), B._dtype_code(g.dtype)
        if kind is B.mona_vector:
            a.n = w.numel()
        else:
            a.m, a.n = w.shape
    return bytes(out)


@pytest.mark.parametrize("as_list", [list, tuple])
def test_filled_like_by_hand(as_list):
    shapes = [(3, 5), (1, 1), (70, 1), (1, 64), (128, 256)]
    for wd, gd in ((F, F), (H, F), (H, H), (F, H)):
        w = as_list(torch.zeros(s, dtype=wd) for s in shapes)
        g = as_list(torch.zeros(s, dtype=gd) for s in shapes)
        assert bytes(B.make_matrices(w, g)) == by_hand(B.mona_matrix, w, g)
        assert bytes(B.make_vectors(w, g)) == by_hand(B.mona_vector, w, g)
        arr = (C.c_void_p * len(w))()
        code = B._dtype_code(gd)
        assert B._load_helper().mona_fill_slots(w, g, len(w), code, C.addressof(arr)) == 1
        assert list(arr) == [t.data_ptr() for t in g]
        assert B._load_helper().mona_fill_slots(w, g, len(w), 1 - code, C.addressof(arr)) == 0
    # parameters, views into a larger array, a dimension more
    p = [torch.nn.Parameter(torch.zeros(4, 6)), torch.zeros(10, 8)[2:7], torch.zeros(0, 3)]
    g = [torch.zeros(4, 6), torch.ones(5, 8), torch.zeros(0, 3)]
    assert bytes(B.make_matrices(p, g)) == by_hand(B.mona_matrix, p, g)
    v = [torch.zeros(2, 3, 4), torch.zeros(())]
    assert bytes(B.make_vectors(v, v)) == by_hand(B.mona_vector, v, v)


def test_refused_as_before():
    w = [torch.zeros(4, 6), torch.zeros(8, 2)]
    for make in (B.make_matrices, B.make_vectors):
        for bad in (torch.zeros(6, 4), torch.zeros(6, 4).t(), torch.zeros(24), torch.zeros(4, 12)[:, ::2]):
            with pytest.raises(ValueError):
                make(w, [bad, w[1]])
        with pytest.raises(TypeError):
            make(w, [w[0].double(), w[1]])
        with pytest.raises(IndexError):
            make(w, w[:1])
        with pytest.raises(ValueError):
            make([torch.zeros(6, 4).t()], [torch.zeros(4, 6)])
        assert len(make(w, w + w)) == 2                       # gradients beyond the parameters are not looked at
    with pytest.raises(ValueError):
        B.make_matrices([torch.zeros(4)], [torch.zeros(4)])
    with pytest.raises(AttributeError):
        B.make_vectors([torch.zeros(4)], [3.0])
