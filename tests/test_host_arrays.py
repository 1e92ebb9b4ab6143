"""Host arrays of the binding: every form of argument gives numpy's int32 or
int64 contents, or numpy's error."""
import ctypes as C

import numpy as np
import pytest
import torch

gs = pytest.importorskip("paper_2108_12430_amd.gwstream")

FORMS = {
    "list": [3, -1, 2**31 - 1],
    "one": [7],
    "numpy ints": list(np.arange(5)),
    "bools": [True, False],
    "floats": [1.7, -2.9],
    "mixed": [1, np.float64(2.5)],
    "tuple": (4, 5, 6),
    "range": range(6),
    "int64 array": np.arange(9),
    "int32 array": np.arange(9, dtype=np.int32),
    "strided": np.arange(20)[::3],
    "reversed": np.arange(7)[::-1],
    "columns": np.arange(12).reshape(3, 4).T,
    "float array": np.array([1.5, 2.5]),
    "tensor": torch.arange(4),
    "list of tensors": [torch.tensor(3), torch.tensor(4)],
    "nested": [[1, 2], [3, 4]],
    "empty": [],
}


@pytest.mark.parametrize("fn,dtype", [(gs._host_i32, np.int32), (gs._host_i64, np.int64)])
@pytest.mark.parametrize("form", FORMS)
def test_host_array_matches_numpy(form, fn, dtype):
    want = np.ascontiguousarray(np.asarray(FORMS[form], dtype=dtype))
    keep, addr = fn(FORMS[form])
    assert len(keep) == len(want)
    if want.size:
        got = np.frombuffer(C.string_at(addr, want.nbytes), dtype=dtype)
        np.testing.assert_array_equal(got, want.reshape(-1))


@pytest.mark.parametrize("bad,error", [([2**31], OverflowError), (["x"], ValueError), ([None], TypeError),
                                       ([[1], [2, 3]], ValueError)])
def test_host_array_refuses_what_numpy_refuses(bad, error):
    with pytest.raises(error):
        np.asarray(bad, dtype=np.int32)
    with pytest.raises(error):
        gs._host_i32(bad)
