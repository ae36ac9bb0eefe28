"""CPU test of the binding's argument marshalling: weight tables in every form callers pass them in."""
import numpy as np
import pytest

import paper_1907_02818_amd as lib

TABLE = [[[float(9 * i + 3 * j + k) - 13.5 for k in range(3)] for j in range(3)] for i in range(3)]


@pytest.mark.parametrize("form", ["list", "tuple", "array", "f32", "transposed", "tensor", "rows of arrays", "flat", "ints"])
def test_weight_tables_flatten_in_order(form):
    import torch
    a = np.array(TABLE)
    w = {"list": TABLE, "tuple": tuple(tuple(tuple(r) for r in p) for p in TABLE), "array": a, "f32": a.astype(np.float32),
         "transposed": np.ascontiguousarray(a.transpose(2, 1, 0)).transpose(2, 1, 0), "tensor": torch.tensor(TABLE),
         "rows of arrays": [[np.array(r) for r in p] for p in TABLE], "flat": a.ravel().tolist(),
         "ints": np.arange(27).reshape(3, 3, 3)}[form]
    want = list(range(27)) if form == "ints" else a.ravel().tolist()
    assert [float(v) for v in lib._flatten(w)] == want


def test_scalars_and_empty_tables_flatten():
    assert lib._flatten(2.5) == [2.5] and lib._flatten(np.float32(2.5)) == [2.5]
    assert lib._flatten([]) == [] and lib._flatten([[], [1]]) == [1]
