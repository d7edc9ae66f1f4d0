"""Array inputs that the Python binding takes (CPU only)."""
import numpy as np
import pytest


@pytest.mark.parametrize("form", ["list", "scalar", "0-d", "1-d", "strided", "float64", "byte-swapped", "read-only"])
def test_query_plan_takes_any_array_form(form):
    import paper_2606_26441_amd as gs
    base = [np.array([v], np.float32) for v in (1.5, 2.0, 0.25)]
    make = {
        "list": lambda a: a.tolist(),
        "scalar": lambda a: float(a[0]),
        "0-d": lambda a: np.array(a[0], np.float32),
        "1-d": lambda a: a,
        "strided": lambda a: np.repeat(a, 2)[::2],
        "float64": lambda a: a.astype(np.float64),
        "byte-swapped": lambda a: a.astype(a.dtype.newbyteorder()),
        "read-only": lambda a: np.frombuffer(a.tobytes(), np.float32),
    }[form]
    assert gs.query_plan_host("fp32", *[make(a) for a in base]) == gs.query_plan_host("fp32", *base)
