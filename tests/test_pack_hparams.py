"""The native conversion of suggestions to records against the Python one, field by field."""
import collections

import numpy as np
import pytest

from paper_2012_04201_amd import binding as bb

FULL = {"hidden": [3, 70000], "solver": "sgd", "nesterov": True, "batch_size": 7, "epochs": 9, "lr": 0.1, "alpha": 1,
        "momentum": 0.5, "beta1": 0.8, "beta2": 0.7, "eps": 0, "seed": 2 ** 64 - 1, "power_t": 0.25, "tol": 1e-4,
        "n_iter_no_change": 3, "validation_fraction": 0.2}
ODD = [{}, FULL, dict(FULL, hidden=()), dict(FULL, hidden=(5, 4, 3, 2, 1)), dict(FULL, hidden=np.array([4, 5])),
       dict(FULL, hidden=[np.int64(6)]), dict(FULL, solver="adam", nesterov=0), dict(FULL, seed=-1), dict(FULL, seed=np.uint64(2 ** 63)),
       dict(FULL, batch_size=3.9, lr=np.float32(0.3), epochs=np.int32(4)), dict(FULL, lr=float("inf"), alpha=True),
       dict(FULL, batch_size=2 ** 35 + 5, epochs=-2), collections.OrderedDict(FULL), dict(FULL, tol="1e-3"), {"solver": "rmsprop"},
       {"".join(["l", "r"]): 0.5, "name": "extra"}, {"name": 1, 5: 2, "lr": 0.5}]


@pytest.mark.parametrize("wrap", [list, tuple, collections.deque])
def test_records_are_those_of_the_python_conversion(wrap):
    want = (bb.HParams * len(ODD))()
    for h, d in zip(want, ODD):
        bb._set_hparams(h, d)
    got = bb.make_hparams(wrap(ODD))
    for i in range(len(ODD)):
        for name, _ in bb.HParams._fields_:
            a, b = getattr(got[i], name), getattr(want[i], name)
            assert (list(a), name) == (list(b), name) if name == "hidden" else (a, name) == (b, name), (i, name)


@pytest.mark.parametrize("bad", [{"lr": None}, {"hidden": 3}, {"batch_size": "x"}, None, {"lr": 10 ** 400}])
def test_what_is_no_suggestion_is_still_an_error(bad):
    with pytest.raises((TypeError, ValueError, AttributeError, OverflowError)):
        bb.make_hparams([FULL, bad, FULL])
