"""Which models the full-batch kernel takes (no GPU needed: on the recording runtime, which names the kernels launched)."""
import re

import pytest

from test_full_batch_kernel import SHAPES
from test_host_launches import child  # noqa: F401


def kernels(child, n, d, c, shapes, batch):  # noqa: F811
    """[(kernel, its template arguments)] of a call's training launches, and the class that the library names for the first model."""
    names, cls = child("""
        n, d, c, shapes, batch = %r
        rc = L.bbo_mlp_cv_eval(P(4096), P(4096), C.c_int64(n), d, c, P(4096), 5, records(shapes, batch), len(shapes), 0, P(4096),
                               P(4096), P(0), P(4096), C.c_size_t(1 << 40), P(900))
        assert rc == 0
        print(json.dumps([[l[5] for l in log() if l[0] == "launch"],
                          L.bbo_mlp_kernel_class(C.c_int64(n), d, c, records(shapes, batch), 0)]))
    """ % ((n, d, c, shapes, batch),))
    found = [re.match(r"_ZN\S*?(k_train\w*?)I((?:Li\d+E)+)E", x) for x in names]
    return [(m.group(1), tuple(int(v) for v in re.findall(r"Li(\d+)E", m.group(2)))) for m in found if m], cls


@pytest.mark.parametrize("n,d,c,h", SHAPES)
def test_the_shapes_of_its_tests_reach_the_kernel(child, n, d, c, h):  # noqa: F811
    """All but the last three of them, with the batch size 0, n or more; none with a row less."""
    other = (n, d, c, h) in SHAPES[-3:]
    for batch in (0, n, 2 * n):
        found, cls = kernels(child, n, d, c, [[h]], batch)
        assert [k for k, _ in found] == ["k_train_small" if other else "k_train_full"] and cls == 1
        if not other:
            assert found[0][1] == (d // 16 + 1, -(-h // 16), max(c, 1), 4 if n <= 80 else 8)
    found, cls = kernels(child, n, d, c, [[h]], n - 1)
    assert [k for k, _ in found] == ["k_train_small"] and cls == 1


def test_few_models_of_several_widths_share_a_launch(child):  # noqa: F811
    shapes = [[8], [16], [17], [32], [40], [48], [5]]
    assert kernels(child, 150, 6, 2, shapes, 0)[0] == [("k_train_full", (1, 3, 2, 8))]
    assert sorted(kernels(child, 150, 6, 2, shapes * 20, 0)[0]) == [("k_train_full", (1, t, 2, 8)) for t in (1, 2, 3)]


def test_every_compiled_variant_is_reached(child):  # noqa: F811
    compiled, launched = child("""
        rt.hr_kernel.restype = C.c_char_p
        compiled, i = [], 0
        while rt.hr_kernel(i):
            compiled.append(rt.hr_kernel(i).decode())
            i += 1
        launched = []
        for n in (20, 120, 400):
            for d in (3, 20):
                for h in (9, 25, 41, 57):
                    for c in (1, 2, 3, 4):
                        rc = L.bbo_mlp_cv_eval(P(4096), P(4096), C.c_int64(n), d, c, P(4096), 5, records([[h]], 0), 1, 0, P(4096),
                                               P(4096), P(0), P(4096), C.c_size_t(1 << 40), P(900))
                        launched += [l[5] for l in log() if l[0] == "launch"]
        print(json.dumps([compiled, launched]))
        """)
    full = {x for x in compiled if "k_train_full" in x}
    assert len(full) == 44 and full == {x for x in launched if "k_train_full" in x}
