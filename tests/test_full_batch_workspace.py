"""Workspace of the kernel for full batches (no GPU needed: on the recording runtime)."""
from test_host_launches import child  # noqa: F401


def test_a_workspace_made_for_full_batches_holds_the_same_models_at_any_batch_size(child):  # noqa: F811
    """The full-batch kernel's models need less room than the same models with smaller batches."""
    tried, short = child("""
        def room(n, d, c, shapes, batch):
            out = C.c_size_t(0)
            rc = L.bbo_mlp_workspace_bytes(C.c_int64(n), d, c, 5, records(shapes, batch), len(shapes), 0, C.byref(out))
            assert rc == 0, L.bbo_mlp_last_error()
            return out.value
        tried, short = 0, []
        for n, d, c, h in ((43, 21, 0, 32), (80, 15, 3, 16), (500, 18, 3, 24), (150, 4, 3, 20), (400, 31, 2, 32), (300, 4, 1, 64)):
            for count in (1, 7, 250):
                shapes = [[h - i % 3] for i in range(count)]
                for batch in (1, 16, n - 1):
                    tried += 1
                    if room(n, d, c, shapes, 0) < room(n, d, c, shapes, batch):
                        short.append((n, d, c, h, count, batch))
        print(json.dumps([tried, short]))
        """)
    assert tried == 54 and not short
