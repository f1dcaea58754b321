"""The launch plans, on the host: where the tables and the scratch lie in a workspace, and the record of
the tables that calls left in workspaces."""
import random

from host_probe import plans, run


def forward_cases():
    r = random.Random(3)
    out = []
    for d, M, S in ((128, 128, 128), (128, 128, 63), (128, 100, 128), (128, 128, 255), (64, 64, 127), (32, 16, 31)):
        for bf16 in (0, 1):
            for B, H in ((1, 16), (2, 16), (16, 1), (17, 1), (3, 7)):
                for L in (1, 64, 960, 1000, 1018 * 64, 65536, r.randrange(1, 70000)):
                    out.append(("f", B, H, L, d, M, S, bf16, 0, 0))
    return out


def test_tables_of_one_key_lie_in_one_place_before_the_scratch():
    """A call with reuse_tables finds the tables of an earlier one by the key alone, so plans with
    equal keys must agree on every table's place, and no scratch may lie before a table."""
    cases = forward_cases()
    places = {}
    for c, p in zip(cases, plans(cases)):
        if p is None:
            continue
        assert max(p["tables"]) <= p["summ"] <= p["total"], c
        first = places.setdefault(p["key"], (p["tables"], c))
        assert first[0] == p["tables"], (c, first[1])
    assert len(places) > 20


def test_records_of_tables_end_where_another_call_writes():
    script = [
        ("build 0 1000 100 7", None), ("keep 0 1000 500 7", 1),
        ("keep 0 1000 500 8", 0), ("keep 0 1000 500 7", 0),     # other tables in the same workspace
        ("build 0 1000 100 7", None), ("build 1 1000 100 9", None),
        ("keep 0 1000 100 7", 1), ("keep 1 1000 100 9", 1),     # each device its own
        ("build 0 5000 100 3", None),
        ("write 0 1100 3900", None), ("keep 0 1000 100 7", 1), ("keep 0 5000 100 3", 1),  # between the two
        ("write 0 400 601", None), ("keep 0 1000 100 7", 0),    # the first byte of the tables
        ("write 0 5099 1", None), ("keep 0 5000 100 3", 0),     # the last one
        ("build 0 3000 100 5", None), ("keep 0 2000 900 6", 0), ("keep 0 3000 100 5", 1),
        ("keep 0 2000 1001 6", 0), ("keep 0 3000 100 5", 0),    # a workspace inside another call's scratch
    ]
    script += [(f"build 0 {10000 + 10 * i} 5 {i}", None) for i in range(70)]  # more than are recorded
    script += [("keep 0 10000 5 0", 0), ("keep 0 10690 5 69", 1)]
    got = run("records", [x for x, _ in script])
    assert [int(x) for x in got] == [y for _, y in script if y is not None]
