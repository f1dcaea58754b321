"""The launch plans, on the host: where the tables and the scratch lie in a workspace."""
import random

from host_probe import plans


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
