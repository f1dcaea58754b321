"""The launch plans, on the host: where the tables and the scratch lie in a workspace, the record of the
tables that calls left in workspaces, and which products of a layer the library forms itself."""
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


def test_segments_of_the_one_unit_kernels_run_in_one_round():
    """256 compute units (the host's default).  With two or three workgroups to a compute unit the
    segments fill two, and never start a second round; whether so many fit is a matter of
    registers as well as of LDS (float32 at d = 128 takes the register file for one)."""
    def nseg(units, d, M, S, bf16, chunk, anchor=0):
        return plans([("f", 1, units, 1024, d, M, S, bf16, chunk, anchor)])[0]["nseg"]

    for anchor in (0, 1):
        assert [nseg(u, 128, 16, 31, 0, 16, anchor) for u in (100, 128, 200, 256, 400)] == [3, 2, 2, 1, 1]
        assert [nseg(u, 128, 16, 31, 1, 32, anchor) for u in (100, 128, 200, 256, 400)] == [5, 4, 2, 2, 1]
    assert [nseg(u, 64, 16, 31, 1, 16) for u in (128, 200, 256, 300, 384, 385, 511)] == [4, 2, 2, 2, 2, 1, 1]
    cases = [("f", 1, u, 2000, d, M, S, bf16, chunk, 0) for u in (5, 100, 171, 255, 257, 300, 390, 511) for d in (32, 64, 128)
             for M, S in ((16, 31), (32, 63), (64, 64), (64, 127)) for bf16 in (0, 1) for chunk in (16, 32, 64, 128)]
    for c, p in zip(cases, plans(cases)):
        if p is not None and not p["pair"] and p["nseg"] > 1 and c[2] > 256:
            assert c[2] * p["nseg"] <= 768, (c, p["nseg"])


def test_segments_for_two_workgroups_keep_the_scan_short():
    """Few sequences in short chunks: twice the segments only where that halves a workgroup's chunks, and
    no scan gets much longer than with half of them."""
    def nseg(units, L, d, M, S, bf16, chunk):
        return plans([("f", 1, units, L, d, M, S, bf16, chunk, 0)])[0]["nseg"]

    assert nseg(4, 8000, 64, 64, 127, 1, 16) == 125 and nseg(4, 2000, 64, 64, 127, 1, 16) == 63
    assert nseg(6, 3500, 64, 32, 63, 1, 32) == 37 and nseg(12, 3500, 64, 64, 127, 1, 16) == 37
    assert nseg(2, 30000, 32, 16, 31, 1, 16) == 125 and nseg(1, 14000, 32, 32, 63, 0, 16) == 438
    for units in (1, 2, 3, 5, 7, 12, 31, 64):
        for L in (300, 2000, 3500, 9000, 30000, 60000):
            n = nseg(units, L, 64, 32, 63, 1, 32)
            assert units * n <= 512 and (n <= 128 or units <= 3)


def test_products_that_the_vendor_library_takes():
    """The own kernel does not split a reduction, so past 1024 it loses at any number of tokens, and widths of 256
    and 512 go back to the library once many tokens hide its start."""
    takes = lambda m, n, k: run("products", [f"{m} {n} {k}"]) == ["1"]
    assert takes(1, 96, 32) and takes(10 ** 6, 1152, 384) and takes(4000, 1920, 640) and takes(1000, 3072, 1024)
    assert takes(32768, 768, 256) and takes(8192, 512, 512) and not takes(65536, 256, 256)
    assert not takes(16384, 1536, 512) and not takes(8528, 640, 640)
    for m in (1, 16, 200, 500, 4000):
        assert not takes(m, 3 * 1536, 1536) and not takes(m, 2048, 2048)
    assert not takes(4000, 1024, 1024) and not takes(8000, 2304, 768) and not takes(8, 12, 64) and not takes(0, 96, 32)
