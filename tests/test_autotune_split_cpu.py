"""The autotuner's split-x2 candidates against the kernels that are built, and what ``tune`` keeps of them, on the
CPU (the timing is replaced)."""
import json
import os
import re

import pytest

import synthetic as S
from paper_2211_10185_amd import autotune as A

SIZES = list(S.smooth_even_sizes(32, 256))


def all_candidates(N, prec, k):
    return A.candidates(N, prec, k) + A.more_candidates(N, prec, k)


def built_variants():
    """(N, precision) -> the variants of the shape table that a flag can select (4 is the A/B update's own)."""
    src = open(os.path.join(A.HERE, "csrc", "split_passes.h")).read()
    rows = re.findall(r"^    \{(\d+), ([01]), (\d), ", src, re.M)
    assert len(rows) > 100
    out = {}
    for n, p, v in rows:
        if v != "4":
            out.setdefault((int(n), int(p)), set()).add(int(v))
    return out


def test_every_built_variant_is_a_candidate_and_no_other():
    built = built_variants()
    for N in SIZES:
        for prec in (0, 1):
            offered = {c["split_variant"] for c in all_candidates(N, prec, 3) if c["split"]}
            assert offered == built.get((N, prec), set()), (N, prec)


@pytest.mark.parametrize("k", [1, 2, 3])
def test_tune_times_and_records_every_candidate(tmp_path, monkeypatch, k):
    path = str(tmp_path / "tuning.json")
    monkeypatch.setattr(A, "_device_name", lambda: "test")
    monkeypatch.setattr(A, "_cache", None)
    for prec in (0, 1):
        for N in SIZES:
            cands = all_candidates(N, prec, k)
            assert len({A.schedule_name(c) for c in cands}) == len(cands), (N, prec)
            # each in turn is the fastest, and is what the entry says
            for want in cands:
                monkeypatch.setattr(A, "time_schedule", lambda N, p, k, s, steps: 1.0 if s == want else 2.0)
                if os.path.exists(path):
                    os.remove(path)
                e = A.tune([N], precisions=(prec,), states=(k,), path=path, verbose=False)[A.key(N, prec, k)]
                assert len(e["us_per_step"]) == len(cands), (N, prec)
                assert (e["split"], e["rowcol"], e["groups"], e["split_variant"]) == (
                    want["split"], want["rowcol"], want["groups"], want.get("split_variant", 0)), (N, prec)


@pytest.mark.parametrize("N", [64, 108, 128, 150, 162, 180, 250, 256])
def test_tuning_again_keeps_the_roundings_of_complex64(tmp_path, monkeypatch, N):
    """A faster schedule with other factors of x2 does not take an entry over; one with the same does."""
    path = str(tmp_path / "tuning.json")
    monkeypatch.setattr(A, "_device_name", lambda: "test")
    monkeypatch.setattr(A, "_cache", None)
    cands = all_candidates(N, 0, 3)
    for old in cands:
        entry = dict(old, split_variant=old.get("split_variant", 0))
        same = [c for c in cands if A.rounding(c, N, 0) == A.rounding(old, N, 0)]
        assert old in same
        for out in (path, str(tmp_path / "other.json")):
            with open(path, "w") as f:
                json.dump({"entries": {A.key(N, 0, 3): entry}}, f)
            # the others are faster than all of its kind, and of its kind the last one is
            times = {A.schedule_name(c): 5.0 - i / 100 if c in same else 1.0 for i, c in enumerate(cands)}
            monkeypatch.setattr(A, "time_schedule", lambda N, p, k, s, steps: times[A.schedule_name(s)])
            e = A.tune([N], precisions=(0,), states=(3,), path=out, verbose=False, keep=path)[A.key(N, 0, 3)]
            assert sorted(e["us_per_step"]) == sorted(A.schedule_name(c) for c in same)
            assert A.schedule_name(e) == A.schedule_name(same[-1])


def test_roundings_follow_the_factors_of_the_shape_table():
    src = open(os.path.join(A.HERE, "csrc", "split_passes.h")).read()
    n1 = {(int(n), int(v)): int(f) for n, v, f in re.findall(r"^    \{(\d+), 0, (\d), (\d+), ", src, re.M) if v != "4"}
    for N in SIZES:
        if N < 96:
            continue
        for c in all_candidates(N, 0, 1):
            for d in all_candidates(N, 0, 1):
                if c["split"] and d["split"]:
                    same = n1[N, c["split_variant"]] == n1[N, d["split_variant"]]
                    assert (A.rounding(c, N, 0) == A.rounding(d, N, 0)) == same, (N, c, d)


def test_states_of_the_size_of_the_cache_run_on_one_stream(tmp_path, monkeypatch):
    path = str(tmp_path / "tuning.json")
    e = {"rowcol": False, "single_stream": False, "groups": 3, "split": True, "split_variant": 0}
    plane = dict(e, split=False)
    with open(path, "w") as f:
        json.dump({"entries": {"162/0/2": e, "160/1/2": e, "180/0/2": plane}}, f)
    monkeypatch.setenv("QFDTD_TUNING", path)
    monkeypatch.setattr(A, "_cache", None)
    for N, prec, k, groups in [(162, 0, 7, 3), (162, 0, 8, 1), (160, 1, 4, 3), (180, 0, 6, 3)]:
        s = A.schedule_for(N, 2, prec, k)
        assert (s["groups"], s["single_stream"]) == (groups, groups == 1), (N, prec, k)
        assert s["split_variant"] == 0 and not s["rowcol"]
    A._cache = None


def test_ab_rule_names_kernels_that_are_built():
    built = built_variants()
    for N in SIZES:
        for prec in (0, 1):
            for k in (1, 2, 3, 8):
                e = A.ab_schedule(N, prec, k)
                if e is not None:
                    assert e["split_variant"] in built[N, prec] and 1 <= e["groups"] <= k
    # the sizes and state counts whose second shape was measured to be the better one
    assert [A.ab_schedule(120, 1, k)["split_variant"] for k in (1, 3)] == [1, 0]


def test_ab_update_keeps_row_and_column_passes_that_a_complex64_cache_asks_for():
    plane = {"rowcol": False, "single_stream": True, "groups": 1, "split": False, "split_variant": 0}
    rowcol = dict(plane, rowcol=True)
    assert A.ab_schedule_for(64, 0, 1, rowcol) == rowcol
    assert A.ab_schedule_for(64, 0, 1, plane) == A.ab_schedule(64, 0, 1)
    assert A.ab_schedule_for(100, 1, 1, rowcol) == A.ab_schedule(100, 1, 1)      # complex128: faster, within 1e-14
    assert A.ab_schedule_for(160, 0, 3, dict(plane, split=True)) == plane        # no split-x2 kernels: as before
