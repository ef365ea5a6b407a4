"""Which tiles a call of the reduce takes, asked of the host's rule on the CPU: that the GPU tests
that are about one kernel run that kernel, and that regions which may be hit unevenly do not take
the slim tiles where those lose."""
import itertools
import os
import shutil
import subprocess

import numpy as np
import pytest

import test_gpu_reduce_dense as dense
import test_gpu_reduce_slim as slim
import test_gpu_reduce_tiles as tiles
import test_gpu_reduce_wide as wide

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CUS = 256


@pytest.fixture(scope="module")
def forms(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no g++")
    exe = tmp_path_factory.mktemp("forms") / "shape_of"
    subprocess.run([gxx, "-O2", "-std=c++17", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_2201_07598_amd", "csrc"),
                    os.path.join(ROOT, "tests", "cabi", "shape_of.cpp"), "-o", str(exe)], check=True)

    def ask(calls):                                  # (B, width, capacity, P) -> "form kind slots"
        text = "".join(f"{B} {width} {capacity} {P} {CUS}\n" for B, width, capacity, P in calls)
        out = subprocess.run([str(exe)], input=text, capture_output=True, text=True, check=True).stdout.splitlines()
        assert len(out) == len(calls)
        return out
    return ask


def test_cases_about_slim_tiles_take_them(forms):
    calls = [(slim.LONG_B, slim.LONG_WIDTH, c, P) for P, *_ in slim.LONG_CASES for c in slim.LONG_CAPACITIES]
    calls += [(slim.WINDOW_B, slim.WINDOW_WIDTH, slim.WINDOW_CAPACITY, P) for P, *_ in slim.WINDOW_CASES]
    assert set(forms(calls)) == {"slim sparse 98304"}
    full = forms([(slim.FULL_B, slim.FULL_WIDTH, slim.FULL_CAPACITY, P) for P, *_ in slim.FULL_CASES])
    assert all(f.startswith("slim ranked") and int(f.split()[2]) >= 39_000 for f in full)
    kinds = forms([(slim.kind_batch(width), width, capacity, P) for P, width, _, _, _, capacity in slim.KIND_CASES])
    assert all(f.startswith("slim") for f in kinds) and len(set(kinds)) > 3
    P, width, B = slim.VALUES_CALL
    assert forms([(B, width, slim.VALUES_CAPACITY, P)]) == ["slim ranked 65536"]
    P, width, B, cap = slim.REPLAY_CALL
    assert forms([(B, width, cap, P)]) == ["slim ranked 65536"]


def test_cases_about_wide_tiles_take_them(forms):
    got = forms([(wide.B, wide.WIDTH, capacity, P) for _, P, capacity, _, _ in wide.CASES])
    for case, form in zip(wide.CASES, got):
        assert form.startswith(case[0]) and int(form.split()[2]) >= 44_000, (case, form)
    B, P, width, capacity = wide.FULL
    assert forms([(B, width, capacity, P)]) == ["wide4 sparse 98304"]


@pytest.mark.parametrize("calls", [
    # 33 to 63 contributions, tiles planned full or for more hits than collide in one window (hit
    # unevenly 0.67 to 1.0 times as fast in slim tiles)
    [(186, 400_000, int(s * 400_000), 40) for s in (0.06, 0.1, 0.15, 0.2, 0.3)],
    [(1_000, 44_237, 6_768, 46), (1_300, 50_627, 11_900, 40), (60, 739_221, 123_000, 60), (900, 56_643, 13_200, 50)],
    # 64 to 128, planned full (30 % in common 0.92, log-normal stretches 0.93)
    [(400, 150_000, int(s * 150_000), P) for P in (64, 128) for s in (0.1, 0.15, 0.3)],
    [(27, 1_600_000, int(s * 1_600_000), 64) for s in (0.1, 0.2, 0.3)],
    # few, a good part of the slots hit
    [(100, 1_600_001, int(s * 1_600_001), P) for P in (5, 6, 7) for s in (0.201, 0.3, 0.39)],
    [(100, 1_600_001, int(s * 1_600_001), P) for P in (3, 4) for s in (0.101, 0.15)],
])
def test_no_slim_tiles_where_uneven_regions_lose(forms, calls):
    assert [f for f in forms(calls) if f.startswith("slim")] == []


def test_slim_tiles_where_they_gain(forms):
    calls = [(490, 1_597_315, 249_000, 16), (373, 5_250_000, 342_000, 64), (400, 400_000, 12_000, 40), (400, 800_000, 24_000, 100),
             (60, 3_000_001, 120_000, 4), (60, 2_000_001, 380_000, 12),
             (100, 1_600_001, 460_000, 16), (114, 3_437_500, 1_100_000, 32)]
    assert [f for f in forms(calls) if not f.startswith("slim")] == []


def batches_of(test, module, monkeypatch):
    """The (B, width, capacity, P) of every batch that a parametrised GPU test would run."""
    got, none = [], np.zeros(0, np.uint32)
    monkeypatch.setattr(module, "run_batch",
                        lambda regions, P, width, capacity, **_: got.append((len(regions), width, capacity, P)))
    for name in ("some", "clustered"):
        if hasattr(module, name):
            monkeypatch.setattr(module, name, lambda *_: none)
    marks = [m.args for m in getattr(test, "pytestmark", []) if m.name == "parametrize"]
    for values in itertools.product(*(a[1] for a in marks)):
        kw = {}
        for (names, _), v in zip(marks, values):
            names = names.split(",")
            kw.update(zip(names, v if len(names) > 1 else [v]))
        test(**kw)
    return got


@pytest.mark.parametrize("module,test,kernels", [
    (tiles, "test_wide_tiles_in_batches", {"narrow ranked", "narrow sparse", "slim ranked", "wide4 ranked", "wide4 dense"}),
    (tiles, "test_wide_tiles_with_more_hits_than_they_have_room_for", {"narrow sparse"}),
    (tiles, "test_windows_of_a_tile", {"narrow sparse", "narrow dense"}),
    (dense, "test_edges_of_dense_tiles", {"narrow dense", "narrow ranked", "wide4 dense"}),
    (dense, "test_dense_copy_of_wide_dense_tiles", {"wide4 dense"})])
def test_kernels_that_other_tests_run(forms, monkeypatch, module, test, kernels):
    calls = batches_of(getattr(module, test), module, monkeypatch)
    assert {" ".join(f.split()[:2]) for f in forms(calls)} == kernels


def test_kernels_of_entries_beyond_a_chunk(forms):
    cases = next(m.args[1] for m in tiles.test_entries_beyond_a_chunk.pytestmark if m.args[0] == "P,units")
    for P in sorted({P for P, _ in cases}):
        lone, batch = forms([(1, 900_001, 60_000, P), (36, 900_001, 120_000, P)])
        assert lone.startswith("narrow sparse")
        assert batch.startswith("narrow ranked" if P <= 32 else "wide5 ranked" if P < 64 else "wide4 ranked"), (P, batch)
