"""The dispatch rules of the projections, asked on the host (tests/tile_rules_audit.cpp compiles the header that the library
compiles): every shape of the GPU tests that is there for one kernel still goes to that kernel."""
import os
import shutil
import subprocess

import pytest

from paper_2104_12470_amd import workloads as wl
from tests import tile_shapes as ts

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    exe = tmp_path_factory.mktemp("rules") / "tile_rules_audit"
    subprocess.run([cxx, "-std=c++17", "-O1", "-Wall", "-Wextra", "-Werror", os.path.join(ROOT, "tests", "tile_rules_audit.cpp"), "-o", str(exe)],
                   check=True)

    def run(questions):
        out = subprocess.run([str(exe)], input="".join(f"{w} {M} {N} {K}\n" for w, M, N, K in questions), capture_output=True, text=True, check=True)
        answers = out.stdout.splitlines()
        assert len(answers) == len(questions)
        return answers
    return run


def test_operator_shapes_take_the_kernel_they_are_there_for(ask):
    want = [(("route", M, N, K), r) for M, K, N, r in ts.LARGE_TILES]
    want += [(("bias", M, N, K), r) for M, K, N, r, _ in ts.ROWS_STREAM] + [(("route", M, N, K), r) for M, K, N, _, r in ts.ROWS_STREAM]
    want += [(("mapped", M, N, K), r) for M, K, N, _, _, r in ts.STRIDED]                 # rows with strides are never sliced either
    got = ask([q for q, _ in want])
    assert [(q, r) for (q, _), r in zip(want, got)] == want
    tiles = {r for _, r in want}
    for name in ("256x256 x2", "192x128 x2", "128x128 x2", "128x128 x2, shared schedule", "128x64 x3", "96x128 x4", "128x128 x3", "192x128 x3", "128x256 x3", "64x64 x3",
                 "rows 32", "rows 64", "rows 128", "64x128 x3"):
        assert name in tiles, f"no operator test for {name}"


def test_layer_shapes_take_the_kernel_they_are_there_for(ask):
    seen = set()
    for w, routes in ts.LAYERS:
        T, H, F = int(sum(wl.lengths(w))), w.hidden, w.ffn
        sizes = {"qkv": (T, 3 * H, H), "o": (T, H, H), "ffn1": (T, F, H), "ffn2": (T, H, F)}
        for name, want in routes.items():
            if name in ("o", "ffn2"):
                assert ask([("ranges", *sizes[name])]) == ["1"], (w.name, name)
            assert ask([("mapped", *sizes[name])]) == [want], (w.name, name, T)
            seen.add((want, "qkv" if name == "qkv" else "gelu" if name == "ffn1" else "res"))
    assert {("192x128 x3", "qkv"), ("192x128 x3", "res"), ("128x128 x3", "qkv"), ("128x256 x3", "qkv"), ("128x256 x3", "gelu")} <= seen


def test_the_weight_stream_takes_no_call_that_it_slows_down(ask):
    """17 to 128 rows without a cut, shapes measured slower as a stream of weights (by 4 to 60 %) than on the kernels they have
    otherwise: an output too narrow to fill the CUs, cached weights under 65 rows and more or in a part-filled second round, a
    vocabulary.  And shapes that it serves better stay with it."""
    slower = [("route", M, N, K) for M, N, K in ((75, 6144, 6144), (109, 7808, 7808), (105, 7936, 7936), (110, 7872, 31488), (68, 8192, 8192), (68, 18432, 8192),
                                                 (33, 7168, 4096), (92, 16704, 6272), (102, 13440, 4480), (64, 20480, 2048), (40, 20480, 4096), (64, 36864, 2048),
                                                 (26, 19968, 4992), (24, 50304, 2048), (64, 50304, 2432), (52, 50304, 7552), (100, 50304, 4096), (128, 65536, 8192))]
    slower += [("mapped", 100, 12288, 4096), ("mapped", 128, 16384, 4096), ("mapped_once", 66, 36864, 4096)]
    assert not any(r.startswith("rows") for r in ask(slower)), dict(zip(slower, ask(slower)))
    better = [("route", M, N, K) for M, N, K in ((20, 6912, 2304), (32, 20480, 4096), (48, 12288, 4096), (64, 16384, 4096), (64, 49152, 12288), (64, 65536, 4096), (28, 50304, 4096),
                                                 (100, 40960, 8192), (128, 36864, 12288))]
    better += [("mapped_once", 100, 12288, 4096), ("mapped_once", 128, 16384, 4096), ("mapped_once", 68, 16384, 4096), ("mapped", 48, 12288, 4096)]
    assert all(r.startswith("rows") for r in ask(better)), dict(zip(better, ask(better)))


def test_room_for_the_sums_of_cut_projections(ask):
    """The workspace asks for a dozen row counts; every one up to the capacity is covered."""
    sizes = [(H, K) for H in (64, 256, 768, 960, 1024, 1600, 1984, 2048, 3072, 4096, 5120, 8192, 12288, 16384) for K in (H, 4 * H, 8192)]
    got = ask([("sums", M, H, K) for H, K in sizes for M in (1, 16, 17, 31, 32, 33, 48, 64, 65, 100, 128, 129, 255, 256, 257, 640, 1000, 1023, 1024, 1025, 3000)])
    assert all(a.split()[0] == a.split()[1] for a in got)
    assert sum(a != "0 0" for a in got) > 100


def test_only_as_many_sequences_as_a_wave_counts_are_put_in_order(ask):
    """Two lengths per lane of a wave: 128 sequences.  The operators take up to 65535, whose order stays the batch's."""
    taken = [("longest_first", *q) for q in ((2, 129, 512), (48, 32, 1516), (128, 3, 777), (128, 65535, 4096))]
    left = [("longest_first", *q) for q in ((1, 1000, 512), (2, 128, 4096), (48, 32, 511), (129, 2, 512), (129, 96, 4096), (200, 8, 1024), (300, 1, 512), (65535, 65535, 4096))]
    assert ask(taken) == ["1"] * len(taken) and ask(left) == ["0"] * len(left)


def test_creating_a_handle_costs_microseconds():
    """Sizing a layer's workspace is a few dozen arithmetic rules: one query stays below the price of a walk over a thousand row
    counts (17 us where this takes one)."""
    import time

    from paper_2104_12470_amd import eet
    cfg = eet.make_config(1024, 16, 4096, 8, 512, 1024)
    best = 1e9
    for _ in range(50):
        t = time.perf_counter()
        for _ in range(20):
            eet.eet_workspace_bytes(cfg)
        best = min(best, (time.perf_counter() - t) / 20)
    assert best < 8e-6, f"{best * 1e6:.1f} us"
