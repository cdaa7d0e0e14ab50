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
    for name in ("256x256 x2", "192x128 x2", "128x128 x2", "128x64 x3", "96x128 x4", "128x128 x3", "192x128 x3", "128x256 x3", "64x64 x3",
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
