"""The Linear Relation calls stay inside the workspace that their queries ask
for: the C-ABI layer with its launches replaced by a probe of the arguments
(tests/workspace_probe.cpp), on the CPU."""
from __future__ import annotations

import ctypes
import os
import subprocess

import pytest

from paper_2608_20172_amd import binding as R
from paper_2608_20172_amd import build
from tests.linear_shapes import BF16_KERNELS

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
BASE, GB = 0x7F0000000000, 1 << 33


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    out = tmp_path_factory.mktemp("probe")
    objs = [os.path.join(build.BUILD_DIR, s + ".o") for s in build.SOURCES]
    if not all(os.path.exists(o) for o in objs):
        build.build()
    probe, path = str(out / "probe.o"), str(out / "librelation_probe.so")
    for cmd in ([build.hipcc(), *build.COMMON, *build.DEVICE_FLAGS, "-x", "hip", "-c",
                 os.path.join(ROOT, "tests", "workspace_probe.cpp"), "-o", probe],
                # the probe's definitions come first and stand
                [build.hipcc(), f"--offload-arch={build.ARCH}", "-shared", "-fPIC", "-Wl,--allow-multiple-definition",
                 "-o", path, probe, *objs, "-L/opt/rocm/lib", "-lrocblas", "-Wl,-rpath,/opt/rocm/lib"]):
        r = subprocess.run(cmd, capture_output=True, text=True)
        assert r.returncode == 0, r.stderr[-3000:]
    dll = ctypes.CDLL(path)
    for name, (res, args) in R._SIGS.items():
        if name.startswith("relation_linear") or name == "relation_last_error":
            fn = getattr(dll, name)
            fn.restype, fn.argtypes = res, args
    dll.probe_used.restype, dll.probe_used.argtypes = ctypes.c_int64, [ctypes.c_size_t]
    return dll


def _used(lib, B, H, T, D, dtype, backward, gated, rope):
    """(bytes the query asks for, bytes the launched kernels would use)"""
    p = ctypes.byref(R.RelProblem(B, H, T, D, dtype, 1, 2.0, 0.0, H * T * D, T * D, D))
    a = [BASE + i * GB for i in range(12)]
    name = f"relation_linear_{'gated_' if gated else ''}{'bwd' if backward else 'fwd'}"
    query = getattr(lib, name + "_workspace_bytes")
    size = query(p, rope) if gated else query(p)
    ws = BASE + 64 * GB
    gate = [a[4], a[5], rope, 1e4] if gated else []
    outs = [a[6], a[7], a[8], a[9], a[10]] + ([a[11], a[11] + GB // 2] if gated else []) if backward else [a[6], a[7]]
    st = getattr(lib, name)(p, a[0], a[1], a[2], a[3], *gate, *outs, ws, size, None)
    assert st == R.REL_OK, lib.relation_last_error()
    return size, lib.probe_used(ws)


@pytest.mark.parametrize("D", [32, 64, 128])
def test_calls_stay_inside_the_queried_workspace(lib, D):
    """Every even RoPE width, problems of one head and up, lengths on both sides
    of chunk, segment and routing edges, forward and backward, both types."""
    ropes = range(0, D + 1, 8 if D == 128 else 2)
    taken = set()
    for B, H in ((1, 1), (1, 2), (3, 1), (2, 8), (8, 8), (65, 8)):
        for T in (1, 63, 64, 65, 129, 512, 513, 1024, 1025, 1089, 4097):
            for dtype in (R.REL_BF16, R.REL_F32):
                for backward in (False, True):
                    for gated, rope in [(False, 0)] + [(True, r) for r in (ropes if T <= 129 else (0, D // 2 - 2 if D < 128 else 40, D))]:
                        size, used = _used(lib, B, H, T, D, dtype, backward, gated, rope)
                        taken.add((dtype, backward, bool(lib.probe_bf16_kernels())))
                        assert 0 <= used <= size, (B, H, T, D, dtype, backward, gated, rope, used, size)
    assert {(R.REL_BF16, False, True), (R.REL_BF16, True, True), (R.REL_F32, True, False)} <= taken


@pytest.mark.parametrize("D", [32, 64, 128])
@pytest.mark.parametrize("H", [1, 7, 64, 520])
def test_workspace_for_a_sequence_serves_shorter_ones(lib, D, H):
    for backward in (False, True):
        last = 0
        for T in list(range(1, 70)) + list(range(70, 2300, 13)):
            p = ctypes.byref(R.RelProblem(1, H, T, D, R.REL_BF16, 1, 2.0, 0.0, H * T * D, T * D, D))
            size = getattr(lib, f"relation_linear_gated_{'bwd' if backward else 'fwd'}_workspace_bytes")(p, 24)
            assert size >= last, (T, size, last)
            last = size


# (B H, T, D, gated, rope, backward) -> linear_bf16.hip's kernels; both sides of each line of linear_bf16_route
ROUTES = [
    ((1, 64, 32, True, 24, True), True), ((2, 300, 32, False, 0, False), True),
    ((2, 64, 64, False, 0, False), True), ((2, 65, 64, False, 0, False), False), ((32, 1024, 64, True, 0, False), False),
    ((33, 1024, 64, True, 0, False), True), ((2, 1025, 64, False, 0, False), True),
    ((64, 1024, 64, True, 60, False), False), ((65, 1024, 64, True, 60, False), True), ((2, 300, 64, True, 64, False), True),
    ((16, 1024, 64, False, 0, True), False), ((17, 1024, 64, False, 0, True), True), ((1, 1025, 64, False, 0, True), True),
    ((16, 1024, 64, True, 60, True), False), ((17, 1024, 64, True, 60, True), True), ((2, 64, 64, True, 60, True), True),
    ((10, 512, 64, True, 64, True), False), ((11, 512, 64, True, 64, True), True), ((2, 128, 64, True, 64, True), True),
    ((1, 576, 64, True, 64, True), True),
    ((16, 1024, 128, False, 0, False), False), ((17, 1024, 128, False, 0, False), True), ((8, 1088, 128, False, 0, False), False),
    ((10, 1088, 128, False, 0, False), True), ((1, 2112, 128, False, 0, False), True), ((2, 64, 128, True, 80, False), True),
    ((8, 1088, 128, True, 80, False), False), ((1, 1088, 128, True, 128, False), True), ((4, 300, 128, True, 128, False), False),
    ((10, 1024, 128, False, 0, True), False), ((10, 1088, 128, False, 0, True), True), ((4, 1024, 128, True, 80, True), False),
    ((4, 1088, 128, True, 80, True), True), ((32, 64, 128, True, 0, True), False), ((33, 64, 128, True, 0, True), True),
]


@pytest.mark.parametrize("problem,bf16_kernels", ROUTES)
def test_which_kernels_take_a_bf16_problem(lib, problem, bf16_kernels):
    H, T, D, gated, rope, backward = problem
    _used(lib, 1, H, T, D, R.REL_BF16, backward, gated, rope)
    assert bool(lib.probe_bf16_kernels()) == bf16_kernels
    _used(lib, 1, H, T, D, R.REL_F32, backward, gated, rope)
    assert not lib.probe_bf16_kernels()


def test_shapes_of_the_gpu_tests_take_the_bf16_kernels(lib):
    for H, T, D, rope, _ in BF16_KERNELS:
        for backward in (False, True):
            _used(lib, 1, H, T, D, R.REL_BF16, backward, True, rope)
            assert lib.probe_bf16_kernels(), (H, T, D, rope, backward)
