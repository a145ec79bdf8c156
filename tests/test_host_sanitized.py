"""libsig's host logic under AddressSanitizer and UndefinedBehaviorSanitizer (CPU only, nothing is launched).

The planner, the plan checks, the footprint query and the gradient's segment rule are index and size arithmetic that
decides LDS sizes and grid shapes.  Every translation unit of the library is compiled for the host only (hipcc
--cuda-host-only, a few seconds) with both sanitizers, the device code objects they would embed are replaced by empty
bundles, and tests/host_sweep.cpp drives the host-only entry points over some ten thousand seeded shapes and
twenty thousand arbitrary plans.  The run fails on any sanitizer report and on any broken invariant (the planner's own
plan refused by the plan check, LDS above the library's limit, a grid beyond 2^31 - 1, ...).

tests/host_launches.cpp makes calls over a HIP runtime of its own: which kernels they launch, and what they do where scratch
cannot be had.
"""
import json
import os
import re
import subprocess
from concurrent.futures import ThreadPoolExecutor

import pytest

from paper_2501_08455_amd import build as lib_build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CLANGXX = "/opt/rocm/lib/llvm/bin/clang++"


@pytest.fixture(scope="module")
def linked(tmp_path_factory):
    """linked(program, *link flags): the library's host code and tests/<program> with both sanitizers, as an executable."""
    if not os.path.exists(CLANGXX):
        pytest.skip("no ROCm clang++ here")
    tmp_path = tmp_path_factory.mktemp("host")
    flags = ["--cuda-host-only", "-O1", "-g", "-std=c++17", "-fPIC", "-fno-omit-frame-pointer",
             "-Xarch_host", "-fsanitize=address", "-Xarch_host", "-fsanitize=undefined",
             "-Xarch_host", "-fno-sanitize-recover=all", "-Wno-unused-command-line-argument",
             "-I" + os.path.join(ROOT, "include"), "-I" + lib_build.CSRC]

    def compile_one(src):
        obj = str(tmp_path / (os.path.splitext(src)[0] + ".o"))
        res = subprocess.run([lib_build._hipcc()] + flags + ["-c", os.path.join(lib_build.CSRC, src), "-o", obj],
                             capture_output=True, text=True)
        return obj, res

    with ThreadPoolExecutor(max_workers=8) as pool:
        results = list(pool.map(compile_one, lib_build.SOURCES))
    for obj, res in results:
        if res.returncode != 0 and "sanitize" in res.stderr and "unsupported" in res.stderr:
            pytest.skip("this toolchain has no host sanitizer runtime")
        assert res.returncode == 0, res.stderr[-3000:]
    objs = [obj for obj, _ in results]
    # the host objects refer to the device code objects that a full build embeds: empty offload bundles stand in
    undefined = subprocess.run(["nm", "-u"] + objs, capture_output=True, text=True).stdout
    stubs = sorted(set(re.findall(r"__hip_fatbin_[0-9a-f]+", undefined)))
    stub_c = tmp_path / "fatbin_stubs.c"
    stub_c.write_text("".join('__attribute__((aligned(4096))) const char %s[32] = "__CLANG_OFFLOAD_BUNDLE__";\n' % s
                              for s in stubs))

    def link(program):
        exe = str(tmp_path / os.path.splitext(program)[0])
        res = subprocess.run([CLANGXX, "-fsanitize=address", "-fsanitize=undefined", "-fno-sanitize-recover=all", "-g",
                              "-D__HIP_PLATFORM_AMD__=1", "-isystem", "/opt/rocm/include",
                              "-I" + os.path.join(ROOT, "include"), os.path.join(ROOT, "tests", program),
                              "-x", "c", str(stub_c), "-x", "none"] + objs +
                             ["-L/opt/rocm/lib", "-lamdhip64", "-Wl,-rpath,/opt/rocm/lib", "-o", exe],
                             capture_output=True, text=True)
        assert res.returncode == 0, res.stderr[-3000:]
        return exe

    return link


def run(exe, *args, calls=""):
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0:abort_on_error=0:verify_asan_link_order=0",
               UBSAN_OPTIONS="print_stacktrace=1:halt_on_error=1")
    ran = subprocess.run([exe] + list(args), input=calls, capture_output=True, text=True, env=env, timeout=600)
    assert ran.returncode == 0, (ran.returncode, ran.stdout[-4000:] + ran.stderr[-4000:])
    return ran.stdout


def test_host_logic_runs_clean_under_sanitizers(linked):
    assert "host sweep ok" in run(linked("host_sweep.cpp"))


@pytest.fixture(scope="module")
def launches(linked, tmp_path_factory):
    """launches([(bytes to be had, "f" or "b", B, L, d, depth, stream), ...]): (status, allocations refused, kernels) of each call."""
    exe = linked("host_launches.cpp")
    registers = tmp_path_factory.mktemp("registers") / "registers"
    reported = json.load(open(lib_build.RESOURCES)) if os.path.exists(lib_build.RESOURCES) else {}
    registers.write_text("".join("%s %d\n" % (name, use["VGPRs"] + use.get("AGPRs", 0)) for unit in reported.values() for name, use in unit.items()))

    def answers(calls):
        out = run(exe, str(registers), calls="".join("%d %s %d %d %d %d %d\n" % call for call in calls)).splitlines()
        assert len(out) == len(calls)
        return [(int(line.split()[0]), int(line.split()[1]), line.split()[2:]) for line in out]

    return answers


PLENTY = 1 << 40
OK, ALLOC = 0, 3

# bytes to be had, call, status, kernel (None: nothing is launched)
SCARCE = [
    # the reduced rows of the first: 2 * 39 * 12 * 14 floats; the general sweep needs less
    (48000, "b", (2, 40, 12, 3, 1), OK, "sig_backward_general"), (PLENTY, "b", (2, 40, 12, 3, 1), OK, "sig_stream_depth3"),
    (0, "b", (2, 40, 11, 3, 1), ALLOC, None),
    # a path in one workgroup; what lies before a stretch folded again
    (0, "b", (1, 1500, 6, 2, 1), OK, "sig_stream_depth2"), (0, "f", (1, 1400, 10, 4, 1), OK, "sig_split_rows"),
    # segments, which no call does without
    (0, "f", (1, 2000, 6, 5, 0), ALLOC, None), (0, "b", (1, 600, 5, 4, 1), ALLOC, None),
]


def test_calls_that_cannot_have_scratch_return(launches):
    """... and leave the context to other threads (host_launches.cpp makes such a call behind each)."""
    got = launches([(most, way) + call for most, way, call, _, _ in SCARCE])
    for (most, way, call, status, kernel), (rc, refused, kernels) in zip(SCARCE, got):
        assert rc == status and (refused > 0) == (most < PLENTY), (way, call, rc, refused)
        assert any(kernel in k for k in kernels) if kernel else not kernels, (way, call, kernels)


# call, kernel: the routes that the cases of tests/test_gpu_*.py name, and the calls beside them
ROUTES = [
    ("b", (2, 45001, 9, 3, 1), "sig_backward_tiled"), ("b", (600, 3500, 5, 3, 1), "sig_backward_tiled"), ("b", (3, 40001, 10, 3, 1), "sig_backward_tiled"),
    ("b", (300, 1500, 10, 4, 1), "sig_backward_sliced"), ("b", (700, 700, 5, 4, 1), "sig_backward_tiled"), ("b", (24, 1700, 10, 3, 1), "sig_backward_segment_affine"),
    ("b", (1, 600, 10, 4, 1), "sig_backward_segment_affine"), ("b", (3000, 500, 7, 3, 1), "sig_backward_chunked"), ("b", (17000, 100, 7, 3, 1), "sig_backward_tiled"),
    ("b", (8200, 500, 3, 3, 1), "sig_backward_chunked"), ("b", (16500, 256, 5, 3, 1), "sig_backward_tiled"), ("b", (8200, 128, 2, 6, 1), "sig_backward_kernel"),
    ("b", (40, 60, 13, 3, 1), "sig_backward_general"), ("b", (2, 11, 21, 2, 1), "sig_backward_general"), ("b", (2, 11, 12, 4, 1), "sig_backward_general"),
    ("b", (2, 11, 11, 2, 1), "sig_stream_depth2"), ("b", (2, 60000, 10, 2, 1), "sig_stream_depth2"), ("b", (17000, 100, 10, 2, 1), "sig_stream_depth2"),
    ("b", (1, 5200000, 20, 2, 1), "sig_stream_depth2"), ("b", (1, (1 << 30) + 2, 2, 2, 1), "sig_backward_general"), ("b", (40, 60, 12, 3, 1), "sig_stream_depth3"),
    ("b", (10000, 3, 10, 2, 0), "sig_backward_kernel"), ("b", (2, 60000, 10, 2, 0), "sig_bracket_depth2"), ("b", (1, 150, 10, 5, 0), "sig_backward_segment"),
    ("f", (64, 256, 4, 4, 1), "sig_stream_rows"), ("f", (40, 90, 12, 3, 1), "sig_stream_rows"), ("f", (1500, 40, 16, 2, 1), "sig_depth2_rows"),
    ("f", (2, 700, 9, 4, 1), "sig_split_rows"), ("f", (4096, 256, 4, 4, 1), "sig_on_chip_kernel"), ("f", (8, 500, 12, 4, 1), "sig_level"),
]


def test_calls_take_the_kernels_that_the_gpu_tests_name(launches):
    got = launches([(PLENTY, way) + call for way, call, _ in ROUTES])
    wrong = [(way, call, kernel, kernels) for (way, call, kernel), (rc, _, kernels) in zip(ROUTES, got) if rc != OK or not any(kernel in k for k in kernels)]
    assert not wrong, wrong
