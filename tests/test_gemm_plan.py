"""The GEMM planner on the host (no GPU): plan.cpp, api.cpp and validate.cpp
built with g++ and test stand-ins for the kernel launchers, so that a call which
passes every check reports SPEC_ERR_HIP instead of launching."""

import collections
import ctypes
import os
import random
import shutil
import subprocess
import time

import pytest

from paper_2606_18502_amd import _lib
from tests import gemm_shapes

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2606_18502_amd", "csrc")
ROCM_INCLUDE = "/opt/rocm/include"

PLAIN, STATS, SILU = 0, 1, 2
Plan = collections.namedtuple("Plan", "kind splits krot m_tiles n_tiles bn groups workspace")


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    if shutil.which("g++") is None or not os.path.isdir(ROCM_INCLUDE):
        pytest.skip("g++ or the HIP headers are not available")
    out = str(tmp_path_factory.mktemp("plan") / "libplan.so")
    srcs = [os.path.join(CSRC, f) for f in ("api.cpp", "validate.cpp", "plan.cpp")]
    srcs += [os.path.join(ROOT, "tests", "hostsan", f) for f in ("launch_stubs.cpp", "plan_abi.cpp")]
    res = subprocess.run(["g++", "-std=c++17", "-O2", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__",
                          f"-I{ROCM_INCLUDE}", f"-I{os.path.join(ROOT, 'include')}", *srcs, "-o", out],
                         capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    h = _lib.declare(ctypes.CDLL(out))
    h.test_plan_gemm.argtypes = [ctypes.c_int64] * 3 + [ctypes.c_int] * 2 + [ctypes.c_void_p]
    h.test_plan_gemm.restype = None
    h.test_plan_search.argtypes = h.test_plan_gemm.argtypes
    h.test_plan_search.restype = None
    h.test_plan_many.argtypes = [ctypes.c_int64] * 3 + [ctypes.c_int] * 2
    h.test_plan_many.restype = ctypes.c_int64
    return h


def plan(lib, M, N, K, epilogue=PLAIN, may_split=True):
    out = (ctypes.c_int64 * 8)()
    lib.test_plan_gemm(M, N, K, epilogue, int(may_split), out)
    return Plan(*out)


def k_starts(lib, p, N, K):
    """The K-step at which each column's sum starts, for columns 0, 16, 32, ...
    (every tile is a multiple of 16 columns wide)."""
    return [lib.test_k_start(c // p.bn * p.bn, K // 128) if p.krot else 0 for c in range(0, N, 16)]


def shapes(seed, count):
    rng = random.Random(seed)
    for _ in range(count):
        yield rng.randint(1, 512), 8 * rng.randint(512, 5120), 128 * rng.randint(1, 112)


def test_statistics_and_unsplit_plain_walk_k_alike(lib):
    """The logits stored with their statistics are the unsplit plain GEMM's bit
    for bit: both sum every column's products in the same order."""
    fixed = [(33, 32896, 8192), (59, 38296, 6656), (320, 128256, 4096), (8, 128256, 4096), (80, 32000, 4096)]
    for M, V, K in fixed + list(shapes(1, 30000)):
        s, u = plan(lib, M, V, K, STATS), plan(lib, M, V, K, PLAIN, may_split=False)
        if s.krot or u.krot:
            assert k_starts(lib, s, V, K) == k_starts(lib, u, V, K), (M, V, K, s, u)


@pytest.mark.parametrize("N", [12288, 14336, 16384, 24576, 28672])
def test_wide_decode_linears_stagger(lib, N):
    """One or two M-tiles that read 192 or more N-tiles start K at staggered
    steps, whether or not their tile kind has a statistics epilogue."""
    seen = set()
    for M in range(1, 321):
        p = plan(lib, M, N, 4096)
        if p.splits == 1 and p.m_tiles <= 2 and p.n_tiles >= 192 and p.bn != 224:
            assert p.krot == 1, (M, N, p)
            seen.add(p.kind)
    assert len(seen) >= (2 if N < 28672 else 4), seen
    assert plan(lib, 8, 28672, 4096).krot == 1 and plan(lib, 80, 28672, 4096).krot == 1
    assert plan(lib, 80, 6144, 4096).krot == 0


@pytest.mark.parametrize("M,N,K,tile", [
    (65, 6144, 4096, (11, 1)), (80, 6144, 4096, (11, 1)),       # QKV of a small verify batch: 13.0 us as (10, 2), 12.2 so
    (80, 7168, 4096, (11, 1)), (160, 4096, 4096, (11, 1)), (160, 4096, 3584, (11, 1)), (144, 3000, 9984, (8, 3)),
])
def test_splits_that_cost_more_than_they_gain(lib, M, N, K, tile):
    """Shapes at which a K split of the 80x64 or the 160x64 tile measured slower
    than the named kind and split."""
    p = plan(lib, M, N, K)
    assert (p.kind, p.splits) == tile, p


HIP, UNSUPPORTED, WORKSPACE, ALIGN = 7, 3, 6, 5


def logit_stats_status(lib, M, V, K, lda, ldw):
    """The status of a call whose pointers are never followed (stand-in launchers)."""
    A, ld = 0x1000, (V + 7) // 8 * 8
    return lib.spec_fp8_gemm_logit_stats(A, lda, A, 0, A, ldw, A, 0, M, V, K, ctypes.c_float(0.7), A, ld, A,
                                         lib.spec_logit_stats_count(M, V, K), None)


@pytest.mark.parametrize("M,V,K,limited", [
    (320, 128256, 4096, True), (310, 128200, 4096, True), (320, 32064, 4096, True), (300, 32008, 256, True),
    (71, 66200, 4096, False),                  # M <= 80 (the planner takes 160 x 384 all the same)
    (100, 128256, 4096, False), (321, 128256, 4096, False), (1000, 128256, 4096, False), (320, 128256, 4224, False), (320, 12000, 4096, False),
    (320, 28672, 4096, False),                 # 160 x 224 tiles stream no more rows
])
def test_long_strides_of_the_lm_head(lib, M, V, K, limited):
    """Strides past a tile's 4 GiB are refused for the stated shapes only, and
    do not depend on the tile that the estimate picks."""
    lda, ldw = ((1 << 32) - 128) // 159 // 16 * 16, ((1 << 32) - 128) // 383 // 16 * 16
    want = UNSUPPORTED if limited else HIP
    assert logit_stats_status(lib, M, V, K, lda, ldw) == HIP             # the longest that the tile addresses
    assert logit_stats_status(lib, M, V, K, lda + 16, K) == want
    assert logit_stats_status(lib, M, V, K, K, ldw + 16) == want


def gemm_status(lib, M, N, K, ws=None, nbytes=0):
    A = 0x1000
    return lib.spec_fp8_gemm(A, K, A, 0, A, K, A, 0, M, N, K, A, (N + 7) // 8 * 8, 0, ws, nbytes, None)


def test_a_workspace_is_required_where_k_is_split(lib):
    """Decode-sized projections always report a size; only a call that splits
    K is refused without one, and an unsplit one never looks at it."""
    seen = collections.Counter()
    decode = [(M, N, K) for M in (1, 8, 64, 80, 81, 128, 200, 320) for N, K in
              ((6144, 4096), (4096, 4096), (4096, 14336), (1024, 4096), (4096, 1024), (2048, 8192))]
    for M, N, K in decode + [(640, 4096, 14336), (1000, 4096, 14336)]:
        required = N < 12288 and ((M <= 80 and K >= 2048 and -(-M // 64) * -(-N // 64) <= 128)
                                  or (80 < M <= 320 and K >= 256 and (N <= 4096 or K >= 2 * N)))
        p = plan(lib, M, N, K)
        need = lib.spec_fp8_gemm_workspace_bytes(M, N, K)
        if required:
            assert need > 0, (M, N, K)
        refused = required and p.splits > 1
        assert gemm_status(lib, M, N, K) == (WORKSPACE if refused else HIP), (M, N, K, p)
        assert gemm_status(lib, M, N, K, 0x1000, max(need, 1) - 1) == (WORKSPACE if refused else HIP)
        assert gemm_status(lib, M, N, K, 0x1008, need) == (ALIGN if refused else HIP)
        seen[required, p.splits > 1] += 1
    assert seen[True, True] and seen[True, False] and seen[False, True]
    assert plan(lib, 320, 4096, 4096).splits == 1 and lib.spec_fp8_gemm_workspace_bytes(320, 4096, 4096) > 0


def test_the_unrolled_planner_finds_what_a_search_finds(lib):
    out = (ctypes.c_int64 * 2)()
    rng = random.Random(5)
    for i in range(12000):
        M = int(round(2 ** rng.uniform(0, 13)))
        N, K = int(round(2 ** rng.uniform(3, 17.2))), 128 * int(round(2 ** rng.uniform(0, 7)))
        for epilogue, may_split in ((PLAIN, True), (PLAIN, False), (STATS, True), (SILU, True)):
            N8 = N if epilogue != SILU else N // 16 * 16 + 16
            lib.test_plan_search(M, N8, K, epilogue, int(may_split), out)
            p = plan(lib, M, N8, K, epilogue, may_split)
            if p.m_tiles * p.n_tiles * 4 <= 4096 or out[1] == 1:         # (beyond the tickets no plan splits)
                assert (p.kind, p.splits) == tuple(out), (M, N8, K, epilogue, may_split)


@pytest.mark.parametrize("M,N,K", [(64, 4096, 14336), (80, 4096, 14336), (320, 4096, 14336)])
def test_planning_is_short(lib, M, N, K):
    """A plan is on the host path of every call (about 3 us in all)."""
    reps, best = 2000, 1e9
    for _ in range(20):
        t = time.perf_counter()
        lib.test_plan_many(M, N, K, PLAIN, reps)
        best = min(best, time.perf_counter() - t)
    assert best / reps < 0.4e-6, best / reps


@pytest.mark.parametrize("epilogue,shapes", [
    (SILU, gemm_shapes.SILU), (STATS, gemm_shapes.STATS), (PLAIN, gemm_shapes.SPLIT)], ids=["silu", "stats", "split"])
def test_parity_shapes_reach_their_kernels(lib, epilogue, shapes):
    for (M, N, K), want in shapes:
        p = plan(lib, M, 2 * N if epilogue == SILU else N, K, epilogue)
        assert (p.kind, p.splits, p.krot) == want, (M, N, K, p)


def test_every_kernel_has_a_parity_shape(lib):
    """Each kind and epilogue that a plan can reach, K split and staggered
    starts among them, is named by a parity test."""
    from tests.test_gpu_gemm_tiles import SHAPES
    plain = {(p.kind, p.splits > 1) for p in (plan(lib, *s) for s in SHAPES)}
    assert {k for k, split in plain if not split} == set(range(13))
    assert {w[0] for _, w in gemm_shapes.SPLIT} | {k for k, split in plain if split} >= {3, 4, 5, 6, 7, 8, 9, 10, 11, 12}
    named = {(e, w[0], w[2]) for e, t in ((SILU, gemm_shapes.SILU), (STATS, gemm_shapes.STATS)) for _, w in t}
    rng = random.Random(9)
    for _ in range(20000):
        M = int(round(2 ** rng.uniform(0, 12)))
        N, K = 16 * int(round(2 ** rng.uniform(1, 13))), 128 * int(round(2 ** rng.uniform(0, 7)))
        for e in (SILU, STATS):
            p = plan(lib, M, N, K, e)
            assert (e, p.kind, p.krot) in named, (e, M, N, K, p)
        p = plan(lib, M, N, K)
        assert p.splits == 1 or p.kind >= 3, (M, N, K, p)
