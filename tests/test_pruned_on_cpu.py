"""The layer step over the candidates that can still be minimal (csrc/gbmw_pruned.h) on the CPU: its
source compiled for the host, a fiber per lane (tests/host_wave), under AddressSanitizer, against
the oracle bit for bit.  No GPU: an access out of range ends a child process here, not a device."""
import os
import subprocess

import numpy as np
import pytest

import gbmw_inputs as gi
import oracle
import pins

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2307_02031_amd", "csrc")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    exe = tmp_path_factory.mktemp("host_wave") / "pruned"
    src = os.path.join(HERE, "host_wave")
    # no stack instrumentation: the fibers' stacks are not the sanitizer's
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-w", "-ffp-contract=off", "-fsanitize=address",
                    "--param", "asan-stack=0", "-D__HIPCC__", "-I", src, "-I", CSRC, os.path.join(src, "pruned.cpp"),
                    "-o", str(exe)], check=True)
    return exe


def run(program, tmp_path, p, unit, records):
    """Tables and records of one instance; unit: groups of 64 budgets per wave (0: four waves share one)."""
    L, S, E = int(p.L[0]), p.S, p.E
    src, dst = tmp_path / "in", tmp_path / "out"
    with open(src, "wb") as f:
        np.array([S, E, L, unit, records], np.int32).tofile(f)
        for a, t in ((p.c, np.float32), (p.M, np.int32), (p.R, np.float32)):
            np.ascontiguousarray(a, t).tofile(f)
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0:halt_on_error=1")
    r = subprocess.run([str(program), str(src), str(dst)], env=env, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[:3000]
    with open(dst, "rb") as f:
        C = np.fromfile(f, np.float32, L * (E + 1) * S).reshape(L, E + 1, S)
        A = np.fromfile(f, np.uint8, L * (E + 1) * S).reshape(L, E + 1, S)
    return C, A


def check(program, tmp_path, p, unit, records):
    C, A = run(program, tmp_path, p, unit, records)
    ref = oracle.solve_problem(p, 0, keep_C=True, keep_A=True, nthreads=4)
    for l in range(int(p.L[0])):
        pins.assert_same_f32(C[l], ref.C[l], f"{p.name} unit {unit} records {records} C layer {l}")
        assert np.array_equal(A[l], ref.A[l]), f"{p.name} unit {unit} records {records} A layer {l}"


SHAPES = [(0, 1), (0, 0), (1, 1), (4, 0), (4, 1)]         # (groups per wave, records)


@pytest.mark.parametrize("S", [17, 40, 64, 70, 130, 255])
def test_a_group_that_no_plan_reaches_yet(program, tmp_path, S):
    """The two words of a column speak for 64 budgets of their own, which may end beyond the group that
    reads them: every column can look like a candidate although none is finite up to the group's end.
    More of them than a wave keeps go to the whole workgroup, whose second look then leaves none."""
    for first, then, E in ((70, 60, 300), (40, 30, 200), (70, 60, 127), (40, 30, 100)):   # the last group whole / cut by E
        p = gi.random_instance(7000 + S, 4, S, E, M_rng=(1, 9), R_rng=(0.0, 4.0))
        p.M[0], p.M[1] = first, then
        for unit, records in SHAPES[:4]:
            check(program, tmp_path, p, unit, records)


def broken(S, seed):
    """Inputs that a solve refuses once it has run (device arrays are checked by its own kernels)."""
    st = gi.Stream(40 + seed)
    p = gi.random_instance(7300 + S + seed, 4, S, 600, M_rng=(0, 3), R_rng=(0.0, 4.0))
    p.M[0] = 70
    if seed == 0:
        p.R[2] = np.nan                                   # more columns start to fit in a group than a wave keeps
    else:
        what = np.array([np.nan, -np.inf, np.inf, -1e30, -0.0, 1e38], np.float32)
        for a, n in ((p.c.reshape(-1), 2 * seed), (p.R.reshape(-1), p.R.size // 2 ** seed)):
            a[st.integers(n, 0, a.size - 1)] = what[st.integers(n, 0, 5)]
        bad = np.array([-1, -2 ** 31, 2 ** 31 - 1, 601, 64], np.int64)
        p.M.reshape(-1)[st.integers(6, 0, p.M.size - 1)] = bad[st.integers(6, 0, 4)]
        p.R[2, st.integers(S // 2, 0, S - 1)] = np.nan
    return p


@pytest.mark.parametrize("S", [12, 40, 70, 130])
def test_refused_inputs_are_read_and_written_in_range(program, tmp_path, S):
    """NaN, negative and infinite costs and memories out of every range: whatever the values are, no
    kernel leaves its buffers (the results are not looked at, the library hands none out)."""
    for seed in range(5):
        for unit, records in SHAPES:
            run(program, tmp_path, broken(S, seed), unit, records)


def signed_zeros(S, L, E, seed):
    rs = np.random.RandomState(seed)
    p = gi.random_instance(seed, L, S, E, M_rng=(0, 70), R_rng=(0.0, 1.0))
    p.c[:] = np.where(rs.rand(*p.c.shape) < 0.5, np.float32(-0.0), np.where(rs.rand(*p.c.shape) < 0.6, np.float32(0.0), p.c))
    p.R[:] = np.where(rs.rand(*p.R.shape) < 0.7, np.float32(-0.0), p.R)
    return p


@pytest.mark.parametrize("S", [9, 33, 65, 129])
def test_the_sign_of_a_zero_is_the_lowest_index_s(program, tmp_path, S):
    """Costs of -0.0 are accepted; 0.0 and -0.0 are equal candidates, and the sum of the lowest index is
    kept with its sign, also where that changes inside a group that begins and ends alike."""
    for seed, E in ((1, 5), (2, 127), (3, 500)):
        for unit, records in ((0, 1), (1, 0), (4, 1)):
            check(program, tmp_path, signed_zeros(S, 4, E, 100 * S + seed), unit, records)
