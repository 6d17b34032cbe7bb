"""Set-up when device memory runs short, on the host: libdcg.so linked with a
HIP runtime whose device memory is host memory under a capacity and whose
kernels do nothing (tests/native), so that allocations can be made to fail one
by one.

The dense matrices of the coarse cycles are optional: a set-up that cannot have
one (128 MiB, and 805 MB of scratch where it is made by products) succeeds
without it and holds what it would hold otherwise.  A set-up that fails gives
back all it took and leaves nothing that a later one holds twice."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
NATIVE = os.path.join(ROOT, "tests", "native")
PKG = os.path.join(ROOT, "paper_2606_13429_amd")
MATRIX = 4096 * 4096 * 8
OK, ENOMEM = 0, -2


@pytest.fixture(scope="session")
def program(tmp_path_factory):
    lib = os.path.join(PKG, "libdcg.so")
    if not os.path.exists(lib):
        pytest.skip("libdcg.so is not built")
    exe = str(tmp_path_factory.mktemp("alloc") / "alloc_main")
    subprocess.run(["g++", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    os.path.join(NATIVE, "fake_hip.cpp"), os.path.join(NATIVE, "alloc_main.cpp"), "-o", exe,
                    "-rdynamic", "-Wl,--unresolved-symbols=ignore-in-shared-libs", lib, "-Wl,-rpath," + PKG,
                    "-lpthread", "-ldl"], check=True)

    def run(*args):
        out = subprocess.run([exe] + [str(a) for a in args], check=True, capture_output=True, text=True,
                             timeout=120).stdout
        return {k: int(v) for k, v in (line.split() for line in out.splitlines())}
    return run


def _clean(r):
    assert r["clean_status"] == OK and r["clean_left"] == 0
    assert r["left_bytes"] == 0 and r["left_objects"] == 0 and r["bad_frees"] == 0 and r["device"] == 0


# the set-ups that keep a matrix
SETUPS = [("omg", 32), ("3d", 16), ("fp64", 64), ("mixed", 64)]


@pytest.mark.parametrize("what,n", SETUPS)
@pytest.mark.parametrize("short", [1, MATRIX])
def test_setup_without_the_memory_of_the_matrix(program, what, n, short):
    r = program("room", what, n, short)
    assert r["clean_matrices"] == 1
    assert r["status"] == OK and r["matrices"] == 0 and r["last_error"] == 0
    # the FP64 inverses that the mixed form makes its matrix with may be there or not
    slack = 4 << 20 if what == "mixed" else 0
    assert r["clean_bytes"] - MATRIX - slack <= r["bytes"] <= r["clean_bytes"] - MATRIX
    _clean(r)


@pytest.mark.parametrize("what,n,calls", [
    ("omg", 32, (0, 20, 70)), ("3d", 16, (0, 10, 40)), ("fp64", 64, (0, 12, 25, 27, 50)),
    ("mixed", 64, (0, 12, 24, 27, 30, 50))])
def test_a_failed_setup_gives_everything_back(program, what, n, calls):
    r = program("fail", what, n, *calls)
    assert r["refused"] == r["again_ok"] == r["again_equal"] == len(calls)
    _clean(r)


GIB = 1 << 30


@pytest.mark.parametrize("n,fp32,budget,matrix", [
    (64, 0, 0, 0),               # what dcg_server_group_bytes says
    (64, 1, 0, 0),
    (64, 1, 2 * GIB - 1, 0),     # below 16 matrices
    (64, 0, 2 * GIB, 1),
    (64, 1, 2 * GIB, 1),
    (32, 0, 2 * GIB, 0),         # two levels
    (512, 1, 0, 0),              # a group above 2 GiB that fits without the matrix only
])
def test_server_admits_what_group_bytes_says(program, n, fp32, budget, matrix):
    """The matrix is no part of what a group needs: a budget of dcg_server_group_bytes
    holds the group at every size, and with room for it the cycles use it."""
    r = program("budget", n, fp32, budget)
    assert r["status"] == OK
    assert (r["products"] > 0) == bool(matrix)
    assert r["left_bytes"] == 0 and r["left_objects"] == 0 and r["bad_frees"] == 0


def test_matrices_make_room_for_a_group(program):
    """A third group that fits beside two running ones without their matrices is
    admitted while they run."""
    r = program("shared", 2 * GIB)
    assert r["taken"] == 1
    assert r["admitted"] == 1 and r["running"] == 2
    assert r["over_budget"] <= 0
    assert r["status_64"] == r["status_128"] == r["status_256"] == OK
    assert r["left_bytes"] == 0 and r["left_objects"] == 0 and r["bad_frees"] == 0


GROUP_256_VECTORS = 7            # as large as a matrix each


def test_matrix_goes_with_the_group_that_was_charged_for_it(program):
    """Freed with its group, also where a handle without a matrix holds the mesh."""
    r = program("evicted", 2 * GIB)
    assert r["handle"] == r["status"] == r["status_256"] == r["status_again"] == OK
    assert r["with_64"] == 1 and r["with_256"] == 2 + GROUP_256_VECTORS
    assert r["after"] == 1 + GROUP_256_VECTORS
    assert r["left_bytes"] == 0 and r["left_objects"] == 0 and r["bad_frees"] == 0


def test_prepared_matrix_stays_within_the_budget(program):
    """What prepare() made is freed when the group that comes has no room for it."""
    r = program("prepared", 2 * GIB)
    assert r["status_256"] == r["status_128"] == r["prepare"] == r["status"] == OK
    assert r["before"] == 1 + GROUP_256_VECTORS and r["prepared"] == r["before"] + 1
    assert r["after"] == GROUP_256_VECTORS
    assert r["over_budget"] <= 0
    assert r["left_bytes"] == 0 and r["left_objects"] == 0 and r["bad_frees"] == 0


@pytest.mark.parametrize("started", [0, 3])
def test_set_up_where_threads_cannot_be_started(program, started):
    r = program("threads", started)
    assert r["clean_status"] == r["status"] == OK and r["equal"] == 1
