"""The library's host code without a GPU, on a HIP runtime that only records (recorded_hip.c): what a call leaves behind when one of
its HIP calls fails, and what it launches."""
import json
import os
import subprocess
import sys

import pytest

from paper_2511_15898_amd.build import LIB_PATH, build_library

HERE = os.path.dirname(os.path.abspath(__file__))

# Runs in a process of its own: its HIP symbols must come before those of any runtime that is loaded already.
PROGRAM = r'''
import ctypes as C, json, sys
hip = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
hip.recorded_log.restype = C.c_char_p
lib = C.CDLL(sys.argv[2])

def create(B, V, k, n):
    h = C.c_void_p()
    assert lib.gr_create(C.byref(h), B, V, k, n, None) == 0
    return h
def log():
    return hip.recorded_log().decode().split("\n")[:-1]
def buffer(n):
    return (C.c_double * n)()

def walk(h, S, K, L, V, k):
    rows = buffer(S * K * L * V // 2 + 1)
    ints = [(C.c_int * (S * L))() for _ in range(4)]
    return lib.gr_tree_walk(h, rows, rows, None, (C.c_int * (S * K * L))(), (C.c_float * (S * L))(), S, K, L, V, k, C.c_float(1e-4), *ints, None)
def solve(h, B, V, n, k):
    rows, out = buffer(B * V // 2 + 1), buffer(B)
    return lib.gr_solve(h, rows, rows, n, k, C.c_float(1e-4), B, V, out, out, None)
def verify(h, B):
    return lib.gr_verify(h, buffer(64 * B), buffer(B), buffer(B), buffer(B), None)
def sweep(h, B, V, ks, ns):
    rows, out = buffer(B * V // 2 + 1), buffer(B * 128)
    return lib.gr_accept_sweep(h, rows, rows, (C.c_int * len(ks))(*ks), len(ks), (C.c_int * len(ns))(*ns), len(ns), B, V, out, out, None)

result = {}
exec(sys.argv[3])
print(json.dumps(result))
'''


@pytest.fixture(scope="module")
def recorded(tmp_path_factory):
    if not os.path.exists(LIB_PATH):
        build_library()
    so = str(tmp_path_factory.mktemp("recorded") / "librecorded_hip.so")
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-o", so, os.path.join(HERE, "recorded_hip.c")], check=True)

    def run(body):
        r = subprocess.run([sys.executable, "-c", PROGRAM, so, LIB_PATH, body], capture_output=True, text=True, timeout=120)
        assert r.returncode == 0, r.stdout + r.stderr
        return json.loads(r.stdout)
    return run


@pytest.mark.parametrize("V, k", [(1024, 32), (1024, 300)])
@pytest.mark.parametrize("call, after", [("to_host", 0), ("synchronize", 0), ("to_device", 0)])
def test_a_walk_that_fails_leaves_no_policy_and_nothing_in_flight(recorded, V, k, call, after):
    """A batch of a walk is read through row offsets, so what it leaves in the handle is no policy of the caller's rows; and the
    staging that its copies use belongs to the next call."""
    r = recorded(f"""
h = create(4, {V}, {k}, 3)
result["whole"] = walk(h, 4, 3, 2, {V}, {k})
hip.recorded_clear()
hip.recorded_fail(b"{call}", {after})
result["rc"] = walk(h, 4, 3, 2, {V}, {k})
result["log"] = log()
result["verify"] = verify(h, 4)
""")
    EHIP, ESTATE = -4, -3
    assert r["whole"] == 0 and r["rc"] == EHIP
    assert r["verify"] == ESTATE
    assert r["log"][-1].startswith("synchronize"), r["log"]


@pytest.mark.parametrize("k", [32, 300])
@pytest.mark.parametrize("call", ["solve(h, 4, 1024, 3, {k})", "walk(h, 4, 3, 2, 1024, {k})", "sweep(h, 4, 1024, [10, {k}], [1, 2])", "verify(h, 4)"])
def test_a_failed_call_leaves_no_error_to_the_next(recorded, k, call):
    """Whichever of a call's launches, copies and waits fails: that call reports it, and a valid one after it does not."""
    call = call.format(k=k)
    r = recorded(f"""
h = create(4, 1024, 300, 3)
assert solve(h, 4, 1024, 3, {k}) == 0
hip.recorded_clear()
assert {call} == 0
steps, result["seen"] = log(), []
for i, line in enumerate(steps):
    name = line.split()[0]
    if name not in ("launch", "to_device", "to_host", "synchronize"):
        continue
    assert solve(h, 4, 1024, 3, {k}) == 0
    hip.recorded_clear()
    hip.recorded_fail(name.encode(), sum(x.split()[0] == name for x in steps[:i]))
    rc = {call}
    hip.recorded_clear()
    result["seen"].append([line, rc, solve(h, 4, 1024, 3, {k}), verify(h, 4)])
""")
    assert len(r["seen"]) >= 1
    for line, failed, solved, verified in r["seen"]:
        assert failed == -4 and solved == 0 and verified == 0, (line, failed, solved, verified)


def test_a_walk_without_memory_for_its_batch_goes_by_levels_and_the_next_one_asks_again(recorded):
    """Sequences of two paths, all of them the same: 4 nodes to a level, where the handle has 4 rows.  A walk of more nodes than the scratch
    holds asks for more, a smaller one for nothing."""
    r = recorded("""
h = create(4, 1024, 32, 2)
assert walk(h, 1, 1, 1, 1024, 32) == 0              # one node: staging only
def batch(S, L, fail=False):
    hip.recorded_clear()
    if fail:
        hip.recorded_fail(b"malloc", 0)
    assert walk(h, S, 2, L, 1024, 32) == 0
    rows = [int(x.split()[2]) for x in log() if x.startswith("launch") and "solve_kernel" in x]
    return rows[0], sum(x.startswith("malloc") for x in log())
result["got"] = [batch(4, 3, True), batch(4, 3), batch(4, 3), batch(4, 9), batch(4, 3)]
""")
    assert r["got"] == [[4, 1], [12, 1], [12, 0], [36, 1], [12, 0]], r


def test_a_refused_walk_leaves_the_policy_of_the_last_solve(recorded):
    r = recorded("""
h = create(4, 1024, 32, 3)
result["solve"] = solve(h, 4, 1024, 3, 32)
result["walk"] = walk(h, 4, 3, 2, 1024, 0)          # no workspace for a support this large
result["verify"] = verify(h, 4)
""")
    assert r == {"solve": 0, "walk": -1, "verify": 0}


@pytest.mark.parametrize("V, ks, launches", [(300, [10, 0], 1), (8192, [300, 0], 1), (8192, [300], 1), (8193, [10, 4096], 1), (8193, [10, 4097], 1),
                                             (70000, [300], 1), (70000, [300, 0], 1)])
def test_a_grid_launches_what_its_support_needs(recorded, V, ks, launches):
    """A grid of large supports is one launch: one that has nothing to do costs a call of few rows as much as one that has."""
    r = recorded(f"""
h = create(1, {V}, 0, 4)
hip.recorded_clear()
result["rc"] = sweep(h, 1, {V}, {ks}, [1, 2, 4])
result["log"] = log()
""")
    assert r["rc"] == 0 and all(line.startswith("launch ") for line in r["log"]), r
    assert len(r["log"]) == launches, r["log"]


@pytest.mark.parametrize("max_n", [1, 2, 3, 5, 16])
@pytest.mark.parametrize("B", [1, 256, 257, 320, 321, 448, 449])
def test_a_handle_sets_up_the_kernels_that_its_calls_launch(recorded, max_n, B):
    """A kernel with more than 64 KB of dynamic LDS needs its limit raised on the device: for every draft count of the handle, batches on
    both workgroup sizes, supports in LDS and in HBM, grids, and walks whose batches hold more rows than the handle."""
    r = recorded(f"""
h = create({B}, 600, 0, {max_n})
for n in range(1, {max_n} + 1):
    for k in (20, 300):
        assert solve(h, {B}, 600, n, k) == 0 and verify(h, {B}) == 0
assert sweep(h, {B}, 600, [10, 0], [1, 2]) == 0
if {B} == 320:
    paths = (C.c_int * (240 * {max_n} * 2))(*[i % 2 * (i // 2 % 7) for i in range(240 * {max_n} * 2)])   # one token at level 0, so two nodes a sequence
    rows, ints = buffer(240 * {max_n} * 600 + 1), [(C.c_int * 480)() for _ in range(4)]
    hip.recorded_clear()
    assert lib.gr_tree_walk(h, rows, rows, None, paths, (C.c_float * 480)(), 240, {max_n}, 2, 600, 20, C.c_float(1e-4), *ints, None) == 0
    result["batch"] = [x.split()[1:] for x in log() if "solve_kernel" in x]
result["over"] = hip.recorded_over()
""")
    assert r["over"] == 0
    if B == 320:
        # more rows than the handle, and than have a compute unit each: the small workgroup, then the large one for the rows that it leaves (of all with
        # more than 8 drafts there is one kernel)
        sizes = [512 if "Li512E" in kernel else 256 for kernel, rows in r["batch"]]
        assert sizes == ([256, 512] if max_n <= 8 else [256]) and all(rows == "480" for _, rows in r["batch"]), r["batch"]
