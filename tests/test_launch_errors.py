"""A launch that fails, at every place of every chain of launches: the call says so, and nothing that would have run on what that launch did not
write is launched after it.  The runtime's launch call is replaced (launch_shim.c): no GPU, no kernel runs, pointers are never read."""
import ctypes
import json
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
FG_ERR_LAUNCH = 5

CHAINS = {
    "all pairs": ("knn", 1000, 3, 1, 10, 0),
    "group kernel": ("knn", 6000, 4, 1, 20, 0),
    "group kernel, two passes": ("knn", 20000, 8, 1, 100, 0),
    "few points, votes": ("knn", 24000, 3, 4, 12, 0),
    "few tiles": ("knn", 60000, 3, 1, 16, 0),
    "tile or group kernel": ("knn", 100000, 4, 2, 40, 0),
    "tile or group kernel, two passes": ("knn", 100000, 3, 1, 100, 0),
    "ranked": ("knn", 1000000, 3, 10, 32, 0),
    "ordered, leaf and tile kernel": ("knn", 1200000, 2, 5, 16, 0),
    "ordered, two passes": ("knn", 1200000, 2, 5, 80, 0),
    "leaf kernel": ("knn", 200000, 8, 1, 64, 0),
    "leaf kernel, two passes": ("knn", 300000, 6, 1, 70, 0),
    "leaf kernel, direction flags": ("knn", 200000, 6, 1, 70, 1),
    "tile kernel, direction flags": ("knn", 100000, 4, 2, 40, 1),
    "counted": ("counted", 100000, 3, 1, 20, 0),
    "backward, binned": ("bwd", 20000, 3, 1, 16, 1),
    "backward, plain": ("bwd", 20000, 3, 1, 16, 0),
    "index matrices": ("oc", 20000, 0, 2, 16, 1),
    "index matrices without scratch": ("oc", 20000, 0, 2, 16, 0),
}

# (child: ctypes alone, so that nothing else uses the replaced calls)
CHILD = """
import ctypes, json, sys
lib = ctypes.CDLL(sys.argv[1])
shim = ctypes.CDLL(None)
i32, i64, sz = ctypes.c_int32, ctypes.c_int64, ctypes.c_size_t
P = lambda: ctypes.c_void_p(1 << 20)
big = sz(1 << 40)
def call(kind, n, d, s, k, flag):
    if kind == "knn":
        return lib.fg_binned_select_knn_dir(P(), P(), P() if flag else None, i64(n), i32(d), i32(s), i32(k), i32(0), i32(0), P(), P(), P(), big, None)
    if kind == "counted":
        return lib.fg_binned_select_knn_counted(P(), P(), i64(n), i32(d), i32(s), i32(k), i32(0), i32(0), P(), P(), P(), P(), big, None)
    if kind == "bwd":
        return lib.fg_knn_backward(P(), P(), P(), P() if flag else None, i64(n), i32(d), i32(s), i32(k), P(), P() if flag else None, big, None)
    return lib.fg_oc_helper(P(), P(), P(), P(), i64(n), i64(40), i32(s), i32(100), i32(n // s), i32(1), i32(1), P(), P(), P() if flag else None, big, None)
out = {}
for name, args in json.loads(sys.argv[2]).items():
    rows = []
    fail = 0
    while True:
        shim.shim_reset(fail)
        status = call(*args)
        rows.append((fail, status, shim.shim_made()))
        fail += 1
        if fail > rows[0][2]: break
    out[name] = rows
print(json.dumps(out))
"""


@pytest.fixture(scope="module")
def answers(tmp_path_factory):
    from paper_2511_10442_amd import binding
    binding.lib()                                        # built if it is not there
    shim = str(tmp_path_factory.mktemp("shim") / "launch_shim.so")
    subprocess.check_call(["gcc", "-O1", "-shared", "-fPIC", "-o", shim, os.path.join(HERE, "launch_shim.c")])
    r = subprocess.run([sys.executable, "-c", CHILD, binding.LIB_PATH, json.dumps(CHAINS)], capture_output=True, text=True,
                       env=dict(os.environ, LD_PRELOAD=shim), timeout=100)
    assert r.returncode == 0, r.stdout + r.stderr
    return json.loads(r.stdout.splitlines()[-1])


@pytest.mark.parametrize("name", list(CHAINS))
def test_first_error_ends_the_chain(answers, name):
    rows = answers[name]
    assert rows[0][1] == 0 and rows[0][2] >= 1, rows[0]
    for fail, status, made in rows[1:]:
        assert status == FG_ERR_LAUNCH and made == fail, "launch %d of %d failed: status %d, %d launches" % (fail, rows[0][2], status, made)
