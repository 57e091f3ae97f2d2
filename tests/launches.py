"""What the library's calls launch, without a GPU: the runtime's launch call is replaced (launch_shim.c) in a child process that
makes the calls; pointers are never read."""
import functools
import json
import os
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))

# (ctypes alone, so that nothing else uses the replaced calls)
CHILD = """
import ctypes, json, re, sys
lib = ctypes.CDLL(sys.argv[1])
shim = ctypes.CDLL(None)
shim.shim_name.restype = ctypes.c_char_p
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
out = []
for args, every in json.loads(sys.stdin.read()):
    shim.shim_reset(0)
    status = call(*args)
    made = shim.shim_made()
    names = [re.search("k_[a-z_]*[a-z]", shim.shim_name(i).decode()).group() for i in range(made)]
    rows = []
    for fail in range(1, made + 1 if every else 0):
        shim.shim_reset(fail)
        rows.append((fail, call(*args), shim.shim_made()))
    out.append((status, names, rows))
print(json.dumps(out))
"""


@functools.lru_cache(maxsize=None)
def _shim():
    shim = os.path.join(tempfile.mkdtemp(), "launch_shim.so")
    subprocess.check_call(["gcc", "-O1", "-shared", "-fPIC", "-o", shim, os.path.join(HERE, "launch_shim.c")])
    return shim


def launches(calls, every_failure=False):
    """calls: (kind, n, d, n_segments, k, flag) each.  For each (status, names of the kernels launched, and with every_failure one (number of the
    launch that failed, status, launches made) per launch)."""
    from paper_2511_10442_amd import binding
    binding.lib()                                        # built if it is not there
    r = subprocess.run([sys.executable, "-c", CHILD, binding.LIB_PATH], input=json.dumps([(c, every_failure) for c in calls]), capture_output=True,
                       text=True, env=dict(os.environ, LD_PRELOAD=_shim()), timeout=100)
    assert r.returncode == 0, r.stdout + r.stderr
    return json.loads(r.stdout.splitlines()[-1])
