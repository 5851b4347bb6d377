"""Runs calls of the library on a recording HIP runtime (hip_record.cpp), in a process of their own: which kernels
they launch and which copies they make, without a GPU."""
import json
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))

PRELUDE = """
import ctypes, json, sys
stub = ctypes.CDLL(sys.argv[1], ctypes.RTLD_GLOBAL)
stub.record_take.restype = ctypes.c_char_p
sys.path.insert(0, sys.argv[2])
import paper_2407_04656_amd as lz
def fail_launch(after):
    stub.record_fail_launch(after)
def calls():
    return stub.record_take().decode().splitlines()
class At:
    "A tensor as the binding sees one: an address."
    def __init__(self, address): self.address = address
    def data_ptr(self): return self.address
    def is_contiguous(self): return True
def code(f, *args, **kw):
    try:
        f(*args, **{'stream': 0, **kw})
    except lz.LzError as e:
        return e.code
    return 0
calls()
"""


def recorded(tmp_path, body):
    """Runs `body`, which has `lz`, `At(address)`, `calls()` (what was asked since the last time), `code(call, ...)` (its status) and
    `fail_launch(n)` (the launch after n more fails), and assigns `out`; returns `out`."""
    so = os.path.join(str(tmp_path), "hip_record.so")
    if not os.path.exists(so):
        subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-o", so, os.path.join(HERE, "hip_record.cpp")], check=True)
    text = PRELUDE + body + "\nprint('\\n' + json.dumps(out))\n"
    done = subprocess.run([sys.executable, "-c", text, so, os.path.dirname(HERE)], capture_output=True, text=True, timeout=300)
    assert done.returncode == 0, done.stderr
    return json.loads(done.stdout.splitlines()[-1])
