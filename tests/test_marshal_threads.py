"""The native marshalling on the CPU: its source built once more for tensors on the CPU, calling functions of this test."""
import os
import subprocess
import sys

import pytest

from paper_2603_05353_amd import build

FUNCTIONS = r"""
#include <atomic>
#include <cstdlib>
#include <new>
#include <unistd.h>
static std::atomic<int> entered{0};
extern "C" int slow(void *, void *, const int *, long, int) { entered = 1; usleep(400000); return 0; }
extern "C" int throwing(void *, void *, const int *, long, int) { throw std::bad_alloc(); }
extern "C" int is_entered() { return entered; }
extern "C" void linger_at_exit() { atexit([] { usleep(1500000); }); }
"""

PROGRAM = """
import ctypes, importlib.machinery, importlib.util, sys, threading, time
import torch
loader = importlib.machinery.ExtensionFileLoader("_ifkv_marshal", sys.argv[1])
marshal = importlib.util.module_from_spec(importlib.util.spec_from_file_location("_ifkv_marshal", sys.argv[1], loader=loader))
loader.exec_module(marshal)
lib = ctypes.CDLL(sys.argv[2])
address = lambda f: ctypes.cast(f, ctypes.c_void_p).value
x, pos = torch.zeros(3, 2, 64), torch.zeros(3, dtype=torch.int32)
caller = lambda f: marshal.Caller(1, False, 4, 2, 64, 128, 64, *[address(f)] * 7)
"""

DAEMON = PROGRAM + """
lib.linger_at_exit()  # the process is still there when the thread comes back
threading.Thread(target=caller(lib.slow).rope_rows, args=(x, pos), daemon=True).start()
while not lib.is_entered():
    time.sleep(0.01)
print("leaves", flush=True)
"""

THROWS = PROGRAM + """
try:
    caller(lib.throwing).rope_rows(x, pos)
except RuntimeError as e:
    print("leaves", e, flush=True)
"""


@pytest.fixture(scope="module")
def built(tmp_path_factory):
    d = tmp_path_factory.mktemp("marshal")
    with open(os.path.join(build.CSRC, "marshal.cpp")) as f:
        text = f.read()
    assert text.count("t.is_cuda()") == 1
    src, module, functions = str(d / "marshal_cpu.cpp"), str(d / "_ifkv_marshal.so"), str(d / "functions.so")
    with open(src, "w") as f:
        f.write(text.replace("t.is_cuda()", "t.is_cpu()"))
    r = subprocess.run(build.marshal_command(src, module), capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run(["g++", "-shared", "-fPIC", "-x", "c++", "-", "-o", functions], input=FUNCTIONS, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    return module, functions


@pytest.mark.parametrize("program", [DAEMON, THROWS], ids=["a-daemon-thread-that-comes-back-after-the-end", "a-call-that-throws"])
def test_what_unwinds_does_not_abort_the_process(built, program):
    """A thread that returns from the library while the interpreter ends is taken off its stack, as out of a ctypes call; a C++
    exception becomes a Python one."""
    r = subprocess.run([sys.executable, "-c", program, *built], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.startswith("leaves"), (r.returncode, r.stdout, r.stderr[-2000:])
