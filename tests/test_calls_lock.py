"""The interpreter lock in the native marshalling: it is not held while the library runs or memory is allocated, and a thread that
cannot have it back because the interpreter ends goes quietly.  csrc/nm_calls.cpp is compiled for CPU tensors (the device's name exchanged in
its text) beside a library whose entries only look at the lock; each test is a process of its own."""
import os
import subprocess
import sys
import sysconfig

import pytest

from paper_2409_09708_amd import build as nm_build

LIBRARY = r"""
#include <unistd.h>
#include <atomic>
#include <stdexcept>
#include <c10/core/CPUAllocator.h>
static std::atomic<int> entered{0}, held{0};
extern "C" int look_pause = 0;  // microseconds
extern "C" int looks() { return entered; }
extern "C" int looks_held() { return held; }
extern "C" int look() {
  held += PyGILState_Check();
  ++entered;
  if (look_pause) usleep(look_pause);
  return 0;
}
struct Allocator final : c10::Allocator {  // of every tensor, those that Python makes among them
  c10::Allocator* plain = c10::GetCPUAllocator();
  c10::DataPtr allocate(size_t n) override {
    look();
    if (n > 1000000) throw std::runtime_error("no memory of that size");
    return plain->allocate(n);
  }
  void copy_data(void* to, const void* from, size_t n) const override { plain->copy_data(to, from, n); }
};
extern "C" void look_at_allocations() { c10::SetCPUAllocator(new Allocator, 255); }
extern "C" size_t kilobyte() { return 1024; }
"""

SETUP = r"""
import ctypes, importlib.machinery, importlib.util, sys, threading, time
import torch
path = sys.argv[1]
loader = importlib.machinery.ExtensionFileLoader("_nm_calls", path)
calls = importlib.util.module_from_spec(importlib.util.spec_from_loader("_nm_calls", loader))
loader.exec_module(calls)
own = ctypes.CDLL(path)
at = lambda name: ctypes.cast(getattr(own, name), ctypes.c_void_p).value
table = {n: at("look") for n in ("nm_prune", "nm_prune_scored", "nm_pack", "nm_unpack", "nm_linear_forward",
                                 "nm_linear_forward_prepared", "nm_linear_forward_static")}
table.update(nm_values_bytes=at("kilobyte"), nm_index_bytes=at("kilobyte"), nm_spmm_workspace_bytes=at("kilobyte"))
def raise_status(status):
    raise RuntimeError(status)
calls.bind(table, raise_status, lambda nbytes, device, stream: torch.empty(nbytes, dtype=torch.uint8))
class Stream:
    cuda_stream = 0
s = Stream()
W, words = torch.zeros(8, 64, dtype=torch.bfloat16), torch.zeros(8, 4, dtype=torch.int32)
score = W.float()
def prune():
    return calls.prune(W, 2, 4, None, s)
def forward():
    return calls.forward(W, words, 64, 2, 4, W, None, None, None, None, s, 0)
"""


@pytest.fixture(scope="module")
def cpu_edition(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("calls")
    with open(os.path.join(nm_build.CSRC, "nm_calls.cpp")) as f:
        text = f.read().replace("CUDA", "CPU").replace("is_cuda", "is_cpu")
    source, out = str(tmp / "nm_calls.cpp"), str(tmp / "_nm_calls.so")
    with open(source, "w") as f:
        f.write(text + LIBRARY)
    nm_build.compile_calls(source, out)
    return out


def run(path, script):
    return subprocess.run([sys.executable, "-c", SETUP + script, path], capture_output=True, text=True, timeout=120)


@pytest.mark.parametrize("call", ["prune", "forward"])
def test_thread_in_a_call_while_the_interpreter_ends(cpu_edition, call):
    """The thread's call returns after the interpreter has begun to end, and while that still goes on."""
    done = run(cpu_edition, f"call = {call}\n" + r"""
class Last:
    def __del__(self, wait=time.sleep):
        wait(2)
        print("ended", flush=True)
last = Last()
ctypes.c_int.in_dll(own, "look_pause").value = 1000000
threading.Thread(target=call, daemon=True).start()
while not own.looks():
    time.sleep(0.01)
""")
    assert done.returncode == 0 and "ended" in done.stdout, (done.returncode, done.stderr[-500:])


def test_allocations_and_library_calls_release_the_lock(cpu_edition):
    done = run(cpu_edition, r"""
own.look_at_allocations()
for call, looks in ((prune, 2), (lambda: calls.prune_scored(score, 2, 4, s), 2), (lambda: calls.pack(W, 2, 4, None, s), 3),
                    (lambda: calls.unpack(W, words, 128, 2, 4, s), 2), (forward, 3)):
    before = own.looks()
    assert call() is not NotImplemented
    assert (own.looks() - before, own.looks_held()) == (looks, 0), (own.looks() - before, own.looks_held())
try:  # a refused allocation arrives as an exception, and the thread has the lock again
    calls.unpack(W, words, 1 << 30, 2, 4, s)
except RuntimeError as e:
    assert "no memory of that size" in str(e)
    print("raised")
prune()
""")
    assert done.returncode == 0 and "raised" in done.stdout, (done.returncode, done.stderr[-500:])
