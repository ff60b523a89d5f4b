"""Host and device memory by the HIP runtime's own log of a child process: the
allocation-free cut entry point makes no allocating call, device or pinned host
memory, not even as a process's first call into the library, and what the library
keeps from threads that have ended is given back by sclap_trim_memory."""
import os
import re
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CHILD = """
import ctypes, os
import numpy as np
import paper_1404_4797_amd as sc

L = sc.load()

def device(a):  # HIP's own entry points, found through the library
    p = ctypes.c_void_p()
    assert L.hipMalloc(ctypes.byref(p), ctypes.c_size_t(a.nbytes)) == 0
    assert L.hipMemcpy(p, ctypes.c_void_p(a.ctypes.data), ctypes.c_size_t(a.nbytes), 1) == 0
    return p

n = 4096  # a ring
xadj = device(2 * np.arange(n + 1, dtype=np.int64))
adj = device(np.stack([(np.arange(n) - 1) % n, (np.arange(n) + 1) % n], 1).astype(np.int32))
part = device((np.arange(n) // 1024).astype(np.int32))
g = sc.Graph(n, xadj, adj, None, None)
cut, bw = ctypes.c_int64(0), np.zeros(4, dtype=np.int64)
for call in ("sclap_cut_dev_noalloc", "sclap_cut_dev"):
    os.write(2, ("BEGIN %s\\n" % call).encode())
    st = getattr(L, call)(ctypes.byref(g), part, 4, ctypes.addressof(cut), bw.ctypes.data, None)
    os.write(2, ("END %s\\n" % call).encode())
    assert st == 0 and cut.value == 4 and bw.tolist() == [1024] * 4

import threading

def work():
    c, b = ctypes.c_int64(0), np.zeros(4, dtype=np.int64)
    assert L.sclap_cut_dev(ctypes.byref(g), part, 4, ctypes.addressof(c), b.ctypes.data, None) == 0

os.write(2, b"BEGIN threads\\n")
for _ in range(2):  # the second thread takes over what the first one left
    t = threading.Thread(target=work)
    t.start()
    t.join()
os.write(2, b"END threads\\n")
os.write(2, b"BEGIN trim\\n")
assert L.sclap_trim_memory() == 0
os.write(2, b"END trim\\n")
work()
assert L.sclap_trim_memory() == 0
"""


@pytest.fixture(scope="module")
def calls():
    """The HIP calls that the child's log shows between BEGIN and END of a name."""
    import paper_1404_4797_amd as m
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    m.load()
    r = subprocess.run([sys.executable, "-c", CHILD], cwd=ROOT, capture_output=True, text=True, timeout=100,
                       env={**os.environ, "AMD_LOG_LEVEL": "3"})
    assert r.returncode == 0, r.stderr[-2000:]

    def between(name):
        text = r.stderr[r.stderr.index("BEGIN %s\n" % name):r.stderr.index("END %s\n" % name)]
        return re.findall(r"\b(hip\w+) ?\(", text)
    return between


def test_first_call_allocates_nothing(calls):
    assert any("Malloc" in c for c in calls("sclap_cut_dev"))  # the log shows such calls
    seen = calls("sclap_cut_dev_noalloc")
    assert any("Launch" in c for c in seen) and not any("Alloc" in c or "Malloc" in c for c in seen), seen


def test_trim_frees_what_ended_threads_left(calls):
    assert calls("threads").count("hipHostMalloc") == 1 and "hipHostFree" not in calls("threads")
    assert calls("trim").count("hipHostFree") == 1
