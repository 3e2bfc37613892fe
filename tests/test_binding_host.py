"""The Python binding's use of the interpreter lock and of its workspaces, on the CPU.

A stub (binding_stub.cpp) stands in for the stream look-up and for the library's calls,
and fake tensors for the GPU's. Each check runs in a process of its own, since a fault here ends the process.
"""

import os
import subprocess
import sys
import textwrap

import pytest
import torch
from torch.utils import cpp_extension

from paper_2608_00531_amd import build as pbuild

HERE = os.path.dirname(os.path.abspath(__file__))

PRELUDE = """
import ctypes, sys, warnings
warnings.simplefilter("ignore")                      # fake tensors' pointers
stub = ctypes.CDLL(sys.argv[1], ctypes.RTLD_GLOBAL)  # before the binding's own libraries
import torch
from torch._subclasses import FakeTensorMode
import paper_2608_00531_amd as pc
"""


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("stub") / "stub.so")
    cmd = ["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI, "-I", pbuild.INCLUDE]
    for path in cpp_extension.include_paths("cuda"):
        cmd += ["-isystem", path]
    res = subprocess.run(cmd + [os.path.join(HERE, "binding_stub.cpp"), "-o", out], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    return out


def child(stub, code, *args):
    res = subprocess.run([sys.executable, "-c", PRELUDE + textwrap.dedent(code), stub, *args],
                         cwd=os.path.dirname(HERE), capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stdout + res.stderr
    return res.stdout.split()


@pytest.mark.parametrize("name", ["margins", "margins_noalloc", "margins_accept", "margins_accept_tree",
                                  "tree_attn", "accept", "repair_tree", "commit"])
def test_tensors_without_storage_raise(stub, name):
    """A tensor under vmap has no data pointer: every call says so and the process lives."""
    out = child(stub, """
        with FakeTensorMode():
            f = lambda *s: torch.zeros(3, *s, device="cuda")
            i = lambda *s: torch.zeros(3, *s, dtype=torch.int32, device="cuda")
            x, n, t, m = f(2, 4, 16), i(2), i(2, 4), f(2, 4)
            q, k, off = f(2, 4, 2, 64), f(40, 2, 64), torch.zeros(3, 2, dtype=torch.int64, device="cuda")
            fn, args = {
                "margins": (pc.cure_margins, [x]),
                "margins_noalloc": (pc.cure_margins_noalloc, [x]),
                "margins_accept": (lambda x, t, n: pc.cure_margins_accept(x, t, t, n, n, 4), [x, t, n]),
                "margins_accept_tree": (lambda t, n: pc.cure_margins_accept(x[0], t, t, n, n, 4), [t, n]),
                "tree_attn": (lambda q, k, off, n, t: pc.cure_tree_attn(q, k, k, off, n, n, t, [8, 8], [4, 4], 1.0),
                              [q, k, off, n, t]),
                "accept": (lambda t, n: pc.cure_accept(t, t, t, n, n, 4), [t, n]),
                "repair_tree": (lambda x, m, t, n: pc.cure_repair_tree(x, m, t, n, t, 4, 2, 1.0), [x, m, t, n]),
                "commit": (lambda k, off, n, t: pc.cure_commit(k, k, off, n, n, t, n, t, n, 4), [k, off, n, t]),
            }[sys.argv[2]]
            try:
                torch.vmap(fn)(*args)
            except RuntimeError as e:
                print("refused" if "data pointer" in str(e) else e)
        """, name)
    assert out == ["refused"]


def test_calls_of_threads_on_one_stream_do_not_interleave(stub):
    """A call's kernels hand data on through the stream's workspace, or through the library's scratch
    array: no other call on it may enqueue between them."""
    out = child(stub, """
        import threading
        errors = []
        def work(k):
            try:
                with FakeTensorMode():
                    f = lambda *s: torch.zeros(*s, device="cuda")
                    i = lambda *s: torch.zeros(*s, dtype=torch.int32, device="cuda")
                    x, n, t, off = f(2, 8, 40000), i(2), i(2, 8), torch.zeros(2, dtype=torch.int64, device="cuda")
                    q, c = f(2, 8, 2, 64), f(3000, 2, 64)
                    calls = [lambda: pc.cure_margins(x), lambda: pc.cure_margins_accept(x, t, t, n, n, 8),
                             lambda: pc.cure_margins_noalloc(x),
                             lambda: pc.cure_repair_tree(x, f(2, 8), t, n, t, 8, 2, 1.0),
                             lambda: pc.cure_tree_attn(q, c, c, off, n, n, t, [1000, 1000], [8, 8], 1.0, kv_split=3)]
                    for j in range(2 * len(calls)):
                        calls[(j + (k % 2)) % len(calls)]()
            except Exception as e:
                errors.append(repr(e))
        threads = [threading.Thread(target=work, args=(k,)) for k in range(6)]
        for t in threads: t.start()
        for t in threads: t.join()
        print(stub.stub_calls(), stub.stub_overlaps(), *errors)
        """)
    assert out == ["60", "0"]


def test_a_workspace_that_was_handed_out_stays_allocated(stub):
    """A captured graph replays with the workspace's address, whatever larger calls come after it. The
    buffers kept for that are bounded by the one in use."""
    out = child(stub, """
        from torch.multiprocessing.reductions import StorageWeakRef
        from torch.utils._python_dispatch import TorchDispatchMode
        seen = []                                    # the byte buffers that were allocated
        class Watch(TorchDispatchMode):
            def __torch_dispatch__(self, func, types, args=(), kwargs=None):
                t = func(*args, **(kwargs or {}))
                if isinstance(t, torch.Tensor) and t.dtype == torch.uint8:
                    ref = StorageWeakRef(t.untyped_storage())
                    if not any(ref == r for r, _ in seen):
                        seen.append((ref, t.numel()))
                return t
        with FakeTensorMode(), Watch():
            for batch in (1, 2, 3, 40, 41, 90):
                pc.cure_margins(torch.zeros(batch, 8, 40000, device="cuda"))
            need = pc.lib().cure_margins_workspace_size(90, 8, 40000)
        print(any(r.expired() for r, _ in seen), len(seen), seen[-1][1] >= need,
              sum(n for _, n in seen[:-1]) <= seen[-1][1])
        """)
    assert out[0] == "False" and int(out[1]) >= 3 and out[2:] == ["True", "True"]
