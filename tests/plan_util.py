"""The library's planner, asked by tests (plan_queries.cpp, built against the library's own header and linked with it)."""
from __future__ import annotations

import ctypes
import functools
import os
import subprocess
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))


def compile_queries(out_dir: str, library: str) -> str:
    out = os.path.join(out_dir, "plan_queries.so")
    subprocess.run([os.environ.get("CXX", "g++"), "-std=c++17", "-O1", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-isystem", "/opt/rocm/include",
                    "-o", out, os.path.join(HERE, "plan_queries.cpp"), library], check=True)
    return out


def declare(lib):
    num, nums = ctypes.c_int, ctypes.POINTER(ctypes.c_int)
    for name, restype in (("two_pass_faster", num), ("two_pass_supported", num), ("two_pass_workspace_bytes", ctypes.c_size_t)):
        getattr(lib, name).argtypes, getattr(lib, name).restype = [nums] + [num] * 7, restype
    for name, restype in (("prefill_workspace_bytes", ctypes.c_size_t), ("prefill_least_workspace_bytes", ctypes.c_size_t), ("prefill_wide_taken", num)):
        getattr(lib, name).argtypes, getattr(lib, name).restype = [num] * 6, restype
    ptr = ctypes.c_void_p
    lib.prefill_cut.argtypes, lib.prefill_cut.restype = [num] * 6 + [nums], None
    lib.prefill_batched_cut.argtypes, lib.prefill_batched_cut.restype = [nums] + [num] * 7 + [nums], None
    lib.prefill_batched_cost.argtypes, lib.prefill_batched_cost.restype = [nums] + [num] * 6, ctypes.c_double
    lib.prefill_batched_workspace_bytes.argtypes, lib.prefill_batched_workspace_bytes.restype = [nums] + [num] * 6, ctypes.c_size_t
    ptrs = ctypes.POINTER(ptr)
    lib.launch_large_batched.argtypes, lib.launch_large_batched.restype = [ptr, ptrs, ptr, ptrs, ptrs, ptrs, nums] + [num] * 7 + [ptr] * 3 + [num], num
    lib.launch_large.argtypes, lib.launch_large.restype = [ptr] * 7 + [num] * 7 + [ptr, ctypes.c_size_t, ptr, ptr, num], num
    return lib


@functools.lru_cache(maxsize=None)
def queries():
    from paper_2601_22716_amd import binding
    binding.library()
    with tempfile.TemporaryDirectory() as d:
        return declare(ctypes.CDLL(compile_queries(d, binding.library_path())))


def takes_two_passes(M, Ns, K, r, bits, f32, act=False, lib=None):
    return bool((lib or queries()).two_pass_faster((ctypes.c_int * len(Ns))(*Ns), len(Ns), M, K, r, bits, int(f32), int(act)))


def cut(M, N, K, r, bits, f32, lib=None):
    """The large-M kernel's tiles and the number of parts that meet in each: (tokens, rows, parts)."""
    out = (ctypes.c_int * 3)()
    (lib or queries()).prefill_cut(M, N, K, r, bits, int(f32), out)
    return tuple(out)


def batched_cuts(M, Ns, K, r, bits, f32, lib=None):
    """... of the matrices of one launch, and how many of the parts one workgroup takes: [(tokens, rows, parts, walk), ..]."""
    lib, cuts = lib or queries(), []
    for l in range(len(Ns)):
        out = (ctypes.c_int * 4)()
        lib.prefill_batched_cut((ctypes.c_int * len(Ns))(*Ns), len(Ns), M, K, r, bits, int(f32), l, out)
        cuts.append(tuple(out))
    return cuts


def batched_cost(M, Ns, K, r, bits, f32, lib=None):
    """The planner's estimate of that launch, us."""
    return (lib or queries()).prefill_batched_cost((ctypes.c_int * len(Ns))(*Ns), len(Ns), M, K, r, bits, int(f32))
