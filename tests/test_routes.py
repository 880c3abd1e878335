"""Which kernels a call launches and which memory it asks for, through the C ABI on the CPU: the library's host side runs against a
stand-in for the HIP runtime (hip_double.cpp), each case in a process of its own, so that the library's workspace starts
unallocated."""
import ctypes
import json
import os
import subprocess
import sys

import pytest

from tests import plan_util

HERE = os.path.dirname(os.path.abspath(__file__))

PREAMBLE = """
import ctypes, json, sys
double, library, queries, arg = sys.argv[1], sys.argv[2], sys.argv[3], json.loads(sys.argv[4])
sys.path.insert(0, sys.argv[5])
rt = ctypes.CDLL(double, ctypes.RTLD_GLOBAL)
lib = ctypes.CDLL(library)
from tests import plan_util
plan = plan_util.declare(ctypes.CDLL(queries))
rt.double_launched.restype = ctypes.c_char_p
rt.double_largest_allocation.argtypes = [ctypes.c_size_t]
lib.lords_workspace_zero_bytes.restype = ctypes.c_size_t
vp, front = ctypes.c_void_p, lib.lords_workspace_zero_bytes()
at = lambda i: (1 << 32) + (i << 24)                       # (addresses: nothing is read)
each = lambda i, n: (vp * n)(*[at(i + l) for l in range(n)])


def launched():
    # kernels launched since the last call of this, the template's arguments left out
    names = rt.double_launched().decode().split()
    rt.double_forget_launches()
    return [n[n.index("lords") + 5:].lstrip("0123456789").split("_kernel")[0] for n in names]


def matmul(M, N, K, r, bits, f32):
    return lib.lords_matmul(vp(at(0)), vp(at(1)), vp(at(2)), vp(at(3)), vp(at(4)), vp(at(5)), M, N, K, r, bits, int(f32), 1, None)


def batched(Ns, M, K, r, bits, f32):
    n = len(Ns)
    return lib.lords_matmul_batched(vp(at(0)), each(10, n), vp(at(1)), each(20, n), each(30, n), each(40, n), (ctypes.c_int * n)(*Ns),
                                    n, M, K, r, bits, int(f32), 1, None)


def gate_up(M, N, K, r, bits, f32):
    return lib.lords_gate_up(vp(at(0)), vp(at(1)), vp(at(2)), vp(at(3)), vp(at(4)), vp(at(5)), vp(at(6)), vp(at(7)), vp(at(8)), M, N, K, r, bits,
                             int(f32), 1, None)
"""


@pytest.fixture(scope="module")
def routes(tmp_path_factory):
    from paper_2601_22716_amd import binding
    d = str(tmp_path_factory.mktemp("routes"))
    double = os.path.join(d, "hip_double.so")
    subprocess.run([os.environ.get("CXX", "g++"), "-std=c++17", "-O1", "-shared", "-fPIC", "-o", double, os.path.join(HERE, "hip_double.cpp")], check=True)
    queries = plan_util.compile_queries(d, binding.library_path())

    def run(body, arg=None):
        r = subprocess.run([sys.executable, "-c", PREAMBLE + body, double, binding.library_path(), queries, json.dumps(arg), os.path.dirname(HERE)],
                           capture_output=True, text=True, timeout=120)
        assert r.returncode == 0, (r.returncode, r.stderr[-2000:])
        return json.loads(r.stdout.strip().splitlines()[-1])
    return run


@pytest.mark.parametrize("L,N,M,K,r,f32", [
    (8, 1024, 2048, 36864, 64, True), (8, 4096, 8192, 36864, 100, False), (4, 1024, 4096, 73728, 64, True), (3, 1024, 4096, 98304, 43, True),
    (2, 1024, 8192, 147456, 64, True), (7, 1024, 2048, 36864, 64, True), (6, 1000, 3000, 49152, 63, True)])
def test_batched_two_passes_of_many_columns(routes, L, N, M, K, r, f32):
    """Matrices of so many columns that a tile of each is more than the scratch for the dequantised weights holds: as many of
    them at a time as it does hold."""
    out = routes("""
Ns, (M, K, r, bits, f32) = [arg["N"]] * arg["L"], arg["rest"]
alone = plan_util.takes_two_passes(M, Ns[:1], K, r, bits, f32, lib=plan)
most = max(n for n in range(1, len(Ns) + 1) if plan.two_pass_supported((ctypes.c_int * n)(*Ns[:n]), n, M, K, r, bits, int(f32), 0))
print(json.dumps([alone, most, batched(Ns, M, K, r, bits, f32), launched()]))
""", dict(L=L, N=N, rest=[M, K, r, 4, f32]))
    alone, most, status, kernels = out
    assert alone and status == 0
    assert kernels[::2] == ["dequant_operand"] * (len(kernels) // 2) and kernels[1::2] == ["operand_gemm"] * (len(kernels) // 2)
    assert most < L or (L, K) == (7, 36864)
    assert len(kernels) >= 2 * -(-L // most)


def test_two_pass_scratch_of_any_batch(routes):
    """The scratch asked for is positive for every batch, and at most what is set aside where the batch is supported."""
    out = routes("""
import random
rng, bad = random.Random(11), []
for _ in range(4000):
    L = rng.randint(1, 8)
    Ns = (ctypes.c_int * L)(*[int(2 ** rng.uniform(0, 15)) for _ in range(L)])
    K, f32 = 32 * int(2 ** rng.uniform(0, 14.5)), rng.randint(0, 1)
    a = (Ns, L, int(2 ** rng.uniform(7, 13)), K, rng.randint(1, 42 if f32 else 128), rng.choice([2, 3, 4]), f32, 0)
    size = plan.two_pass_workspace_bytes(*a)
    if size <= 0 or plan.two_pass_supported(*a) and size > 128 << 20:
        bad.append([list(Ns), K, size])
print(json.dumps(bad))
""")
    assert out == []


def test_batched_call_without_joint_scratch_does_nothing_twice(routes):
    """One matrix goes in two passes, the others share tiles, whose scratch together is not to be had: each matrix is computed once."""
    out = routes("""
Ns, (M, K, r, bits, f32) = [6144] + [3000] * 7, (1000, 4096, 100, 4, 0)
takes = lambda n: plan_util.takes_two_passes(M, [n], K, r, bits, f32, lib=plan)
parts = [plan.prefill_workspace_bytes(M, n, K, r, bits, f32) for n in Ns]
need = plan.two_pass_workspace_bytes((ctypes.c_int * 1)(Ns[0]), 1, M, K, r, bits, f32, 0)
room = need + front + (33 << 20)                            # (33 MB: what fp32 factors keep beside the first block, and alignment)
rt.double_largest_allocation(room)
print(json.dumps([takes(Ns[0]), takes(Ns[1]), min(parts[1:]), max(parts), sum(parts[1:]), room, batched(Ns, M, K, r, bits, f32), launched()]))
""")
    first, second, least, most, joint, room, status, kernels = out
    assert first and not second and 0 < least and most < room < joint and status == 0
    assert kernels.count("dequant_operand") == 1 and kernels.count("operand_gemm") == 1
    assert kernels.count("prefill") + kernels.count("prefill_wide") == 7


@pytest.mark.parametrize("call", ["matmul(2000, 6144, 4096, 64, 4, True)", "matmul(2000, 6144, 4096, 100, 4, False)", "matmul(1500, 11008, 4096, 48, 4, False)",
                                  "batched([6144, 3000, 3001], 2000, 4096, 64, 4, True)", "batched([3000] * 4, 1000, 4096, 100, 4, False)"])
def test_memory_that_is_not_there_is_not_asked_for_on_every_call(routes, call):
    """Beside an allocator that has left room for little, a call that can do with less asks for more once in a thousand times; once
    there is room it has it again."""
    out = routes("""
matmul(4, 512, 4096, 8, 4, False), launched()               # (the first block)
rt.double_largest_allocation(front + (40 << 20))
asked = rt.double_allocations_asked
call = lambda: eval(arg)
first = [call(), launched(), asked()]
status = [call() for _ in range(500)]
few = [max(status), launched()[-len(first[1]):], asked()]
rt.double_largest_allocation(1 << 40)
status = [call() for _ in range(1100)]
print(json.dumps([first, few, [max(status), launched()[-1], asked()]]))
""", call)
    first, few, again = out
    assert first[0] == few[0] == again[0] == 0
    assert few[1] == first[1]
    assert first[2] >= 3 and few[2] == first[2]             # (the first block and two attempts)
    assert again[2] == few[2] + 1
    if "True" in call or "matmul(2000" in call:
        assert "operand_gemm" not in first[1] and again[1] == "operand_gemm"


def test_refused_memory_that_a_call_needs_is_asked_for_every_time(routes):
    """A call that cannot do with less is refused, and served as soon as there is room, whatever was refused before."""
    out = routes("""
rt.double_largest_allocation(1 << 20)
refused = [matmul(100, 8000, 4096, 32, 4, False), matmul(2000, 6144, 4096, 64, 4, True), matmul(1500, 11008, 4096, 48, 4, False)]
rt.double_largest_allocation(1 << 40)
print(json.dumps([refused, matmul(100, 8000, 4096, 32, 4, False), matmul(2000, 6144, 4096, 64, 4, True)]))
""")
    assert out == [[6, 6, 6], 0, 0]


@pytest.mark.parametrize("M,N,K,r,bits", [(411, 7402, 1376, 4, 4), (83, 22668, 2336, 27, 3), (411, 14000, 4096, 20, 4)])
def test_parts_that_meet_are_optional(routes, M, N, K, r, bits):
    """Tiles that several workgroups finish together ask for more memory than other cuts of the work: where it is not to be had a
    call runs with less, also in a caller's workspace of what the other cuts need and while the stream is captured."""
    out = routes("""
M, N, K, r, bits = arg
asks = front + plan.prefill_workspace_bytes(M, N, K, r, bits, 0)
in_ws = lambda size: lib.lords_matmul_ws(vp(at(0)), vp(at(1)), vp(at(2)), vp(at(3)), vp(at(4)), vp(at(5)), M, N, K, r, bits, 0, 1, None, 0, vp(at(9)),
                                         ctypes.c_size_t(size))
rt.double_largest_allocation(50 << 20)                      # (32 MiB of it for products with fp32 factors)
short = [matmul(M, N, K, r, bits, False), launched()]
caller = [in_ws(front), in_ws(asks), launched()]
rt.double_capturing(1)
print(json.dumps([asks > front + (20 << 20), short, caller, matmul(M, N, K, r, bits, False), launched()]))
""", [M, N, K, r, bits])
    assert out == [True, [0, ["prefill"]], [0, 0, ["prefill"] * 2], 0, ["prefill"]]


@pytest.mark.parametrize("capturing", [0, 1])
def test_gate_up_with_room_for_1024_tokens(routes, capturing):
    """Without the scratch for its weights a pair keeps the gate of 2048 tokens in memory, or of 1024: with room for
    1024 a call of a few more is served, captured too."""
    out = routes("""
M, N, K, r = 1112, 6144, 8192, 64
takes = plan_util.takes_two_passes(M, [N, N], K, r, 4, True, act=True, lib=plan)
most = front + 1024 * N * 4 + 4096
matmul(4, 512, 4096, 8, 4, False)                           # (the first block)
rt.double_largest_allocation(most)
if arg:
    gate_up(1024, N, K, 8, 4, True)                        # (grows the block to that)
    rt.double_capturing(1)
launched()
print(json.dumps([takes, gate_up(M, N, K, r, 4, True), launched()]))
""", capturing)
    takes, status, kernels = out
    assert takes and status == 0
    assert kernels == ["prefill"] * 4


def test_a_pair_whose_gate_is_not_to_be_had_stays_refused(routes):
    """Two passes need no gate in memory, but a pair that the large-M kernel's way has no memory for is not to be accepted for it."""
    out = routes("""
rt.double_largest_allocation(1 << 38)
takes = [plan_util.takes_two_passes(2048, [n, n], 32, 8, 4, False, act=True, lib=plan) for n in (1 << 20, 1 << 26)]
print(json.dumps([takes, gate_up(2048, 1 << 26, 32, 8, 4, False), launched()]))
""")
    assert out == [[True, False], 6, []]


@pytest.mark.parametrize("Ns,rest,first", [
    ([2305, 1545, 5312, 658, 1443, 480], [143, 640, 5, 2, 1], False), ([3722, 2776, 4485, 354], [516, 864, 38, 4, 0], False),
    ([3129, 1837, 2122, 649], [647, 864, 18, 2, 1], False), ([2452, 1975], [2296, 704, 22, 3, 1], True)])
def test_batched_matrices_stay_in_one_launch_where_that_is_faster(routes, Ns, rest, first):
    """Matrices that alone leave much of the chip idle are one launch of the large-M kernel, beside each other: two passes are
    to beat that launch, not the sum of launches that each idle; also where one alone would go in two passes."""
    out = routes("""
Ns, (M, K, r, bits, f32) = arg
print(json.dumps([[plan_util.takes_two_passes(M, [n], K, r, bits, f32, lib=plan) for n in Ns], batched(Ns, M, K, r, bits, f32), launched()]))
""", [Ns, rest])
    alone, status, kernels = out
    assert alone == [first] + [False] * (len(Ns) - 1) and status == 0
    assert set(kernels) <= {"prefill", "prefill_wide"} and len(kernels) <= 2


def test_batched_matrices_go_in_two_passes_together(routes):
    """... and two passes where they are the faster way, with them matrices that alone would not take them."""
    out = routes("""
Ns, (M, K, r, bits, f32) = [4096, 1024, 1024], (2048, 4096, 64, 4, 1)
print(json.dumps([[plan_util.takes_two_passes(M, [n], K, r, bits, f32, lib=plan) for n in Ns], batched(Ns, M, K, r, bits, f32), launched()]))
""")
    alone, status, kernels = out
    assert status == 0 and kernels == ["dequant_operand", "operand_gemm"]


@pytest.mark.parametrize("Ns,rest,most", [
    ([4096, 1024, 1024], [256, 4096, 32, 4, 0], 41), ([4096, 1024, 1024], [1024, 4096, 32, 4, 0], 105), ([2048, 512, 512], [1024, 2048, 32, 4, 0], 38),
    ([1600, 400, 400], [651, 1600, 11, 4, 0], 34), ([1216] * 3, [943, 1216, 16, 4, 0], 28), ([1088] * 3, [1360, 1088, 9, 4, 0], 30)])
def test_matrices_cut_into_parts_do_not_queue_for_the_chip(routes, Ns, rest, most):
    """Tiles that fill the chip in parts where their matrix is alone are taken with fewer workgroups beside others: at most an
    eighth over the estimates of the launches without parts (us), and one launch."""
    out = routes("""
Ns, (M, K, r, bits, f32) = arg
print(json.dumps([plan_util.batched_cost(M, Ns, K, r, bits, f32, lib=plan), batched(Ns, M, K, r, bits, f32), launched()]))
""", [Ns, rest])
    cost, status, kernels = out
    assert cost <= 1.125 * most and status == 0 and kernels == ["prefill"]


@pytest.mark.parametrize("M,N,K,r,bits", [(330, 6528, 2496, 15, 4), (362, 3008, 1216, 23, 4), (385, 2464, 1088, 29, 3), (282, 3456, 1216, 12, 4), (260, 7264, 1920, 8, 2)])
def test_pairs_that_two_passes_serve_faster_go_there(routes, M, N, K, r, bits):
    """Pairs of which the large-M kernel's tiles would meet in parts, 10 to 18 % slower than two passes."""
    out = routes("""
M, N, K, r, bits = arg
status = lib.lords_gate_up(*[vp(at(i)) for i in range(9)], M, N, K, r, bits, 0, 1, None)
print(json.dumps([plan_util.cut(M, N, K, r, bits, 0, lib=plan)[2] > 0, status, launched()]))
""", [M, N, K, r, bits])
    assert out == [True, 0, ["dequant_operand", "operand_gemm"]]


@pytest.mark.parametrize("M,N,K,r,bits,f32,pieces", [
    (2049, 67, 160, 20, 2, 0, [2048, 1]), (2073, 65, 160, 20, 2, 0, [2048, 25]), (2098, 65, 160, 20, 4, 1, [2048, 50]), (1028, 943, 4480, 20, 3, 0, [1024, 4]),
    (1114, 3866, 8608, 8, 2, 0, [1024, 90]), (1025, 67, 160, 32, 4, 0, [1025]), (4101, 72, 4704, 60, 2, 0, [2048, 2048, 5])])
def test_pieces_of_a_pair(routes, M, N, K, r, bits, f32, pieces):
    """The pieces that a pair of many tokens goes in: two launches of the large-M kernel each, one of a few-token kernel for a few."""
    status, kernels = routes("print(json.dumps([gate_up(*arg), launched()]))", [M, N, K, r, bits, f32])
    assert status == 0 and kernels.count("prefill") == 2 * sum(p > 16 for p in pieces)
    assert len([k for k in kernels if k.startswith(("decode", "gemv"))]) == sum(p <= 16 for p in pieces)
