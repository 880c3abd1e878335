"""Ranks that are not a multiple of eight and row counts that are not a multiple of four on every kernel that reads rows
of B as 16-byte operands: the load that is moved back at the array's end, factors of fewer than eight entries in all,
entries of the next row (or infinities in it) that must not count, and outputs stored four at a time."""
import numpy as np
import pytest

import lords_inputs as li
from oracle import lords_oracle as onp

pytestmark = pytest.mark.gpu

Y_TOL, Y_MAX_TOL = 5e-3, 2e-2


@pytest.fixture(scope="module")
def gpu():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from tests import gpu_util
    return gpu_util


def check(Y, want, what):
    mx = onp.max_abs_over_rms(Y, want)
    print(f"   {what}: max/rms={mx:.2e}", flush=True)
    assert np.isfinite(Y).all(), what
    # (below 16 outputs the Frobenius ratio is one sample of the element-wise error, which is checked)
    assert mx <= Y_MAX_TOL and (want.size < 16 or onp.rel_fro(Y, want) <= Y_TOL), (what, mx)


@pytest.mark.parametrize("M", [1, 2, 5, 16, 40])
@pytest.mark.parametrize("N,r", [(1, 1), (1, 7), (1, 9), (2, 3), (7, 1), (9, 1), (17, 4), (33, 5), (66, 7), (131, 15), (259, 31), (66, 33),
                                 (513, 45), (30, 63), (130, 65), (67, 100), (35, 127)])
def test_products(gpu, M, N, r):
    print(f"ragged M={M} N={N} r={r}", flush=True)
    K, bits = 1184, 2 + (N + r) % 3
    cs = li.make_case("tiny", M=M, N=N, K=K, bits=bits, r=r, factor_dtype="bf16", seed=21 + r)
    want = onp.matmul(cs.X_f32, cs.codes, cs.codebook, cs.B_f32, cs.A_f32, cs.bits)
    check(gpu.DeviceCase(cs).matmul(), want, "product")


@pytest.mark.parametrize("M", [1, 2, 4])
@pytest.mark.parametrize("N,r", [(50, 5), (50, 20), (50, 45), (50, 70)])
def test_a_row_of_infinities_stays_in_its_row(gpu, M, N, r):
    """The 16 bytes fetched for a row reach into the next one: its values must not enter, not even times zero."""
    import torch
    cs = li.make_case("tiny", M=M, N=N, K=544, bits=4, r=r, factor_dtype="bf16", seed=22)
    d = gpu.DeviceCase(cs)
    clean = d.matmul()
    d.B = d.B.clone()
    d.B[17] = float("inf")
    d.B[49] = float("nan")
    Y = d.matmul()
    keep = [n for n in range(N) if n not in (17, 49)]
    np.testing.assert_array_equal(Y[:, keep], clean[:, keep])
    assert not np.isfinite(Y[:, 17]).any() and np.isnan(Y[:, 49]).all()


@pytest.mark.parametrize("M", [1, 3, 16])
@pytest.mark.parametrize("N", [1, 2, 3, 5, 1025, 2047])
def test_gate_up_and_batched(gpu, M, N):
    """Several matrices in one launch (shared tickets, read-back of four rows at a time) with ragged N and rank."""
    import torch
    import paper_2601_22716_amd as L
    K, r, bits = 2112, 13, 4
    cg = li.make_case("tiny", M=M, N=N, K=K, bits=bits, r=r, factor_dtype="bf16", seed=23)
    cu = li.make_case("tiny", M=M, N=N, K=K, bits=bits, r=r, factor_dtype="bf16", seed=24)
    dg, du = gpu.DeviceCase(cg), gpu.DeviceCase(cu)
    G = onp.matmul(cg.X_f32, cg.codes, cg.codebook, cg.B_f32, cg.A_f32, bits)
    U = onp.matmul(cg.X_f32, cu.codes, cu.codebook, cu.B_f32, cu.A_f32, bits)
    Yg, Yu = (torch.full((M, N), float("nan"), device="cuda") for _ in range(2))
    L.lords_matmul_batched(dg.X, [dg.codes, du.codes], dg.codebook, [dg.B, du.B], [dg.A, du.A], [Yg, Yu], [N, N], M, K, r, bits)
    H = torch.full((M, N), float("nan"), device="cuda")
    L.lords_gate_up(dg.X, dg.codes, dg.B, dg.A, du.codes, du.B, du.A, dg.codebook, H, M, N, K, r, bits)
    torch.cuda.synchronize()
    check(Yg.cpu().numpy(), G, "batched, first")
    check(Yu.cpu().numpy(), U, "batched, second")
    # |silu'| <= 1.1 and |silu(g)| <= |g|: the gates of the two products carried through
    silu = G / (1 + np.exp(-G))
    rms = lambda a: float(np.sqrt(np.mean(a * a)))
    bound = 1.05 * Y_MAX_TOL * (1.1 * rms(G) * np.abs(U) + rms(U) * np.abs(silu)) + 1e-6
    assert np.all(np.abs(H.cpu().numpy() - silu * U) <= bound)


@pytest.mark.parametrize("M,N,K,r,bits,fdt", [(17, 1, 288, 8, 4, "bf16"), (40, 131, 544, 32, 2, "bf16"), (130, 257, 416, 48, 3, "f32" ),
                                              (130, 514, 1056, 13, 3, "f32"), (257, 1027, 416, 32, 4, "bf16"),
                                              (1025, 67, 160, 32, 4, "bf16"), (1039, 33, 1184, 20, 3, "bf16"), (1030, 35, 160, 10, 4, "f32"),
                                              # several pieces, at an odd offset of H: 2048 and a few, 2048 and some, 1024 and a few
                                              (2049, 67, 160, 20, 2, "bf16"), (2073, 65, 160, 20, 2, "bf16"), (2098, 65, 160, 20, 4, "f32"), (1028, 943, 4480, 20, 3, "bf16"),
                                              # ranks beyond the large-M kernel: both products, then the element-wise pass, 1024 tokens at a time
                                              (40, 131, 288, 136, 4, "bf16"), (1100, 67, 160, 136, 3, "bf16"), (40, 35, 288, 65, 2, "f32"), (1100, 66, 160, 65, 4, "f32")])
def test_gate_up_of_many_tokens(gpu, M, N, K, r, bits, fdt):
    """The up product's large-M kernel reads the gate's sums four columns at a time and multiplies by their silu: last
    rows and columns, half tiles, pieces of a call (how many: test_routes.py).  Pairs in two passes are test_gpu_two_pass.py's, those
    whose tiles meet test_gpu_meet.py's."""
    from tests import plan_util
    assert not plan_util.takes_two_passes(M, [N, N], K, r, bits, fdt == "f32", act=True)
    import torch
    import paper_2601_22716_amd as L
    cg = li.make_case("tiny", M=M, N=N, K=K, bits=bits, r=r, factor_dtype=fdt, seed=25)
    cu = li.make_case("tiny", M=M, N=N, K=K, bits=bits, r=r, factor_dtype=fdt, seed=26)
    dg, du = gpu.DeviceCase(cg), gpu.DeviceCase(cu)
    G = onp.matmul(cg.X_f32, cg.codes, cg.codebook, cg.B_f32, cg.A_f32, bits)
    U = onp.matmul(cg.X_f32, cu.codes, cu.codebook, cu.B_f32, cu.A_f32, bits)
    H = torch.full((M, N), float("nan"), device="cuda")
    L.lords_gate_up(dg.X, dg.codes, dg.B, dg.A, du.codes, du.B, du.A, dg.codebook, H, M, N, K, r, bits)
    torch.cuda.synchronize()
    silu = G / (1 + np.exp(-G))
    rms = lambda a: float(np.sqrt(np.mean(a * a)))
    bound = 1.05 * Y_MAX_TOL * (1.1 * rms(G) * np.abs(U) + rms(U) * np.abs(silu)) + 1e-6
    assert np.all(np.abs(H.cpu().numpy() - silu * U) <= bound)
