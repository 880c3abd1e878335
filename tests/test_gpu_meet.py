"""Products of many tokens whose tiles are cut into two, four or eight parts that several workgroups finish together, through
the C ABI: against the fp64 oracle, and run to run bit for bit.  Gates as for lords_matmul.

Sizes: every tile shape, each with the numbers of parts that its plans have (the tokens and rows of a tile and the parts stand beside
each case and are asked of the planner), K tiles that the parts do not divide (a unit more or less each), ragged last K
tiles, token counts at which the last slices of a tile have no tokens (17, 33, 65, 129 ...), rows off the tiles.
"""
import sys

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


@pytest.mark.parametrize("M,N,K,r,bits,fdt,cut", [
    (17, 4096, 4096, 32, 4, "bf16", (128, 128, 8)), (33, 3001, 4000, 7, 3, "bf16", (128, 128, 8)), (65, 4099, 3104, 32, 2, "bf16", (128, 256, 8)),
    (128, 4096, 4096, 20, 4, "bf16", (128, 128, 8)), (129, 1003, 2016, 10, 3, "bf16", (256, 128, 8)),
    (300, 1024, 4096, 32, 4, "bf16", (256, 128, 8)), (445, 1882, 2016, 10, 4, "bf16", (256, 128, 4)),
    (1795, 1765, 2176, 10, 2, "bf16", (256, 128, 2)), (2047, 1021, 2080, 31, 4, "bf16", (256, 128, 2)),
    (261, 8714, 1984, 20, 4, "bf16", (256, 256, 2)), (262, 4165, 1344, 8, 4, "bf16", (256, 256, 4)), (264, 2174, 2720, 8, 4, "bf16", (256, 256, 8)),
    (18, 16643, 1696, 8, 3, "bf16", (128, 256, 2)), (17, 6325, 928, 8, 3, "bf16", (128, 128, 4)), (17, 8379, 960, 60, 3, "bf16", (128, 256, 4)), (100, 1999, 2592, 48, 3, "bf16", (128, 128, 8)),
    (500, 4096, 1056, 48, 4, "bf16", (128, 128, 2)), (237, 3699, 1568, 87, 4, "bf16", (128, 128, 4)), (18, 4495, 1952, 96, 4, "bf16", (128, 256, 8)),
    (100, 4096, 4096, 10, 4, "f32", (128, 128, 8)), (19, 3045, 2048, 40, 3, "f32", (128, 128, 8)), (705, 2284, 2624, 7, 2, "f32", (128, 256, 4)),
    (135, 5466, 1184, 8, 3, "f32", (128, 256, 2)), (26, 4453, 1952, 20, 4, "f32", (128, 256, 8)), (86, 3869, 2304, 64, 4, "f32", (64, 128, 4)),
    (17, 14575, 1088, 60, 4, "f32", (64, 128, 2)), (500, 4096, 1056, 16, 3, "f32", (128, 128, 2)), (250, 16000, 4128, 60, 2, "bf16", (128, 256, 2))])
def test_parts_that_meet(gpu, M, N, K, r, bits, fdt, cut):
    from tests import plan_util
    assert plan_util.cut(M, N, K, r, bits, fdt == "f32") == cut and not plan_util.takes_two_passes(M, [N], K, r, bits, fdt == "f32")
    print(f"parts that meet M={M} N={N} K={K} r={r} bits={bits} factors={fdt}", flush=True)
    sys.stdout.flush()
    c = li.make_case("tiny", M=M, N=N, K=K, r=r, bits=bits, factor_dtype=fdt, seed=81, signed_factors=True)
    d = gpu.DeviceCase(c)
    Y = d.matmul()
    rows = np.unique(np.r_[np.random.default_rng(1).integers(0, N, 24), 0, N - 1])
    want = onp.matmul_rows(c.X_f32, c.codes, c.codebook, c.B_f32, c.A_f32, bits, rows)
    assert np.isfinite(Y).all()
    rf, mx = onp.rel_fro(Y[:, rows], want), onp.max_abs_over_rms(Y[:, rows], want)
    assert rf <= Y_TOL and mx <= Y_MAX_TOL, (rf, mx)
    for _ in range(3):
        np.testing.assert_array_equal(d.matmul(), Y)


def test_parts_that_meet_in_one_launch_of_several_matrices(gpu):
    """... and each matrix of a batched call has the bits of its single call."""
    import torch
    import paper_2601_22716_amd as L
    M, K, r, bits, Ns = 300, 4000, 32, 4, [4096, 1024, 1000]
    dev = [gpu.DeviceCase(li.make_case("tiny", M=M, N=N, K=K, bits=bits, r=r, factor_dtype="bf16", seed=85 + i)) for i, N in enumerate(Ns)]
    want = [d.matmul(X=dev[0].X, M=M) for d in dev]
    Ys = [torch.full((M, N), float("nan"), device="cuda") for N in Ns]
    L.lords_matmul_batched(dev[0].X, [d.codes for d in dev], dev[0].codebook, [d.B for d in dev], [d.A for d in dev], Ys, Ns, M, K, r, bits)
    torch.cuda.synchronize()
    for Y, w in zip(Ys, want):
        np.testing.assert_array_equal(Y.cpu().numpy(), w)


@pytest.mark.parametrize("M,N,K,r,bits,fdt,cut", [
    (1700, 4099, 4128, 9, 2, "bf16", (256, 256, 2)), (250, 5123, 4128, 20, 4, "bf16", (256, 128, 4)), (205, 5122, 4096, 16, 3, "bf16", (256, 128, 4)),
    (256, 5119, 5120, 32, 4, "bf16", (256, 256, 8)), (30, 4093, 4096, 20, 4, "bf16", (128, 128, 8)), (70, 4097, 4096, 20, 4, "bf16", (128, 256, 8)),
    (17, 14337, 4096, 7, 3, "bf16", (128, 256, 4)),
    (500, 4095, 1056, 48, 4, "bf16", (128, 128, 2)), (705, 2282, 2624, 7, 2, "f32", (128, 256, 4)), (86, 3869, 2304, 64, 4, "f32", (64, 128, 4))])
def test_parts_left_to_others(gpu, M, N, K, r, bits, fdt, cut):
    """Workgroups that do not wait, or hardly, leave their shares of a tile to others: the same bits, with and without a gate, in
    both output types, and the counts back at zero."""
    import torch
    import paper_2601_22716_amd as L
    from tests import plan_util
    print(f"parts left to others M={M} N={N} K={K} r={r} bits={bits} factors={fdt}", flush=True)
    q, f32 = plan_util.queries(), fdt == "f32"
    assert plan_util.cut(M, N, K, r, bits, f32) == cut
    d = gpu.DeviceCase(li.make_case("tiny", M=M, N=N, K=K, r=r, bits=bits, factor_dtype=fdt, seed=91, signed_factors=True))
    front, part = L.lords_workspace_zero_bytes(), q.prefill_workspace_bytes(M, N, K, r, bits, int(f32))
    ws = torch.zeros(front + part, dtype=torch.uint8, device="cuda")
    gate = torch.randn(M * N + 4, device="cuda")                # (read four columns at a time)
    stream = torch.cuda.current_stream().cuda_stream

    def launch(dtype, gate_at, polls):
        Y = torch.full((M, N), float("nan"), dtype=dtype, device="cuda")
        ws[front:] = 255                                        # (not a number: a part that is read before it is written shows)
        assert q.launch_large(d.X.data_ptr(), d.codes.data_ptr(), d.codebook.data_ptr(), d.B.data_ptr(), d.A.data_ptr(), Y.data_ptr(), gate_at, M, N, K, r,
                              bits, int(f32), int(dtype == torch.float32), ws.data_ptr() + front, part, ws.data_ptr(), stream, polls) == 0
        torch.cuda.synchronize()
        assert not ws[:front].any()
        return Y

    for gate_at in (None, gate.data_ptr()):
        for dtype in (torch.float32, torch.bfloat16):
            want = launch(dtype, gate_at, 1 << 20)
            assert torch.isfinite(want).all()
            for polls in (0, 1, 3):
                assert torch.equal(launch(dtype, gate_at, polls), want), (gate_at is not None, dtype, polls)
    ref = torch.from_numpy(d.matmul()).cuda()
    assert torch.equal(launch(torch.float32, None, 0), ref)


@pytest.mark.parametrize("M,N,K,r,bits,fdt,hdt,cut", [
    (28, 14595, 800, 96, 4, "bf16", "f32", (128, 128, 2)), (19, 2626, 1952, 20, 3, "bf16", "bf16", (128, 128, 8)), (18, 2699, 2016, 60, 2, "bf16", "f32", (128, 128, 8)),
    (18, 16643, 1696, 8, 3, "bf16", "bf16", (128, 256, 2)), (17, 6325, 928, 8, 3, "bf16", "f32", (128, 128, 4)), (17, 8379, 960, 60, 3, "bf16", "f32", (128, 256, 4)), (128, 4099, 4096, 16, 4, "bf16", "f32", (128, 256, 8)),
    (129, 6927, 928, 20, 3, "bf16", "f32", (256, 128, 2)), (257, 682, 928, 20, 3, "bf16", "bf16", (256, 128, 4)), (258, 278, 2624, 8, 3, "bf16", "f32", (256, 128, 8)),
    (140, 8490, 1440, 32, 2, "bf16", "f32", (256, 256, 4)), (269, 2053, 2624, 32, 2, "bf16", "bf16", (256, 256, 8)), (559, 10975, 512, 20, 3, "bf16", "f32", (256, 256, 0)),
    (18, 14345, 800, 32, 4, "f32", "f32", (128, 128, 2)), (19, 3045, 2048, 40, 3, "f32", "bf16", (128, 128, 8)), (135, 5466, 1184, 8, 3, "f32", "f32", (128, 256, 2)),
    (26, 4453, 1952, 20, 4, "f32", "bf16", (128, 256, 8)), (25, 6481, 928, 60, 3, "f32", "f32", (64, 128, 4))])
def test_gate_up_whose_products_meet(gpu, M, N, K, r, bits, fdt, hdt, cut):
    """The up product's workgroups multiply their slices by the gate's silu: sampled rows of the matrices, the last ones among them,
    against the oracle, with the bound that the gates of the two products carry through (|silu'| <= 1.1, |silu(g)| <= |g|)."""
    import torch
    import paper_2601_22716_amd as L
    from tests import plan_util
    print(f"pair M={M} N={N} K={K} r={r} bits={bits} factors={fdt} out={hdt}", flush=True)
    f32 = fdt == "f32"
    assert plan_util.cut(M, N, K, r, bits, f32) == cut and not plan_util.takes_two_passes(M, [N, N], K, r, bits, f32, act=True)
    cg, cu = (li.make_case("tiny", M=M, N=N, K=K, r=r, bits=bits, factor_dtype=fdt, seed=101 + i, signed_factors=True) for i in range(2))
    dg, du = gpu.DeviceCase(cg), gpu.DeviceCase(cu)
    H = torch.full((M, N), float("nan"), dtype=torch.float32 if hdt == "f32" else torch.bfloat16, device="cuda")
    L.lords_gate_up(dg.X, dg.codes, dg.B, dg.A, du.codes, du.B, du.A, dg.codebook, H, M, N, K, r, bits)
    torch.cuda.synchronize()
    rows = np.unique(np.r_[np.random.default_rng(2).integers(0, N, 40), 0, N - 3, N - 2, N - 1])
    G, U = (onp.matmul_rows(cg.X_f32, c.codes, c.codebook, c.B_f32, c.A_f32, bits, rows) for c in (cg, cu))
    silu = G / (1 + np.exp(-G))
    rms = lambda a: float(np.sqrt(np.mean(a * a)))
    want = silu * U
    bound = 1.05 * Y_MAX_TOL * (1.1 * rms(G) * np.abs(U) + rms(U) * np.abs(silu)) + 1e-6 + (0.0 if hdt == "f32" else 2.0 ** -8) * np.abs(want)
    assert torch.isfinite(H).all() and np.all(np.abs(H.float().cpu().numpy()[:, rows] - want) <= bound)


@pytest.mark.parametrize("M,N,K,r,bits", [(411, 7402, 1376, 4, 4), (83, 22668, 2336, 27, 3)])
def test_without_room_for_parts_that_meet(gpu, M, N, K, r, bits):
    """A caller's workspace of the front alone: whole tiles.  Their sums of K fp32 additions are taken in another order (about
    sqrt(K) 2^-24 of their rms)."""
    import torch
    import paper_2601_22716_amd as L
    d = gpu.DeviceCase(li.make_case("tiny", M=M, N=N, K=K, r=r, bits=bits, factor_dtype="bf16", seed=97, signed_factors=True))
    ws = torch.zeros(L.lords_workspace_zero_bytes(), dtype=torch.uint8, device="cuda")
    Y = torch.full((M, N), float("nan"), device="cuda")
    L.lords_matmul_ws(d.X, d.codes, d.codebook, d.B, d.A, Y, M, N, K, r, bits, ws)
    torch.cuda.synchronize()
    assert not ws.any() and onp.rel_fro(Y.cpu().numpy(), d.matmul()) <= 1e-5
