"""Products of many tokens that go in two passes (weights dequantised once into scratch, then a product that reads them),
through the C ABI: against the fp64 oracle on sampled rows, and bit for bit against the large-M kernel on whole tiles, which
performs the same operations in the same order.  Gates as for lords_matmul.

Sizes: the smallest at which the planner takes two passes, off the tiles in every direction (tokens and rows not multiples
of 256, 128, 16 or 4, an odd number of K tiles, a ragged last one), every padded contraction, ranks that are not multiples
of 4 or 8.
"""
import sys

import numpy as np
import pytest

import lords_inputs as li
from oracle import lords_oracle as onp
from tests import plan_util
from tests.plan_util import takes_two_passes

pytestmark = pytest.mark.gpu

Y_TOL, Y_MAX_TOL = 5e-3, 2e-2


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def gpu():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from tests import gpu_util
    return gpu_util


def check_rows(Y, c, X_f32, bits, what, seed=0, count=24):
    rows = np.unique(np.concatenate([np.random.default_rng(seed).integers(0, c.N, count), [0, c.N - 1]]))
    want = onp.matmul_rows(X_f32, c.codes, c.codebook, c.B_f32, c.A_f32, bits, rows)
    rf, mx = onp.rel_fro(Y[:, rows], want), onp.max_abs_over_rms(Y[:, rows], want)
    say(f"   {what}: rel_fro={rf:.2e} max/rms={mx:.2e}")
    assert np.isfinite(Y).all(), what
    assert rf <= Y_TOL and mx <= Y_MAX_TOL, (what, rf, mx)


def by_whole_tiles(d, M):
    """The large-M kernel with a workspace that has no room for parts (its front alone); a bf16 case must need none."""
    import torch
    import paper_2601_22716_amd as L
    front = L.lords_workspace_zero_bytes()
    assert d.B.dtype == torch.float32 or L.lords_workspace_bytes(M, d.N, d.K, d.r, d.bits, L.LORDS_BF16) <= front
    ws = torch.zeros(front, dtype=torch.uint8, device="cuda")
    Y = torch.full((M, d.N), float("nan"), device="cuda")
    L.lords_matmul_ws(d.X, d.codes, d.codebook, d.B, d.A, Y, M, d.N, d.K, d.r, d.bits, ws)
    torch.cuda.synchronize()
    return Y.cpu().numpy()


def plan_has_whole_tiles(M, N, K, r, bits, fdt):
    return fdt == "f32" or plan_util.queries().prefill_workspace_bytes(M, N, K, r, bits, 0) == 0


# The last column: the large-M kernel's own plan has whole tiles (or, with fp32 factors, makes do with them), so that it can be
# compared with bit for bit.  Every padded contraction is, and at 128 every code width; one and two K tiles too.
@pytest.mark.parametrize("M,N,K,r,bits,fdt,compared", [
    (3000, 777, 544, 64, 4, "f32", True), (3001, 1030, 672, 43, 3, "f32", True), (4097, 1500, 544, 41, 2, "f32", True),
    (3000, 2999, 1056, 16, 4, "f32", True), (4097, 2999, 4128, 10, 3, "f32", True),
    (3329, 3622, 96, 64, 4, "f32", True), (4881, 2458, 32, 50, 2, "f32", True), (2456, 5853, 128, 63, 3, "f32", True), (3329, 3622, 160, 62, 4, "f32", True),
    (3000, 2999, 544, 99, 2, "bf16", False), (3001, 3002, 672, 128, 4, "bf16", False), (3000, 2999, 2080, 45, 3, "bf16", True),
    (2747, 3331, 544, 99, 2, "bf16", True), (3232, 2361, 672, 128, 4, "bf16", True), (3911, 2361, 544, 70, 3, "bf16", True),
    (2049, 4001, 2208, 64, 2, "bf16", True), (3000, 2999, 2208, 31, 4, "bf16", True), (3000, 2999, 2208, 8, 3, "bf16", True)])
def test_two_pass_product(gpu, M, N, K, r, bits, fdt, compared):
    say(f"two passes M={M} N={N} K={K} r={r} bits={bits} factors={fdt}")
    assert takes_two_passes(M, [N], K, r, bits, fdt == "f32")
    assert plan_has_whole_tiles(M, N, K, r, bits, fdt) == compared
    c = li.make_case("tiny", M=M, N=N, K=K, r=r, bits=bits, factor_dtype=fdt, seed=3, signed_factors=True)
    d = gpu.DeviceCase(c)
    Y = d.matmul()
    check_rows(Y, c, c.X_f32, bits, "Y")
    if compared:
        np.testing.assert_array_equal(Y, by_whole_tiles(d, M))


@pytest.mark.parametrize("M,N,K,r,bits,fdt", [(3001, 1030, 672, 43, 3, "f32"), (3911, 2361, 544, 70, 3, "bf16"), (2049, 4001, 2208, 64, 2, "bf16")])
def test_two_pass_infinities_and_nan(gpu, M, N, K, r, bits, fdt):
    """Infinities and NaN in X and in the factors come out where the large-M kernel has them; the tokens and rows that
    have none are the finite ones of the oracle."""
    say(f"two passes, infinities M={M} N={N} K={K} r={r} bits={bits} factors={fdt}")
    assert takes_two_passes(M, [N], K, r, bits, fdt == "f32")
    c = li.make_case("tiny", M=M, N=N, K=K, r=r, bits=bits, factor_dtype=fdt, seed=8, signed_factors=True)
    d = gpu.DeviceCase(c)
    finite = d.matmul()
    inf, nan = float("inf"), float("nan")
    tokens, rows = [0, 255, 256, M // 2, M - 1], [0, 15, 300, N - 1]
    for m, k, v in zip(tokens, (K - 1, 0, 127, K // 2, K - 9), (inf, -inf, nan, inf, -inf)):
        d.X[m, k] = v
    for n, j, v in zip(rows, (0, r - 1, r // 2, r - 1), (nan, inf, -inf, inf)):
        d.B[n, j] = v
    Y = d.matmul()
    np.testing.assert_array_equal(Y, by_whole_tiles(d, M))
    assert not np.isfinite(Y[tokens]).any() and not np.isfinite(Y[:, rows]).any()
    keep = np.ix_(np.setdiff1d(np.arange(M), tokens), np.setdiff1d(np.arange(N), rows))
    np.testing.assert_array_equal(Y[keep], finite[keep])
    d.A[r - 1, K - 1] = inf                                  # (every weight of the last column)
    Y = d.matmul()
    np.testing.assert_array_equal(Y, by_whole_tiles(d, M))
    assert not np.isfinite(Y).any()


def test_two_pass_slab_tiles_and_bf16_output(gpu):
    """Codes in the slab-tile layout give the bits of the canonical rows; bf16 outputs are the rounded fp32 ones."""
    import torch
    import paper_2601_22716_amd as L
    M, N, K, r, bits = 3000, 2999, 544, 99, 3
    say("two passes, slab tiles")
    assert takes_two_passes(M, [N], K, r, bits, False)
    c = li.make_case("tiny", M=M, N=N, K=K, r=r, bits=bits, factor_dtype="bf16", seed=4, signed_factors=True)
    d = gpu.DeviceCase(c)
    tiled = torch.empty(L.lords_repack_bytes(N, K, bits), dtype=torch.uint8, device="cuda")
    L.lords_repack(d.codes, tiled, N, K, bits)
    Y32 = torch.full((M, N), float("nan"), device="cuda")
    Y16 = torch.full((M, N), float("nan"), device="cuda", dtype=torch.bfloat16)
    L.lords_matmul_repacked(d.X, tiled, d.codebook, d.B, d.A, Y32, M, N, K, r, bits)
    L.lords_matmul(d.X, d.codes, d.codebook, d.B, d.A, Y16, M, N, K, r, bits)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(Y32.cpu().numpy(), d.matmul())
    assert torch.equal(Y32.bfloat16(), Y16)


@pytest.mark.parametrize("M,N,K,compared", [(1300, 19000, 4128, False), (1201, 19000, 4128, True), (1300, 33000, 2080, True)])
def test_two_pass_in_chunks(gpu, M, N, K, compared):
    """W larger than the scratch: rows in chunks, the last one ragged."""
    import torch
    r, bits = 128, 2
    say(f"two passes in chunks N={N} K={K}")
    assert takes_two_passes(M, [N], K, r, bits, False) and ((N + 15) // 16) * ((K + 127) // 128) * 4096 > 128 << 20
    c = li.make_case("tiny", M=M, N=N, K=K, r=r, bits=bits, factor_dtype="bf16", seed=5, signed_factors=True)
    d = gpu.DeviceCase(c)
    Y = d.matmul()
    check_rows(Y, c, c.X_f32, bits, "Y")
    assert plan_has_whole_tiles(M, N, K, r, bits, "bf16") == compared
    if compared:
        np.testing.assert_array_equal(Y, by_whole_tiles(d, M))
    del d
    torch.cuda.empty_cache()


@pytest.mark.parametrize("M,Ns,K,r,bits,fdt", [
    (3000, [2999, 500, 777], 544, 64, 4, "f32"), (4096, [3000, 40, 3001], 1056, 99, 3, "bf16"), (3000, [2999, 300], 2208, 64, 2, "bf16"),
    (2296, [2452, 1975], 704, 22, 3, "f32")])
def test_two_pass_batched(gpu, M, Ns, K, r, bits, fdt):
    """Several matrices, some of which alone would not go in two passes (of the last ones none does together): the single
    calls' bits; from a captured graph too."""
    import torch
    import paper_2601_22716_amd as L
    say(f"two passes batched M={M} Ns={Ns} K={K} r={r} bits={bits} factors={fdt}")
    assert takes_two_passes(M, [Ns[0]], K, r, bits, fdt == "f32")
    cases = [li.make_case("tiny", M=M, N=n, K=K, r=r, bits=bits, factor_dtype=fdt, seed=7 + i, signed_factors=True) for i, n in enumerate(Ns)]
    dev = [gpu.DeviceCase(c) for c in cases]
    out = [torch.full((M, n), float("nan"), device="cuda") for n in Ns]

    def call():
        L.lords_matmul_batched(dev[0].X, [d.codes for d in dev], dev[0].codebook, [d.B for d in dev], [d.A for d in dev], out, Ns, M, K, r, bits)
    call()
    torch.cuda.synchronize()
    single = [d.matmul(X=dev[0].X, M=M) for d in dev]
    for l, (c, o) in enumerate(zip(cases, out)):
        check_rows(o.cpu().numpy(), c, cases[0].X_f32, bits, f"matrix {l}", seed=l)
        np.testing.assert_array_equal(o.cpu().numpy(), single[l], err_msg=f"matrix {l}")
    graph, stream = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    with torch.cuda.graph(graph, stream=stream):
        call()
    for rep in range(3):
        for o in out:
            o.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        for l, o in enumerate(out):
            np.testing.assert_array_equal(o.cpu().numpy(), single[l], err_msg=f"replay {rep}, matrix {l}")
        dev[-1].matmul(X=dev[0].X, M=M)                      # eager work between the replays


def test_two_pass_batched_in_groups(gpu):
    """Eight matrices of 36864 columns, a tile of each of which is more than the scratch holds: the single calls' bits."""
    import torch
    import paper_2601_22716_amd as L
    M, N, K, r, bits = 2049, 600, 36864, 64, 4
    say("two passes batched in groups")
    assert takes_two_passes(M, [N], K, r, bits, True)
    dev = [gpu.DeviceCase(li.make_case("tiny", M=M if i == 0 else 1, N=N, K=K, r=r, bits=bits, factor_dtype="f32", seed=61 + i, signed_factors=True))
           for i in range(8)]
    out = [torch.full((M, N), float("nan"), device="cuda") for _ in dev]
    L.lords_matmul_batched(dev[0].X, [d.codes for d in dev], dev[0].codebook, [d.B for d in dev], [d.A for d in dev], out, [N] * 8, M, K, r, bits)
    torch.cuda.synchronize()
    for l, (d, o) in enumerate(zip(dev, out)):
        np.testing.assert_array_equal(o.cpu().numpy(), d.matmul(X=dev[0].X, M=M), err_msg=f"matrix {l}")


@pytest.mark.parametrize("M,N,K,r,bits,fdt", [(3000, 2999, 544, 64, 4, "f32"), (3001, 2002, 1056, 99, 3, "bf16"), (1025, 20011, 4128, 128, 2, "bf16"), (2049, 2002, 1120, 64, 4, "bf16"),
                                                (2243, 617, 288, 21, 2, "bf16"), (2049, 1990, 416, 32, 3, "bf16"), (4100, 1031, 320, 7, 4, "bf16"), (2557, 2003, 1696, 9, 3, "f32")])
def test_two_pass_gate_up(gpu, M, N, K, r, bits, fdt):
    """The pair against silu(gate) * up formed from the two single products, whose sums it has: fp32 silu and product, so
    a few units of 2^-24 and of the exponential's error, relative to the element."""
    import torch
    import paper_2601_22716_amd as L
    say(f"two passes gate/up M={M} N={N} K={K} r={r} bits={bits} factors={fdt}")
    assert takes_two_passes(M, [N, N], K, r, bits, fdt == "f32", act=True)
    dev = [gpu.DeviceCase(li.make_case("tiny", M=M, N=N, K=K, r=r, bits=bits, factor_dtype=fdt, seed=11 + i, signed_factors=True)) for i in range(2)]
    ga, up = dev
    G, U = (torch.from_numpy(d.matmul(X=ga.X, M=M)).double() for d in dev)
    H = torch.full((M, N), float("nan"), device="cuda")
    L.lords_gate_up(ga.X, ga.codes, ga.B, ga.A, up.codes, up.B, up.A, ga.codebook, H, M, N, K, r, bits)
    torch.cuda.synchronize()
    want = G * torch.sigmoid(G) * U
    # (the sums may be cut otherwise where a single product shares tiles: 1e-6 of their rms)
    bound = 4e-6 * want.abs() + 4e-6 * (G.square().mean().sqrt() * U.abs() + U.square().mean().sqrt() * G.abs()) + 1e-12
    assert bool(((H.cpu().double() - want).abs() <= bound).all())


@pytest.mark.parametrize("fdt,r", [("f32", 64), ("bf16", 99)])
def test_two_pass_backward_input(gpu, fdt, r):
    """The gradient of the input is the forward product of the transposed layer."""
    import torch
    import paper_2601_22716_amd as L
    M, N, K, bits = 3000, 544, 2976, 4
    say(f"two passes backward factors={fdt} r={r}")
    assert takes_two_passes(M, [K], N, r, bits, fdt == "f32")
    c = li.make_case("tiny", M=M, N=N, K=K, r=r, bits=bits, factor_dtype=fdt, seed=9, signed_factors=True)
    d = gpu.DeviceCase(c)
    codes_t = torch.empty((K, L.lords_row_bytes(N, bits)), dtype=torch.uint8, device="cuda")
    L.lords_transpose_codes(d.codes, codes_t, N, K, bits)
    dY = torch.randn((M, N), generator=torch.Generator(device="cuda").manual_seed(1), device="cuda").bfloat16()
    dX = torch.full((M, K), float("nan"), device="cuda")
    L.lords_backward_input(dY, codes_t, d.codebook, d.B, d.A, dX, M, N, K, r, bits)
    torch.cuda.synchronize()
    Wh = c.codebook.astype(np.float64)[d.unpack()] * (c.B_f32.astype(np.float64) @ c.A_f32.astype(np.float64))
    want = dY.float().cpu().numpy().astype(np.float64) @ Wh
    rf, mx = onp.rel_fro(dX.cpu().numpy(), want), onp.max_abs_over_rms(dX.cpu().numpy(), want)
    say(f"   dX: rel_fro={rf:.2e} max/rms={mx:.2e}")
    assert rf <= Y_TOL and mx <= Y_MAX_TOL, (rf, mx)
