"""The large-M kernel's form with one wave per SIMD (bf16 factors of rank 33 .. 64, 256 x 256 tiles), through the C ABI, against the
fp64 oracle on sampled rows; whole tiles and tiles shared by several workgroups, in runs shorter and longer than a tile.
Gates as for lords_matmul.

Sizes: the planner takes this form at them, and they are off the tiles in every direction: tokens and rows that are no
multiples of 256, 64, 16 or 4, K tiles of every raggedness (32, 64 and 96 columns left over), one K tile alone, ranks at both
ends of the range and odd ones, both code layouts, both output types.
"""
import sys

import numpy as np
import pytest

import lords_inputs as li
from oracle import lords_oracle as onp
from tests import plan_util

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


def taken(*problem):
    return bool(plan_util.queries().prefill_wide_taken(*problem, 0))


def check_rows(Y, c, bits, what, seed=0):
    rows = np.unique(np.concatenate([np.random.default_rng(seed).integers(0, c.N, 40), [0, c.N - 1], np.arange(max(0, c.N - 20), c.N)]))
    want = onp.matmul_rows(c.X_f32, c.codes, c.codebook, c.B_f32, c.A_f32, bits, rows)
    rf, mx = onp.rel_fro(Y[:, rows], want), onp.max_abs_over_rms(Y[:, rows], want)
    say(f"   {what}: rel_fro={rf:.2e} max/rms={mx:.2e}")
    assert np.isfinite(Y).all(), what
    assert rf <= Y_TOL and mx <= Y_MAX_TOL, (what, rf, mx)


SHAPES = [(3001, 2999, 96, 49, 2), (2049, 4097, 416, 33, 4), (257, 28001, 544, 63, 4), (1500, 7001, 2144, 37, 3),
          (3001, 2999, 3072, 64, 4), (2049, 4097, 4128, 45, 3), (201, 20002, 4192, 64, 2), (1500, 2999, 8288, 40, 3),
          (1001, 9003, 3072, 50, 4), (511, 9003, 8288, 61, 2)]


@pytest.mark.parametrize("M,N,K,r,bits", SHAPES)
def test_wide_product(gpu, M, N, K, r, bits):
    import torch
    import paper_2601_22716_amd as L
    say(f"wide M={M} N={N} K={K} r={r} bits={bits}")
    c = li.make_case("tiny", M=M, N=N, K=K, r=r, bits=bits, factor_dtype="bf16", seed=21, signed_factors=True)
    d = gpu.DeviceCase(c)
    # (a caller's workspace: the large-M kernel alone, whatever else the library would take)
    need = L.lords_workspace_bytes(M, N, K, r, bits, L.LORDS_BF16)
    assert taken(M, N, K, r, bits)
    ws = torch.zeros(need, dtype=torch.uint8, device="cuda")
    for rep in range(2):                                       # (the counters of shared tiles are left at zero)
        Y = torch.full((M, N), float("nan"), device="cuda")
        L.lords_matmul_ws(d.X, d.codes, d.codebook, d.B, d.A, Y, M, N, K, r, bits, ws)
        torch.cuda.synchronize()
        if rep == 0:
            first = Y
    assert torch.equal(first, Y)
    check_rows(Y.cpu().numpy(), c, bits, "Y")
    Y16 = torch.full((M, N), float("nan"), device="cuda", dtype=torch.bfloat16)
    L.lords_matmul_ws(d.X, d.codes, d.codebook, d.B, d.A, Y16, M, N, K, r, bits, ws)
    assert torch.equal(Y16, Y.bfloat16())


def test_wide_slab_tiles_gate_and_batch(gpu):
    """The other ways into it: the slab-tile layout, several matrices in a launch, the up product that multiplies by the
    gate's silu: the bits of the single products (silu and product in fp32: see the two-pass tests' bound)."""
    import torch
    import paper_2601_22716_amd as L
    M, N, K, r, bits = 300, 28001, 1056, 45, 3
    say("wide: slab tiles, pair, batch")
    assert taken(M, N, K, r, bits)
    dev = [gpu.DeviceCase(li.make_case("tiny", M=M, N=N, K=K, r=r, bits=bits, factor_dtype="bf16", seed=31 + i, signed_factors=True)) for i in range(2)]
    a, b = dev
    single = [torch.from_numpy(d.matmul(X=a.X, M=M)).cuda() for d in dev]
    tiled = torch.empty(L.lords_repack_bytes(N, K, bits), dtype=torch.uint8, device="cuda")
    L.lords_repack(a.codes, tiled, N, K, bits)
    Y = torch.full((M, N), float("nan"), device="cuda")
    L.lords_matmul_repacked(a.X, tiled, a.codebook, a.B, a.A, Y, M, N, K, r, bits)
    assert torch.equal(Y, single[0])
    out = [torch.full((M, N), float("nan"), device="cuda") for _ in dev]
    L.lords_matmul_batched(a.X, [d.codes for d in dev], a.codebook, [d.B for d in dev], [d.A for d in dev], out, [N, N], M, K, r, bits)
    for o, s in zip(out, single):
        assert torch.equal(o, s)
    H = torch.full((M, N), float("nan"), device="cuda")
    L.lords_gate_up(a.X, a.codes, a.B, a.A, b.codes, b.B, b.A, a.codebook, H, M, N, K, r, bits)
    G, U = (s.double() for s in single)
    want = G * torch.sigmoid(G) * U
    assert bool(((H.double() - want).abs() <= 4e-6 * want.abs() + 1e-12).all())


@pytest.mark.parametrize("M,N,K,r,bits", [(250, 28672, 8160, 33, 2), (201, 20002, 4192, 64, 2)])
def test_wide_smaller_workspace(gpu, M, N, K, r, bits):
    """These tiles' parts are twice as large as those of 128-token tiles.  A workspace that holds the latter is accepted all the
    same and the cut made for it; a smaller one is refused."""
    import torch
    import paper_2601_22716_amd as L
    least = L.lords_workspace_zero_bytes() + plan_util.queries().prefill_least_workspace_bytes(M, N, K, r, bits, 0)
    say(f"wide, smaller workspace M={M} N={N} K={K} r={r} bits={bits}: {least}")
    assert least < L.lords_workspace_bytes(M, N, K, r, bits, L.LORDS_BF16)
    c = li.make_case("tiny", M=M, N=N, K=K, r=r, bits=bits, factor_dtype="bf16", seed=23, signed_factors=True)
    d = gpu.DeviceCase(c)
    room = torch.zeros(least + 4096, dtype=torch.uint8, device="cuda")
    room[least:] = 77                                          # (nothing behind it is written)
    Y = torch.full((M, N), float("nan"), device="cuda")
    with pytest.raises(L.LordsError):
        L.lords_matmul_ws(d.X, d.codes, d.codebook, d.B, d.A, Y, M, N, K, r, bits, room[:least - 256])
    for _ in range(2):
        L.lords_matmul_ws(d.X, d.codes, d.codebook, d.B, d.A, Y, M, N, K, r, bits, room[:least])
    torch.cuda.synchronize()
    assert bool((room[least:] == 77).all())
    check_rows(Y.cpu().numpy(), c, bits, "Y")


@pytest.mark.parametrize("M,N,K,r,bits", [(257, 28001, 544, 63, 4), (1001, 9003, 3072, 50, 4)])
def test_wide_infinities_and_nan(gpu, M, N, K, r, bits):
    """Infinities and NaN in X and in the factors stay with their tokens and rows; the others keep their bits."""
    say(f"wide, infinities M={M} N={N} K={K} r={r} bits={bits}")
    assert taken(M, N, K, r, bits) and not plan_util.takes_two_passes(M, [N], K, r, bits, 0)
    d = gpu.DeviceCase(li.make_case("tiny", M=M, N=N, K=K, r=r, bits=bits, factor_dtype="bf16", seed=8, signed_factors=True))
    finite = d.matmul()
    inf, nan = float("inf"), float("nan")
    tokens, rows = [0, 255, 256, M // 2, M - 1], [0, 15, 300, N - 1]
    for m, k, v in zip(tokens, (K - 1, 0, 127, K // 2, K - 9), (inf, -inf, nan, inf, -inf)):
        d.X[m, k] = v
    for n, j, v in zip(rows, (0, r - 1, r // 2, r - 1), (nan, inf, -inf, inf)):
        d.B[n, j] = v
    Y = d.matmul()
    assert not np.isfinite(Y[tokens]).any() and not np.isfinite(Y[:, rows]).any()
    keep = np.ix_(np.setdiff1d(np.arange(M), tokens), np.setdiff1d(np.arange(N), rows))
    np.testing.assert_array_equal(Y[keep], finite[keep])
    d.A[r - 1, K - 1] = inf                                  # (every weight of the last column)
    assert not np.isfinite(d.matmul()).any()
