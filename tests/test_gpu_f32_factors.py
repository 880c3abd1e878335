"""fp32 factors on the few-token and large-M kernels: the split into bf16 parts at the edges of the contraction
lengths (3 r = 32, 64, 128, 192), ragged rows and columns, and the calls that have no scratch to share tiles in."""
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
    rf, mx = onp.rel_fro(Y, want), onp.max_abs_over_rms(Y, want)
    print(f"   {what}: rel_fro={rf:.2e} max/rms={mx:.2e}", flush=True)
    assert np.isfinite(Y).all(), what
    assert rf <= Y_TOL and mx <= Y_MAX_TOL, (what, rf, mx)


@pytest.mark.parametrize("r", [1, 10, 11, 21, 22, 42, 43, 64, 65])
@pytest.mark.parametrize("M,N,K,bits", [(1, 270, 544, 4), (2, 17, 2080, 3), (16, 515, 1312, 2), (17, 129, 288, 4),
                                        (130, 1030, 416, 3), (300, 700, 1184, 2)])
def test_products_at_the_edges(gpu, M, N, K, bits, r):
    print(f"f32 factors M={M} N={N} K={K} bits={bits} r={r}", flush=True)
    cs = li.make_case("tiny", M=M, N=N, K=K, bits=bits, r=r, factor_dtype="f32", seed=11, signed_factors=True)
    want = onp.matmul(cs.X_f32, cs.codes, cs.codebook, cs.B_f32, cs.A_f32, cs.bits)
    check(gpu.DeviceCase(cs).matmul(), want, "product")


@pytest.mark.parametrize("r", [4, 16, 40, 60])
def test_low_parts_of_the_factors_are_used(gpu, r):
    """X = the first rows of the identity returns single weights: integer levels and the scale are exact but for the
    dropped Blo * Alo and the rounded low parts (2^-16 of each positive term), the fp32 sums (3 r additions of 2^-24) and
    the one rounding of the weight to bf16, whose 8 significant bits round by up to 2^-8 of a value just above a power of
    two.  Without the low parts each factor would be off by up to 2^-8 as well."""
    import torch
    K, N, M = 544, 200, 160
    cs = li.make_case("tiny", M=M, N=N, K=K, bits=4, r=r, factor_dtype="f32", seed=12, codebook="int")
    d = gpu.DeviceCase(cs)
    d.X = torch.eye(K, device="cuda", dtype=torch.bfloat16)[:M].contiguous()
    want = onp.dequant(cs.codes, cs.codebook, cs.B_f32, cs.A_f32, cs.bits)[:, :M].T
    Y = d.matmul()
    assert np.all(np.abs(Y - want) <= (2.0 ** -8 + 2.0 ** -14) * np.abs(want) + 1e-30)


@pytest.mark.parametrize("M,N,K,r", [(300, 4096, 1056, 16), (200, 1030, 2080, 40)])
def test_front_only_workspace_is_enough(gpu, M, N, K, r):
    """A large-M call with fp32 factors runs in a workspace of the front alone (whole tiles), as it does under capture
    before anything larger was handed out."""
    import torch
    import paper_2601_22716_amd as L
    cs = li.make_case("tiny", M=M, N=N, K=K, bits=4, r=r, factor_dtype="f32", seed=13, signed_factors=True)
    d = gpu.DeviceCase(cs)
    want = onp.matmul(cs.X_f32, cs.codes, cs.codebook, cs.B_f32, cs.A_f32, cs.bits)
    ws = torch.zeros(L.lords_workspace_zero_bytes(), dtype=torch.uint8, device="cuda")
    Y = torch.full((M, N), float("nan"), dtype=torch.float32, device="cuda")
    L.lords_matmul_ws(d.X, d.codes, d.codebook, d.B, d.A, Y, M, N, K, r, 4, ws)
    torch.cuda.synchronize()
    check(Y.cpu().numpy(), want, "front only")
    assert not ws.any().item(), "the front is left at zero"
