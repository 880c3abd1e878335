"""Calls that cannot have the workspace they would like: what follows a refused allocation, and the forms that run with less.
A copy of the library, loaded beside it, stands for a program that has not grown its workspace yet."""
import shutil

import numpy as np
import pytest

import lords_inputs as li

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from tests import gpu_util
    return gpu_util


@pytest.fixture
def fresh_library(tmp_path, monkeypatch):
    """The binding's calls go to a library whose workspace is still unallocated."""
    from paper_2601_22716_amd import binding
    copy = str(tmp_path / "liblords_fresh.so")
    shutil.copy(binding.library_path(), copy)
    monkeypatch.setattr(binding, "_LIB_PATH", copy)
    monkeypatch.setattr(binding, "_lib", None)


def captured(call):
    import torch
    stream = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=stream):
        call()
    return graph


def test_refused_allocation_leaves_no_error_behind(gpu, fresh_library):
    """A gate/up product whose fp32 gate would take 512 GiB is refused before anything is launched; the calls after it are
    none the wiser."""
    import torch
    import paper_2601_22716_amd as L
    cs = li.make_case("tiny", M=40, N=512, K=256, bits=4, r=8, factor_dtype="bf16", seed=51)
    d = gpu.DeviceCase(cs)
    want = d.matmul()
    with pytest.raises(L.LordsError) as e:      # (the small arrays are never read: the call ends at its workspace)
        L.lords_gate_up(d.X, d.codes, d.B, d.A, d.codes, d.B, d.A, d.codebook, d.X, 2048, 1 << 26, 32, 8, 4)
    assert e.value.status == 6
    np.testing.assert_array_equal(d.matmul(), want)
    assert torch.ones(3, device="cuda").sum().item() == 3


@pytest.mark.parametrize("fdt,r", [("bf16", 32), ("f32", 16)])
def test_batched_call_without_its_joint_scratch(gpu, fresh_library, fdt, r):
    """Captured after each matrix alone was warmed up, a batched call of many tokens finds room for the largest matrix's
    partial sums but not for all of them together: it runs matrix by matrix, with the same results."""
    import torch
    import paper_2601_22716_amd as L
    M, K, bits, Ns = 300, 2080, 4, [4096, 3000, 4099]
    dev = [gpu.DeviceCase(li.make_case("tiny", M=M, N=N, K=K, bits=bits, r=r, factor_dtype=fdt, seed=52 + i)) for i, N in enumerate(Ns)]
    X = dev[0].X
    want = [d.matmul(X=X) for d in dev]
    Ys = [torch.empty((M, N), device="cuda") for N in Ns]

    front = L.lords_workspace_zero_bytes()
    scratch = [L.lords_workspace_bytes(M, N, K, r, bits, L.LORDS_F32 if fdt == "f32" else L.LORDS_BF16) - front for N in Ns]
    assert sum(scratch) > 1.5 * (max(scratch) + front)          # (a grown workspace has half as much to spare)

    def call():
        L.lords_matmul_batched(X, [d.codes for d in dev], dev[0].codebook, [d.B for d in dev], [d.A for d in dev], Ys, Ns, M, K, r, bits)

    graph = captured(call)
    for rep in range(3):
        for Y in Ys:
            Y.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        for Y, w in zip(Ys, want):
            np.testing.assert_array_equal(Y.cpu().numpy(), w, err_msg=f"replay {rep}")
        np.testing.assert_array_equal(dev[1].matmul(X=X), want[1])            # eager work between the replays
    call()                                                                   # ... and now the joint launch
    torch.cuda.synchronize()
    for Y, w in zip(Ys, want):
        np.testing.assert_array_equal(Y.cpu().numpy(), w)


def test_f32_factor_products_do_not_depend_on_what_was_allocated(gpu, fresh_library):
    """Products of many tokens with fp32 factors, captured while the library holds its smallest workspace, and the same calls
    after it has grown: the same bits."""
    import torch
    import paper_2601_22716_amd as L
    M, N, K, r, bits = 300, 4096, 1056, 16, 4
    d = gpu.DeviceCase(li.make_case("tiny", M=M, N=N, K=K, bits=bits, r=r, factor_dtype="f32", seed=55, signed_factors=True))
    codes_t = torch.empty((K, L.lords_row_bytes(N, bits)), dtype=torch.uint8, device="cuda")
    L.lords_transpose_codes(d.codes, codes_t, N, K, bits)
    dY = torch.randn((M, N), device="cuda").to(torch.bfloat16)
    Y, dX, H = torch.empty((M, N), device="cuda"), torch.empty((M, K), device="cuda"), torch.empty((M, 1024), device="cuda")

    def call():
        L.lords_matmul(d.X, d.codes, d.codebook, d.B, d.A, Y, M, N, K, r, bits)
        L.lords_backward_input(dY, codes_t, d.codebook, d.B, d.A, dX, M, N, K, r, bits)
        L.lords_gate_up(d.X, d.codes, d.B, d.A, d.codes, d.B, d.A, d.codebook, H, M, 1024, K, r, bits)

    d.matmul(M=1, X=d.X[:1].contiguous())                   # (the front has to be there before a capture)
    graph = captured(call)
    results = []
    for rep in range(3):
        for out in (Y, dX, H):
            out.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        results.append([out.cpu().numpy() for out in (Y, dX, H)])
        if rep == 0:                                        # grows the workspace
            gpu.DeviceCase(li.make_case("tiny", M=300, N=4099, K=2080, bits=4, r=32, factor_dtype="bf16", seed=56)).matmul()
    call()
    torch.cuda.synchronize()
    results.append([out.cpu().numpy() for out in (Y, dX, H)])
    for other in results[1:]:
        for a, b in zip(results[0], other):
            assert np.isfinite(a).all()
            np.testing.assert_array_equal(a, b)
    # ... and those of a caller's workspace of the size asked for, and of a larger one
    need = L.lords_workspace_bytes(M, N, K, r, bits, L.LORDS_F32)
    for size in (need, need + (64 << 20)):
        ws = torch.zeros(size, dtype=torch.uint8, device="cuda")
        L.lords_matmul_ws(d.X, d.codes, d.codebook, d.B, d.A, Y, M, N, K, r, bits, ws)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(Y.cpu().numpy(), results[0][0])


def replays(graph, outs, between):
    """Outputs of three replays, eager work between them."""
    import torch
    results = []
    for _ in range(3):
        for out in outs:
            out.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        results.append([out.float().cpu().numpy() for out in outs])
        between()
    for other in results[1:]:
        for a, b in zip(results[0], other):
            np.testing.assert_array_equal(a, b)
    return results[0]


@pytest.mark.parametrize("fdt,r", [("f32", 64), ("bf16", 64), ("bf16", 99)])
def test_two_passes_without_their_scratch(gpu, fresh_library, fdt, r):
    """Captured while the library's workspace has no room for the dequantised weights, products that go in two passes run by whole
    tiles: the bits of the eager calls after it."""
    import torch
    import paper_2601_22716_amd as L
    from tests import plan_util
    M, N, K, bits, f32 = 2049, 4003, 2208, 4, fdt == "f32"
    d = gpu.DeviceCase(li.make_case("tiny", M=M, N=N, K=K, bits=bits, r=r, factor_dtype=fdt, seed=71, signed_factors=True))
    e = gpu.DeviceCase(li.make_case("tiny", M=1, N=4001, K=K, bits=bits, r=r, factor_dtype=fdt, seed=72, signed_factors=True))
    # ... and the gradient of the input of a layer with the transposed sizes
    b = gpu.DeviceCase(li.make_case("tiny", M=1, N=K, K=4032, bits=bits, r=r, factor_dtype=fdt, seed=73, signed_factors=True))
    codes_t = torch.empty((b.K, L.lords_row_bytes(b.N, bits)), dtype=torch.uint8, device="cuda")
    L.lords_transpose_codes(b.codes, codes_t, b.N, b.K, bits)
    for n in (N, e.N, b.K):
        assert plan_util.takes_two_passes(M, [n], K, r, bits, f32) and n * K * 2 > 16 << 20        # (the first block: 16 MiB)
    Y, dX = torch.empty((M, N), device="cuda"), torch.empty((M, b.K), device="cuda")
    Ys = [torch.empty((M, n), device="cuda") for n in (N, e.N)]

    def call():
        L.lords_matmul(d.X, d.codes, d.codebook, d.B, d.A, Y, M, N, K, r, bits)
        L.lords_matmul_batched(d.X, [d.codes, e.codes], d.codebook, [d.B, e.B], [d.A, e.A], Ys, [N, e.N], M, K, r, bits)
        L.lords_backward_input(d.X, codes_t, d.codebook, b.B, b.A, dX, M, b.N, b.K, r, bits)

    d.matmul(M=1, X=d.X[:1].contiguous())                   # (the front has to be there before a capture)
    outs = [Y, *Ys, dX]
    got = replays(captured(call), outs, lambda: d.matmul(M=1, X=d.X[:1].contiguous()))
    call()
    torch.cuda.synchronize()
    for g, out in zip(got, outs):
        assert np.isfinite(g).all()
        np.testing.assert_array_equal(g, out.cpu().numpy())


@pytest.mark.parametrize("fdt,r,bits", [("f32", 64, 4), ("bf16", 99, 3), ("bf16", 64, 2)])
def test_gate_up_in_two_passes_without_its_scratch(gpu, fresh_library, fdt, r, bits):
    """Captured with room for the gate of 2048 tokens but not for the dequantised weights: 2048 tokens and then the others by
    whole tiles, the bits of the eager call after it."""
    import torch
    import paper_2601_22716_amd as L
    from tests import plan_util
    M, N, K = 2200, 1502, 4128
    assert plan_util.takes_two_passes(M, [N, N], K, r, bits, fdt == "f32", act=True)
    assert 2 * N * K * 2 > 16 << 20 > 2048 * N * 4 + L.lords_workspace_zero_bytes()
    ga, up = (gpu.DeviceCase(li.make_case("tiny", M=M if i == 0 else 1, N=N, K=K, bits=bits, r=r, factor_dtype=fdt, seed=75 + i, signed_factors=True)) for i in range(2))
    H, H16 = torch.empty((M, N), device="cuda"), torch.empty((M, N), device="cuda", dtype=torch.bfloat16)

    def call():
        for out in (H, H16):
            L.lords_gate_up(ga.X, ga.codes, ga.B, ga.A, up.codes, up.B, up.A, ga.codebook, out, M, N, K, r, bits)

    ga.matmul(M=1, X=ga.X[:1].contiguous())
    got = replays(captured(call), [H, H16], lambda: ga.matmul(M=1, X=ga.X[:1].contiguous()))
    call()
    torch.cuda.synchronize()
    assert np.isfinite(got[0]).all()
    np.testing.assert_array_equal(got[0], H.cpu().numpy())
    np.testing.assert_array_equal(got[1], H16.float().cpu().numpy())


def test_wide_tiles_without_room_for_their_parts(gpu, fresh_library):
    """Ranks 33 to 64: a product whose 256-token tiles would share 64 MiB of parts is cut for what there is.  Its sums may then
    differ from the full plan's by the order of their 8160 fp32 additions (about sqrt(8160) 2^-24 = 5e-6 of their rms)."""
    import torch
    import paper_2601_22716_amd as L
    from oracle import lords_oracle as onp
    from tests import plan_util
    M, N, K, r, bits = 250, 28672, 8160, 33, 2
    q = plan_util.queries()
    assert q.prefill_workspace_bytes(M, N, K, r, bits, 0) > 32 << 20 and q.prefill_least_workspace_bytes(M, N, K, r, bits, 0) < 8 << 20
    d = gpu.DeviceCase(li.make_case("tiny", M=M, N=N, K=K, bits=bits, r=r, factor_dtype="bf16", seed=79, signed_factors=True))
    Y = torch.empty((M, N), device="cuda")

    def call():
        L.lords_matmul(d.X, d.codes, d.codebook, d.B, d.A, Y, M, N, K, r, bits)

    d.matmul(M=1, X=d.X[:1].contiguous())
    got, = replays(captured(call), [Y], lambda: d.matmul(M=1, X=d.X[:1].contiguous()))
    call()
    torch.cuda.synchronize()
    full = Y.cpu().numpy()
    assert np.isfinite(got).all() and onp.rel_fro(got, full) <= 1e-5
