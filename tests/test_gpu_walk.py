"""Several matrices in one launch whose tiles are cut into parts, of which a workgroup takes two, four or eight one after the other:
every matrix has the bits of its single call, whoever waits for whom, and the counts are back at zero."""
import ctypes

import pytest

import lords_inputs as li

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,Ns,K,r,bits,fdt,cut", [
    # 256 x 256 tiles; 256 x 128; 128-token tiles; 64 (six times 32 columns); a tile one workgroup's, or shared by two or four
    (266, [5515, 3085, 1529, 1830], 1344, 5, 3, "bf16", (256, 256, 4, 2)), (268, [836, 2401, 1327], 5056, 8, 2, "bf16", (256, 256, 8, 2)),
    (1115, [1865, 3479, 2831], 1824, 20, 4, "bf16", (256, 256, 2, 2)),
    (268, [703, 460, 3970, 1905], 1152, 14, 2, "bf16", (256, 128, 2, 2)), (257, [261, 1957, 1886, 116], 1024, 22, 3, "bf16", (256, 128, 4, 2)),
    (277, [343, 3946, 432, 1671], 1408, 20, 3, "bf16", (256, 128, 4, 4)), (262, [2195, 612, 127, 3047], 2656, 5, 4, "bf16", (256, 128, 8, 4)),
    (305, [293, 407, 338, 157], 4352, 11, 4, "bf16", (256, 128, 8, 2)),
    (24, [4487, 2353, 175, 4240], 2688, 4, 4, "bf16", (128, 128, 8, 8)), (273, [2748, 3472, 4233, 1212], 992, 53, 4, "bf16", (128, 256, 2, 2)),
    (486, [2134, 2157], 928, 84, 2, "bf16", (128, 256, 4, 2)), (135, [591, 2925, 1285, 100], 1024, 105, 4, "bf16", (128, 128, 4, 2)),
    (283, [2325, 4338, 4280], 2208, 5, 3, "f32", (128, 256, 4, 4)), (204, [530, 777, 1027, 2475], 1952, 39, 2, "f32", (128, 128, 8, 4)),
    (97, [3952, 2837], 1024, 46, 3, "f32", (64, 128, 4, 4)), (220, [2037, 193, 224], 960, 58, 2, "f32", (64, 128, 4, 2))])
def test_several_parts_by_one_workgroup(M, Ns, K, r, bits, fdt, cut):
    import torch
    import paper_2601_22716_amd as L
    from tests import gpu_util, plan_util
    print(f"several parts M={M} Ns={Ns} K={K} r={r} bits={bits} factors={fdt}", flush=True)
    q, f32, n = plan_util.queries(), fdt == "f32", len(Ns)
    assert cut in plan_util.batched_cuts(M, Ns, K, r, bits, f32) and not plan_util.takes_two_passes(M, Ns, K, r, bits, f32)
    dev = [gpu_util.DeviceCase(li.make_case("tiny", M=M, N=N, K=K, bits=bits, r=r, factor_dtype=fdt, seed=85 + i, signed_factors=True)) for i, N in enumerate(Ns)]
    X, codebook = dev[0].X, dev[0].codebook
    front, part = L.lords_workspace_zero_bytes(), q.prefill_batched_workspace_bytes((ctypes.c_int * n)(*Ns), n, M, K, r, bits, int(f32))
    ws = torch.zeros(front + part, dtype=torch.uint8, device="cuda")
    each = lambda ts: (ctypes.c_void_p * n)(*[t.data_ptr() for t in ts])
    for dtype in (torch.float32, torch.bfloat16):
        want = [torch.full((M, N), float("nan"), dtype=dtype, device="cuda") for N in Ns]
        for d, N, Y in zip(dev, Ns, want):
            L.lords_matmul(X, d.codes, codebook, d.B, d.A, Y, M, N, K, r, bits)
        Ys = [torch.full((M, N), float("nan"), dtype=dtype, device="cuda") for N in Ns]
        L.lords_matmul_batched(X, [d.codes for d in dev], codebook, [d.B for d in dev], [d.A for d in dev], Ys, Ns, M, K, r, bits)
        torch.cuda.synchronize()
        for l in range(n):
            assert torch.isfinite(want[l]).all() and torch.equal(Ys[l], want[l]), (dtype, l)
        for polls in (0, 1, 1 << 20):
            ws[front:] = 255                                    # (not a number: a part that is read before it is written shows)
            for Y in Ys:
                Y.fill_(float("nan"))
            assert q.launch_large_batched(X.data_ptr(), each([d.codes for d in dev]), codebook.data_ptr(), each([d.B for d in dev]), each([d.A for d in dev]), each(Ys),
                                          (ctypes.c_int * n)(*Ns), n, M, K, r, bits, int(f32), int(dtype == torch.float32), ws.data_ptr() + front, ws.data_ptr(),
                                          torch.cuda.current_stream().cuda_stream, polls) == 0
            torch.cuda.synchronize()
            assert not ws[:front].any()
            for l in range(n):
                assert torch.equal(Ys[l], want[l]), (dtype, polls, l)
