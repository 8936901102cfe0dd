"""GPU parity of the stage-load GEMM (bf16 MFMA, fp32 accumulate) against the fp64 oracle."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import paper_2409_06941_amd as fr          # noqa: E402
from oracle.gemm import gemm_nt            # noqa: E402
from workloads import gemm_inputs          # noqa: E402


def _to_dev_bf16(x32):
    bits = gemm_inputs.bf16_bits(x32).view(np.int16)
    return torch.from_numpy(bits).cuda()


# from two tiles to more than two tiles per CU; tile counts that are and are not multiples of the 8 XCDs
@pytest.mark.parametrize("M,N,K", [(256, 256, 64), (256, 512, 192), (768, 256, 4096), (512, 1280, 320),
                                   (2048, 8192, 128), (1024, 16384 + 256, 192)])
def test_gemm_matches_oracle(M, N, K):
    print("gemm", M, N, K, flush=True)
    a, b = gemm_inputs.operands(M, N, K, seed=M + N + K)
    A, B = _to_dev_bf16(a), _to_dev_bf16(b)
    Cm = torch.zeros((M, N), dtype=torch.int16, device="cuda")
    fr.fr_gemm_bf16(A, B, Cm, M, N, K, torch.cuda.current_stream())
    torch.cuda.synchronize()
    got = gemm_inputs.bits_to_f32(Cm.cpu().numpy().view(np.uint16)).astype(np.float64)
    want = gemm_nt(a, b)
    # result = bf16 rounding (relative 2^-8 at most, half an ulp of 8 bits) of an fp32-accumulated sum whose own
    # error is bounded by K * 2^-24 * sum|a||b| <= K * 2^-24 * K (|a|, |b| < 1)
    bound = np.abs(want) * 2.0 ** -8 + K * K * 2.0 ** -24 + 1e-30
    assert np.all(np.abs(got - want) <= bound)
    # and it must be the nearest bf16 for nearly every entry (loose accumulation differences aside)
    nearest = gemm_inputs.bf16_round(want.astype(np.float32)).astype(np.float64)
    assert np.mean(got == nearest) > 0.98


# sizes on both sides of the lines between the tiles as the choice draws them on 256 units, through the public call
@pytest.mark.parametrize("M,N,K", [(256, 256, 64), (512, 768, 448), (256, 512, 2624), (512, 256, 4160), (1024, 1536, 512),
                                   (1280, 1536, 1216), (2048, 4096, 320), (2048, 4096, 1088), (4352, 3840, 1216), (3328, 4608, 64)])
def test_every_tile_shape_matches_oracle(M, N, K):
    test_gemm_matches_oracle(M, N, K)


# every tile, whatever the choice would be: one, two and three k-tiles, odd and even counts, counts that do not divide by
# four (K in four parts), and a band of rows that is cut short
@pytest.mark.parametrize("tile", range(7))
@pytest.mark.parametrize("M,N,K", [(256, 256, 64), (256, 512, 128), (512, 256, 192), (256, 256, 320), (512, 768, 448), (1280, 512, 512), (256, 256, 1216)])
def test_each_tile_matches_oracle(tile, M, N, K):
    print("gemm tile", tile, M, N, K, flush=True)
    a, b = gemm_inputs.operands(M, N, K, seed=M + N + K)
    A, B = _to_dev_bf16(a), _to_dev_bf16(b)
    Cm = torch.zeros((M, N), dtype=torch.int16, device="cuda")
    f = fr.lib().fr_gemm_bf16_tile
    f.argtypes = [ctypes.c_void_p] * 3 + [ctypes.c_int32] * 4 + [ctypes.c_void_p]
    assert f(A.data_ptr(), B.data_ptr(), Cm.data_ptr(), M, N, K, tile, torch.cuda.current_stream().cuda_stream) == fr.FR_OK
    torch.cuda.synchronize()
    got = gemm_inputs.bits_to_f32(Cm.cpu().numpy().view(np.uint16)).astype(np.float64)
    want = gemm_nt(a, b)
    assert np.all(np.abs(got - want) <= np.abs(want) * 2.0 ** -8 + K * K * 2.0 ** -24 + 1e-30)      # as in test_gemm_matches_oracle
    assert f(A.data_ptr(), B.data_ptr(), Cm.data_ptr(), M, N, K, 7, None) == fr.FR_ERR_ARG


def test_streams_with_few_units_and_captured_graphs():
    # the choice of a tile asks the stream for its units: a masked stream, and a stream that is capturing
    M, N, K = 512, 2816, 320
    a, b = gemm_inputs.operands(M, N, K, seed=3)
    A, B = _to_dev_bf16(a), _to_dev_bf16(b)
    Cm = torch.zeros((M, N), dtype=torch.int16, device="cuda")
    want = gemm_nt(a, b)
    bound = np.abs(want) * 2.0 ** -8 + K * K * 2.0 ** -24 + 1e-30

    def check():
        torch.cuda.synchronize()
        got = gemm_inputs.bits_to_f32(Cm.cpu().numpy().view(np.uint16)).astype(np.float64)
        assert np.all(np.abs(got - want) <= bound)
        Cm.zero_()
    for cus in (8, 64):
        print("units", cus, flush=True)
        ctx = fr.Context(device_id=0, cu_count=cus)
        torch.cuda.synchronize()
        fr.fr_gemm_bf16(A, B, Cm, M, N, K, ctx.fr_side_stream())
        check()
        ctx.fr_destroy()
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        fr.fr_gemm_bf16(A, B, Cm, M, N, K, torch.cuda.current_stream())
    for _ in range(3):
        graph.replay()
        check()


def test_identity_and_shape_errors():
    M = N = K = 256
    a, _ = gemm_inputs.operands(M, N, K, seed=1)
    eye = np.eye(N, K, dtype=np.float32)
    A, B = _to_dev_bf16(a), _to_dev_bf16(eye)
    Cm = torch.zeros((M, N), dtype=torch.int16, device="cuda")
    fr.fr_gemm_bf16(A, B, Cm, M, N, K, torch.cuda.current_stream())
    torch.cuda.synchronize()
    assert np.array_equal(Cm.cpu().numpy().view(np.uint16), gemm_inputs.bf16_bits(a))     # exact
    for shape in [(250, 256, 64), (256, 100, 64), (256, 256, 72), (0, 256, 64)]:
        with pytest.raises(fr.FreeRideError) as e:
            fr.fr_gemm_bf16(A, B, Cm, *shape, torch.cuda.current_stream())
        assert e.value.code == fr.FR_ERR_ARG


def test_gpt_load_bursts_run_and_report_flops():
    layers, h, ffn, T = 2, 512, 2048, 256
    need = fr.Load.fr_load_workspace_bytes(fr.FR_LOAD_GPT, layers, h, ffn, T)
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    load = fr.Load(fr.FR_LOAD_GPT, layers, h, ffn, T, workspace=ws, seed=7, stream=torch.cuda.current_stream())
    fp, bp = load.fr_load_flops()
    per_layer = 2 * T * (3 * h * h + h * h + 2 * h * ffn)
    assert fp == layers * per_layer and bp == 2 * fp
    load.fr_load_fp(torch.cuda.current_stream())
    load.fr_load_bp(torch.cuda.current_stream())
    torch.cuda.synchronize()
    load.fr_load_destroy()
    with pytest.raises(fr.FreeRideError):
        fr.Load(fr.FR_LOAD_GPT, layers, h, ffn, T, workspace=ws[: need // 2], seed=7)
