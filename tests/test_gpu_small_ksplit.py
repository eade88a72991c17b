"""Register-staged GEMM kernels: K sliced over workgroups, tiles of 64 and 128,
operands at every row alignment, and K tails inside a tile.  Bit-exact."""
import numpy as np
import pytest

from oracle import oracle as orc
from paper_2606_09905_amd import qx

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# batch, M, N, K: below and from eight K tiles, slices with a short last one,
# one row or column, many tiles (no slices), 128 x 128 tiles, K within 32
SHAPES = [(1, 1, 1, 448), (1, 1, 1, 449), (1, 20, 48, 4096), (1, 65, 63, 1001), (3, 22, 20, 700), (1, 17, 129, 8191),
          (1, 31, 2049, 577), (20, 1025, 49, 48), (6, 2049, 33, 129), (70, 60, 65, 200), (80, 64, 64, 72), (70, 17, 136, 40), (2, 300, 200, 130), (1, 1100, 1000, 29), (5, 130, 257, 33), (1, 64, 64, 24575)]
ROUTES = [("i8_direct", 127), ("f16_exact", 256), ("f16_exact", 1024), ("i8_karatsuba", 8000), ("i8_offset4", 32768)]


def ints(rng, shape, lo, hi, dtype):
    a = rng.integers(lo, hi, shape, dtype=np.int64, endpoint=True)
    a[rng.random(shape) < 0.2] = lo          # the extremes, often
    return a.astype(dtype)


def run(ex, A, B):
    with ex:
        out = ex.run([torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda()])
        again = ex.run([torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda()])
        torch.cuda.synchronize()
    assert torch.equal(out, again)
    return out.cpu().numpy()


@pytest.mark.parametrize("b,M,N,K", SHAPES)
@pytest.mark.parametrize("route,bound", ROUTES)
def test_i16(b, M, N, K, route, bound):
    rng = np.random.default_rng(M + N + K)
    hi = min(bound, 32767)
    A, B = ints(rng, (b, M, K), -bound, hi, np.int16), ints(rng, (b, K, N), -bound, hi, np.int16)
    C = run(qx.Executor.gemm_i16i32(M, N, K, b, bound, bound, route), A, B)
    assert np.array_equal(C, orc.gemm_i16i32(A, B))


@pytest.mark.parametrize("b,M,N,K", SHAPES)
def test_s24(b, M, N, K):
    rng = np.random.default_rng(M + N + K)
    A = ints(rng, (b, M, K), -(1 << 31), (1 << 31) - 1, np.int32)
    B = ints(rng, (b, K, N), -(1 << 31), (1 << 31) - 1, np.int32)
    C = run(qx.Executor.gemm_i32_s24(M, N, K, b, "s24_i8limb"), A, B)
    assert np.array_equal(C, orc.gemm_i32_s24(A, B))


@pytest.mark.parametrize("M,N,K,bound", [(50, 70, 449, 256), (50, 70, 1500, 256), (700, 801, 500, 1024)])
def test_no_alloc_call(M, N, K, bound):
    rng = np.random.default_rng(K)
    A, B = ints(rng, (M, K), -bound, bound - 1, np.int16), ints(rng, (K, N), -bound, bound - 1, np.int16)
    a, b = torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda()
    C = torch.full((M, N), 7, dtype=torch.int32, device="cuda")
    qx.check(qx.lib().qgemm_i16i32_noalloc(a.data_ptr(), b.data_ptr(), C.data_ptr(), M, N, K, 1, bound, bound,
                                           torch.cuda.current_stream().cuda_stream))
    torch.cuda.synchronize()
    assert np.array_equal(C.cpu().numpy(), orc.gemm_i16i32(A, B))


def test_conv_small_output():
    rng = np.random.default_rng(3)
    x, w = ints(rng, (1, 33, 7, 9), -127, 127, np.int16), ints(rng, (40, 33, 5, 5), -127, 127, np.int16)
    y = qx.conv2d_gemm(torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda(), 1, 2, 127, 127)
    torch.cuda.synchronize()
    ref = torch.nn.functional.conv2d(torch.from_numpy(x).double(), torch.from_numpy(w).double(), padding=2)
    assert np.array_equal(y.cpu().numpy(), ref.numpy().astype(np.int64).astype(np.int32))


def test_empty_output_of_a_long_sum():
    # no tile to slice: the planner must not divide by their number
    assert qx.plan_conv2d(0, 64, 9, 9, 16, 3, 3, 1, 1, 127, 127)["kernels"] == 0
    assert qx.plan_conv2d_t("i32", 0, 64, 9, 9, 16, 3, 3, 1, 1)["kernels"] == 0
    for M, N in ((0, 5), (5, 0)):
        assert qx.plan_gemm_i16i32(M, N, 4096, 1, 127, 127)["kernels"] == 0
        assert qx.plan_gemm_i32_s24(M, N, 4096)["kernels"] == 0


@pytest.mark.parametrize("N,Ci,H,W,Co,k,stride", [(2, 16, 9, 11, 16, 3, 1), (1, 48, 6, 5, 3, 1, 1), (1, 49, 6, 5, 3, 1, 2),
                                                  (3, 60, 7, 7, 15, 4, 1)])
def test_conv_i32_few_channels(N, Ci, H, W, Co, k, stride):
    # long sums over few pixels go through the limbs, short ones stay direct
    rng = np.random.default_rng(Ci)
    x = ints(rng, (N, Ci, H, W), -(1 << 23), (1 << 23) - 1, np.int32)
    w = ints(rng, (Co, Ci, k, k), -(1 << 23), (1 << 23) - 1, np.int32)
    auto = qx.conv2d_gemm_t(torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda(), stride, k // 2)
    with qx.Executor.conv2d_t("i32", N, Ci, H, W, Co, k, k, stride, k // 2, "s24_valu") as ex:
        direct = ex.run([torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda()])
        torch.cuda.synchronize()
    assert torch.equal(auto, direct)
    assert np.array_equal(auto.cpu().numpy(), orc.conv2d_s24(x, w, stride, k // 2))


@pytest.mark.parametrize("batch,M,N,K", [(1, 33, 33, 250001), (1, 64, 4161, 1025), (8, 61, 64, 8193), (1, 250, 256, 4300)])
def test_flushing_bounds_sliced(batch, M, N, K):
    assert qx.plan_gemm_i16i32(M, N, K, batch, 1024, 1024)["route_name"] == "f16_exact"
    rng = np.random.default_rng(K)
    A, B = ints(rng, (batch, M, K), -1024, 1024, np.int16), ints(rng, (batch, K, N), -1024, 1024, np.int16)
    C = run(qx.Executor.gemm_i16i32(M, N, K, batch, 1024, 1024), A, B)
    assert np.array_equal(C, orc.gemm_i16i32(A, B))


@pytest.mark.parametrize("M,N,K", [(1024, 1024, 257), (700, 801, 500)])
def test_flushing_bounds_large(M, N, K):
    # bounds whose chunk is under one K tile: three int8 products when large
    assert qx.plan_gemm_i16i32(M, N, K, 1, 1024, 1024)["route_name"] == "i8_karatsuba"
    rng = np.random.default_rng(K)
    A, B = ints(rng, (1, M, K), -1024, 1024, np.int16), ints(rng, (1, K, N), -1024, 1024, np.int16)
    C = run(qx.Executor.gemm_i16i32(M, N, K, 1, 1024, 1024), A, B)
    assert np.array_equal(C, orc.gemm_i16i32(A, B))
