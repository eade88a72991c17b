"""FP32 kernels on the bf16 matrix cores: every float as three bf16 terms.

The elementwise bound is the a-priori one of fp32 sums in any order, u = 2^-24
per term; the dropped product (l l, at most 2^-34 of the whole) lies inside it,
and a sum of one product rounds as an fp32 multiplication does.  The split of a
scaled value is exact down to the last subnormal bit of a float, so small values
take no other path than ordinary ones; where a sum is not finite (infinities,
NaN, overflow of the scaled sums) the fp32 matrix cores give it again.
"""
import numpy as np
import pytest

from oracle import oracle as orc
from paper_2606_09905_amd import qx

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
U = 2.0 ** -24


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    assert qx.lib() is not None


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def host(t):
    torch.cuda.synchronize()
    return t.cpu().numpy()


def core_bound(Q, K, V):
    d, L = Q.shape[1], Q.shape[0]
    return (d + L + 4) * U * ((np.abs(Q).astype(np.float64) @ np.abs(K).astype(np.float64).T) @ np.abs(V))


# both workgroup sizes (128 and 256 queries), one and several key splits, one
# key block, a last block of one key and of 31
@pytest.mark.parametrize("L,d", [(1, 64), (33, 32), (63, 128), (129, 96), (160, 64), (4095, 64), (4128, 64),
                                 (8193, 32), (2817, 96), (2080, 128)])
def test_core(L, d):
    rng = np.random.default_rng(L + d)
    Q, K, V = ((rng.standard_normal((L, d)) * d ** -0.5).astype(np.float32) for _ in range(3))
    O = host(qx.attn_core(dev(Q), dev(K), dev(V)))
    assert (np.abs(O - orc.attn_f64(Q, K, V)) <= core_bound(Q, K, V)).all()


@pytest.mark.parametrize("L", [96, 4352])
# exact at every size a float can have: subnormal operands, terms and products,
# and sums that the scales take to 2^96 and beyond
@pytest.mark.parametrize("scales", [(2.0 ** 40, 2.0 ** -40, 1.0), (1.0, 1.0, 1e-36), (2.0 ** -70, 2.0 ** 60, 1e10),
                                    (2.0 ** -39,) * 3, (2.0 ** 28,) * 3, (1e-13, 1e-13, 1.0), (2.0 ** -60, 2.0 ** -60, 1.0),
                                    (1e-41, 1e20, 1e20), (2.0 ** -72, 2.0 ** -72, 2.0 ** 90), (1e18, 1e-40, 1e18),
                                    (2.0 ** 31, 2.0 ** 31, 2.0 ** 31), (2.0 ** 45, 2.0 ** 45, 1e-30)])
def test_core_ranges(L, scales):
    rng = np.random.default_rng(L)
    Q, K, V = ((rng.standard_normal((L, 64)) * s).astype(np.float32) for s in scales)
    O = host(qx.attn_core(dev(Q), dev(K), dev(V)))
    # results below the smallest normal number lose up to its half ulp per term,
    # and so do scores, each of which is multiplied by a value
    floor = L * 2.0 ** -149 + 64 * 2.0 ** -149 * np.abs(V).astype(np.float64).sum(axis=0)
    assert (np.abs(O - orc.attn_f64(Q, K, V)) <= core_bound(Q, K, V) + floor).all()


@pytest.mark.parametrize("L", [70, 4352])
@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan])
def test_core_not_finite(L, value):
    rng = np.random.default_rng(L)
    Q, K, V = ((rng.standard_normal((L, 64)) * 0.125).astype(np.float32) for _ in range(3))
    V[L - 2, 5] = value
    Q[7, 3] = value
    O = host(qx.attn_core(dev(Q), dev(K), dev(V)))
    with np.errstate(invalid="ignore"):
        R = (Q.astype(np.float64) @ K.astype(np.float64).T) @ V.astype(np.float64)
    ok = np.ones_like(O, dtype=bool)
    ok[7], ok[:, 5] = False, False          # row 7 sums infinities of both signs: NaN
    assert np.isnan(O[7]).all()
    rows = np.arange(L) != 7
    assert np.array_equal(np.isnan(O[rows, 5]), np.isnan(R[rows, 5]))
    if not np.isnan(value):
        assert np.array_equal(O[rows, 5], R[rows, 5])
    Q[7, 3], V[L - 2, 5] = 0.0, 0.0
    bound = core_bound(Q, K, V)
    assert (np.abs(O[ok] - R[ok]) <= bound[ok]).all()


# One non-zero product a sum.  Every step is exact but the smaller terms' sum
# (2^-7 of the product at most, rounded to 2^-24 of itself) and the last
# addition (half an ulp).  0x1.00ff8p0 = 1 + 2^-8 - 2^-17 has the largest
# second and third terms.
HALF_ULP = 0.5 + 2.0 ** -6


def ulps(y, r):
    return np.abs(y - r) / 2.0 ** (np.floor(np.log2(np.abs(r))) - 23)


@pytest.mark.parametrize("k,Ci,Co", [(3, 64, 128), (1, 32, 33)])
def test_conv_one_product(k, Ci, Co):
    rng = np.random.default_rng(Ci)
    x = rng.standard_normal((4, Ci, 28, 28)).astype(np.float32)
    w = np.zeros((Co, Ci, k, k), np.float32)
    w[np.arange(Co), np.arange(Co) % Ci, k // 2, k // 2] = rng.standard_normal(Co)
    w[0, 0, k // 2, k // 2] = x[0, 0, 0, 0] = float.fromhex("0x1.00ff8p0")
    y = host(qx.conv2d_gemm_t(dev(x), dev(w), 1, k // 2))
    r = conv_ref(x, w, 1, k // 2)
    assert (r != 0).all() and ulps(y, r).max() <= HALF_ULP


@pytest.mark.parametrize("d", [32, 64, 96, 128])
def test_core_one_product(d):
    # one key, one coordinate: (q k) v, each product to half an ulp
    rng = np.random.default_rng(d)
    for i in range(8):
        Q, K, V = np.zeros((1, d), np.float32), np.zeros((1, d), np.float32), rng.standard_normal((1, d)).astype(np.float32)
        Q[0, i], K[0, i] = rng.standard_normal(2) if i else [float.fromhex("0x1.00ff8p0")] * 2
        O = host(qx.attn_core(dev(Q), dev(K), dev(V)))
        S = np.float32(Q[0, i]) * np.float64(K[0, i])
        # S to half an ulp, then S's float times V to half an ulp
        s = np.array([np.float32(S), np.nextafter(np.float32(S), np.float32(np.inf)),
                      np.nextafter(np.float32(S), np.float32(-np.inf))], np.float32)
        s = s[ulps(s.astype(np.float64), S) <= HALF_ULP]
        err = np.stack([ulps(O, np.float64(t) * V) for t in s]).max(axis=(1, 2))
        assert err.min() <= HALF_ULP


def test_conv_constant_operands():
    # the dropped terms of equal operands share one sign
    c = np.float32(float.fromhex("0x1.00ff8p0"))
    x, w = np.full((1, 32, 9, 9), c), np.full((64, 32, 1, 1), c)
    y = host(qx.conv2d_gemm_t(dev(x), dev(w)))
    assert ulps(y, conv_ref(x, w, 1, 0)).max() <= HALF_ULP


def sdpa_ref(Q, K, V, scale, causal):
    return orc.sdpa_f64(Q, K, V, scale, causal)


# the merged maximum of a row whose first key splits are masked, one wave and
# eight, blocks past a wave's last query, ragged d on both workgroup sizes
@pytest.mark.parametrize("BH,L,d,causal", [(1, 32, 64, True), (3, 97, 33, True), (1, 1025, 64, True),
                                           (40, 257, 64, True), (9, 512, 80, True), (5, 1290, 31, False),
                                           (4, 1281, 128, True), (2, 1100, 96, False)])
def test_softmax(BH, L, d, causal):
    rng = np.random.default_rng(BH + L + d)
    Q, K, V = (rng.standard_normal((BH, L, d)).astype(np.float32) for _ in range(3))
    O = host(qx.sdpa_f32(dev(Q), dev(K), dev(V), d ** -0.5, causal))
    R = sdpa_ref(Q, K, V, d ** -0.5, causal)
    # a score's error, (d + 4) u |q||k| scale, is the relative error of its exponential
    s = (d + 4) * U * d ** -0.5 * np.abs(Q).max() * np.abs(K).max() * d + 8 * U
    assert np.abs(O - R).max() <= (2 * s + L * U) * np.abs(V).max()
    assert np.linalg.norm(O - R) <= 4e-6 * np.linalg.norm(R)


@pytest.mark.parametrize("L", [64, 2000])
def test_softmax_small_probabilities(L):
    # Probabilities of 2^-115 beside a maximum whose value is 0.  scale ln 2
    # makes the base-2 scores the keys' numbers, which are eighths: exact, so a
    # probability is off by its exponential's error alone (about an ulp).
    rng = np.random.default_rng(L)
    Q, K, V = np.zeros((1, L, 32), np.float32), np.zeros((1, L, 32), np.float32), rng.standard_normal((1, L, 32))
    V = (V * 1e30).astype(np.float32)
    Q[..., 0] = 1.0
    K[0, 1:, 0] = -112 - rng.integers(0, 96, L - 1) / 8
    V[0, 0] = 0.0
    scale = float(np.float32(np.log(2.0)))
    assert np.float32(scale * 1.4426950408889634) == 1.0
    O = host(qx.sdpa_f32(dev(Q), dev(K), dev(V), scale, False))
    P = 2.0 ** K[0, :, 0].astype(np.float64)
    R, A = P @ V[0].astype(np.float64), P @ np.abs(V[0]).astype(np.float64)
    assert (np.abs(O[0] - R) <= (8 + L / 32 + 8) * U * A).all()


@pytest.mark.parametrize("BH,L", [(2, 100), (20, 512)])
def test_softmax_ranges(BH, L):
    d = 64
    rng = np.random.default_rng(L)
    Q, K, V = (rng.standard_normal((BH, L, d)).astype(np.float32) for _ in range(3))
    V0 = V.copy()
    V[0] *= 1e-37
    V[1] *= 1e30                        # some sums overflow at the split's scale
    K[1, 3, 5] = 1e-33
    K[0, L - 1, 0] = np.inf             # an infinite score of either sign
    O = host(qx.sdpa_f32(dev(Q), dev(K), dev(V), 0.125, True))
    K[1, 3, 5] = 0.0
    last = Q[0, L - 1, 0]
    K[0, L - 1, 0] = 0.0
    R = sdpa_ref(Q, K, V0, 0.125, True)
    assert np.linalg.norm(O[0, :L - 1] / np.float64(1e-37) - R[0, :L - 1]) <= 2e-5 * np.linalg.norm(R[0, :L - 1])
    assert np.linalg.norm(O[1] / np.float64(1e30) - R[1]) <= 4e-6 * np.linalg.norm(R[1])
    if BH > 2:
        assert np.linalg.norm(O[2:] - R[2:]) <= 4e-6 * np.linalg.norm(R[2:])
    if last > 0:
        assert np.isnan(O[0, L - 1]).all()      # exp(inf - inf)


# N, C_in, H, W, C_out, K, stride, pad: one tile and many, C_out and pixels off
# the tiles' edges, K splits with a short last one and outputs not a multiple
# of 4, stride 2, tap ranges that start inside a tap's channels
CONV = [(1, 32, 1, 1, 1, 1, 1, 0), (1, 64, 7, 9, 33, 3, 1, 1), (3, 96, 5, 7, 65, 3, 2, 1), (1, 256, 7, 7, 130, 3, 1, 1),
        (2, 160, 13, 11, 63, 5, 1, 2), (7, 32, 56, 57, 128, 3, 1, 1), (1, 224, 3, 3, 5, 3, 1, 0)]


def conv_ref(x, w, stride, pad):
    t = [torch.from_numpy(a.astype(np.float64)) for a in (x, w)]
    return torch.nn.functional.conv2d(*t, stride=stride, padding=pad).numpy()


@pytest.mark.parametrize("case", CONV)
def test_conv(case):
    N, Ci, H, W, Co, k, stride, pad = case
    rng = np.random.default_rng(sum(case))
    x = rng.standard_normal((N, Ci, H, W)).astype(np.float32)
    w = rng.standard_normal((Co, Ci, k, k)).astype(np.float32)
    y = host(qx.conv2d_gemm_t(dev(x), dev(w), stride, pad))
    bound = (Ci * k * k + 4) * U * conv_ref(np.abs(x), np.abs(w), stride, pad)
    assert (np.abs(y - conv_ref(x, w, stride, pad)) <= bound).all()
    assert np.array_equal(y, host(qx.conv2d_gemm_t(dev(x), dev(w), stride, pad)))


@pytest.mark.parametrize("case", [CONV[2], CONV[3], CONV[6]])
@pytest.mark.parametrize("scales", [(2.0 ** -61, 2.0 ** -61), (2.0 ** -99, 2.0 ** -20), (2.0 ** 40, 2.0 ** 40),
                                    (2.0 ** 57, 2.0 ** 57), (1e-41, 1e10), (1e25, 1e-44), (2.0 ** -75, 2.0 ** -75)])
def test_conv_ranges(case, scales):
    N, Ci, H, W, Co, k, stride, pad = case
    rng = np.random.default_rng(sum(case))
    x = (rng.standard_normal((N, Ci, H, W)) * scales[0]).astype(np.float32)
    w = (rng.standard_normal((Co, Ci, k, k)) * scales[1]).astype(np.float32)
    y = host(qx.conv2d_gemm_t(dev(x), dev(w), stride, pad))
    R, A = conv_ref(x, w, stride, pad), conv_ref(np.abs(x), np.abs(w), stride, pad)
    assert (np.abs(y.astype(np.float64) - R) <= Ci * k * k * (U * A + 2.0 ** -149) + 4 * U * A).all()


def best_time(ex, inputs):
    out = torch.empty(ex.out_shape, dtype=ex.out_dtype, device="cuda")
    times = []
    for _ in range(6):
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        a.record()
        for _ in range(10):
            ex.run(inputs, out)
        b.record()
        torch.cuda.synchronize()
        times.append(a.elapsed_time(b))
    return min(times)


def test_small_values_take_the_same_path():
    # a call that goes to the fp32 matrix cores' path takes 2.5 to 4.5 times as long
    g = torch.Generator(device="cuda").manual_seed(5)
    Q, K, V = (torch.randn((16, 2048, 64), generator=g, device="cuda") for _ in range(3))
    with qx.Executor.sdpa_f32(16, 2048, 64, 0.125, True) as ex:
        t = best_time(ex, [Q, K, V])
        K2, V2 = K.clone(), V.clone()
        K2[:, 5, 3], V2[:, 7, 1] = 1e-33, 1e-40
        assert best_time(ex, [Q, K2, V2]) < 2 * t
    with qx.Executor.attn("f32", 4096, 64, 0) as ex:
        q, k, v = (t.reshape(-1, 64)[:4096].contiguous() for t in (Q, K, V))
        assert best_time(ex, [q * 1e-13, k * 1e-13, v * 1e-13]) < 2 * best_time(ex, [q, k, v])
    x, w = torch.randn((8, 64, 56, 56), generator=g, device="cuda"), torch.randn((128, 64, 3, 3), generator=g, device="cuda")
    with qx.Executor.conv2d_t("f32", 8, 64, 56, 56, 128, 3, 3, 1, 1) as ex:
        t = best_time(ex, [x, w])
        w[5::64, 1, 0, 0] = 1e-40
        assert best_time(ex, [x, w]) < 2 * t


@pytest.mark.parametrize("case", [CONV[2], CONV[3], CONV[5]])
@pytest.mark.parametrize("value", [np.inf, np.nan, 3e-38, 1e25])
def test_conv_out_of_range(case, value):
    N, Ci, H, W, Co, k, stride, pad = case
    rng = np.random.default_rng(sum(case))
    x = rng.standard_normal((N, Ci, H, W)).astype(np.float32)
    w = rng.standard_normal((Co, Ci, k, k)).astype(np.float32)
    x[N - 1, 3, 2, 1] = value
    w[Co // 2, Ci - 1, k - 1, 0] = value
    y = host(qx.conv2d_gemm_t(dev(x), dev(w), stride, pad))
    with np.errstate(invalid="ignore"):
        R, A = conv_ref(x, w, stride, pad), conv_ref(np.abs(x), np.abs(w), stride, pad)
    fin = np.isfinite(R)
    assert np.array_equal(np.isfinite(y), fin)
    assert np.array_equal(np.isnan(y), np.isnan(R))
    assert (np.abs(y[fin].astype(np.float64) - R[fin]) <= (Ci * k * k + 4) * U * A[fin]).all()
