"""LeNet pipeline: group edges of the pooled convolutions (images per workgroup
1, 2, 4, 8 and a short last group) and the extremes of the 24-bit operands,
whose weight limbs carry into a fourth one.  Bit-exact against the oracle."""
import numpy as np
import pytest

from oracle import oracle as orc
from paper_2606_09905_amd import qx

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
SHAPES = ((6, 1, 5, 5), (16, 6, 5, 5), (400, 120), (120, 84), (84, 10))


@pytest.mark.parametrize("B", [2, 255, 513, 1027, 2049])
@pytest.mark.parametrize("kind", ["full", "top", "bottom"])
def test_lenet_edges(B, kind):
    rng = np.random.default_rng(B)
    lo, hi = {"full": (-(1 << 31), (1 << 31) - 1), "top": ((1 << 23) - 200, (1 << 23) - 1),
              "bottom": (-(1 << 23), -(1 << 23) + 200)}[kind]
    x = rng.integers(lo, hi, (B, 1, 32, 32), dtype=np.int32, endpoint=True)
    ws = [rng.integers(lo, hi, s, dtype=np.int32, endpoint=True) for s in SHAPES]
    with qx.Executor.lenet_i32(B) as ex:
        y = ex.run([torch.from_numpy(a).cuda() for a in (x, *ws)])
        torch.cuda.synchronize()
    assert np.array_equal(y.cpu().numpy(), orc.lenet_i32(x, *ws))
