"""Shapes at the edges of the launch rules: short rows of the row scan, attention launches that leave
compute units to spare."""
import numpy as np
import pytest

from synth import workloads as W
from oracle import draft_entropy_topk, pipeline as P

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def G():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import gpu_util
    return gpu_util


@pytest.mark.parametrize("V", [65, 500, 640, 641, 1024, 4096, 8192, 8193, 12000])
@pytest.mark.parametrize("R,K", [(17, 10), (40, 3), (20, 64)])
def test_short_rows(G, R, V, K):
    """Rows that leave waves, or 16-lane groups, of the first tile without a value: the threshold must
    come from groups that hold one.  Tied and masked rows among them."""
    rs = np.random.RandomState(R + V)
    x = (rs.randn(R, V) * np.exp(rs.uniform(np.log(0.3), np.log(8.0), size=(R, 1)))).astype(np.float32)
    x[1] = 1.5
    x[2, 3:] = -np.inf
    x[3] = np.round(x[3])
    want = draft_entropy_topk(x, K, 1.0)
    got = G.run_entropy(x, K, 1.0)
    assert np.array_equal(got["topk_idx"], want["topk_idx"])
    for k in ("ent_topk", "ent_full"):
        assert G.entropy_err(got[k], want[k]) <= 1.0, k
