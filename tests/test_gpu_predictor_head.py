"""The predictor's head at the edges of its layers: outputs are taken 64 at a time, inputs in groups of four and in parts per wave,
requests four or eight to a work-group, softmax rows 16 lanes wide, prefixes within or beyond one row of 16 lanes.  Against the
fp64 reference; the tolerance and its derivation are those of test_gpu_predictor.py."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from paper_2605_06472_amd import workloads as W                                    # noqa: E402
from tests.test_gpu_predictor import DevicePredictor, _check                       # noqa: E402


@pytest.mark.parametrize("B", [5, 1025])                   # four requests per work-group with a ragged last one, eight likewise
@pytest.mark.parametrize("V,d,hidden,K,L", [
    (1, 32, 1, 1, 1),            # one of everything: a hidden layer of a quarter group, two outputs
    (2, 32, 63, 8, 16),          # padding of W_b's last group reaches past its own place in the workspace
    (15, 64, 64, 4, 17),         # 64 outputs exactly, a softmax row of 16, a prefix past one row of lanes
    (16, 64, 65, 3, 33),         # one past each
    (32, 128, 129, 2, 64),       # three chunks of hidden units: two parts, two waves without an item
    (64, 128, 255, 8, 5),        # 520 outputs: more chunks than waves
    (63, 64, 193, 8, 15),        # 512 outputs: as many
])
def test_layer_edges(V, d, hidden, K, L, B):
    print("head", V, d, hidden, K, L, B, flush=True)
    m = W.predictor_model(700 + V, V=V, d=d, d_x=128, hidden=hidden, K=K)
    b = W.predictor_batch(m, seed=800 + hidden, B=B, L=L)
    b.prefix_len[0] = 0
    b.prefix_len[-1] = L                                   # (the drawn prefix may be shorter)
    b.prefix[-1] = [(3 * i) % V for i in range(L)]
    _check(m, b, DevicePredictor(m, L, max_batch=B).forward(b), "V=%d d=%d hidden=%d K=%d L=%d B=%d" % (V, d, hidden, K, L, B))
