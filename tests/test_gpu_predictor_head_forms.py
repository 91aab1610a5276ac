"""The predictor's head kernel where its two forms meet (four requests per work-group up to a batch of 1024, eight above)
and at the remainders of its layers.  Tolerance as derived in test_gpu_predictor.py."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from paper_2605_06472_amd import workloads as W                       # noqa: E402
from tests.test_gpu_predictor import DevicePredictor, _check          # noqa: E402


@pytest.mark.parametrize("V,d,d_x,hidden,K,L,B", [
    (8, 64, 512, 64, 3, 16, 1023),        # four per work-group, the last one short
    (8, 64, 512, 64, 3, 16, 1025),        # eight per work-group, one request in the last
    (32, 128, 272, 255, 4, 33, 1029),     # 132 outputs: three chunks of 64 in two parts; 255 hidden units: the last group of four is padded
    (32, 128, 272, 255, 4, 33, 9),        # the same with four per work-group
    (64, 128, 256, 256, 8, 64, 1100),     # the largest tables, which take more than one load per thread and 64 KiB of LDS; 520 outputs: a ninth chunk for eight waves
    (1, 32, 64, 1, 1, 1, 1030),           # one agent, one hidden unit, one prefix slot
])
def test_forms_match_reference(V, d, d_x, hidden, K, L, B):
    m = W.predictor_model(500 + V, V=V, d=d, d_x=d_x, hidden=hidden, K=K)
    b = W.predictor_batch(m, seed=600 + B, B=B, L=L)
    got = DevicePredictor(m, L, max_batch=B).forward(b)
    _check(m, b, got, "V=%d d=%d hidden=%d K=%d L=%d B=%d" % (V, d, hidden, K, L, B))
