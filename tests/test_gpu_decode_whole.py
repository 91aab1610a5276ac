"""Paged decode where the slicing and the product's instruction change: contexts left whole beside cut ones, every head ratio (one or two
groups of four heads, or sixteen columns), lists around 64 and 128 requests.  Both entry points, which must agree bit for bit; bounds of
every decode test."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from paper_2605_06472_amd import binding, workloads as W          # noqa: E402
from tests.gpu_util import DeviceBatch, assert_close, to_numpy     # noqa: E402

CALLS = {
    "short": lambda B: [1 + (7 * r) % 80 for r in range(B)],               # five pages at most: whole in any call
    "six_pages": lambda B: [81 + r % 16 for r in range(B)],                # one more
    "whole": lambda B: [500 + (13 * r) % 400 for r in range(B)],
    "skewed": lambda B: [17 + (r * r * 37) % (2000 if B < 100 else 1000) for r in range(B)],   # (inside the static limits)
}


@pytest.mark.parametrize("hq,hkv,d", [(2, 2, 128), (4, 2, 64), (8, 2, 128), (16, 2, 64), (16, 2, 128), (16, 1, 64), (32, 2, 128)])
@pytest.mark.parametrize("batch,call", [(1, "six_pages"), (1, "whole"), (7, "skewed"), (30, "whole"), (64, "short"), (65, "six_pages"), (128, "short"),
                                        (129, "skewed")])
def test_whole_and_cut_contexts(oracle, batch, call, hq, hkv, d):
    lens = CALLS[call](batch)
    print("whole", batch, call, hq, hkv, d, flush=True)
    b = W.ragged_small(900 + batch, "bf16", Hq=hq, Hkv=hkv, d=d, prefix_lens=tuple(n - 1 for n in lens), new_lens=(1,) * batch,
                       num_pages=sum((n + 15) // 16 for n in lens) + 8)
    db = DeviceBatch(b)
    ctx = np.asarray(lens, np.int32)
    want = oracle.decode(b.q, b.kv_pool, b.block_table, ctx)
    outs = []
    for entry in (binding.paged_decode, binding.paged_decode_static, binding.paged_decode):
        out = torch.full_like(db.q, 7.0)
        entry(db.shape, db.q, db.kv_pool, db.block_table, ctx, out)
        outs.append(out)
    torch.cuda.synchronize()
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])
    assert_close(W.to_f64(to_numpy(outs[0])), want, "bf16", "%s of %d" % (call, batch))
