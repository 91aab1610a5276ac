"""The fp32 attention's distance from fp64 on short contexts, where the dot products' rounding is most of it: no further than
a plain evaluation in fp32 with four interleaved chains per dot product (as the kernel that came before this one had)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from paper_2605_06472_amd import workloads as W          # noqa: E402
from tests.gpu_util import DeviceBatch                    # noqa: E402


def _plain(b):
    """softmax(q k / sqrt(d)) v with every product-sum rounded to fp32 (fma), keys in order."""
    f, d64 = np.float32, np.float64
    c = f(f(1.4426950408889634) * (f(1) / np.sqrt(f(b.d))))
    out, off = np.zeros(b.q.shape, f), 0
    for r in range(b.B):
        p, n = int(b.prefix_lens[r]), int(b.new_lens[r])
        pages = b.kv_pool[b.block_table[r, :-(-p // b.P)]]
        K, V = (np.concatenate([pages[:, i].transpose(0, 2, 1, 3).reshape(-1, b.Hkv, b.d)[:p], new[off:off + n]])
                for i, new in ((0, b.k_new), (1, b.v_new)))
        for h in range(b.Hq):
            k, v, q = K[:, h * b.Hkv // b.Hq], V[:, h * b.Hkv // b.Hq], b.q[off:off + n, h]
            acc = np.zeros((4, n, p + n), f)
            for i in range(b.d):
                acc[i % 4] = (acc[i % 4].astype(d64) + np.outer(q[:, i].astype(d64), k[:, i])).astype(f)
            s = (acc[0] + acc[1]) + (acc[2] + acc[3])
            s[np.arange(p + n)[None] > p + np.arange(n)[:, None]] = -np.inf
            w = np.exp2((s - s.max(1, keepdims=True)) * c)
            den, o = np.zeros(n, f), np.zeros((n, b.d), f)
            for t in range(p + n):
                den = den + w[:, t]
                o = (o.astype(d64) + np.outer(w[:, t].astype(d64), v[t])).astype(f)
            out[off:off + n, h] = o * (f(1) / den)[:, None]
        off += n
    return out


@pytest.mark.parametrize("kw", [dict(Hq=8, Hkv=2, d=128, prefix_lens=(16,) * 4, new_lens=(8, 6, 5, 4)),
                                dict(Hq=6, Hkv=2, d=128, prefix_lens=(30, 20, 10), new_lens=(7, 5, 3)),
                                dict(Hq=4, Hkv=2, d=64, prefix_lens=(29, 12), new_lens=(6, 3))], ids=["d128_g4", "d128_g3", "d64_g2"])
def test_short_contexts_are_no_further_from_fp64_than_a_plain_evaluation(oracle, kw):
    """Root mean square over three batches of some thousand outputs each.  Measured: 0.92 to 0.95 of the plain error with four
    chains per score, 1.05 to 1.3 with two."""
    mine = plain = 0.0
    for seed in (1, 2, 3):
        b = W.ragged_small(seed, "f32", num_pages=96, sigma=1.0, **kw)
        want = oracle.prefill(b.q, b.k_new, b.v_new, b.kv_pool, b.block_table, b.prefix_lens, b.new_lens)
        db = DeviceBatch(b)
        db.prefill()
        torch.cuda.synchronize()
        mine += (np.linalg.norm(db.out_f64() - want) / np.linalg.norm(want)) ** 2
        plain += (np.linalg.norm(_plain(b) - want) / np.linalg.norm(want)) ** 2
    print("error %.3e, plain %.3e" % ((mine / 3) ** 0.5, (plain / 3) ** 0.5))
    assert mine ** 0.5 <= 1.02 * plain ** 0.5
