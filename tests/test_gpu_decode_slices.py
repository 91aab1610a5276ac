"""Paged decode: batches on both sides of what fits a kernel argument and of a search round over requests, contexts that
end on and beside slice edges, requests without context among them; both entry points, which must agree bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from paper_2605_06472_amd import binding, workloads as W          # noqa: E402
from tests.gpu_util import DeviceBatch, assert_close, to_numpy     # noqa: E402

EDGES = (0, 1, 16, 63, 64, 65, 128, 129, 255, 256, 257, 0, 1024, 1025, 2049)


@pytest.mark.parametrize("batch,hq,hkv,d", [(1, 32, 8, 128), (3, 16, 1, 64), (64, 8, 2, 64), (65, 4, 4, 128), (128, 32, 2, 128),
                                            (129, 16, 2, 128), (300, 8, 8, 64)])
def test_decode_batches_and_slice_edges(oracle, batch, hq, hkv, d):
    lens = [EDGES[(3 * r + batch) % len(EDGES)] for r in range(batch)]
    lens[batch // 2] = 4100
    pages = sum((n + 1 + 15) // 16 for n in lens) + 8
    b = W.ragged_small(500 + batch, "bf16", Hq=hq, Hkv=hkv, d=d, prefix_lens=tuple(lens), new_lens=(1,) * batch, num_pages=pages)
    db = DeviceBatch(b)
    want = oracle.decode(b.q, b.kv_pool, b.block_table, b.prefix_lens)
    outs = []
    for entry in (binding.paged_decode, binding.paged_decode_static, binding.paged_decode):
        out = torch.full_like(db.q, 7.0)
        entry(db.shape, db.q, db.kv_pool, db.block_table, np.asarray(lens, np.int32), out)
        outs.append(out)
    torch.cuda.synchronize()
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])
    assert_close(W.to_f64(to_numpy(outs[0])), want, "bf16", "decode of %d" % batch)


@pytest.mark.parametrize("hq,hkv,d,tokens", [(16, 1, 128, 512), (16, 1, 128, 513), (16, 2, 64, 1024), (16, 2, 64, 1025),
                                             (4, 1, 128, 2048), (4, 1, 128, 2049), (2, 2, 64, 8192), (1, 1, 64, 16384), (1, 1, 64, 16385)])
def test_merges_on_both_sides_of_what_one_work_group_holds(oracle, hq, hkv, d, tokens):
    """Slices of 64 tokens: the first of each pair has 64 KiB of output partials per KV head, the second one slice more;
    one short request beside it.  Same bound as every decode test."""
    lens = (tokens - 1, 100)
    b = W.ragged_small(700 + tokens, "bf16", Hq=hq, Hkv=hkv, d=d, prefix_lens=lens, new_lens=(1, 1), num_pages=tokens // 16 + 24)
    db = DeviceBatch(b)
    ctx = np.array([tokens, 100], np.int32)
    want = oracle.decode(b.q, b.kv_pool, b.block_table, ctx)
    outs = []
    for entry in (binding.paged_decode, binding.paged_decode_static, binding.paged_decode):
        out = torch.full_like(db.q, 7.0)
        entry(db.shape, db.q, db.kv_pool, db.block_table, ctx, out)
        outs.append(out)
    torch.cuda.synchronize()
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])
    assert_close(W.to_f64(to_numpy(outs[0])), want, "bf16", "decode of %d tokens" % tokens)


def test_a_merge_whose_weights_do_not_fit_at_once(oracle):
    """256 slices of 16 heads: the merging work-groups hold the weights of 128 slices at a time."""
    tokens = 32768
    b = W.ragged_small(720, "bf16", Hq=32, Hkv=2, d=128, prefix_lens=(tokens - 1,), new_lens=(1,), num_pages=tokens // 16 + 8)
    db = DeviceBatch(b)
    ctx = np.array([tokens], np.int32)
    want = oracle.decode(b.q, b.kv_pool, b.block_table, ctx)
    outs = []
    for entry in (binding.paged_decode, binding.paged_decode_static):
        out = torch.full_like(db.q, 7.0)
        entry(db.shape, db.q, db.kv_pool, db.block_table, ctx, out)
        outs.append(out)
    torch.cuda.synchronize()
    assert torch.equal(outs[0], outs[1])
    assert_close(W.to_f64(to_numpy(outs[0])), want, "bf16", "decode of %d tokens" % tokens)
