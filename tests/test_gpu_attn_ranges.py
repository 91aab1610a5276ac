"""Attention launches whose token blocks are dealt out to several work-groups by ranges of KV tiles (few
token blocks on long contexts): ranges, their partial results and the merge against the oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from paper_2605_06472_amd import binding, workloads as W                       # noqa: E402
from tests.gpu_util import PEAKED_ATOL, DeviceBatch, assert_close, sample_rows, to_numpy   # noqa: E402

CASES = {
    # one row and one more / fewer than a page, a KV tile, a 32-token block; nine tiles is the shortest context that is cut
    "one_row": dict(prefix_lens=(4097,), new_lens=(1,)),
    "tile_edges": dict(prefix_lens=(1023, 1024, 1025), new_lens=(31, 33, 1)),
    "shortest": dict(prefix_lens=(448,), new_lens=(65,)),
    "suffix_ranges": dict(prefix_lens=(3,), new_lens=(700,), Hq=8, Hkv=2),
    "empty_and_cold": dict(prefix_lens=(2500, 0, 900, 0), new_lens=(70, 0, 5, 300), Hq=8, Hkv=2),
    "peaked": dict(prefix_lens=(3301, 77), new_lens=(40, 130), q_scale=8.0),
    "g1": dict(prefix_lens=(2240, 130), new_lens=(200, 129), Hq=2, Hkv=2),
    "g2": dict(prefix_lens=(2240, 130), new_lens=(65, 129), Hq=4, Hkv=2),
    "g8_d64": dict(prefix_lens=(2240, 5), new_lens=(65, 130), Hq=16, Hkv=2, d=64),
    "g16_d64": dict(prefix_lens=(1500,), new_lens=(33,), Hq=16, Hkv=1, d=64),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_ranges_of_keys_match_the_oracle(oracle, name):
    kw = dict(dtype="bf16", Hq=32, Hkv=8, num_pages=480)
    kw.update(CASES[name])
    b = W.ragged_small(140, **kw)
    print("case", name, "B", b.B, "N", b.N, flush=True)
    db = DeviceBatch(b)
    db.prefill()
    torch.cuda.synchronize()
    first = db.out.clone()
    want = oracle.prefill(b.q, b.k_new, b.v_new, b.kv_pool, b.block_table, b.prefix_lens, b.new_lens)
    assert_close(db.out_f64(), want, "bf16", name, atol=PEAKED_ATOL if name == "peaked" else None)
    # from the cached work list, with other values left in the partial-result buffer in between
    other = DeviceBatch(W.ragged_small(141, "bf16", Hq=8, Hkv=2, prefix_lens=(2000,), new_lens=(50,), num_pages=160))
    other.prefill()
    db.out.zero_()
    db.prefill()
    torch.cuda.synchronize()
    assert torch.equal(db.out, first)
    # it is another order of summation than one work-group per token block, and no further from it than the tolerance
    binding.set_attn_waves(4)
    try:
        db.out.zero_()
        db.prefill()
        torch.cuda.synchronize()
    finally:
        binding.set_attn_waves(0)
    assert not torch.equal(db.out, first), "the launch was not cut into ranges"
    assert_close(W.to_f64(to_numpy(db.out)), W.to_f64(to_numpy(first)), "bf16", name + " against one range", atol=PEAKED_ATOL)


SHORT_CASES = {
    # ranges of one, two and three tiles: the partial prefix tile alone in one, suffix tiles alone, 16 and 17 tiles
    "five_tiles": dict(prefix_lens=(200,), new_lens=(64,)),
    "partial_tile": dict(prefix_lens=(301,), new_lens=(8,)),
    "cold": dict(prefix_lens=(0,), new_lens=(300,), Hq=8, Hkv=2),
    "sixteen_tiles": dict(prefix_lens=(960,), new_lens=(33,), Hq=8, Hkv=2),
    "seventeen_tiles": dict(prefix_lens=(1024,), new_lens=(33,), Hq=8, Hkv=2),
    "three_tiles": dict(prefix_lens=(2100, 40), new_lens=(20, 70), Hq=8, Hkv=2, d=64),
    "peaked": dict(prefix_lens=(333,), new_lens=(40,), q_scale=8.0),
    "g1_d64": dict(prefix_lens=(250,), new_lens=(130,), Hq=4, Hkv=4, d=64),
}


@pytest.mark.parametrize("name", sorted(SHORT_CASES))
def test_ranges_of_few_tiles_match_the_oracle(oracle, name):
    """The bounds of the test above: the same path with shorter ranges."""
    kw = dict(dtype="bf16", Hq=32, Hkv=8, num_pages=160)
    kw.update(SHORT_CASES[name])
    b = W.ragged_small(160, **kw)
    db = DeviceBatch(b)
    db.prefill()
    torch.cuda.synchronize()
    first = db.out.clone()
    want = oracle.prefill(b.q, b.k_new, b.v_new, b.kv_pool, b.block_table, b.prefix_lens, b.new_lens)
    assert_close(db.out_f64(), want, "bf16", name, atol=PEAKED_ATOL if name == "peaked" else None)
    db.out.zero_()
    db.prefill()                                      # from the cached work list
    torch.cuda.synchronize()
    assert torch.equal(db.out, first)
    binding.set_attn_waves(4)
    try:
        db.prefill()
        torch.cuda.synchronize()
    finally:
        binding.set_attn_waves(0)
    assert not torch.equal(db.out, first), "the launch was not cut into ranges"


F32_CASES = {
    # row blocks of 128 (token, head) rows, waves of 32, KV tiles of 32 keys: one row, exact blocks, one past, odd ratios
    "one_row": dict(Hq=2, Hkv=1, d=64, prefix_lens=(257,), new_lens=(1,)),
    "no_prefix": dict(Hq=4, Hkv=2, d=64, prefix_lens=(0, 0), new_lens=(64, 65)),
    "block_edges": dict(Hq=8, Hkv=2, d=128, prefix_lens=(31, 32, 33, 0), new_lens=(32, 33, 8, 0)),
    "ratio_3": dict(Hq=6, Hkv=2, d=128, prefix_lens=(500, 63), new_lens=(43, 11)),
    "ratio_5": dict(Hq=5, Hkv=1, d=64, prefix_lens=(95,), new_lens=(77,)),
    "ratio_1": dict(Hq=3, Hkv=3, d=64, prefix_lens=(640, 1), new_lens=(130, 129)),
    "fills_the_chip": dict(Hq=32, Hkv=8, d=64, prefix_lens=(100,), new_lens=(1100,)),
}


@pytest.mark.parametrize("name", sorted(F32_CASES))
def test_fp32_row_blocks_and_ranges(oracle, name):
    b = W.ragged_small(150, "f32", num_pages=96, sigma=1.0, **F32_CASES[name])
    print("case f32", name, "B", b.B, "N", b.N, flush=True)
    db = DeviceBatch(b)
    outs = []
    for k in range(2):                          # built, then from the cached work list
        db.out.fill_(7.0)
        db.prefill()
        torch.cuda.synchronize()
        outs.append(db.out.clone())
    assert torch.equal(outs[0], outs[1])
    want = oracle.prefill(b.q, b.k_new, b.v_new, b.kv_pool, b.block_table, b.prefix_lens, b.new_lens)
    assert_close(db.out_f64(), want, "f32", name)
    binding.set_attn_waves(4)                   # a forced shape of the bf16 kernel: fp32 launches stay whole, too
    try:
        db.prefill()
        torch.cuda.synchronize()
    finally:
        binding.set_attn_waves(0)
    assert torch.equal(db.out, outs[0]) == (name == "fills_the_chip"), "which launches are cut"
    assert_close(db.out_f64(), want, "f32", name + ", whole")


def test_long_blocks_that_leave_cus_idle_are_cut(oracle):
    """280 work-groups of 32 rows / 144 of 64 rows of about 145 tile steps: neither form fills its rounds."""
    b = W.long_history(seed=1017, batch=1, prefix=8200, new=1100, num_pages=640)
    db = DeviceBatch(b)
    db.prefill()
    torch.cuda.synchronize()
    rows = sample_rows(b, per_request=24, unit=32, max_boundaries=16)
    want = oracle.prefill(b.q, b.k_new, b.v_new, b.kv_pool, b.block_table, b.prefix_lens, b.new_lens, rows=rows)
    assert_close(db.out_f64()[rows], want, "bf16", "8200 + 1100")
    cut = db.out.clone()
    for waves in (4, 64):
        binding.set_attn_waves(waves)
        try:
            db.prefill()
            torch.cuda.synchronize()
        finally:
            binding.set_attn_waves(0)
        assert not torch.equal(db.out, cut), "the launch was not cut into ranges"


def test_cut_launches_on_two_streams_at_once(oracle):
    """Partial results are kept per stream: launches that are in flight together, of different lengths and both data types,
    each give the bits they give alone."""
    streams = [torch.cuda.Stream() for _ in range(2)]
    batches = [DeviceBatch(W.ragged_small(170 + k, dtype, num_pages=700, **kw)) for k, (dtype, kw) in enumerate((
        ("bf16", dict(Hq=32, Hkv=8, prefix_lens=(6000,), new_lens=(40,))), ("bf16", dict(Hq=8, Hkv=2, prefix_lens=(3000, 900), new_lens=(33, 70))),
        ("f32", dict(Hq=8, Hkv=2, d=128, sigma=1.0, prefix_lens=(2000,), new_lens=(50,))), ("bf16", dict(Hq=16, Hkv=2, d=64, prefix_lens=(4000,), new_lens=(65,)))))]
    alone = []
    for db in batches:
        db.prefill()
        torch.cuda.synchronize()
        alone.append(db.out.clone())
    outs = [[torch.full_like(db.out, 7.0) for db in batches] for _ in streams]
    torch.cuda.synchronize()
    for _ in range(10):
        for k in range(len(batches)):
            for s, stream in enumerate(streams):
                j = (k + 2 * s) % len(batches)
                batches[j].prefill(stream=stream, out=outs[s][j])
    torch.cuda.synchronize()
    for s in range(len(streams)):
        for j, want in enumerate(alone):
            assert torch.equal(outs[s][j], want), (s, j)


@pytest.mark.parametrize("dtype,heads", [("bf16", (32, 8, 128)), ("bf16", (16, 2, 64)), ("f32", (8, 2, 128))])
def test_a_request_alone_and_in_a_batch(oracle, dtype, heads):
    """The same bits while a work-group shape is forced, whatever else the call holds; rounding apart (twice the oracle's
    bound: either side is within it) where the library splits the one launch and not, or otherwise, the other."""
    b = W.ragged_small(144, dtype, Hq=heads[0], Hkv=heads[1], d=heads[2], prefix_lens=(1500, 40, 700, 0), new_lens=(40, 130, 1, 70), num_pages=320)
    db = DeviceBatch(b)
    off = np.concatenate([[0], np.cumsum(b.new_lens)])

    def alone(r, out):
        sl = slice(int(off[r]), int(off[r + 1]))
        binding.prefix_prefill(db.sub_shape(1), db.q[sl], db.k_new[sl], db.v_new[sl], db.kv_pool, db.block_table[r:r + 1],
                               b.prefix_lens[r:r + 1].copy(), b.new_lens[r:r + 1].copy(), out[sl])

    split = {}
    for waves in (0, 4, 8, 64):
        binding.set_attn_waves(waves)
        try:
            db.out.fill_(7.0)
            db.prefill()
            one_by_one = torch.full_like(db.out, 5.0)
            for r in range(b.B):
                alone(r, one_by_one)
            torch.cuda.synchronize()
        finally:
            binding.set_attn_waves(0)
        split[waves] = (db.out.clone(), one_by_one)
        if waves:
            assert torch.equal(db.out, one_by_one), waves
            assert torch.equal(db.out, split[4][0]), waves
    assert not torch.equal(split[0][1], split[4][1]), "no launch was split"
    atol, rtol = {"bf16": (4e-2, 2e-2), "f32": (2e-5, 2e-5)}[dtype]
    a, c = (W.to_f64(to_numpy(t)) for t in split[0])
    assert np.abs(a - c).max() <= atol and np.linalg.norm(a - c) <= rtol * np.linalg.norm(c)


@pytest.mark.parametrize("prefix,new,heads", [(12001, 37, (32, 8, 128)), (5000, 100, (8, 2, 64)), (7777, 33, (16, 2, 128))])
def test_ranges_do_not_see_where_pages_stand(prefix, new, heads):
    """Ranges begin anywhere in the blocks of 64 page ids that a wave holds, and run across their ends: the same bits wherever
    the pages stand in the pool, and no others if one of them is another page."""
    b = W.ragged_small(145, "bf16", Hq=heads[0], Hkv=heads[1], d=heads[2], prefix_lens=(prefix,), new_lens=(new,), num_pages=prefix // 16 + 40)
    db = DeviceBatch(b)
    db.prefill()
    moved = DeviceBatch(b)
    to = torch.from_numpy(np.random.default_rng(5).permutation(b.num_pages)).cuda()
    moved.kv_pool[to] = db.kv_pool
    moved.block_table.copy_(to[db.block_table.long()].int())
    moved.prefill()
    torch.cuda.synchronize()
    assert torch.equal(moved.out, db.out)
    for tile in range(0, -(-prefix // 64), 7):
        table = moved.block_table.clone()
        moved.block_table[0, 4 * tile] = moved.block_table[0, 4 * tile + 8 if tile < 20 else 4 * tile - 8]
        moved.prefill()
        torch.cuda.synchronize()
        assert not torch.equal(moved.out, db.out), tile
        moved.block_table.copy_(table)


def test_scores_that_run_away_across_ranges(oracle):
    """Scores that climb by ~100 log2 units per 32-key block: the ranges' references differ by thousands."""
    b = W.ragged_small(142, "bf16", prefix_lens=(1100,), new_lens=(40,), num_pages=96)
    d, p = b.d, 1100
    u = np.sign(np.random.default_rng(3).standard_normal(d)).astype(np.float32)
    b.q = W.f32_to_bf16_bits(np.broadcast_to(4.0 * u, W.to_f64(b.q).shape).astype(np.float32))
    t = np.arange(p + 40, dtype=np.float32) + 1.0
    keys = W.f32_to_bf16_bits((0.05 * t)[:, None, None] * np.broadcast_to(u, (p + 40, b.Hkv, d)))
    for tok in range(p):
        b.kv_pool[b.block_table[0, tok // b.P], 0, :, tok % b.P] = keys[tok]
    b.k_new[:] = keys[p:]
    db = DeviceBatch(b)
    db.prefill()
    torch.cuda.synchronize()
    want = oracle.prefill(b.q, b.k_new, b.v_new, b.kv_pool, b.block_table, b.prefix_lens, b.new_lens)
    assert_close(db.out_f64(), want, "bf16", "runaway scores")
