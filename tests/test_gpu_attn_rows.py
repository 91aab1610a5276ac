"""bf16 prefill: rows are (suffix token, query head), 32 to a wave, and key groups share a unit's tiles out, at the sizes where
either can go wrong, against the fp64 oracle (bounds: gpu_util.TOL)."""
import numpy as np
import pytest
import torch

from paper_2605_06472_amd import binding, workloads as W
from tests.gpu_util import DeviceBatch, assert_close, to_numpy

pytestmark = pytest.mark.gpu

HEADS = [(16, 1, 64), (16, 1, 128), (16, 2, 64), (32, 4, 128), (8, 2, 64), (8, 2, 128), (4, 2, 128), (3, 3, 64)]


def edges(G):
    """New tokens around the ends of a wave (32 rows), a work-group (128) and a 64-row unit (256), and one token."""
    rows = {32, 128, 256}
    n = sorted({1} | {max(1, r // G + k) for r in rows for k in (-1, 0, 1)})
    return tuple(n)


@pytest.mark.parametrize("heads", HEADS, ids=lambda h: "%d_%d_%d" % h)
@pytest.mark.parametrize("waves", [0, 4, 8, 64])
def test_row_edges(oracle, heads, waves):
    hq, hkv, d = heads
    new = edges(hq // hkv)
    prefix = tuple((0, 17, 64, 100, 250)[i % 5] for i in range(len(new)))
    b = W.ragged_small(500 + d, "bf16", Hq=hq, Hkv=hkv, d=d, prefix_lens=prefix, new_lens=new, num_pages=600)
    print("rows", heads, waves, new, flush=True)
    db = DeviceBatch(b)
    db.out.fill_(7.0)
    binding.set_attn_waves(waves)
    try:
        db.prefill()
        torch.cuda.synchronize()
    finally:
        binding.set_attn_waves(0)
    want = oracle.prefill(b.q, b.k_new, b.v_new, b.kv_pool, b.block_table, b.prefix_lens, b.new_lens)
    assert_close(db.out_f64(), want, "bf16", "%s %d" % (heads, waves))


# whole launches of two key groups (tests/test_host_routes.py holds that they are): 8 and 9 tiles, a group that ends inside the
# diagonal, rows of few tokens, all ratios
GROUPS = {
    "nine_tiles": dict(Hq=8, Hkv=2, d=128, prefix_lens=(450,) * 24, new_lens=(40,) * 24),
    "eight_tiles_d64": dict(Hq=16, Hkv=2, d=64, prefix_lens=(440,) * 30, new_lens=(20,) * 30),
    "long_suffix": dict(Hq=8, Hkv=2, d=128, prefix_lens=(282, 511), new_lens=(1794, 1700)),
    "g1_few_rows": dict(Hq=8, Hkv=8, d=128, prefix_lens=(600,) * 20, new_lens=tuple(1 + i % 5 for i in range(20))),
}


@pytest.mark.parametrize("name", sorted(GROUPS))
def test_two_key_groups(oracle, name):
    b = W.ragged_small(510, "bf16", num_pages=1400, **GROUPS[name])
    print("groups", name, flush=True)
    db = DeviceBatch(b)
    outs = []
    for _ in range(2):
        db.out.fill_(7.0)
        db.prefill()
        torch.cuda.synchronize()
        outs.append(db.out.clone())
    assert torch.equal(*outs)
    want = oracle.prefill(b.q, b.k_new, b.v_new, b.kv_pool, b.block_table, b.prefix_lens, b.new_lens)
    assert_close(db.out_f64(), want, "bf16", name)


# cut launches whose ranges two key groups share (tests/test_host_routes.py): ranges of an odd number of tiles, the last one shorter,
# rows in one wave and in two work-groups, a short request beside a long one
@pytest.mark.parametrize("heads,prefix,new", [((16, 1, 64), (20001,), (3,)), ((16, 2, 64), (19999,), (20,)), ((8, 2, 64), (20000, 700), (10, 5)),
                                              ((4, 2, 128), (26003,), (1,)), ((16, 2, 128), (26000,), (20,))])
def test_two_key_groups_in_ranges(oracle, heads, prefix, new):
    hq, hkv, d = heads
    b = W.ragged_small(530, "bf16", Hq=hq, Hkv=hkv, d=d, prefix_lens=prefix, new_lens=new, num_pages=1800)
    print("ranges", heads, prefix, new, flush=True)
    db = DeviceBatch(b)
    outs = []
    for _ in range(2):
        db.out.fill_(7.0)
        db.prefill()
        torch.cuda.synchronize()
        outs.append(db.out.clone())
    assert torch.equal(*outs)
    want = oracle.prefill(b.q, b.k_new, b.v_new, b.kv_pool, b.block_table, b.prefix_lens, b.new_lens)
    assert_close(db.out_f64(), want, "bf16", "%s %s" % (heads, prefix))


# cut launches whose blocks have partial results of one, two and four work-groups side by side, an uncut request among them
@pytest.mark.parametrize("heads,prefix,new", [((16, 1, 128), (2100,) * 6 + (9000, 30), (1,) * 6 + (33, 2)), ((16, 1, 64), (3000, 9001, 2500), (9, 40, 1)),
                                              ((32, 2, 128), (1700, 6000, 2040), (8, 65, 17)), ((16, 2, 128), (1900, 8003), (16, 17))])
def test_parts_of_uneven_blocks(oracle, heads, prefix, new):
    hq, hkv, d = heads
    b = W.ragged_small(540, "bf16", Hq=hq, Hkv=hkv, d=d, prefix_lens=prefix, new_lens=new, num_pages=1500)
    print("uneven", heads, prefix, new, flush=True)
    db = DeviceBatch(b)
    outs = []
    for waves in (0, 0, 4):
        db.out.fill_(7.0)
        binding.set_attn_waves(waves)
        try:
            db.prefill()
            torch.cuda.synchronize()
        finally:
            binding.set_attn_waves(0)
        outs.append(db.out.clone())
    assert torch.equal(*outs[:2]) and not torch.equal(outs[0], outs[2]), "the launch was not cut into ranges"
    want = oracle.prefill(b.q, b.k_new, b.v_new, b.kv_pool, b.block_table, b.prefix_lens, b.new_lens)
    assert_close(W.to_f64(to_numpy(outs[0])), want, "bf16", "%s %s" % (heads, prefix))


# launches whose list names the work-groups that exist (tests/test_host_routes.py): every shape, whole, cut, and in two key groups,
# from the list that is built and from the kept one
UNEVEN = [((16, 2, 128), (450,) * 12, tuple(3 + (r * 7) % 38 for r in range(12))), ((32, 2, 64), (0, 700, 30, 64, 129, 1), (30, 1, 65, 7, 16, 33)),
          ((16, 1, 64), (450,) * 40 + (600,) * 40, tuple(1 + (r * 7) % 30 for r in range(80)))]


@pytest.mark.parametrize("heads,prefix,new", UNEVEN)
@pytest.mark.parametrize("waves", [0, 4, 8, 64])
def test_named_work_groups(oracle, heads, prefix, new, waves):
    hq, hkv, d = heads
    b = W.ragged_small(550, "bf16", Hq=hq, Hkv=hkv, d=d, prefix_lens=prefix, new_lens=new, num_pages=3400)
    print("named", heads, len(new), waves, flush=True)
    db = DeviceBatch(b)
    outs = []
    binding.set_attn_waves(waves)
    try:
        for _ in range(3):
            db.out.fill_(7.0)
            db.prefill()
            torch.cuda.synchronize()
            outs.append(db.out.clone())
    finally:
        binding.set_attn_waves(0)
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])
    want = oracle.prefill(b.q, b.k_new, b.v_new, b.kv_pool, b.block_table, b.prefix_lens, b.new_lens)
    assert_close(db.out_f64(), want, "bf16", "%s %d" % (heads, waves))


def test_rows_of_a_wave_more_than_2_gib_apart():
    """300000 heads of 128: a token is 77 MB from the next, so the 32 tokens of a wave are 2.4 GB of Q."""
    heads, d, n = 300000, 128, 32
    assert (n - 1) * heads * d * 2 >= 1 << 31
    print("wide tokens", flush=True)
    g = torch.Generator(device="cuda").manual_seed(7)
    q, k, v = (torch.empty(n, heads, d, dtype=torch.bfloat16, device="cuda").normal_(0, 0.5, generator=g) for _ in range(3))
    pool = torch.zeros(1, 2, heads, 16, d, dtype=torch.bfloat16, device="cuda")
    out = torch.full_like(q, 7.0)
    shape = binding.make_shape(1, heads, heads, d, 16, 1, 2, "bf16")
    binding.prefix_prefill(shape, q, k, v, pool, torch.zeros(1, 2, dtype=torch.int32, device="cuda"), np.array([0], np.int32), np.array([n], np.int32), out)
    torch.cuda.synchronize()
    some = [0, 1, 149999, 299998, 299999]
    q, k, v = (t[:, some].double().cpu().transpose(0, 1) for t in (q, k, v))
    s = (q @ k.transpose(1, 2) / d ** 0.5).masked_fill(torch.ones(n, n).triu(1).bool(), float("-inf"))
    want = (torch.softmax(s, -1) @ v).transpose(0, 1)
    assert_close(out[:, some].double().cpu().numpy(), want.numpy(), "bf16", "wide tokens")


@pytest.mark.parametrize("where", ["first", "second", "both"])
def test_a_key_group_whose_keys_count_nothing(oracle, where):
    """One of the two groups, or all of the prefix, scores -inf: the other one's keys, or the suffix, are the result."""
    b = W.ragged_small(520, "bf16", num_pages=1400, Hq=8, Hkv=2, d=128, prefix_lens=(512,) * 24, new_lens=(40,) * 24)
    lo, hi = {"first": (0, 20), "second": (20, 32), "both": (0, 32)}[where]      # pages; 9 tiles: 5 (20 pages) and 4
    db = DeviceBatch(b)
    q = db.q.view(torch.bfloat16) if db.q.dtype != torch.bfloat16 else db.q
    pool = db.kv_pool.view(torch.bfloat16) if db.kv_pool.dtype != torch.bfloat16 else db.kv_pool
    q[..., 0] = 1.0
    table = db.block_table.long()
    for r in range(b.B):
        pool[table[r, lo:hi], 0, :, :, 0] = float("-inf")
    db.out.zero_()
    db.prefill()
    torch.cuda.synchronize()
    keep = [p for p in range(32) if not lo <= p < hi]
    off = 0
    for r in range(0, b.B, 7):
        n = int(b.new_lens[r])
        off = int(b.new_lens[:r].sum())
        k = torch.cat([pool[table[r, keep], 0].permute(0, 2, 1, 3).reshape(-1, 2, 128), db.k_new[off:off + n]]).float().cpu()
        v = torch.cat([pool[table[r, keep], 1].permute(0, 2, 1, 3).reshape(-1, 2, 128), db.v_new[off:off + n]]).float().cpu()
        qq = q[off:off + n].float().cpu().view(n, 2, 4, 128)
        s = torch.stack([qq[:, h // 4, h % 4] @ k[:, h // 4].T for h in range(8)], 1).double() / 128 ** 0.5
        t = torch.arange(k.shape[0]) - 16 * len(keep)
        s[(t[None, :] > torch.arange(n)[:, None])[:, None, :].expand_as(s)] = float("-inf")
        p = torch.softmax(s, -1)
        want = torch.stack([p[:, h] @ v[:, h // 4].double() for h in range(8)], 1)
        assert_close(db.out[off:off + n].double().cpu().numpy(), want.numpy(), "bf16", "%s request %d" % (where, r))
