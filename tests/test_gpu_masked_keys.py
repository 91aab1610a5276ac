"""Keys whose score is minus infinity for every query (a key's component is -inf where the queries' is positive): they count
nothing, also where a range or slice of the context begins with nothing else, or holds nothing else.  All other scores stand near
-650 in log2 units, so a reference that is not taken from the first scores that count would lose them."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from paper_2605_06472_amd import binding, workloads as W          # noqa: E402
from tests.gpu_util import DeviceBatch, assert_close, to_numpy     # noqa: E402

# [first, last) tokens: whole ranges and pages, the start of a range, single 32-key blocks and single tokens
MASKED = ((64, 400), (448, 500), (512, 544), (600, 601), (704, 1000))


def _set(a, index, value):
    a[index] = W.f32_to_bf16_bits(np.full(1, value, np.float32))[0] if a.dtype == np.uint16 else np.float32(value)


def _masked(seed, dtype, tokens, new, **kw):
    b = W.ragged_small(seed, dtype, prefix_lens=(tokens,), new_lens=(new,), num_pages=tokens // 16 + 20, **kw)
    _set(b.q, (..., 0), 2.0)
    _set(b.q, (..., 1), 16.0)
    keys = [(b.kv_pool, (slice(None), 0)), (b.k_new, (slice(None),))]
    for a, at in keys:
        _set(a, at + (..., 0), 0.0)
        _set(a, at + (..., 1), -320.0 if b.d == 64 else -448.0)
    for lo, hi in MASKED:
        for t in range(lo, min(hi, tokens)):
            _set(b.kv_pool, (b.block_table[0, t // 16], 0, slice(None), t % 16, 0), -np.inf)
    return b


@pytest.mark.parametrize("dtype,heads", [("bf16", (32, 8, 128)), ("bf16", (16, 2, 64)), ("f32", (4, 2, 64)), ("f32", (6, 2, 128))])
def test_prefill_over_keys_that_count_nothing(oracle, dtype, heads):
    b = _masked(900, dtype, 1100, 40, Hq=heads[0], Hkv=heads[1], d=heads[2])
    want = oracle.prefill(b.q, b.k_new, b.v_new, b.kv_pool, b.block_table, b.prefix_lens, b.new_lens)
    assert np.isfinite(want).all()
    db = DeviceBatch(b)
    for waves in (0, 4, 8, 64) if dtype == "bf16" else (0,):
        binding.set_attn_waves(waves)
        try:
            db.out.fill_(7.0)
            db.prefill()
            torch.cuda.synchronize()
        finally:
            binding.set_attn_waves(0)
        # fp32: a score near -450 leaves 2^-24 of itself, 2.7e-5, in its exponent
        got = db.out_f64()
        if dtype == "f32":
            assert np.isfinite(got).all() and np.linalg.norm(got - want) <= 1e-4 * np.linalg.norm(want)
        else:
            assert_close(got, want, dtype, "%s %s, %d waves" % (dtype, heads, waves))


@pytest.mark.parametrize("heads", [(32, 8, 128), (16, 1, 64)])
def test_decode_over_keys_that_count_nothing(oracle, heads):
    b = _masked(901, "bf16", 1100, 1, Hq=heads[0], Hkv=heads[1], d=heads[2])
    want = oracle.decode(b.q, b.kv_pool, b.block_table, b.prefix_lens)
    db = DeviceBatch(b)
    for entry in (binding.paged_decode, binding.paged_decode_static):
        out = torch.full_like(db.q, 7.0)
        entry(db.shape, db.q, db.kv_pool, db.block_table, b.prefix_lens, out)
        torch.cuda.synchronize()
        assert_close(W.to_f64(to_numpy(out)), want, "bf16", "decode %s" % (heads,))
