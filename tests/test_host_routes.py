"""What the library's host side decides and launches, without a GPU: the built libpbkv.so over a runtime that records
launches and runs no kernel (tests/host/).  Each check runs in a process of its own."""
import os
import shutil
import subprocess
import sys

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HOST = os.path.join(ROOT, "tests", "host")
FAKE = 0x1000                                     # a device address that nothing reads


@pytest.fixture(scope="session")
def fake_runtime(tmp_path_factory):
    inc = "/opt/rocm/include"
    if not os.path.exists(os.path.join(inc, "hip", "hip_runtime_api.h")) or not shutil.which("g++"):
        pytest.skip("needs the HIP headers (declarations only) and g++")
    so = str(tmp_path_factory.mktemp("fake") / "libfake_hip.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-w", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I" + inc,
                    "-I" + os.path.join(ROOT, "paper_2605_06472_amd", "csrc"), os.path.join(HOST, "fake_hip.cpp"), "-o", so], check=True)
    return so


@pytest.fixture
def over_fake(fake_runtime):
    def run(check, *args):
        r = subprocess.run([sys.executable, os.path.join(HOST, "fake.py"), fake_runtime, check.__name__, *map(str, args)],
                           capture_output=True, text=True, timeout=300, cwd=ROOT)
        assert r.returncode == 0 and r.stdout.strip().endswith("clean"), (r.stdout + r.stderr)[-3000:]
    return run


def _shape(batch=1, hq=32, hkv=8, d=128, dtype="bf16", width=1 << 20, pages=4096):
    from paper_2605_06472_amd import binding
    return binding.make_shape(batch, hq, hkv, d, 16, pages, width, dtype)


def _prefill(prefix, new, stream=0, **kw):
    from paper_2605_06472_amd import binding
    binding.prefix_prefill(_shape(len(new), **kw), FAKE, FAKE, FAKE, FAKE, FAKE, np.asarray(prefix, np.int32), np.asarray(new, np.int32),
                           FAKE, stream=stream)


def _decode(ctx, stream=0, **kw):
    from paper_2605_06472_amd import binding
    binding.paged_decode(_shape(len(ctx), **kw), FAKE, FAKE, FAKE, np.asarray(ctx, np.int32), FAKE, stream=stream)


def _covers(launches, merges, prefix, new, hq=32, hkv=8, dtype="bf16", **_):
    """Every KV tile of every row block is taken once, by a unit that writes the result or by parts that are merged."""
    G, f32 = hq // hkv, dtype == "f32"
    seen, parts = {}, {}
    for u in (u for l in launches for u in l["units"]):
        req, tok0, p, n, row0, part, kt0, kt1 = u
        assert (p, n, row0) == (prefix[req], new[req], sum(new[:req]))
        waves = launches[0]["waves"]
        T = 128 if f32 else 32 * (8 if waves == 64 else waves) // min(G, 4)
        first, last = (tok0 // G, (min(tok0 + T, n * G) - 1) // G) if f32 else (tok0, min(tok0 + T, n) - 1)
        tiles = (lambda tok: -(-(p + tok) // 32)) if f32 else (lambda tok: -(-p // 64) + -(-tok // 64))
        kt1 = min(kt1, tiles(last + 1))
        assert kt0 < kt1 and kt0 < tiles(first + 1), "a range whose first key some row does not see"
        seen.setdefault((req, tok0), []).append((kt0, kt1, part))
        seen[req, tok0].sort()
        parts[req, tok0] = (T, row0, tiles(last + 1))
    merged = {(m[4], m[0]): m for l in merges for m in l["merged"]}
    rows = [n * (G if f32 else 1) for n in new]
    T = next(iter(parts.values()))[0]
    assert sorted(seen) == [(r, t) for r in range(len(new)) for t in range(0, rows[r], T)]
    for key, ranges in seen.items():
        T, row0, n_tiles = parts[key]
        assert ranges[0][0] == 0 and ranges[-1][1] == n_tiles and all(a[1] == b[0] for a, b in zip(ranges, ranges[1:]))
        if len(ranges) == 1:
            assert ranges[0][2] == -1 and (row0, key[1]) not in merged
        else:
            m = merged.pop((row0, key[1]))
            assert [r[2] for r in ranges] == list(range(m[2], m[2] + m[3])) and m[1] == new[key[0]]
    assert not merged


# ---- device memory runs out -------------------------------------------------------------------------
def check_prefill_without_scratch(fake, dtype):
    """A launch that would be cut takes no partial results when there is no memory for them: it runs whole."""
    kw = dict(dtype=dtype) if dtype == "bf16" else dict(dtype=dtype, hq=8, hkv=2)
    prefix, new = [4000, 7], [33, 5]
    _prefill(prefix, new, **kw)                   # with memory: cut
    (main,), (merge,) = fake.launches("_kernelI")[:1], fake.launches("merge")
    assert "merge" not in main["name"]
    _covers([main], [merge], prefix, new, **kw)
    for repeat in range(2):                       # the second time from whatever the first one kept
        fake.forget()
        fake.limit(4 << 20)                       # another stream: its work lists, but no scratch
        _prefill(prefix, new, stream=0x100, **kw)
        (main,) = fake.launches("attn")
        assert main["merges"] == 0
        if main["units"]:
            _covers([main], [], prefix, new, **kw)
    # a kept list whose scratch has gone: a larger call gave it back and got nothing
    fake.forget()
    fake.limit(None)
    prefix, new = [4000, 9], [33, 5]
    _prefill(prefix, new, stream=0x200, **kw)
    assert fake.launches("merge")
    # nothing is left behind that a later call would take for its own error
    fake.limit(0)
    _decode([16], stream=0)
    fake.limit(None)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_prefill_runs_whole_where_there_is_no_memory_for_partial_results(over_fake, dtype):
    over_fake(check_prefill_without_scratch, dtype)


def check_decode_counters(fake):
    """The one-kernel form at its largest: as many work-groups, all of different (request, KV head) pairs, as there are counters."""
    before = fake.live()
    _decode([40] * 128, hq=8, hkv=8)
    (main,) = fake.launches("decode_")
    assert main["counters"] and main["grid"] == 1024
    _decode([40] * 129, hq=8, hkv=8)
    assert not fake.launches("decode_")[-1]["counters"]
    assert fake.live() - before <= (3 << 20) + 4 * 1024       # work lists, and a word per work-group


def test_decode_counters_are_as_many_as_work_groups(over_fake):
    over_fake(check_decode_counters)


def check_decode_kernels(fake):
    """Which kernel a call takes follows from where its list is and, for lists in memory, from heads and width."""
    for d in (64, 128):
        for hkv, G in ((8, 1), (8, 4), (2, 8), (2, 16)):
            for batch in (1, 64, 65, 128, 129, 500):
                fake.forget()
                _decode([20] * batch, hq=hkv * G, hkv=hkv, d=d, width=2)
                (main,) = fake.launches("decode_")
                kind = "list" if batch <= 128 else "heads" if d == 128 and G > 4 else ""
                assert "decode_bf16_%skernel" % (kind and kind + "_") in main["name"] and "ILi%dE" % d in main["name"], main["name"]
                form = "n1" if d == 64 else {1: "1", 4: "1", 8: "2", 16: "0"}[G]
                assert ("ELi%sE" % form in main["name"].split("kernel")[1]) == (kind != ""), main["name"]


def test_decode_kernels(over_fake):
    over_fake(check_decode_kernels)


def check_decode_without_counters(fake):
    """A decode call that would merge in one kernel merges in two when there is no memory for the counters."""
    _decode([1000])
    assert [l["counters"] != 0 for l in fake.launches("decode_")] == [True]
    fake.forget()
    _prefill([0], [1], stream=0x100)              # another stream, whose work lists have their memory
    fake.limit(8 << 20)                           # enough for partial results, not for the counters too
    fake.forget()
    _decode([1000], stream=0x100)
    assert [l["counters"] for l in fake.launches("decode_")] == [0, 0]
    _decode([1000 + r for r in range(3)] + [0] * 200, hkv=2, hq=8, stream=0x100)
    assert not any(l["counters"] for l in fake.launches("decode_"))


def test_decode_merges_in_two_kernels_where_there_is_no_memory_for_counters(over_fake):
    over_fake(check_decode_without_counters)


# ---- what one stream's scratch comes to ---------------------------------------------------------------
def check_scratch_bound(fake):
    """Launches of long blocks that do not fill their rounds leave the most partial results: growing ones re-allocate a few
    times and end at no more than the header states for a stream (163 MiB, beside 4 MiB for lists and counters)."""
    most = 0
    for prefix in range(30000, 120000, 3000):
        fake.forget()
        _prefill([prefix], [2112])                # 264 units of 64 rows
        main, merge = fake.launches("attn")
        _covers([main], [merge], [prefix], [2112])
        most = max(most, sum(m[3] for m in merge["merged"]) * 8 * 66560)
    assert most > 140e6                           # (half as much again would be past the bound)
    assert fake.live() <= (163 + 4) << 20
    _decode([30000] * 4)                          # a decode call that fits finds its place in the same buffer
    assert fake.live() <= (163 + 4) << 20
    fake.forget()
    stream = 0x100
    for prefix in range(5000, 120000, 500):
        _prefill([prefix], [2112], stream=stream)
    assert fake.count("hipStreamSynchronize") <= 4


def test_scratch_stays_within_its_bound(over_fake):
    over_fake(check_scratch_bound)


# (prefix, new) of many requests and of one, heads: one row group per block beside blocks of several work-groups
UNEVEN = [((6400, 1), 560, (200000, 33), (16, 1, 128)), ((6400, 1), 255, (150000, 40), (32, 2, 128)), ((9000, 3), 240, (120000, 70), (32, 4, 128)),
          ((6400, 1), 255, (150000, 40), (16, 1, 64)), ((7000, 17), 200, (90000, 16), (16, 2, 128))]


def check_scratch_bound_of_uneven_requests(fake):
    """A part takes the room of the work-groups that its own block has, whatever the longest request of the call: the bound holds
    at the head ratios whose blocks are several work-groups, and no two work-groups leave their results in one place."""
    for k, ((p, n), count, one, (hq, hkv, d)) in enumerate(UNEVEN):
        fake.forget()
        stream, before = 0x100 + k, fake.live()
        prefix, new = [p] * count + [one[0]], [n] * count + [one[1]]
        _prefill(prefix, new, hq=hq, hkv=hkv, d=d, stream=stream)
        main, merge = fake.launches("attn")
        assert main["waves"] == 4 and main["merges"] > 0
        _covers([main], [merge], prefix, new, hq=hq, hkv=hkv)
        held = fake.live() - before
        assert held <= (163 + 4) << 20, "%.1f MiB for %s" % (held / 2 ** 20, UNEVEN[k])
        G, bytes_each = hq // hkv, 128 * (d + 2) * 4 * hkv
        units = {(u[0], u[1], u[5]): slot for u, slot in zip(main["units"], main["slots"]) if u[5] >= 0}
        starts = {(sum(new[:r]), t): (r, t) for r, t, _ in units}
        taken = []
        for (tok0, n_new, part0, parts, row0), (slot0, splits) in zip(merge["merged"], merge["places"]):
            req, _ = starts[row0, tok0]
            assert splits == -(-min(32, n_new - tok0) * G // 128)
            for c in range(parts):
                assert units.pop((req, tok0, part0 + c)) == slot0 + c * splits
                taken += range(slot0 + c * splits, slot0 + (c + 1) * splits)
        assert not units and len(set(taken)) == len(taken) and (max(taken) + 1) * bytes_each <= held


def test_scratch_of_uneven_requests_stays_within_its_bound(over_fake):
    over_fake(check_scratch_bound_of_uneven_requests)


def check_scratch_that_cannot_grow(fake):
    """Without memory to grow, the buffer stays for the calls it is large enough for; decode gives it up for its own."""
    _prefill([700], [10])
    (main, merge) = fake.launches("attn")
    fake.limit(4 << 20)
    fake.forget()
    _prefill([60000], [2112])
    assert [l["merges"] for l in fake.launches("attn")] == [0]
    _prefill([700], [10])
    assert fake.launches("attn")[-1]["scratch"] == main["scratch"] and fake.count("hipStreamSynchronize") == 0
    fake.limit(6 << 20)                           # 13 MiB for decode: only together with the 9 MiB that are held
    _decode([30000] * 100, hq=128)
    assert fake.count("hipStreamSynchronize") == 1


def test_scratch_that_cannot_grow(over_fake):
    over_fake(check_scratch_that_cannot_grow)


# ---- the largest calls ----------------------------------------------------------------------------------
def _refused(call, *args, **kw):
    from paper_2605_06472_amd import binding
    try:
        call(*args, **kw)
    except binding.PbkvError as e:
        return e.code
    return 0


def check_largest_bf16_lists(fake):
    """131072 blocks make one launch, one more is refused; lists of 4096 blocks, and every list of ranges, are kept for
    the next call with the same lengths."""
    n = 131072
    _prefill([0] * n, [32] * n, width=2)
    (main,) = fake.launches("attn")
    assert main["tiles"] == n and main["merges"] == 0
    assert _refused(_prefill, [0] * (n + 1), [32] * (n + 1), width=2) == -7
    for prefix, new, kw in (([0] * 4096, [32] * 4096, {}), ([60000], [313 * 64], dict(hq=4, hkv=1)), ([34000], [2112], {})):
        lists = []
        for _ in range(3):
            fake.forget()
            _prefill(prefix, new, **kw)
            lists.append(fake.launches("attn")[0]["list"])
            if not kw and len(new) == 1:
                _covers(fake.launches("attn")[:1], fake.launches("merge"), prefix, new)
        assert lists[1] == lists[2] != lists[0] and fake.count("hipEventRecord") == 0


def check_largest_f32_calls(fake, hq):
    """8388608 new tokens whatever the head ratio (the list of a call was 131072 blocks of 64 tokens), in as many launches as
    the list takes; 64 tokens more are refused, and so are rows past 32 bits."""
    hq = int(hq)
    n, kw = 8388608, dict(hq=hq, hkv=1, d=64, dtype="f32")
    _prefill([0], [n], **kw)
    tok0 = np.concatenate([np.array(l["units"])[:, 1] for l in fake.launches("attn")])
    assert all(l["grid"] * l["threads"] < 1 << 32 and l["merges"] == 0 for l in fake.launches("attn"))
    assert np.array_equal(np.sort(tok0), np.arange(0, n * hq, 128))
    assert _refused(_prefill, [0], [n + 1], **kw) == -7
    assert _refused(_prefill, [0], [n], hq=512, hkv=1, d=64, dtype="f32") == -7
    fake.forget()
    _prefill([0] * 16, [300000] * 16, hq=1024, hkv=512, d=64, dtype="f32")      # grids of many KV heads
    assert sum(l["tiles"] for l in fake.launches("attn")) == 16 * -(-600000 // 128)
    assert _refused(_prefill, [0, 0], [1, 1], hq=1 << 25, hkv=1 << 25, d=64, dtype="f32", pages=2) == -6     # a grid no launch takes


def test_largest_bf16_lists(over_fake):
    over_fake(check_largest_bf16_lists)


@pytest.mark.parametrize("hq", [1, 8])
def test_largest_f32_calls(over_fake, hq):
    over_fake(check_largest_f32_calls, hq)


# ---- streams ----------------------------------------------------------------------------------------------
def check_per_thread_streams(fake):
    """hipStreamPerThread is one handle for a stream per thread: threads share neither partial results, nor counters, nor
    kept lists, and a thread that comes later does not find those of one that is gone."""
    import threading
    PER_THREAD = 2
    seen = []

    def work():
        fake.forget()
        for _ in range(2):
            _prefill([4000], [33], stream=PER_THREAD)
            _decode([1000], stream=PER_THREAD)
            _decode([20] * 200, hkv=1, hq=1, stream=PER_THREAD)
        attn, dec = fake.launches("attn_bf16"), fake.launches("decode_bf16")
        seen.append((attn[1]["scratch"], attn[1]["list"], dec[2]["counters"], dec[3]["list"]))
        assert attn[0]["scratch"] == attn[1]["scratch"] and dec[0]["counters"] == dec[2]["counters"] != 0

    for _ in range(3):
        t = threading.Thread(target=work)
        t.start()
        t.join()
    work()
    assert len(seen) == 4 and all(len(set(column)) == 4 for column in zip(*seen))
    fake.forget()
    _decode([1000], stream=0x100)                 # an ordinary stream is one stream whoever calls
    t = threading.Thread(target=_decode, args=([1000], 0x100))
    t.start()
    t.join()
    a, b = fake.launches("decode_bf16")
    assert a["counters"] == b["counters"]


def test_per_thread_streams_share_nothing(over_fake):
    over_fake(check_per_thread_streams)


def check_fp32_on_many_streams(fake):
    """fp32 prefill goes over any number of streams without a wait: past the eight that keep something it runs whole from
    the ring."""
    kw = dict(dtype="f32", hq=2, hkv=1, d=64)
    for _ in range(2):
        for k in range(12):
            _prefill([256], [64], stream=0x100 + k, **kw)
    assert fake.count("hipDeviceSynchronize") == 0
    merges = [l["merges"] > 0 for l in fake.launches("attn_f32_kernel")]
    assert merges == 2 * (8 * [True] + 4 * [False])
    whole = [l for l in fake.launches("attn_f32_kernel") if not l["merges"]]
    for l in whole:
        _covers([l], [], [256], [64], **kw)
    _prefill([256], [64], stream=0x900)           # bf16 takes the place of the stream used longest ago, as before
    assert fake.count("hipDeviceSynchronize") == 1


def test_fp32_on_many_streams(over_fake):
    over_fake(check_fp32_on_many_streams)


# ---- which launches are cut into ranges of keys -----------------------------------------------------------
# (prefix lengths, new lengths, heads), measured both ways on the GPU: us whole and cut
CUT_OR_WHOLE = {
    "short_cold": ([0, 0, 19], [260] * 3, (8, 2, 128), False),                  # 11.9, 15.3
    "many_short": ([17] * 6, [1281] * 6, (4, 2, 128), False),                    # 29.6, 38.7
    "one_of_two_per_cu": ([400], [805], (32, 2, 128), False),                   # 29.0, 32.3
    "five_tiles_d64": ([225] * 9, [3] * 9, (16, 2, 64), False),                 # 8.0, 8.4
    "turn": ([12001], [37], (32, 8, 128), True),                                # 247, 25
    "long_two_per_cu": ([5086], [718], (32, 8, 128), True),                     # 93.9, 89.8
    "short_turn": ([361], [2], (32, 8, 128), True),                             # 11.6, 10.1
    "ragged_d64": ([1836] * 3, [120, 453, 633], (16, 2, 64), True),             # 34.2, 28.3
    "long_history_that_fills_the_chip": ([32768] * 4, [2048] * 4, (32, 8, 128), False),
    "rounds_not_filled": ([34112], [2112], (32, 8, 128), True),                 # 1456, 1024
}


def check_which_launches_are_cut(fake):
    for name, (prefix, new, (hq, hkv, d), cut) in CUT_OR_WHOLE.items():
        fake.forget()
        _prefill(prefix, new, hq=hq, hkv=hkv, d=d)
        main, merge = fake.launches("attn")[0], fake.launches("merge")
        assert (main["merges"] > 0) == cut, name
        _covers([main], merge, prefix, new, hq=hq, hkv=hkv)


def test_which_launches_are_cut(over_fake):
    over_fake(check_which_launches_are_cut)


# Blocks of fewer work-groups than the longest request's: the launch has those that hold rows (prefix, new, heads, named)
NAMED = {
    "cut_tail_block": ([7278, 7906, 16454], [56, 56, 56], (16, 1, 64), True),
    "cut_uneven": ([8672] * 6, [47, 12, 34, 40, 4, 4], (32, 2, 128), True),
    "whole_64_rows": ([8616] * 27, [13 + 3 * r for r in range(27)], (32, 2, 128), True),
    "whole_4_waves": ([1098] * 59, [3 + r % 22 for r in range(59)], (32, 4, 128), True),
    "one_work_group_each": ([600] * 20, [1 + i % 5 for i in range(20)], (64, 4, 64), False),
    "two_key_groups": ([450] * 40 + [600] * 40, [1 + (r * 7) % 30 for r in range(80)], (16, 1, 64), True),
    "even": ([8672] * 6, [64] * 6, (32, 2, 128), False),
    "few_missing": ([0] * 6, [1900, 1970, 130, 800, 1210, 333], (16, 2, 64), False),               # 1 in 60
    "ratio_4": ([8672] * 6, [47, 12, 34, 40, 4, 4], (32, 8, 128), False),
}


def check_named_work_groups(fake):
    for name, (prefix, new, (hq, hkv, d), named) in NAMED.items():
        G = hq // hkv
        for repeat in range(2):                   # built, then from the kept list
            fake.forget()
            _prefill(prefix, new, hq=hq, hkv=hkv, d=d)
            main = fake.launches("attn_bf16")[0]
            wave_rows = 256 if main["waves"] == 64 else 128
            T = 32 * (8 if main["waves"] == 64 else 4) // min(G, 4)
            exist = [(t, k) for t, u in enumerate(main["units"]) for k in range(-(-min(T, u[3] - u[1]) * G // wave_rows))]
            assert bool(main["named"]) == named and (name != "two_key_groups" or main["threads"] == 512 and not main["merges"]), name
            if named:
                assert main["named"] == exist and main["grid"] == len(exist) * hkv, name
            else:
                splits = max(k for _, k in exist) + 1
                assert main["grid"] == len(main["units"]) * splits * hkv and 32 * len(exist) > 31 * len(main["units"]) * splits, name
        assert fake.count("hipEventRecord") == 0, name


def test_named_work_groups(over_fake):
    over_fake(check_named_work_groups)


# Launches of 64-row units on 256 CUs: cut where their makespan is too far above the even share of the 4-wave units, both counted by
# the work-groups that hold rows (prefix, new, heads; us whole and cut)
ROUNDS = {
    "one_token_two_rounds_and_8": ([12800] * 520, [1] * 520, (16, 1, 128), True),       # 938, 638
    "one_token_d64": ([12800] * 520, [1] * 520, (16, 1, 64), True),                      # 666, 338
    "four_kv_heads": ([12800] * 130, [4] * 130, (32, 4, 128), True),                     # 945, 656
    "half_a_block": ([12800] * 65, [32] * 65, (64, 8, 128), True),                       # 1010, 973
    "three_rounds_filled": ([7000] * 780, [1] * 780, (16, 1, 128), True),                # 741, 520
    "three_rounds_of_full_units": ([7000] * 760, [16] * 760, (16, 1, 128), False),
    "unit_of_eight_rows_d64": ([20619] * 46, [129] * 46, (16, 2, 64), True),             # 719, 617
    "two_kv_heads": ([9867] * 98, [31] * 98, (32, 2, 128), False),                       # +16 % by the cut
    "four_kv_heads_many_units": ([27643] * 15, [188] * 15, (32, 4, 128), True),          # -10 %
    "whole_unit_read_twice": ([12800] * 520, [16] * 520, (16, 1, 128), False),           # 985, 1053
    "whole_unit_read_twice_half_empty": ([12800] * 260, [16] * 260, (16, 1, 128), True), # 629, 563
    "whole_unit_eight_heads": ([12800] * 65, [64] * 65, (32, 8, 128), True),             # 1009, 959
    "whole_unit_d64": ([12800] * 520, [16] * 520, (16, 1, 64), True),                    # 682, 608
}


def check_rounds_of_64_row_units(fake):
    for name, (prefix, new, (hq, hkv, d), cut) in ROUNDS.items():
        fake.forget()
        _prefill(prefix, new, hq=hq, hkv=hkv, d=d)
        main, merge = fake.launches("attn")[0], fake.launches("merge")
        assert (main["merges"] > 0) == cut and main["waves"] == (4 if cut else 64), name
        _covers([main], merge, prefix, new, hq=hq, hkv=hkv)


def test_rounds_of_64_row_units(over_fake):
    over_fake(check_rounds_of_64_row_units)


def check_forced_shape_is_never_cut(fake):
    from paper_2605_06472_amd import binding
    for waves in (4, 8, 64):
        for kw in ({}, dict(dtype="f32", hq=2, hkv=1, d=64)):
            binding.set_attn_waves(waves)
            fake.forget()
            _prefill([4000], [33], **kw)
            assert [l["merges"] for l in fake.launches("attn")] == [0]
            binding.set_attn_waves(0)
            fake.forget()
            _prefill([4000], [33], **kw)
            assert len(fake.launches("attn")) == 2


def test_forced_shape_is_never_cut(over_fake):
    over_fake(check_forced_shape_is_never_cut)


def check_tokens_far_apart(fake):
    """The 4-wave form addresses a wave's 32 / G tokens of Q with 32 bits: from 2 GiB on the call takes the 8-wave form, also
    where the 4-wave form is asked for."""
    from paper_2605_06472_amd import binding
    for G, d in ((1, 128), (1, 64), (2, 128), (16, 128)):
        wide = (1 << 31) // (32 * d * 2)                     # KV heads: 32 / G tokens of G query heads each
        for waves in (0, 4):
            binding.set_attn_waves(waves)
            for heads, expect in ((wide - 1, 4), (wide, 8), (wide + 9000, 8)):
                fake.forget()
                _prefill([0], [33], hq=heads * G, hkv=heads, d=d, width=4, pages=2)
                (main,) = fake.launches("attn")
                assert main["waves"] == expect and main["threads"] == 64 * expect, (heads, waves)
    binding.set_attn_waves(0)


def test_tokens_far_apart_take_a_form_that_reaches_them(over_fake):
    over_fake(check_tokens_far_apart)


# Launches of two key groups per work-group: whole, and the work-groups are of eight waves.
TWO_GROUPS = {
    "nine_tiles": ([450] * 24, [40] * 24, (8, 2, 128), True),
    "eight_tiles_d64": ([440] * 30, [20] * 30, (16, 2, 64), True),
    "long_suffix": ([282, 511], [1794, 1700], (8, 2, 128), True),
    "g1_few_rows": ([600] * 20, [1 + i % 5 for i in range(20)], (8, 8, 128), True),
    "seven_tiles": ([330] * 24, [40] * 24, (8, 2, 128), False),
    "more_units_than_cus": ([1583] * 19, [42] * 19, (32, 8, 128), False),
    "cut": ([12001], [37], (32, 8, 128), False),
}


def check_two_key_groups(fake):
    for name, (prefix, new, (hq, hkv, d), two) in TWO_GROUPS.items():
        for repeat in range(2):                   # built, then from the kept list
            fake.forget()
            _prefill(prefix, new, hq=hq, hkv=hkv, d=d)
            main = fake.launches("attn_bf16")[0]
            assert main["waves"] == 4 and main["threads"] == (512 if two else 256), name
            assert not two or not main["merges"], name


def test_two_key_groups(over_fake):
    over_fake(check_two_key_groups)


# Cut launches of two key groups: long ranges, and CUs left idle (at d = 64 also where they are not).
RANGES_OF_TWO_GROUPS = {
    "one_kv_head_d64": ([20001], [3], (16, 1, 64), True),
    "all_cus_d64": ([32000], [62], (16, 2, 64), True),
    "short_ranges_d64": ([8000], [25], (16, 2, 64), False),
    "two_kv_heads": ([26003], [1], (4, 2, 128), True),
    "all_cus": ([32000], [30], (32, 8, 128), False),
}


def check_two_key_groups_in_ranges(fake):
    for name, (prefix, new, (hq, hkv, d), two) in RANGES_OF_TWO_GROUPS.items():
        for repeat in range(2):
            fake.forget()
            _prefill(prefix, new, hq=hq, hkv=hkv, d=d)
            main, merge = fake.launches("attn_bf16")[0], fake.launches("merge")
            assert main["waves"] == 4 and main["threads"] == (512 if two else 256) and merge, name
            if not repeat:
                _covers([main], merge, prefix, new, hq=hq, hkv=hkv)


def test_two_key_groups_in_ranges(over_fake):
    over_fake(check_two_key_groups_in_ranges)
