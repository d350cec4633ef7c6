"""The launches of a call -- kernels, grids, order -- found without a GPU (see launches.py)."""
import numpy as np
import pytest

from launches import launches_of

QKV_8B = dict(op="forward", dtype=1, hidden=4096, n_q_heads=32, n_kv_heads=8, head_dim=128, rank=16, n_segments=4, n_slots=1024)


def kernels(call):
    assert call["status"] == 0, call
    return [l["kernel"] for l in call["launches"]]


@pytest.mark.parametrize("T", [1, 40, 64, 65, 100, 256])
def test_a_tuning_override_during_a_call_leaves_the_call_whole(T):
    """The override may be set by another host thread at any time: a call that has decided to group and shrink
    inside its projection kernel launches that kernel."""
    plain, torn, after = launches_of([dict(QKV_8B, T=T, n_adapters=4), dict(QKV_8B, T=T, n_adapters=4, tuning_during=[4, 1]),
                                      dict(QKV_8B, T=T, n_adapters=4)])
    assert len(plain["launches"]) == 2, kernels(plain)
    assert torn == plain and after == plain, (kernels(plain), kernels(torn))


@pytest.mark.parametrize("T,hidden", [(1, 4096), (3, 64), (40, 4096), (64, 4096), (65, 4096)])
def test_a_few_rows_start_no_workgroups_for_adapters_they_cannot_use(T, hidden):
    """An entry of the block table holds at least one row: at most T of its ceil(T / 32) + L + 1 are in use."""
    for call, L in zip(launches_of([dict(QKV_8B, T=T, hidden=hidden, n_adapters=L) for L in (1, 8, 32, 128)]), (1, 8, 32, 128)):
        entries = min(-(-T // 32) + L + 1, T)
        if T <= 64:
            assert kernels(call) == ["decode_projection_kernel", "finish_bf16_kernel"]
            ranges = 2 if hidden > 64 else 1
            projection = launches_of([dict(QKV_8B, T=T, hidden=hidden, n_adapters=0)])[0]["launches"][0]["grid"][0] - min(-(-T // 32) + 1, T)
            assert call["launches"][0]["grid"][0] == projection + ranges * entries
        assert call["launches"][1]["grid"][0] == entries, call["launches"][1]


def test_rows_per_tile_of_the_fp32_projection():
    sizes = {(64, 256, 2, 4): 1, (1500, 256, 4, 64): 1, (6000, 256, 4, 64): 2, (32768, 256, 4, 64): 2, (1030, 52, 12, 68): 2, (160, 4096, 32, 128): 2,
             (2930, 1700, 12, 68): 4, (512, 4096, 32, 128): 4}
    calls = [dict(op="forward", dtype=0, T=T, hidden=h, n_q_heads=hq, n_kv_heads=8 if hq == 32 else 2, head_dim=d, n_adapters=0, rank=0,
                  n_segments=1, n_slots=16) for T, h, hq, d in sizes]
    for call, (size, mt) in zip(launches_of(calls), sizes.items()):
        l = [l for l in call["launches"] if l["kernel"] == "gemm_f32_kernel"]
        assert len(l) == 1 and l[0]["ints"] == [mt] and l[0]["grid"][1] == -(-size[0] // (16 * mt)), (size, l)


@pytest.mark.parametrize("dtype", [0, 1])
def test_a_replay_is_the_launches_of_the_call(dtype):
    for T in (1, 64, 200, 300, 3000):
        call = dict(QKV_8B, dtype=dtype, T=T, n_adapters=4)
        once, twice = launches_of([call, dict(call, replays=2)])
        assert once["launches"] and twice["status"] == 0 and twice["launches"] == 2 * once["launches"], (kernels(once), kernels(twice))


# (hidden, query heads, K/V heads, head size, rows, rotation, tile width / 64, 256-row tiles): fused projections whose last rows go in
# tiles of 128 x 128, behind each width of the large ones and all by themselves, down to four slices of the hidden dimension; test_gpu_parity.py
# and test_gpu_rope.py run them.
TAILS = [(512, 5, 2, 40, 1030, False, 4, 1), (512, 60, 2, 128, 1030, False, 3, 4), (192, 22, 3, 128, 1290, False, 2, 3), (512, 24, 8, 128, 700, False, 4, 0),
         (128, 60, 2, 128, 2100, False, 4, 8), (128, 24, 8, 128, 3100, True, 4, 9), (192, 60, 2, 128, 2100, True, 4, 8), (512, 22, 3, 128, 1290, True, 2, 2), (512, 24, 8, 128, 700, True, 4, 0)]


def test_last_rows_of_a_fused_projection_in_small_tiles():
    calls = launches_of([dict(QKV_8B, T=T, hidden=h, n_q_heads=hq, n_kv_heads=hkv, head_dim=d, n_adapters=3, rope=rope) for h, hq, hkv, d, T, rope, _, _ in TAILS])
    up8 = lambda n: -(-n // 8) * 8
    for call, (h, hq, hkv, d, T, rope, width, panels) in zip(calls, TAILS):
        l = call["launches"][-1]
        N = (hq + 2 * hkv) * d
        assert l["kernel"] == "alora_gemm_bf16_kernel" and l["ints"] == [width, 0, int(rope)], l
        assert l["grid"][0] == up8(panels * -(-N // (64 * width))) + up8(-(-(T - 256 * panels) // 128) * -(-N // 128)) and T > 256 * panels, l


CALLS = [dict(QKV_8B, T=T, n_adapters=4, dtype=dtype) for dtype in (0, 1) for T in (1, 200, 700, 3000, 9000)]
READERS = [dict(op="attention", entry=entry, dtype=1, n_tokens=64, n_q_heads=32, n_kv_heads=8, head_dim=128, n_seqs=4, max_blocks=64, block_size=16, n_slots=4096)
           for entry in ("alora_paged_attention", "alora_paged_attention_split", "alora_paged_attention_suffix", "alora_paged_attention_suffix_split")]


def test_an_error_the_program_left_behind_is_not_the_librarys():
    """hipGetLastError holds whatever an earlier call left; neither a call nor a replay fails for it, nor takes it away."""
    calls = [*CALLS, *[dict(c, replays=2) for c in CALLS], *READERS]
    plain = launches_of(calls)
    for call, want in zip(launches_of([dict(c, errors=[101, 0]) for c in calls]), plain):
        assert call["status"] == 0 and call["launches"] == want["launches"] and call["errors"][1] == 101, call


def test_a_launch_that_fails_is_reported_with_its_error():
    both = [call for c in [*CALLS, *READERS] for call in (dict(c, errors=[101, 98]), c)]
    calls = launches_of(both)
    for failed, after in zip(calls[::2], calls[1::2]):
        assert failed["status"] == -4 and failed["launches"] == [] and failed["errors"] == [98, 0], failed
        assert after["status"] == 0, after


def test_planning_a_wide_projection_takes_no_longer_than_a_narrow_one():
    """Half a million tiles are not walked one by one on the host (1.2 ms of it; bound: fifty times what the calls take)."""
    for call in launches_of([dict(QKV_8B, T=2000, hidden=64, n_q_heads=n, n_adapters=4, timed=20) for n in (32, 8000, 60000)]):
        assert call["status"] == 0 and call["host_us"] < 250, call


# Batches whose rows the finishing kernel makes, run by test_gpu_parity.py: (hidden, query heads, K/V heads, head size), rows of the base
# request and of each adapter, ranks.
FINISHED = dict(shape=(1024, 5, 2, 40), entries=[1, 15, 16, 17, 31, 32, 33], infinite=[[10, 3, 20, 17], [40, 3, 33, 24]], ranks=[8, 32, 40, 64])


def test_the_finishing_kernels_cases_reach_it():
    h, hq, hkv, d = FINISHED["shape"]
    sizes = [(rows, r) for rows in [FINISHED["entries"], *FINISHED["infinite"]] for r in FINISHED["ranks"]]
    calls = launches_of([dict(QKV_8B, T=sum(rows), hidden=h, n_q_heads=hq, n_kv_heads=hkv, head_dim=d, n_adapters=len(rows) - 1, rank=r, n_segments=len(rows))
                         for rows, r in sizes])
    for call, (rows, r) in zip(calls, sizes):
        last = call["launches"][-1]
        assert last["kernel"] == "finish_bf16_kernel" and last["ints"][1] == (1 if r <= 32 else 2) and last["grid"][2] == 2, (rows, r, call)


# ---- the row-block reader ------------------------------------------------------------------------
def reader(entry, T, n_seqs, n_q, n_kv, block_size=16):
    return dict(op="attention", entry=entry, dtype=1, n_tokens=T, n_q_heads=n_q, n_kv_heads=n_kv, head_dim=128, n_seqs=n_seqs,
                max_blocks=1024, block_size=block_size, n_slots=1 << 20)


def cut_of(call):
    """(group size, wavefronts, rows per range, workgroups per range) of a recorded reader call."""
    l = call["launches"][0]
    assert l["kernel"] == "paged_attention_blocks_kernel", l
    G, waves, _ = l["ints"]
    assert l["block"][0] == 64 * waves
    return G, waves, l["args"][0], l["args"][1]


def longest_chain(runs, G, waves, rows_per_range, wgs):
    """Row blocks one workgroup takes at most, for runs of (first position, rows) laid one after the other in a batch."""
    rbg = 32 * waves // G
    at, lead = 0, []
    for first, rows in runs:
        pos = first + np.arange(rows)
        lead += list(at + np.flatnonzero((pos % rbg == 0) | (np.arange(rows) == 0)))
        at += rows
    per_range = np.bincount(np.array(lead) // rows_per_range)
    return int(-(-per_range.max() // wgs)), len(lead)


UNEVEN = {"chunk-2048+32": [(2048, 2048)] + [(4095, 1)] * 32, "chunk-1024+16": [(7168, 1024)] + [(8191, 1)] * 16,
          "4x512+32": [(3584, 512)] * 4 + [(4095, 1)] * 32, "decode-first": [(4095, 1)] * 32 + [(1000, 2048)],
          "5x61": [(8129 + 7 * i, 61) for i in range(5)]}


@pytest.mark.parametrize("n_q,n_kv", [(32, 8), (64, 8), (16, 8), (8, 8)])
@pytest.mark.parametrize("runs", UNEVEN.values(), ids=UNEVEN.keys())
def test_no_workgroup_of_the_reader_takes_several_contexts_one_after_the_other(runs, n_q, n_kv):
    """A prompt chunk beside decode rows: the workgroup with the most row blocks is the length of the call."""
    T = sum(r for _, r in runs)
    for table_rows in (len(runs), 256):
        (call,) = launches_of([reader("alora_paged_attention_suffix", T, table_rows, n_q, n_kv)])
        G, waves, rows_per_range, wgs = cut_of(call)
        chain, blocks = longest_chain(runs, G, waves, rows_per_range, wgs)
        assert chain == 1, (chain, blocks, waves, rows_per_range, wgs)


def test_no_workgroup_takes_two_parts_one_after_the_other():
    runs = UNEVEN["chunk-1024+16"]
    (call,) = launches_of([reader("alora_paged_attention_suffix_split", 1040, len(runs), 32, 8)])
    G, waves, rows_per_range, wgs = cut_of(call)
    assert len(call["launches"]) == 2 and longest_chain(runs, G, waves, rows_per_range, wgs)[0] == 1


def test_the_cut_of_a_reader_call_and_its_workspace():
    rng = np.random.default_rng(5)
    sizes = [(int(np.exp(rng.uniform(0, np.log(2e5)))), int(rng.integers(1, 400)), int(rng.choice([1, 2, 4, 8])), int(rng.choice([1, 2, 8, 16])))
             for _ in range(60)] + [(1, 1, 8, 1), (1024, 1, 4, 1), (1025, 1, 4, 1), (2048, 1, 1, 64), (2049, 1, 1, 64)]
    for entry in ("alora_paged_attention_suffix", "alora_paged_attention_suffix_split"):
        for (T, n, G, n_kv), call in zip(sizes, launches_of([reader(entry, T, n, G * n_kv, n_kv) for T, n, G, n_kv in sizes])):
            assert call["status"] == 0
            _, waves, rows_per_range, wgs = cut_of(call)
            behind = -(-(32 * waves // G) // 64) * 64      # rows of the next range that a block may reach into
            assert rows_per_range % 64 == 0 and 64 <= rows_per_range <= 256 * waves - behind and 1 <= wgs <= max(T, 1)
            ranges, parts = -(-T // rows_per_range), call["launches"][0]["grid"][0] // (-(-T // rows_per_range) * wgs * n_kv)
            assert call["launches"][0]["grid"][0] == ranges * wgs * n_kv * parts and 1 <= parts <= 32
            assert (parts > 1) == (len(call["launches"]) == 2)
            if ranges > 1:     # whole blocks, and whole turns over the chip's 32 shader engines of workgroups that may find none
                assert rows_per_range % (32 * waves // G) == 0 and (wgs - rows_per_range * G // (32 * waves)) * n_kv * parts % 32 == 0
            assert call["workspace"] == (T * G * n_kv * parts * 130 * 4 if parts > 1 else 0)


@pytest.mark.parametrize("runs,n_q,n_kv,waves", [
    ([(16383, 1)] * 8, 32, 8, 8), ([(1997, 4)] * 16, 32, 8, 8), ([(16320, 64)] * 4, 8, 8, 8), ([(8142, 50)] * 6, 8, 8, 8),       # few short blocks
    ([(4095, 1)] * 64, 32, 8, 4), ([(16320, 64)] * 4, 32, 8, 4), ([(4091, 5)] * 32, 64, 8, 4),     # more than one per CU, or long runs
    ([(0, 128)] * 100, 32, 8, 4), ([(2301, 700)] * 12, 32, 8, 4),                                  # prompts that start and store often
    ([(14336, 2048)] * 4, 32, 8, 8), ([(7168, 1024)] * 4, 64, 8, 8)])
def test_wavefronts_of_the_reader(runs, n_q, n_kv, waves):
    (call,) = launches_of([reader("alora_paged_attention_suffix", sum(r for _, r in runs), len(runs), n_q, n_kv)])
    assert cut_of(call)[1] == waves


def test_a_reader_call_in_one_part_is_the_call_without_parts():
    """The suffix_split call promises to be the suffix call, same launch, where nothing is cut."""
    rng = np.random.default_rng(9)
    sizes = [(2048, 2, 4, 8), (1024, 1, 8, 8), (4096, 4, 4, 8), (1600, 8, 8, 8), (256, 256, 8, 64), (4096, 256, 1, 16)]
    sizes += [(int(rng.integers(500, 9000)), int(rng.integers(1, 300)), int(rng.choice([1, 2, 4, 8])), int(rng.choice([4, 8, 16]))) for _ in range(40)]
    calls = [reader("alora_paged_attention_suffix" + e, T, n, G * n_kv, n_kv) for T, n, G, n_kv in sizes for e in ("_split", "")]
    out = launches_of(calls)
    whole = [(a, b) for a, b in zip(out[::2], out[1::2]) if len(a["launches"]) == 1]
    assert len(whole) >= 20 and all(a == b for a, b in whole), [(a, b) for a, b in whole if a != b][:3]


# (group, K/V heads, block size, contexts, query rows, in parts, wavefronts): every instantiation of the row-block kernel, where the sizes
# lead to it; test_gpu_attention.py runs them.
CUTS = [
    # long runs, whole contexts: eight wavefronts from 1024 rows a sequence and two workgroups per CU on, else four
    (1, 64, 16, [2100], [2079], False, 8), (2, 64, 16, [1300, 900], [1290, 800], False, 8), (4, 32, 12, [1200], [1100], False, 8),
    (8, 16, 16, [1153], [1030], False, 8), (8, 16, 16, [900, 400], [700, 399], False, 4), (1, 2, 16, [700, 260], [640, 258], False, 4),
    (2, 2, 20, [129, 640, 127], [111, 549, 109], False, 4), (4, 2, 16, [700, 257, 95], [600, 221, 82], False, 4),
    # short runs, whole contexts: eight where their blocks fit the chip at once, else four
    (1, 8, 16, [300, 900, 41], [100, 127, 3], False, 8), (2, 4, 12, [500, 77], [60, 1], False, 8), (4, 8, 16, [1000, 513, 64], [32, 5, 1], False, 8),
    (8, 2, 16, [400, 30, 199], [16, 1, 9], False, 8), (1, 64, 16, [130, 90, 60, 200, 155], [3, 1, 60, 99, 2], False, 4),
    (2, 64, 16, [130, 90, 60, 200, 155], [3, 1, 60, 64, 2], False, 4), (4, 64, 20, [130, 90, 60, 200, 155], [3, 1, 31, 32, 2], False, 4),
    (8, 64, 16, [130, 90, 60, 200, 155], [3, 1, 16, 9, 2], False, 4),
    # contexts in parts: eight wavefronts for long runs, four for short ones
    (1, 2, 16, [900, 500], [300, 201], True, 8), (2, 2, 12, [900, 500], [150, 65], True, 8), (4, 2, 16, [200, 65, 63], [171, 56, 54], True, 8),
    (8, 1, 16, [1100, 33, 900], [943, 28, 771], True, 8), (1, 2, 20, [1500, 300], [100, 28], True, 4), (2, 2, 16, [1500, 300], [40, 64], True, 4),
    (4, 2, 16, [2000, 301], [32, 17], True, 4), (8, 1, 16, [1700, 64], [16, 1], True, 4)]


def test_the_reader_cases_run_on_the_gpu_reach_every_instantiation():
    calls = launches_of([reader("alora_paged_attention_suffix" + ("_split" if parts else ""), sum(rows), len(rows), g * n_kv, n_kv, block_size=bs)
                         for g, n_kv, bs, lens, rows, parts, waves in CUTS])
    for call, (g, n_kv, bs, lens, rows, parts, waves) in zip(calls, CUTS):
        assert cut_of(call)[:2] == (g, waves) and (len(call["launches"]) == 2) == parts, (g, n_kv, rows, parts, call["launches"])
    got = {(tuple(c["launches"][0]["ints"]), len(c["launches"]) == 2) for c in calls}
    for parts in (False, True):
        assert {(i[0], i[1]) for i, p in got if p == parts} == {(g, w) for g in (1, 2, 4, 8) for w in (4, 8)}
        assert {(i[1], i[2]) for i, p in got if p == parts} == {(w, pow2) for w in (4, 8) for pow2 in (0, 1)}


# (group, K/V heads, block size, contexts, query rows, wavefronts): contexts in parts whose number the kernel settles, since more blocks
# than rows fill are likely; single rows, runs that end inside a block, unequal contexts; test_gpu_attention.py runs them.
COUNTED = [(1, 8, 16, [300 + 41 * i for i in range(9)], [1] * 9, 4), (2, 8, 20, [40, 2100, 700, 33, 1], [3, 1, 7, 33, 1], 4),
           (4, 2, 16, [64 * i + 1 for i in range(10)], [1] * 10, 4), (8, 2, 12, [5000] + [200] * 11, [2] + [3] * 11, 4),
           (1, 8, 16, [900, 1500], [150, 140], 8), (2, 8, 20, [900, 1500], [150, 140], 8), (4, 8, 16, [1200, 700, 90], [100, 61, 33], 8),
           (8, 8, 12, [500, 3900], [50, 70], 8)]


def test_parts_are_counted_by_the_kernel_only_where_they_may_not_fit_the_chip():
    merge = "paged_attention_merge_kernel"
    calls = launches_of([reader("alora_paged_attention_suffix_split", sum(rows), len(rows), g * n_kv, n_kv, block_size=bs) for g, n_kv, bs, _, rows, _ in COUNTED])
    for call, case in zip(calls, COUNTED):
        assert cut_of(call)[1] == case[5] and call["launches"][1]["kernel"] == merge and call["launches"][1]["ints"] == [128, 1, 1], (case, call)
    for call in launches_of([reader("alora_paged_attention_suffix_split", T, n, 32, 8) for T, n in [(1, 1), (2, 2), (4, 2), (16, 1), (256, 4)]]):
        assert call["launches"][1]["kernel"] == merge and call["launches"][1]["ints"] == [128, 1, 0], call


def test_a_workspace_that_holds_the_fewer_parts_is_enough():
    """What a call of the reader in parts by rows cannot do without follows from its rows and heads alone: not from how
    long the block tables are, how many, or how large the cache is."""
    name = "alora_paged_attention_split"
    for T in (2, 5, 8, 16, 17, 100, 127):
        fewer, more = min(32, -(-1024 // (T * 8))), min(32, -(-2048 // (T * 8)))
        enough = T * 32 * fewer * 130 * 4
        wide = dict(reader(name, T, T, 32, 8))
        others = [dict(wide, n_seqs=max(1, T - 1)), dict(wide, max_blocks=16), dict(wide, n_slots=4096)]
        calls = launches_of([wide, dict(wide, give=enough), dict(wide, give=enough - 1), *others, *[dict(o, give=enough) for o in others]])
        assert calls[0]["status"] == 0 and calls[0]["workspace"] == T * 32 * more * 130 * 4
        assert calls[0]["launches"][0]["grid"][0] == T * 8 * more
        for c in (calls[1], *calls[3:]):
            assert c["status"] == 0 and c["launches"][0]["grid"][0] == T * 8 * fewer, (T, c)
            assert c["launches"][1]["kernel"] == "paged_attention_merge_kernel" and c["launches"][1]["ints"] == [128, 1, 0], (T, c)
        assert all(c["workspace"] == enough for c in calls[3:6])
        if fewer < more:
            assert calls[2]["status"] == -3 and not calls[2]["launches"]
    # sized for the largest call of a program, two rows a sequence, then one row each
    large = launches_of([reader(name, 32, 16, 32, 8)])[0]["workspace"]
    (call,) = launches_of([dict(reader(name, 16, 16, 32, 8), give=large)])
    assert call["status"] == 0 and call["launches"][0]["grid"][0] == 16 * 8 * 8


def test_small_fp32_calls_of_one_launch_fit_the_chip():
    """(hidden, query heads, K/V heads, head size, rows): one launch up to two workgroups per compute unit, shrink and projection from there on."""
    sizes = {(48, 16, 4, 64, 336): True, (48, 16, 4, 64, 337): False, (256, 32, 8, 64, 160): True, (256, 32, 8, 64, 161): False, (48, 32, 8, 64, 186): False,
             (4, 8, 2, 32, 1360): True, (4, 8, 2, 32, 1361): False, (256, 1, 1, 8, 8192): True, (256, 1, 1, 8, 8193): False,
             (64, 180, 9, 128, 16): True, (64, 184, 8, 128, 16): False, (64, 248, 4, 128, 1): False}      # (the last two in tiles of 32 rows)
    calls = launches_of([dict(op="forward", dtype=0, T=T, hidden=h, n_q_heads=hq, n_kv_heads=hkv, head_dim=d, n_adapters=4, rank=16, n_segments=4, n_slots=16 * T)
                         for h, hq, hkv, d, T in sizes])
    for call, (size, one) in zip(calls, sizes.items()):
        own = [k for k in kernels(call) if k in ("shrink_f32_kernel", "gemm_f32_kernel")]
        assert own == (["gemm_f32_kernel"] if one else ["shrink_f32_kernel", "gemm_f32_kernel"]), (size, kernels(call))


# (rows, K/V heads, positions a table has room for, in parts): calls of the per-row reader that take its kernels for contexts read once, 1, in order of
# length, 2, and in parts of which long contexts have more, 3; test_gpu_attention.py runs them with every type, head size, group and kind of block size.
ONCE = {(60, 4, 480, False): 1, (140, 4, 960, False): 2, (70, 4, 4800, True): 3, (9, 4, 960, True): 1}


def test_the_per_row_readers_cases_reach_every_kernel_for_contexts_read_once():
    for bf16 in (1, 0):
        for (n, n_kv, room, parts), kind in ONCE.items():
            for d, bs in ((64, 16), (128, 24)):
                slots = (104 << 20) // (n_kv * d * (4 if bf16 else 8)) // bs * bs
                (call,) = launches_of([dict(op="attention", entry="alora_paged_attention" + ("_split" if parts else ""), dtype=bf16, n_tokens=n, n_q_heads=n_kv,
                                            n_kv_heads=n_kv, head_dim=d, n_seqs=n, max_blocks=room // bs, block_size=bs, n_slots=slots)])
                assert call["status"] == 0 and call["launches"][0]["contexts"] == (kind if bf16 or kind > 1 else 0), (n, room, parts, bf16, call)
                assert len(call["launches"]) == (2 if parts else 1) and (not parts or call["launches"][1]["ints"] == [d, bf16, int(kind == 3)]), call
