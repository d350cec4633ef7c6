"""GPU parity of the paged-cache reader (alora_paged_attention) against the fp64 oracle
(oracle/attention.py: causal softmax attention, Sec. 2.1), through the C ABI.

Slots no context covers hold NaN in every case, so a read outside a row's causal context shows up
as a NaN in the output."""
import numpy as np
import pytest
import torch

from oracle import attention as oatt
from paper_2512_17910_amd import binding as ab
from paper_2512_17910_amd import workloads as wl
from test_launches import COUNTED, CUTS, ONCE
from gpu_util import TOL, maxnorm_rel, raw_bits, to_dev, to_f64

pytestmark = pytest.mark.gpu


class DeviceCase:
    def __init__(self, c: wl.AttentionCase, scale: float = 0.0):
        self.c = c
        self.q = to_dev(c.q, c.dtype)
        self.kc = to_dev(c.k_cache, c.dtype)
        self.vc = to_dev(c.v_cache, c.dtype)
        self.bt = torch.from_numpy(c.block_tables).to("cuda")
        self.seq = torch.from_numpy(c.token_seq_ids).to("cuda")
        self.pos = torch.from_numpy(c.token_positions).to("cuda")
        self.out = torch.full_like(self.q, float("nan"))
        self.dims = ab.make_attn_dims(self.q, self.kc, self.bt, c.n_q_heads, c.n_kv_heads, c.head_dim, c.block_size, scale)

    def run(self):
        ab.alora_paged_attention(self.q, self.kc, self.vc, self.bt, self.seq, self.pos, self.out, self.dims)
        torch.cuda.synchronize()
        return self.out

    def oracle(self, rows=None, scale=None):
        c = self.c
        return oatt.paged_attention(wl.widen_f64(c.q, c.dtype), wl.widen_f64(c.k_cache, c.dtype),
                                    wl.widen_f64(c.v_cache, c.dtype), c.block_tables, c.token_seq_ids,
                                    c.token_positions, c.block_size, c.n_q_heads, c.n_kv_heads, c.head_dim,
                                    scale=scale, rows=rows)


def _ragged_lens(seed, n, hi):
    rng = np.random.default_rng(seed)
    lens = rng.integers(1, hi + 1, n)
    lens[0] = 1                       # a context of one position
    lens[1] = hi
    return lens


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("group", [1, 2, 4, 8])
def test_matches_the_oracle_on_ragged_contexts(dtype, head_dim, group):
    n_kv = 2
    lens = _ragged_lens(100 + group + head_dim, 9, 333)
    rows = [1, 3, 1, 2, 1, 5, 1, 1, 4]
    for bs in (16, 5):                # a power of two and not
        c = wl.attention_case(f"ragged-{dtype}-d{head_dim}-g{group}-bs{bs}", dtype, lens, rows, n_kv * group, n_kv,
                              head_dim, bs, seed=wl.SEED ^ (head_dim * 8 + group))
        print(f"[case] {c.name} T={c.T} lens={list(lens)}", flush=True)
        d = DeviceCase(c)
        assert ab.alora_paged_attention_validate(d.bt, d.seq, d.pos, d.dims) == ab.ALORA_OK
        out = to_f64(d.run())
        assert np.isfinite(out).all()
        assert maxnorm_rel(out, d.oracle()) <= TOL[dtype]


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_long_contexts_and_explicit_scale(dtype):
    lens = [5000, 4097, 4096, 63, 64, 65, 1023]
    c = wl.attention_case(f"long-{dtype}", dtype, lens, [2, 1, 1, 1, 1, 1, 1], 8, 2, 128, 16, seed=wl.SEED ^ 77)
    print(f"[case] {c.name}", flush=True)
    d = DeviceCase(c, scale=0.05)
    out = to_f64(d.run())
    assert np.isfinite(out).all()
    assert maxnorm_rel(out, d.oracle(scale=0.05)) <= TOL[dtype]


def test_contexts_of_sixteen_thousand_positions():
    """The long-context shape of the reader's benchmark (--long): 32 query / 8 K/V heads of 128, contexts
    of 16384 and 8193 positions, every output element against the oracle."""
    c = wl.attention_case("16k", "bf16", [16384, 8193, 12000], [1, 2, 1], 32, 8, 128, 16, seed=wl.SEED ^ 91)
    d = DeviceCase(c)
    out = to_f64(d.run())
    assert np.isfinite(out).all()
    assert maxnorm_rel(out, d.oracle()) <= TOL["bf16"]


def test_peaked_scores_do_not_overflow():
    """Large score ranges: keys scaled so that scores span hundreds; the running maximum keeps every power
    of two in range."""
    c = wl.attention_case("peaked", "bf16", [700, 300, 40], [1, 2, 3], 4, 1, 128, 16, seed=wl.SEED ^ 5, kv_std=6.0)
    d = DeviceCase(c)
    out = to_f64(d.run())
    assert np.isfinite(out).all()
    assert maxnorm_rel(out, d.oracle()) <= TOL["bf16"]


def test_rows_of_one_sequence_see_exactly_their_causal_context():
    """A projected suffix: 40 consecutive rows of one sequence.  Changing the cached K/V of position j
    changes rows at positions >= j and leaves the rows before it bit-identical."""
    c = wl.attention_case("suffix", "bf16", [200, 90], [40, 1], 8, 2, 64, 16, seed=wl.SEED ^ 9)
    d = DeviceCase(c)
    base = raw_bits(d.run()).copy()
    assert maxnorm_rel(to_f64(d.out), d.oracle()) <= TOL["bf16"]
    j = 180                                             # row index 20 of the suffix (positions 160..199)
    slot = int(c.block_tables[0][j // 16]) * 16 + j % 16
    d.vc[slot] += 1.0
    d.kc[slot] *= -1.0
    after = raw_bits(d.run())
    rows_before = np.flatnonzero((c.token_seq_ids == 0) & (c.token_positions < j))
    rows_after = np.flatnonzero((c.token_seq_ids == 0) & (c.token_positions >= j))
    assert rows_before.size == 20 and rows_after.size == 20
    assert np.array_equal(after[rows_before], base[rows_before])
    assert all((after[r] != base[r]).any() for r in rows_after)
    other = np.flatnonzero(c.token_seq_ids == 1)
    assert np.array_equal(after[other], base[other])


def test_two_calls_give_the_same_bits_and_the_stream_argument_is_honoured():
    c = wl.attention_case("repeat", "bf16", _ragged_lens(3, 40, 900), [1] * 40, 32, 8, 128, 16, seed=wl.SEED ^ 21)
    d = DeviceCase(c)
    first = raw_bits(d.run()).copy()
    d.out.fill_(float("nan"))
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    ab.alora_paged_attention(d.q, d.kc, d.vc, d.bt, d.seq, d.pos, d.out, d.dims, stream=side)
    side.synchronize()
    assert np.array_equal(raw_bits(d.out), first)


def test_out_of_range_indices_are_reported_and_never_dereferenced():
    c = wl.attention_case("bad-indices", "bf16", [50, 60, 70], [1, 1, 1], 4, 2, 64, 16, seed=wl.SEED ^ 33)
    d = DeviceCase(c)
    good = to_f64(d.run()).copy()
    n_blocks = c.k_cache.shape[0] // 16
    # a sequence id outside the table, a negative position: rows of zeros
    seq = c.token_seq_ids.copy()
    seq[0] = 7
    pos = c.token_positions.copy()
    pos[1] = -3
    d.seq.copy_(torch.from_numpy(seq))
    d.pos.copy_(torch.from_numpy(pos))
    assert ab.alora_paged_attention_validate(d.bt, d.seq, d.pos, d.dims) == ab.ALORA_EDATA
    out = to_f64(d.run())
    assert (out[0] == 0).all() and (out[1] == 0).all()
    assert np.array_equal(out[2], good[2])
    # table entries outside the cache inside a context: those positions are left out of the softmax
    d.seq.copy_(torch.from_numpy(c.token_seq_ids))
    d.pos.copy_(torch.from_numpy(c.token_positions))
    bt = c.block_tables.copy()
    bt[2, 1] = n_blocks + 5          # positions 16..31 of sequence 2
    bt[2, 3] = -1                    # positions 48..63
    d.bt.copy_(torch.from_numpy(bt))
    assert ab.alora_paged_attention_validate(d.bt, d.seq, d.pos, d.dims) == ab.ALORA_EDATA
    out = to_f64(d.run())
    assert np.isfinite(out).all()
    keep = np.r_[0:16, 32:48, 64:70]
    kc, vc = wl.widen_f64(c.k_cache, "bf16"), wl.widen_f64(c.v_cache, "bf16")
    slots = oatt.context_slots(c.block_tables[2], 70, 16)[keep]
    dense_bt = np.arange((len(keep) + 15) // 16, dtype=np.int32)[None, :]
    kd = np.zeros((dense_bt.size * 16, kc.shape[1])); kd[:len(keep)] = kc[slots]
    vd = np.zeros((dense_bt.size * 16, vc.shape[1])); vd[:len(keep)] = vc[slots]
    ref = oatt.paged_attention(wl.widen_f64(c.q, "bf16")[2:3], kd, vd, dense_bt, np.zeros(1, np.int32),
                               np.asarray([len(keep) - 1], np.int32), 16, 4, 2, 64)
    assert maxnorm_rel(out[2:3], ref) <= TOL["bf16"]
    assert np.array_equal(out[:2], good[:2])


def test_empty_batch_is_a_no_op():
    c = wl.attention_case("empty", "bf16", [20], [1], 4, 2, 64, 16, seed=wl.SEED ^ 41)
    d = DeviceCase(c)
    dims = ab.make_attn_dims(d.q[:0], d.kc, d.bt, 4, 2, 64, 16)
    ab.alora_paged_attention(d.q[:0], d.kc, d.vc, d.bt, d.seq[:0], d.pos[:0], d.out[:0], dims)
    torch.cuda.synchronize()
    assert torch.isnan(d.out).all()


def test_decode_batch_at_benchmark_size_on_sampled_rows():
    """The reader's benchmark configuration (256 decode rows, 32 query / 8 K/V heads of 128, contexts up
    to 2048): every row finite, 24 sampled rows against the oracle."""
    rng = np.random.default_rng(8)
    lens = rng.integers(2, 2049, 256)
    c = wl.attention_case("decode-256", "bf16", lens, [1] * 256, 32, 8, 128, 16, seed=wl.SEED ^ 55)
    d = DeviceCase(c)
    out = to_f64(d.run())
    assert np.isfinite(out).all()
    rows = np.r_[np.argmax(lens), np.argmin(lens), rng.choice(256, 22, replace=False)]
    assert maxnorm_rel(out[rows], d.oracle(rows=rows)) <= TOL["bf16"]


@pytest.mark.parametrize("dtype,head_dim,group", [("bf16", 128, 4), ("f32", 64, 2), ("bf16", 64, 8), ("bf16", 128, 1)])
def test_split_contexts_match_the_oracle_and_the_single_pass(dtype, head_dim, group):
    """Few rows: every context is cut into up to 32 parts that a second kernel combines.  Ragged contexts
    (shorter than one part, exactly on part boundaries, thousands of positions), against the oracle and,
    to summation order, against the one-workgroup-per-row call; two calls give the same bits."""
    lens = [1, 3, 64, 65, 4096, 4097, 1000, 2048 * 3 + 17]
    c = wl.attention_case(f"split-{dtype}-{head_dim}-{group}", dtype, lens, [1, 2, 1, 1, 1, 3, 1, 1], 2 * group, 2, head_dim,
                          16, seed=wl.SEED ^ (77 + group))
    d = DeviceCase(c)
    nbytes = ab.alora_paged_attention_workspace_bytes(d.dims)
    assert nbytes > 0
    ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    ab.alora_paged_attention_split(d.q, d.kc, d.vc, d.bt, d.seq, d.pos, d.out, d.dims, ws)
    torch.cuda.synchronize()
    got = to_f64(d.out)
    bits = raw_bits(d.out).copy()
    assert np.isfinite(got).all()
    assert maxnorm_rel(got, d.oracle()) <= TOL[dtype]
    single = to_f64(d.run())
    assert maxnorm_rel(got, single) <= TOL[dtype]
    ws.fill_(0xFF)                                  # leftovers in the workspace do not matter
    d.out.fill_(float("nan"))
    ab.alora_paged_attention_split(d.q, d.kc, d.vc, d.bt, d.seq, d.pos, d.out, d.dims, ws)
    torch.cuda.synchronize()
    assert np.array_equal(raw_bits(d.out), bits)
    with pytest.raises(ab.AloraError):
        ab.alora_paged_attention_split(d.q, d.kc, d.vc, d.bt, d.seq, d.pos, d.out, d.dims, ws[: nbytes - 16])


def test_split_call_on_a_large_batch_is_the_single_pass():
    c = wl.attention_case("split-large", "bf16", _ragged_lens(4, 140, 300), [1] * 140, 32, 8, 128, 16, seed=wl.SEED ^ 23)
    d = DeviceCase(c)
    assert ab.alora_paged_attention_workspace_bytes(d.dims) == 0          # 140 rows x 8 K/V heads fill the chip
    first = raw_bits(d.run()).copy()
    d.out.fill_(float("nan"))
    ab.alora_paged_attention_split(d.q, d.kc, d.vc, d.bt, d.seq, d.pos, d.out, d.dims, None)
    torch.cuda.synchronize()
    assert np.array_equal(raw_bits(d.out), first)


def _run_suffix(d):
    d.out.fill_(float("nan"))
    ab.alora_paged_attention_suffix(d.q, d.kc, d.vc, d.bt, d.seq, d.pos, d.out, d.dims)
    torch.cuda.synchronize()
    return d.out


@pytest.mark.parametrize("group", [1, 2, 4, 8])
def test_suffix_rows_share_their_context_and_match_the_oracle(group):
    """Runs of consecutive rows (projected suffixes of 1..70 rows starting at arbitrary positions), single
    decode rows in between, contexts from 1 to thousands of positions, block sizes 16 and 5: every row
    against the oracle; uncovered slots hold NaN."""
    lens = [1, 40, 333, 64, 2500, 97, 1031]
    rows = [1, 40, 70, 1, 33, 5, 8]
    for bs in (16, 5):
        c = wl.attention_case(f"suffix-g{group}-bs{bs}", "bf16", lens, rows, 2 * group, 2, 128, bs, seed=wl.SEED ^ (300 + group))
        print(f"[case] {c.name} T={c.T}", flush=True)
        d = DeviceCase(c)
        out = to_f64(_run_suffix(d))
        assert np.isfinite(out).all()
        assert maxnorm_rel(out, d.oracle()) <= TOL["bf16"]


def test_suffix_call_on_a_decode_batch_and_on_interleaved_rows():
    """No two batch rows continue each other: every row is a block of its own."""
    rng = np.random.default_rng(5)
    lens = rng.integers(1, 700, 60)
    c = wl.attention_case("suffix-decode", "bf16", lens, [1] * 60, 32, 8, 128, 16, seed=wl.SEED ^ 61)
    d = DeviceCase(c)
    out = to_f64(_run_suffix(d))
    assert maxnorm_rel(out, d.oracle()) <= TOL["bf16"]
    # rows of two sequences interleaved (positions consecutive per sequence, but not in the batch)
    c2 = wl.attention_case("suffix-interleaved", "bf16", [300, 300], [16, 16], 8, 2, 128, 16, seed=wl.SEED ^ 62)
    order = np.arange(32).reshape(2, 16).T.reshape(-1)
    c2.q, c2.token_seq_ids, c2.token_positions = c2.q[order], c2.token_seq_ids[order], c2.token_positions[order]
    d2 = DeviceCase(c2)
    out2 = to_f64(_run_suffix(d2))
    assert maxnorm_rel(out2, d2.oracle()) <= TOL["bf16"]


def _mixed_batch(seed, n_q, n_kv, min_rows):
    """Decode rows and projected suffixes of 2..70 rows side by side, short contexts: at least min_rows rows."""
    rng = np.random.default_rng(seed)
    rows, lens = [], []
    while sum(rows) < min_rows:
        r = 1 if rng.random() < 0.6 else int(rng.integers(2, 71))
        rows.append(r)
        lens.append(r + int(rng.integers(0, 150)))
    return wl.attention_case(f"suffix-mixed-{n_q}-{n_kv}", "bf16", lens, rows, n_q, n_kv, 128, 16, seed=wl.SEED ^ seed)


@pytest.mark.parametrize("heads", [(8, 8), (32, 8)])
def test_suffix_call_on_a_batch_large_enough_for_whole_row_blocks_per_workgroup(heads):
    """More than 8192 rows x 8 K/V heads: a workgroup then owns 32 batch rows and works through every block
    that starts among them (decode rows: up to 32 blocks, runs: one or two), with the permuted range index
    where a block spans several ranges (group size 1: 128 rows).  Sampled rows against the oracle, all rows
    finite, and all rows equal to the per-row kernel's within the tolerance."""
    c = _mixed_batch(77 + heads[0], heads[0], heads[1], 8300)
    print(f"[case] {c.name} T={c.T}", flush=True)
    d = DeviceCase(c)
    out = to_f64(_run_suffix(d)).copy()
    assert np.isfinite(out).all()
    per_row = to_f64(d.run())
    assert maxnorm_rel(out, per_row) <= TOL["bf16"]
    rng = np.random.default_rng(5)
    rows = np.unique(np.concatenate([rng.integers(0, c.T, 400), np.arange(64), np.arange(c.T - 64, c.T)]))
    assert maxnorm_rel(out[rows], d.oracle(rows=rows)) <= TOL["bf16"]


def test_suffix_call_at_benchmark_size_on_sampled_rows():
    """The row-block reader's benchmark shape (4 sequences of 16384 positions, the last 2048 of each are query
    rows, 32 query / 8 K/V heads of 128, block size 16): every row finite, 40 sampled rows (first and last
    rows of runs and of row blocks among them) against the oracle; the window of table entries is refilled
    seven times per row block at this length."""
    c = wl.attention_case("suffix-4x16384", "bf16", [16384] * 4, [2048] * 4, 32, 8, 128, 16, seed=wl.SEED ^ 91)
    d = DeviceCase(c)
    out = to_f64(_run_suffix(d))
    assert np.isfinite(out).all()
    rng = np.random.default_rng(9)
    rows = np.unique(np.r_[0, 31, 32, 2047, 2048, 4095 + 33, c.T - 1, rng.choice(c.T, 33, replace=False)])
    assert maxnorm_rel(out[rows], d.oracle(rows=rows)) <= TOL["bf16"]


@pytest.mark.parametrize("group", [1, 4, 8])
def test_suffix_split_cuts_the_context_of_few_row_blocks_into_parts(group):
    """Short suffixes over long contexts (the shape of an aLoRA request): few row blocks, so every block's
    context is cut into parts that a second kernel combines.  Contexts shorter than one part, on part
    boundaries, across several table windows (more than 2048 positions per part); against the oracle, against
    the unsplit call (to summation order), and two calls give the same bits."""
    lens = [5000, 37, 2048 * 3 + 17, 64, 9000, 1]
    rows = [16, 5, 33, 1, 40, 1]
    c = wl.attention_case(f"suffix-split-g{group}", "bf16", lens, rows, 2 * group, 2, 128, 16, seed=wl.SEED ^ (500 + group))
    d = DeviceCase(c)
    nbytes = ab.alora_paged_attention_suffix_workspace_bytes(d.dims)
    assert nbytes > 0
    ws = torch.full((nbytes,), 0xff, dtype=torch.uint8, device="cuda")      # NaN patterns: every entry read is written first
    d.out.fill_(float("nan"))
    ab.alora_paged_attention_suffix_split(d.q, d.kc, d.vc, d.bt, d.seq, d.pos, d.out, d.dims, ws)
    torch.cuda.synchronize()
    got = to_f64(d.out)
    bits = raw_bits(d.out).copy()
    assert np.isfinite(got).all()
    assert maxnorm_rel(got, d.oracle()) <= TOL["bf16"]
    assert maxnorm_rel(got, to_f64(_run_suffix(d))) <= 2.0 ** -7
    d.out.fill_(float("nan"))
    ab.alora_paged_attention_suffix_split(d.q, d.kc, d.vc, d.bt, d.seq, d.pos, d.out, d.dims, ws)
    torch.cuda.synchronize()
    assert np.array_equal(raw_bits(d.out), bits)
    # too small a workspace is refused
    with pytest.raises(ab.AloraError) as e:
        ab.alora_paged_attention_suffix_split(d.q, d.kc, d.vc, d.bt, d.seq, d.pos, d.out, d.dims, ws[:nbytes // 2])
    assert e.value.status == ab.ALORA_EWORKSPACE


def test_suffix_split_on_a_large_batch_is_the_unsplit_call():
    c = _mixed_batch(91, 8, 8, 8300)
    d = DeviceCase(c)
    assert ab.alora_paged_attention_suffix_workspace_bytes(d.dims) == 0
    first = raw_bits(_run_suffix(d)).copy()
    d.out.fill_(float("nan"))
    ab.alora_paged_attention_suffix_split(d.q, d.kc, d.vc, d.bt, d.seq, d.pos, d.out, d.dims, None)
    torch.cuda.synchronize()
    assert np.array_equal(raw_bits(d.out), first)


@pytest.mark.parametrize("seed", range(10))
def test_suffix_calls_on_random_batches_agree_with_the_oracle_and_the_per_row_kernel(seed):
    """Random mixes of decode rows and runs, group sizes 1..8, block sizes that are powers of two, multiples of
    four that are not (12, 20, 24: divisions instead of shifts) and neither (6: served by the per-row kernel),
    contexts up to a few thousand positions; the unsplit and the split call."""
    rng = np.random.default_rng(1000 + seed)
    group = int(rng.choice([1, 2, 4, 8]))
    bs = [4, 12, 16, 20, 64, 24, 8, 6, 32, 128][seed]
    n_seq = int(rng.integers(1, 9))
    rows = [int(rng.choice([1, 1, int(rng.integers(2, 150))])) for _ in range(n_seq)]
    lens = [r + int(rng.integers(0, 2600)) for r in rows]
    c = wl.attention_case(f"suffix-random-{seed}", "bf16", lens, rows, 2 * group, 2, 128, bs, seed=wl.SEED ^ (900 + seed))
    print(f"[case] {c.name} G={group} bs={bs} rows={rows} lens={lens}", flush=True)
    d = DeviceCase(c)
    want = d.oracle()
    per_row = to_f64(d.run()).copy()
    assert maxnorm_rel(per_row, want) <= TOL["bf16"]
    got = to_f64(_run_suffix(d))
    assert np.isfinite(got).all() and maxnorm_rel(got, want) <= TOL["bf16"]
    ws = torch.full((max(ab.alora_paged_attention_suffix_workspace_bytes(d.dims), 16),), 0xff, dtype=torch.uint8, device="cuda")
    d.out.fill_(float("nan"))
    ab.alora_paged_attention_suffix_split(d.q, d.kc, d.vc, d.bt, d.seq, d.pos, d.out, d.dims, ws)
    torch.cuda.synchronize()
    got = to_f64(d.out)
    assert np.isfinite(got).all() and maxnorm_rel(got, want) <= TOL["bf16"]


def test_suffix_call_gives_the_same_bits_on_every_call():
    """The row-block kernel takes no timing-dependent decision: 200 calls on one batch (blocks that need no
    mask, diagonal blocks, single rows), every one bit-identical to the first."""
    c = wl.attention_case("suffix-repeat", "bf16", [200, 90, 700], [40, 1, 65], 8, 2, 128, 16, seed=wl.SEED ^ 9)
    d = DeviceCase(c)
    first = raw_bits(_run_suffix(d)).copy()
    assert maxnorm_rel(to_f64(d.out), d.oracle()) <= TOL["bf16"]
    for it in range(200):
        assert np.array_equal(raw_bits(_run_suffix(d)), first), it


def test_suffix_call_causal_boundaries_bad_indices_and_shapes():
    c = wl.attention_case("suffix-causal", "bf16", [200, 90], [40, 1], 8, 2, 128, 16, seed=wl.SEED ^ 9)
    d = DeviceCase(c)
    base = raw_bits(_run_suffix(d)).copy()
    assert maxnorm_rel(to_f64(d.out), d.oracle()) <= TOL["bf16"]
    j = 180
    slot = int(c.block_tables[0][j // 16]) * 16 + j % 16
    d.vc[slot] += 1.0
    d.kc[slot] *= -1.0
    after = raw_bits(_run_suffix(d))
    before_rows = np.flatnonzero((c.token_seq_ids == 0) & (c.token_positions < j))
    after_rows = np.flatnonzero((c.token_seq_ids == 0) & (c.token_positions >= j))
    assert np.array_equal(after[before_rows], base[before_rows])
    assert all((after[r] != base[r]).any() for r in after_rows)
    # a row with a bad sequence id gets zeros, its neighbours are unaffected
    seq = c.token_seq_ids.copy()
    seq[10] = 99
    d.seq.copy_(torch.from_numpy(seq))
    out = to_f64(_run_suffix(d))
    assert (out[10] == 0).all() and np.isfinite(out).all()
    # fp32 and head_dim 64 are not served by this entry point
    c3 = wl.attention_case("suffix-f32", "f32", [20], [2], 4, 2, 128, 16, seed=wl.SEED ^ 1)
    d3 = DeviceCase(c3)
    with pytest.raises(ab.AloraError):
        ab.alora_paged_attention_suffix(d3.q, d3.kc, d3.vc, d3.bt, d3.seq, d3.pos, d3.out, d3.dims)


# Long runs on workgroups of four wavefronts (blocks of 128 / G rows) that end one row past and one row before a block or a
# sequence's neighbour, on eight where the contexts are cut into parts.
# Bound: the reader's (softmax weights and outputs in bf16).
@pytest.mark.parametrize("group,n_kv,lens,parts", [(1, 64, [1000, 517, 531], False), (8, 16, [385, 1, 639], False), (4, 2, [700, 257, 95], False),
                                                   (2, 2, [129, 640, 127], False), (4, 2, [200, 65, 63], True), (8, 1, [1100, 33, 900], True)])
def test_suffix_rows_with_long_runs(group, n_kv, lens, parts):
    rows = [n - n // 7 for n in lens]
    c = wl.attention_case(f"long-runs-g{group}-{parts}", "bf16", lens, rows, group * n_kv, n_kv, 128, 16, seed=wl.SEED ^ (900 + group))
    print(f"[case] {c.name} T={c.T}", flush=True)
    d = DeviceCase(c)
    if parts:
        ws = torch.empty(max(16, ab.alora_paged_attention_suffix_workspace_bytes(d.dims)), dtype=torch.uint8, device="cuda")
        ab.alora_paged_attention_suffix_split(d.q, d.kc, d.vc, d.bt, d.seq, d.pos, d.out, d.dims, ws)
        torch.cuda.synchronize()
        out = to_f64(d.out)
    else:
        out = to_f64(_run_suffix(d))
    assert np.isfinite(out).all()
    pick = np.unique(np.r_[np.arange(0, c.T, 37), np.cumsum(rows) - 1, np.cumsum(rows)[:-1], [31, 32, 63, 64]])
    pick = pick[pick < c.T]
    assert maxnorm_rel(out[pick], d.oracle(rows=pick)) <= TOL["bf16"]


# Row blocks dealt to the workgroups of a range: decode rows beside a prompt chunk (every one leads a block), and rows of two
# sequences in no order, each a block of its own: many more than workgroups, so that one takes dozens, in two ranges.
# Bound: the reader's (softmax weights and outputs in bf16).
@pytest.mark.parametrize("parts", [False, True], ids=["whole", "parts"])
@pytest.mark.parametrize("kind,group,n_kv", [("chunk+decode", 4, 2), ("decode+chunk", 8, 1), ("shuffled", 2, 1), ("shuffled", 1, 2)])
def test_suffix_row_blocks_that_lie_unevenly(kind, group, n_kv, parts):
    lens, rows = {"chunk+decode": ([1100] + [200 + 9 * i for i in range(40)], [1030] + [1] * 40),
                  "decode+chunk": ([90 + 31 * i for i in range(70)] + [700], [1] * 70 + [650]), "shuffled": ([700, 620], [690, 610])}[kind]
    c = wl.attention_case(f"uneven-{kind}-g{group}", "bf16", lens, rows, group * n_kv, n_kv, 128, 16, seed=wl.SEED ^ (940 + group))
    if kind == "shuffled":
        order = np.random.default_rng(7).permutation(c.T)
        c.q, c.token_seq_ids, c.token_positions = c.q[order].copy(), c.token_seq_ids[order].copy(), c.token_positions[order].copy()
    print(f"[case] {c.name} T={c.T} parts={parts}", flush=True)
    d = DeviceCase(c)
    if parts:
        ws = torch.full((max(16, ab.alora_paged_attention_suffix_workspace_bytes(d.dims)),), 0xff, dtype=torch.uint8, device="cuda")
        d.out.fill_(float("nan"))
        ab.alora_paged_attention_suffix_split(d.q, d.kc, d.vc, d.bt, d.seq, d.pos, d.out, d.dims, ws)
        torch.cuda.synchronize()
        out = to_f64(d.out)
    else:
        out = to_f64(_run_suffix(d))
    assert np.isfinite(out).all()
    pick = np.unique(np.r_[np.arange(0, c.T, 29), np.arange(c.T - 45, c.T), np.arange(0, 75, 2)])
    assert maxnorm_rel(out[pick], d.oracle(rows=pick)) <= TOL["bf16"]


# Every instantiation of the row-block kernel (group size, four or eight wavefronts, block size a power of two or not) with whole
# contexts and with parts; that these sizes lead to them is checked where the launches are recorded.
# Bound: the reader's (softmax weights and outputs in bf16).
@pytest.mark.parametrize("group,n_kv,block_size,lens,rows,parts,waves", CUTS)
def test_suffix_every_cut(group, n_kv, block_size, lens, rows, parts, waves):
    c = wl.attention_case(f"cut-g{group}w{waves}", "bf16", lens, rows, group * n_kv, n_kv, 128, block_size, seed=wl.SEED ^ (980 + group + waves))
    print(f"[case] {c.name} T={c.T} rows={rows} parts={parts}", flush=True)
    d = DeviceCase(c)
    if parts:
        ws = torch.full((max(16, ab.alora_paged_attention_suffix_workspace_bytes(d.dims)),), 0xff, dtype=torch.uint8, device="cuda")
        ab.alora_paged_attention_suffix_split(d.q, d.kc, d.vc, d.bt, d.seq, d.pos, d.out, d.dims, ws)
        torch.cuda.synchronize()
        out = to_f64(d.out)
    else:
        out = to_f64(_run_suffix(d))
    assert np.isfinite(out).all()
    ends = np.cumsum(rows)
    pick = np.unique(np.r_[np.arange(0, c.T, 61), ends - 1, ends[:-1], [1, 31, 32, 63, 64, 127, 128, 255, 256]])
    pick = pick[pick < c.T]
    assert maxnorm_rel(out[pick], d.oracle(rows=pick)) <= TOL["bf16"]


# Parts whose number the kernel settles, with a row that is no row (zeros; it leads a block, whose place in the partial sums has to
# tell the number too).  The workspace holds NaN: a part's place that is read was written.  Bound: the reader's.
@pytest.mark.parametrize("group,n_kv,block_size,lens,rows,waves", COUNTED)
def test_suffix_split_with_counted_parts(group, n_kv, block_size, lens, rows, waves):
    c = wl.attention_case(f"counted-g{group}w{waves}", "bf16", lens, rows, group * n_kv, n_kv, 128, block_size, seed=wl.SEED ^ (1020 + group + waves))
    print(f"[case] {c.name} T={c.T} rows={rows}", flush=True)
    d = DeviceCase(c)
    nbytes = ab.alora_paged_attention_suffix_workspace_bytes(d.dims)
    want = d.oracle()
    for bad in (None, c.T - 1):
        if bad is not None:
            d.seq[bad] = -1
            want[bad] = 0.0
        ws = torch.full((nbytes,), 0xff, dtype=torch.uint8, device="cuda")
        d.out.fill_(float("nan"))
        ab.alora_paged_attention_suffix_split(d.q, d.kc, d.vc, d.bt, d.seq, d.pos, d.out, d.dims, ws)
        torch.cuda.synchronize()
        out = to_f64(d.out)
        assert np.isfinite(out).all() and maxnorm_rel(out, want) <= TOL["bf16"]
        if bad is not None:
            assert not out[bad].any()


# How many parts the kernel settles on: contexts that differ keep all of them, since a workgroup whose part is short takes another;
# alike and short, they go together.  A context in fewer parts than there is room for tells so in its last place.
@pytest.mark.parametrize("n_q,rows,lens,parts", [(8, 212, [7987, 9054, 2831], 11), (16, 219, [6775, 7681, 2401], 6), (32, 1, list(range(500, 2000, 47)), 2)])
def test_suffix_split_parts_of_unequal_contexts(n_q, rows, lens, parts):
    c = wl.attention_case(f"parts-{n_q}x{rows}", "bf16", lens, [rows] * len(lens), n_q, 8, 128, 16, seed=wl.SEED ^ (1040 + n_q))
    d = DeviceCase(c)
    ws = torch.zeros(ab.alora_paged_attention_suffix_workspace_bytes(d.dims), dtype=torch.uint8, device="cuda")
    ab.alora_paged_attention_suffix_split(d.q, d.kc, d.vc, d.bt, d.seq, d.pos, d.out, d.dims, ws)
    room = ws.numel() // (c.T * n_q * 130 * 4)
    last = ws.view(torch.float32).view(c.T, n_q, room, 130)[:, :, room - 1, :2]
    settled = torch.where(last[..., 1] < 0, last[..., 0], float(room)).unique().tolist()
    print(f"[case] {c.name} room for {room} settled {settled}", flush=True)
    assert settled == [parts]
    pick = np.arange(0, c.T, 37)
    assert maxnorm_rel(to_f64(d.out)[pick], d.oracle(rows=pick)) <= TOL["bf16"]


def test_what_the_bits_of_a_row_depend_on():
    """Whole contexts: its own sequence.  In parts also on the other sequences' positions, which settle how many parts there are (then
    equal within the reader's bound); the same call twice gives the same bits either way."""
    lens, rows = [7987, 9054, 2831], [212, 212, 212]
    c = wl.attention_case("bits", "bf16", lens, rows, 8, 8, 128, 16, seed=wl.SEED ^ 1060)
    d = DeviceCase(c)
    ws = torch.zeros(ab.alora_paged_attention_suffix_workspace_bytes(d.dims), dtype=torch.uint8, device="cuda")
    own = slice(424, 636)                # the rows of the third sequence

    def both():
        whole = raw_bits(_run_suffix(d)).copy()
        ws.fill_(0xff)
        ab.alora_paged_attention_suffix_split(d.q, d.kc, d.vc, d.bt, d.seq, d.pos, d.out, d.dims, ws)
        torch.cuda.synchronize()
        return whole, raw_bits(d.out).copy()

    whole, parts = both()
    again = both()
    assert np.array_equal(whole, again[0]) and np.array_equal(parts, again[1])
    d.pos[:424] -= 6000                  # the others' contexts are shorter now
    whole2, parts2 = both()
    assert np.array_equal(whole[own], whole2[own])
    want = oatt.paged_attention(wl.widen_f64(c.q, c.dtype), wl.widen_f64(c.k_cache, c.dtype), wl.widen_f64(c.v_cache, c.dtype), c.block_tables,
                                c.token_seq_ids, c.token_positions, c.block_size, 8, 8, 128, scale=None, rows=np.arange(424, 636, 9))
    for bits in (parts, parts2):
        assert maxnorm_rel(wl.widen_f64(bits[own][::9], "bf16"), want) <= TOL["bf16"]


# One row per sequence over a cache that does not stay in the memory-side cache: contexts are streamed, and where workgroups take
# several turns the longest go first: one run of rows and several, rows that are not valid, contexts all equal, all short but one, none long.
@pytest.mark.parametrize("n,lo,hi,odd", [(300, 1, 900, None), (65, 700, 700, None), (256, 5, 60, 1000), (257, 1, 1023, None), (100, 1, 500, None), (40, 1, 900, None)])
def test_rows_of_streamed_contexts(n, lo, hi, odd):
    print(f"[case] streamed {n} rows of {lo}-{hi}", flush=True)
    rng = np.random.default_rng(1080 + n)
    n_blocks, width = 1600, 64                       # 100 MiB of K and V
    g = torch.Generator(device="cuda").manual_seed(1080 + n)
    kc, vc = (torch.randn(n_blocks * 16, 8 * 128, device="cuda", generator=g).bfloat16() for _ in range(2))
    q = torch.randn(n, 32 * 128, device="cuda", generator=g).bfloat16()
    bt = rng.integers(0, n_blocks, (n, width)).astype(np.int32)      # (sequences share blocks)
    lens = rng.integers(lo, hi + 1, n)
    if odd:
        lens[n // 3] = odd
    seq, pos = rng.permutation(n).astype(np.int32), (lens - 1).astype(np.int32)
    bad = [7, 33]
    seq[bad[0]], pos[bad[1]] = -1, -5
    dbt, dseq, dpos = (torch.from_numpy(a).to("cuda") for a in (bt, seq, pos))
    out = torch.full_like(q, float("nan"))
    ab.alora_paged_attention(q, kc, vc, dbt, dseq, dpos, out, ab.make_attn_dims(q, kc, dbt, 32, 8, 128, 16))
    # more rows than sequences: ordinary loads in batch order, the same arithmetic
    twice = torch.full((2 * n, 32 * 128), float("nan"), device="cuda", dtype=torch.bfloat16)
    q2 = torch.cat([q, q])
    ab.alora_paged_attention(q2, kc, vc, dbt, torch.cat([dseq, dseq]), torch.cat([dpos, dpos]), twice, ab.make_attn_dims(q2, kc, dbt, 32, 8, 128, 16))
    torch.cuda.synchronize()
    assert np.array_equal(raw_bits(out), raw_bits(twice[:n])) and np.array_equal(raw_bits(out), raw_bits(twice[n:]))
    assert not out[bad].any()
    pick = np.array([t for t in range(0, n, 23) if t not in bad])
    want = oatt.paged_attention(to_f64(q), to_f64(kc), to_f64(vc), bt, seq, pos, 16, 32, 8, 128, rows=pick)
    assert maxnorm_rel(to_f64(out)[pick], want) <= TOL["bf16"]


# The same calls with every type, head size, group and kind of block size (test_launches.py: they reach every kernel for contexts read once).
@pytest.mark.parametrize("bs", [16, 24])
@pytest.mark.parametrize("group", [1, 2, 4, 8])
@pytest.mark.parametrize("dtype,d", [("bf16", 64), ("bf16", 128), ("f32", 64), ("f32", 128)])
def test_contexts_read_once_of_every_kind(dtype, d, group, bs):
    for (n, n_kv, room, parts), kind in ONCE.items():
        print(f"[case] once {dtype} d={d} g={group} bs={bs} n={n} room={room} parts={parts}", flush=True)
        rng = np.random.default_rng(1300 + n + group)
        slots = (104 << 20) // (n_kv * d * (4 if dtype == "bf16" else 8)) // bs * bs
        g = torch.Generator(device="cuda").manual_seed(1300 + n + group)
        t = torch.bfloat16 if dtype == "bf16" else torch.float32
        kc, vc = (torch.randn(slots, n_kv * d, device="cuda", generator=g).to(t) for _ in range(2))
        q = torch.randn(n, group * n_kv * d, device="cuda", generator=g).to(t)
        bt = rng.integers(0, slots // bs, (n, room // bs)).astype(np.int32)
        lens = rng.integers(1, room + 1, n)
        lens[:3] = 1, room, room // 2
        seq, pos = rng.permutation(n).astype(np.int32), (lens - 1).astype(np.int32)
        pos[4] = -2
        run, out = _read(q, kc, vc, bt, seq, pos, group * n_kv, n_kv, d, bs, parts)
        run()
        torch.cuda.synchronize()
        assert not out[4].any()
        if not parts:       # more rows than sequences: batch order and ordinary loads, the same arithmetic
            again, twice = _read(torch.cat([q, q]), kc, vc, bt, np.tile(seq, 2), np.tile(pos, 2), group * n_kv, n_kv, d, bs, False)
            again()
            torch.cuda.synchronize()
            assert np.array_equal(raw_bits(out), raw_bits(twice[:n])) and np.array_equal(raw_bits(out), raw_bits(twice[n:]))
        pick = np.array([0, 1, 2, 3, n - 1])
        want = oatt.paged_attention(to_f64(q), to_f64(kc), to_f64(vc), bt, seq, pos, bs, group * n_kv, n_kv, d, rows=pick)
        assert maxnorm_rel(to_f64(out)[pick], want) <= TOL[dtype]
        if parts:           # a workspace that holds the fewer parts
            few, out = _read(q, kc, vc, bt, seq, pos, group * n_kv, n_kv, d, bs, True, n * group * n_kv * min(32, -(-1024 // (n * n_kv))) * (d + 2) * 4)
            few()
            torch.cuda.synchronize()
            assert not out[4].any() and maxnorm_rel(to_f64(out)[pick], want) <= TOL[dtype]


# In parts, by rows: a context is cut into twice the parts where each has at least 512 positions (22 and 11 parts of 12 rows, 8 heads): just,
# just not, and contexts shorter than their parts; a row that is not valid.
def test_parts_of_long_and_short_contexts():
    rng = np.random.default_rng(1090)
    n_blocks, width = 1600, 800
    g = torch.Generator(device="cuda").manual_seed(1090)
    kc, vc = (torch.randn(n_blocks * 16, 8 * 128, device="cuda", generator=g).bfloat16() for _ in range(2))
    lens = np.array([22 * 512, 22 * 512 - 1, 12800, 1, 5, 64, 65, 700, 703, 704, 11, 12000])
    n = len(lens)
    q = torch.randn(n, 32 * 128, device="cuda", generator=g).bfloat16()
    bt = rng.integers(0, n_blocks, (n, width)).astype(np.int32)
    seq, pos = np.arange(n, dtype=np.int32), (lens - 1).astype(np.int32)
    seq[7] = n
    dbt, dseq, dpos = (torch.from_numpy(a).to("cuda") for a in (bt, seq, pos))
    dims = ab.make_attn_dims(q, kc, dbt, 32, 8, 128, 16)
    nbytes = ab.alora_paged_attention_workspace_bytes(dims)
    assert nbytes == n * 32 * 22 * 130 * 4
    out = torch.full_like(q, float("nan"))
    ws = torch.full((nbytes,), 0xff, dtype=torch.uint8, device="cuda")
    print("[case] parts of long and short contexts", flush=True)
    ab.alora_paged_attention_split(q, kc, vc, dbt, dseq, dpos, out, dims, ws)
    torch.cuda.synchronize()
    assert not out[7].any()
    pick = np.delete(np.arange(n), 7)
    want = oatt.paged_attention(to_f64(q), to_f64(kc), to_f64(vc), bt, seq, pos, 16, 32, 8, 128, rows=pick)
    assert maxnorm_rel(to_f64(out)[pick], want) <= TOL["bf16"]


# Few rows per sequence over a cache that does not stay in the memory-side cache: the row-block reader's copies are non-temporal, with eight and
# four wavefronts, in parts as planned and counted; the same bits as over a cache that does, and the oracle's values.
@pytest.mark.parametrize("group", [1, 2, 4, 8])
@pytest.mark.parametrize("n,rows,parts", [(3, 1, False), (70, 3, False), (2, 2, True), (40, 4, True)])
def test_row_blocks_of_streamed_contexts(group, n, rows, parts):
    rng = np.random.default_rng(1100 + group + n)
    n_blocks, small, width = 1600, 1400, 64
    g = torch.Generator(device="cuda").manual_seed(1100 + group + n)
    kc, vc = (torch.randn(n_blocks * 16, 8 * 128, device="cuda", generator=g).bfloat16() for _ in range(2))
    lens = rng.integers(rows, 16 * width + 1, n)
    seq = np.repeat(np.arange(n, dtype=np.int32), rows)
    pos = np.concatenate([np.arange(l - rows, l, dtype=np.int32) for l in lens])
    bt = rng.integers(0, small, (n, width)).astype(np.int32)
    q = torch.randn(n * rows, 8 * group * 128, device="cuda", generator=g).bfloat16()
    dbt, dseq, dpos = (torch.from_numpy(a).to("cuda") for a in (bt, seq, pos))
    outs = []
    for k, v in ((kc, vc), (kc[: small * 16], vc[: small * 16])):
        out = torch.full_like(q, float("nan"))
        dims = ab.make_attn_dims(q, k, dbt, 8 * group, 8, 128, 16)
        print(f"[case] streamed row blocks group={group} {n} x {rows} parts={parts} slots={k.shape[0]}", flush=True)
        if parts:
            ws = torch.full((ab.alora_paged_attention_suffix_workspace_bytes(dims),), 0xff, dtype=torch.uint8, device="cuda")
            ab.alora_paged_attention_suffix_split(q, k, v, dbt, dseq, dpos, out, dims, ws)
        else:
            ab.alora_paged_attention_suffix(q, k, v, dbt, dseq, dpos, out, dims)
        torch.cuda.synchronize()
        outs.append(out)
    assert np.array_equal(raw_bits(outs[0]), raw_bits(outs[1]))
    pick = np.arange(0, n * rows, 1 + n * rows // 12)
    want = oatt.paged_attention(to_f64(q), to_f64(kc), to_f64(vc), bt, seq, pos, 16, 8 * group, 8, 128, rows=pick)
    assert maxnorm_rel(to_f64(outs[0])[pick], want) <= TOL["bf16"]


def _shared_contexts(dtype, hq, hkv, d, bs, lens, groups, prefix, seed):
    """One row per sequence; rows of a group (-1: none) share the cache blocks of their first `prefix` positions.  Returns the same contexts twice: as they
    are, and copied to cache blocks of their own."""
    rng = np.random.default_rng(seed)
    g = torch.Generator(device="cuda").manual_seed(seed)
    nb, pb = -(-np.asarray(lens) // bs), prefix // bs
    table = np.full((len(lens), int(nb.max())), -1, np.int32)
    n_shared = pb * (max(groups) + 1)
    n_blocks = int(n_shared + sum(n - (pb if k >= 0 else 0) for n, k in zip(nb, groups)))
    perm, at = rng.permutation(n_blocks).astype(np.int32), n_shared
    for s, (n, k) in enumerate(zip(nb, groups)):
        own = 0
        if k >= 0:
            table[s, :pb] = perm[k * pb: (k + 1) * pb]
            own = pb
        table[s, own: n] = perm[at: at + n - own]
        at += n - own
    t = torch.bfloat16 if dtype == "bf16" else torch.float32
    pool = max(n_blocks, (104 << 20) // (2 * hkv * d * (2 if dtype == "bf16" else 4)) // bs)      # a cache that outgrows the memory-side one
    kc, vc = (torch.randn(pool * bs, hkv * d, device="cuda", generator=g).to(t) for _ in range(2))
    q = torch.randn(len(lens), hq * d, device="cuda", generator=g).to(t)
    ids = torch.from_numpy(np.concatenate([table[s, :n] for s, n in enumerate(nb)])).long().cuda()
    own_table = np.full_like(table, -1)
    first = np.concatenate([[0], np.cumsum(nb)])
    for s, n in enumerate(nb):
        own_table[s, :n] = first[s] + np.arange(n)
    spare = torch.zeros(max(0, pool - len(ids)) * bs, hkv * d, device="cuda", dtype=t)
    copies = [torch.cat([c.view(pool, bs, -1)[ids].reshape(-1, hkv * d), spare]) for c in (kc, vc)]
    seq, pos = np.arange(len(lens), dtype=np.int32), (np.asarray(lens) - 1).astype(np.int32)
    return q, (kc, vc, table), (*copies, own_table), seq, pos


def _read(q, kc, vc, table, seq, pos, hq, hkv, d, bs, parts, nbytes=None):
    """A call of the reader by rows, bound to its buffers: (the call, its output).  nbytes: the workspace's, else as many as the library asks for."""
    dt, ds, dp = (torch.from_numpy(a).to("cuda") for a in (table, seq, pos))
    out = torch.full_like(q, float("nan"))
    dims = ab.make_attn_dims(q, kc, dt, hq, hkv, d, bs)
    if not parts:
        return lambda: ab.alora_paged_attention(q, kc, vc, dt, ds, dp, out, dims), out
    ws = torch.full((nbytes or max(ab.alora_paged_attention_workspace_bytes(dims), 16),), 0xff, dtype=torch.uint8, device="cuda")
    return lambda: ab.alora_paged_attention_split(q, kc, vc, dt, ds, dp, out, dims, ws), out


# Rows whose contexts share cache blocks (ordinary loads for what is shared, streamed for what is not): the same bits as over copies of their own, and the
# oracle's values.  Groups of all rows, of a few, of some rows only, whole contexts and parts of which some are shared, just half and less.
@pytest.mark.parametrize("dtype,d,group,bs", [("bf16", 128, 1, 16), ("bf16", 128, 2, 24), ("bf16", 128, 4, 16), ("bf16", 64, 8, 16), ("f32", 64, 1, 16), ("f32", 128, 2, 20)])
@pytest.mark.parametrize("n,prefix,parts,of", [(200, 480, False, 200), (160, 480, False, 4), (130, 720, False, 2), (12, 12000, True, 12), (12, 7200, True, 3)])
def test_rows_that_share_contexts(dtype, d, group, bs, n, prefix, parts, of):
    rng = np.random.default_rng(1200 + n + group)
    hkv = 8 if parts else 4
    lens = prefix + rng.integers(1, 6000 if parts else 300, n)
    groups = [i // of if i % 7 else -1 for i in range(n)]
    print(f"[case] shared {dtype} d={d} g={group} bs={bs} n={n} prefix={prefix} parts={parts} of={of}", flush=True)
    q, shared, own, seq, pos = _shared_contexts(dtype, group * hkv, hkv, d, bs, lens, groups, prefix // bs * bs, 1200 + n)
    outs = []
    for kc, vc, table in (shared, own):
        run, out = _read(q, kc, vc, table, seq, pos, group * hkv, hkv, d, bs, parts)
        run()
        torch.cuda.synchronize()
        outs.append(out)
    assert np.array_equal(raw_bits(outs[0]), raw_bits(outs[1]))
    pick = np.arange(0, n, 1 + n // 6)
    want = oatt.paged_attention(to_f64(q), to_f64(shared[0]), to_f64(shared[1]), shared[2], seq, pos, bs, group * hkv, hkv, d, rows=pick)
    assert maxnorm_rel(to_f64(outs[0])[pick], want) <= TOL[dtype]


def _times(calls, rounds=7):
    """The least time of each call, us, measured in turn."""
    best = [float("inf")] * len(calls)
    a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
    for _ in range(rounds):
        for i, call in enumerate(calls):
            call()
            a.record()
            for _ in range(3):
                call()
            b.record()
            b.synchronize()
            best[i] = min(best[i], a.elapsed_time(b) * 1000 / 3)
    return best


def test_a_shared_context_is_not_streamed():
    """12 rows over one prefix of 16K positions, three layers' caches in turn: 97 us a layer, over copies of their own 139.  (Streamed as if each were read
    once: 126.)"""
    lens = 16384 + np.random.default_rng(1230).integers(100, 2000, 12)
    layers = [_shared_contexts("bf16", 8, 8, 128, 16, lens, [0] * 12, 16384, 1230 + i) for i in range(3)]
    calls = [[_read(q, *cache[i], seq, pos, 8, 8, 128, 16, True)[0] for q, *cache, seq, pos in layers] for i in (0, 1)]
    shared, own = _times([lambda c=c: [f() for f in c] for c in calls])
    print(f"[time] shared {shared / 3:.1f} us, copies {own / 3:.1f} us", flush=True)
    assert shared <= 0.82 * own


def test_rows_that_share_a_context_in_pairs_read_it_together():
    """200 rows, each two of the batch over one prefix of 1024 positions: 152 us, over copies of their own 184.  (The longest first, which takes pairs apart: 184.)"""
    lens = 1024 + np.random.default_rng(1240).integers(50, 600, 200)
    layers = [_shared_contexts("bf16", 8, 8, 128, 16, lens, [i // 2 for i in range(200)], 1024, 1240 + i) for i in range(3)]
    calls = [[_read(q, *cache[i], seq, pos, 8, 8, 128, 16, False)[0] for q, *cache, seq, pos in layers] for i in (0, 1)]
    shared, own = _times([lambda c=c: [f() for f in c] for c in calls])
    print(f"[time] pairs {shared / 3:.1f} us, copies {own / 3:.1f} us", flush=True)
    assert shared <= 0.9 * own


# Row blocks of which some contexts are read once (streamed) and others not: runs longer than a block beside single rows under a block table with room for
# more, neighbours over one prefix, parts half of which are shared.  The same bits as over copies of their own, and the oracle's values.
@pytest.mark.parametrize("group", [1, 2, 4, 8])
@pytest.mark.parametrize("rows,groups,table_rows,parts", [([300] + [1] * 40, [-1] * 41, 400, False), ([5] * 30, [0] * 30, 300, False), ([1, 7] * 20, [i // 4 for i in range(40)], 300, False),
                                                          ([130] + [1] * 20, [-1] * 21, 300, True), ([3] * 16, [0] * 16, 200, True), ([8, 1] * 8, [i // 2 if i % 5 else -1 for i in range(16)], 100, True)])
def test_row_blocks_that_share_contexts(group, rows, groups, table_rows, parts):
    prefix = 1600
    lens = prefix + np.random.default_rng(1250 + group).integers(320, 1200, len(rows))
    q, shared, own, _, _ = _shared_contexts("bf16", group * 8, 8, 128, 16, lens, groups, prefix, 1250 + group)
    seq = np.repeat(np.arange(len(rows), dtype=np.int32), rows)
    pos = np.concatenate([np.arange(l - r, l, dtype=np.int32) for l, r in zip(lens, rows)])
    g = torch.Generator(device="cuda").manual_seed(1260)
    q = torch.randn(len(seq), group * 8 * 128, device="cuda", generator=g).bfloat16()
    dseq, dpos = (torch.from_numpy(a).to("cuda") for a in (seq, pos))
    print(f"[case] row blocks sharing group={group} {len(rows)} runs parts={parts}", flush=True)
    outs = []
    for kc, vc, table in (shared, own):
        bt = np.full((table_rows, table.shape[1]), -1, np.int32)
        bt[: len(table)] = table
        dbt, out = torch.from_numpy(bt).to("cuda"), torch.full_like(q, float("nan"))
        dims = ab.make_attn_dims(q, kc, dbt, group * 8, 8, 128, 16)
        assert len(seq) * group <= 32 * table_rows       # (the kernel that streams)
        if parts:
            ws = torch.full((ab.alora_paged_attention_suffix_workspace_bytes(dims),), 0xff, dtype=torch.uint8, device="cuda")
            ab.alora_paged_attention_suffix_split(q, kc, vc, dbt, dseq, dpos, out, dims, ws)
        else:
            ab.alora_paged_attention_suffix(q, kc, vc, dbt, dseq, dpos, out, dims)
        torch.cuda.synchronize()
        outs.append(out)
    assert np.array_equal(raw_bits(outs[0]), raw_bits(outs[1]))
    pick = np.arange(0, len(seq), 1 + len(seq) // 10)
    want = oatt.paged_attention(to_f64(q), to_f64(shared[0]), to_f64(shared[1]), shared[2], seq, pos, 16, group * 8, 8, 128, rows=pick)
    assert maxnorm_rel(to_f64(outs[0])[pick], want) <= TOL["bf16"]


def test_fp32_contexts_are_not_streamed():
    """16 rows at 500 to 1500 positions in fp32, 147 MB a layer, take the time of the same rows and one without a sequence, more rows than sequences, which are not
    taken to read their contexts once: 58 us.  (With non-temporal loads 73.)"""
    lens = np.random.default_rng(1270).integers(500, 1500, 16)
    calls = [[], []]
    for i in range(4):
        q, cache, _, seq, pos = _shared_contexts("f32", 8, 8, 128, 16, lens, [-1] * 16, 0, 1270 + i)
        calls[0].append(_read(q, *cache, seq, pos, 8, 8, 128, 16, False)[0])
        calls[1].append(_read(torch.cat([q, q[:1]]), *cache, np.append(seq, np.int32(-1)), np.append(pos, np.int32(0)), 8, 8, 128, 16, False)[0])
    once, more = _times([lambda c=c: [f() for f in c] for c in calls])
    print(f"[time] fp32 {once / 4:.1f} us, a row more {more / 4:.1f} us", flush=True)
    assert once <= 1.12 * more
