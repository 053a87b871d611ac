"""GPU tests of the persistent unit schedule (launches with several splits).

Which work-group computes a unit, and in which order, must never change a
result: every case is compared with the fp64 oracle, and runs that take the
units in different orders (longest-first plan, plain sequence order above the
plan's batch limit, other batch compositions) must agree bit for bit.
"""
import numpy as np
import pytest
import torch

from paper_2512_22492_amd import binding as B
from paper_2512_22492_amd import workloads

from gpu_util import bf16_to_f64, check_close, decode_extra, device, oracle_ref, run_gpu

pytestmark = pytest.mark.gpu

# batches up to this size take the longest-first plan (it lives in LDS)
PLAN_BATCH_LIMIT = 4096


def problem(hq, hkv, lengths, seed, kv="bf16", layout="hnd", max_pages=None):
    return workloads.make_problem(
        "schedule", batch=len(lengths), num_q_heads=hq, num_kv_heads=hkv,
        lengths=list(lengths), kv_dtype=kv, seed=seed, layout=layout,
        max_pages=max_pages).to(device())


def sub_problem(p, rows):
    """The same sequences (same pages, same pool) as a smaller batch."""
    idx = torch.as_tensor(rows, device=p.q.device)
    return workloads.DecodeProblem(**{**p.__dict__, "batch": len(rows),
                                      "q": p.q[idx].contiguous(),
                                      "block_table": p.block_table[idx].contiguous(),
                                      "seq_lens": p.seq_lens[idx].contiguous()})


def short_lengths(n, seed, hi=300):
    rng = np.random.default_rng(seed)
    L = rng.integers(0, hi + 1, n)
    L[rng.random(n) < 0.05] = 0
    return [int(x) for x in L]


@pytest.mark.parametrize("flags", [0, B.RL_DA_CHECKED])
@pytest.mark.parametrize("batch", [PLAN_BATCH_LIMIT, PLAN_BATCH_LIMIT + 4])
@pytest.mark.parametrize("hq,hkv", [(8, 2), (16, 2)])
def test_large_batches_with_and_without_the_plan(batch, hq, hkv, flags):
    """At the plan's batch limit the plan is largest; one past it the units
    run in sequence order.  Both match the oracle, and a sub-batch (always
    planned) gives the same bits for its sequences."""
    print("case batch", batch, "hq", hq, "hkv", hkv, "flags", flags, flush=True)
    p = problem(hq, hkv, short_lengths(batch, seed=batch + hq), seed=batch + hq)
    got = run_gpu(p, split_tokens=64, flags=flags)
    print(check_close(bf16_to_f64(got), oracle_ref(p), "batch %d G=%d" % (batch, hq // hkv),
                      extra_abs=decode_extra(p, flags)))
    rows = list(range(0, batch, 7))
    part = run_gpu(sub_problem(p, rows), split_tokens=64, flags=flags)
    assert torch.equal(part.view(torch.int16), got[rows].view(torch.int16))


@pytest.mark.parametrize("kv,layout", [("bf16", "hnd"), ("fp8_e4m3", "hnd"), ("bf16", "nhd")])
def test_checked_mode_on_the_persistent_schedule(kv, layout):
    """A checked handle on a launch with many units (longest-first plan): a
    block-table entry out of range and a sequence longer than its table row
    are reported without a fault, and every other sequence's output keeps its
    bits."""
    lengths = [1000 + 37 * (i % 11) for i in range(300)]
    p = problem(8, 2, lengths, seed=71, kv=kv, layout=layout)
    with B.DecodeAttention.for_problem(p, flags=B.RL_DA_CHECKED, split_tokens=64) as attn:
        assert attn.unit_heads() == 1 and attn.split_info(p.max_pages)[1] > 1
        good = run_gpu(p, attn=attn)
        assert attn.check_error() == 0
        print(check_close(bf16_to_f64(good), oracle_ref(p), "checked persistent " + kv + layout,
                          extra_abs=decode_extra(p, B.RL_DA_CHECKED)))
        others = [b for b in range(len(lengths)) if b not in (5, 123)]
        bad_table = p.block_table.clone()
        bad_table[123, 7] = p.num_pages + 5        # inside sequence 123
        q = workloads.DecodeProblem(**{**p.__dict__, "block_table": bad_table})
        got = run_gpu(q, attn=attn)
        assert attn.check_error() & B.RL_DA_DEVERR_PAGE_OUT_OF_RANGE
        assert torch.equal(got[others].view(torch.int16), good[others].view(torch.int16))
        long_lens = p.seq_lens.clone()
        long_lens[5] = p.max_pages * 16 + 1        # longer than its table row
        q = workloads.DecodeProblem(**{**p.__dict__, "seq_lens": long_lens})
        got = run_gpu(q, attn=attn)
        assert attn.check_error() & B.RL_DA_DEVERR_LENGTH_TOO_LONG
        assert torch.equal(got[others].view(torch.int16), good[others].view(torch.int16))


@pytest.mark.parametrize("kv,layout,flags", [
    ("bf16", "hnd", 0), ("bf16", "hnd", B.RL_DA_SCORES_ON_VALU), ("fp8_e4m3", "hnd", 0),
    ("bf16", "nhd", 0), ("fp8_e4m3", "nhd", 0), ("bf16", "nhd", B.RL_DA_PER_HEAD_UNITS)])
def test_degenerate_length_mixes(kv, layout, flags):
    """All sequences empty (only the zero writes run), one long sequence among
    empty ones, one sequence alone, one token each.  Each mix runs as it is
    (few units: one work-group per unit) and padded with empty sequences to
    500 (many units: the longest-first plan); the padded run's rows for the
    original sequences are the same bits."""
    cases = {
        "all_empty": [0] * 37,
        "one_long": [0] * 20 + [5000] + [0] * 20,
        "alone": [4097],
        "one_token_each": [1] * 300,
    }
    for name, lengths in cases.items():
        print("case", kv, layout, flags, name, flush=True)
        # a table at least 64 pages wide: several 16-page splits per row
        width = max(64, max((L + 15) // 16 for L in lengths))
        padded = lengths + [0] * (500 - len(lengths))
        p = problem(8, 2, padded, seed=len(lengths), kv=kv, layout=layout, max_pages=width)
        assert p.max_pages > 16
        # one handle for both runs: the unit family (token-major pools) follows
        # the handle's capacity, and results are batch-invariant for a handle
        with B.DecodeAttention.for_problem(p, flags=flags, split_tokens=256) as attn:
            got_padded = run_gpu(p, attn=attn)
            got = run_gpu(sub_problem(p, list(range(len(lengths)))), attn=attn)
        assert torch.equal(got.view(torch.int16), got_padded[:len(lengths)].view(torch.int16))
        got = bf16_to_f64(got)
        assert np.all(bf16_to_f64(got_padded)[len(lengths):] == 0)
        if max(lengths) == 0:
            assert np.all(got == 0)
            continue
        sub = sub_problem(p, list(range(len(lengths))))
        print(check_close(got, oracle_ref(sub), name, extra_abs=decode_extra(sub, flags)))
        assert np.all(got[np.array(lengths) == 0] == 0)


def test_queue_is_reset_between_launches_of_any_shape():
    """One handle alternates persistent launches of different sizes with
    one-split launches; each result equals a fresh handle's."""
    long_tail = problem(8, 2, [4000, 17, 0, 2500, 900, 33, 1, 3000] * 8, seed=21)
    few = problem(8, 2, [1500, 0, 700], seed=22)
    one_split = problem(8, 2, [200, 90, 250, 3, 0, 16], seed=23)
    max_pages = max(x.max_pages for x in (long_tail, few, one_split))
    runs = [(long_tail, 256), (few, 256), (one_split, 256), (long_tail, 512), (few, 64)]
    fresh = [run_gpu(p, split_tokens=s) for p, s in runs]
    for p, s in runs:
        print(check_close(bf16_to_f64(run_gpu(p, split_tokens=s)), oracle_ref(p), "queue",
                          extra_abs=decode_extra(p, 0)))
    handles = {s: B.DecodeAttention(8, 2, 64, max_pages, split_tokens=s) for s in (64, 256, 512)}
    try:
        for rep in range(3):
            for (p, s), want in zip(runs, fresh):
                got = run_gpu(p, attn=handles[s])
                assert torch.equal(got.view(torch.int16), want.view(torch.int16)), (rep, s)
    finally:
        for h in handles.values():
            h.close()


@pytest.mark.parametrize("kv,layout", [("bf16", "hnd"), ("fp8_e4m3", "nhd")])
@pytest.mark.parametrize("max_batch,lengths", [
    # 2 kv heads: splits of about 512 tokens (16 at most)
    (32, [0, 1, 511, 512, 513, 1025, 4095, 4096, 4097, 8191, 32768, 16, 0, 3000]),
    # 400 pairs: not cut by length
    (200, [4096, 4097, 2049, 6145, 0, 20000, 32768, 7, 20480, 20481]),
])
def test_default_splits_follow_the_sequence_length(max_batch, lengths, kv, layout):
    """Handles with the default split size cut a sequence by its own length.
    Every length at the edges of the rule against the oracle; a sequence's bits
    alone, in a table just wide enough for it, are those of the whole batch."""
    p = problem(8, 2, lengths, seed=101 + max_batch, kv=kv, layout=layout, max_pages=2048)
    with B.DecodeAttention(8, 2, max_batch, 4096, kv_dtype=kv, layout=layout,
                           flags=B.RL_DA_PER_HEAD_UNITS) as attn:
        assert attn.unit_heads() == 1 and attn.split_info(4096) == (4096, 16)
        got = run_gpu(p, attn=attn)
        for b in (len(lengths) - 1, 4, 1):
            one = sub_problem(p, [b])
            one.block_table = one.block_table[:, :max(1, (lengths[b] + 15) // 16)].contiguous()
            assert torch.equal(run_gpu(one, attn=attn).view(torch.int16),
                               got[b:b + 1].view(torch.int16)), b
    print(check_close(bf16_to_f64(got), oracle_ref(p), "by length %d %s" % (max_batch, kv),
                      extra_abs=decode_extra(p, 0)))
    assert np.all(bf16_to_f64(got)[np.array(lengths) == 0] == 0)


@pytest.mark.parametrize("hq,hkv,max_batch", [(8, 2, 65), (32, 2, 33), (4, 1, 300)])
def test_handles_of_many_pairs_keep_whole_splits(hq, hkv, max_batch):
    """Handles of more than 128 (sequence, kv head) pairs, 64 with 16 heads a group,
    divide a sequence as an explicit 4096-token split does, bit for bit."""
    p = problem(hq, hkv, [4097, 0, 30000, 6000, 20481, 12], seed=141 + hq, max_pages=2048)
    with B.DecodeAttention(hq, hkv, max_batch, 4096) as attn, \
            B.DecodeAttention(hq, hkv, max_batch, 4096, split_tokens=4096) as whole:
        got, want = run_gpu(p, attn=attn), run_gpu(p, attn=whole)
    assert torch.equal(got.view(torch.int16), want.view(torch.int16))


def ragged(n, top, seed):
    rng = np.random.default_rng(seed)
    L = np.exp(rng.uniform(0, np.log(top), n)).astype(int)
    L[::9] = 0
    return [int(x) for x in L]


@pytest.mark.parametrize("flags", [0, B.RL_DA_CHECKED])
@pytest.mark.parametrize("hq,hkv,kv,layout", [(8, 2, "bf16", "hnd"), (32, 2, "fp8_e4m3", "hnd"),
                                              (2, 2, "fp8_e4m3", "nhd")])
@pytest.mark.parametrize("max_batch,top,seen", [
    # 64 pairs: up to 32 splits
    (32, 40000, 2500),
    # 128 pairs: more units than the chip holds, splits of 512 to 4096 tokens
    (64, 40000, 2500),
    # 512 pairs: not cut by length
    (256, 24000, 1500),
    # 128 pairs in a table of one default split: a work-group per unit
    (64, 4096, 256),
])
def test_splits_by_length_of_many_sequences(max_batch, top, seen, hq, hkv, kv, layout, flags):
    """Launches that the queue plans, by length (entries of full and last splits by
    class; up to 64 pairs with 16 heads a group) and not, and the static grid of
    a table of one default split, against the oracle; sequences alone, in a
    table as wide as the handle's, give the same bits."""
    lengths = ragged(max_batch, min(top, 4096), seed=max_batch + top)
    lengths[3], lengths[5], lengths[-1] = top, top - 17, min(4097, top)
    lengths[6], lengths[7], lengths[8] = top // 2, top - 3000, top // 3
    print("case", max_batch, top, hq, kv, layout, flags, flush=True)
    p = problem(hq, hkv, lengths, seed=111 + top, kv=kv, layout=layout, max_pages=seen)
    with B.DecodeAttention(hq, hkv, max_batch, 4096, kv_dtype=kv, layout=layout,
                           flags=flags | B.RL_DA_PER_HEAD_UNITS) as attn:
        assert attn.unit_heads() == 1 and attn.split_info(4096) == (4096, 16)
        got = run_gpu(p, attn=attn)
        for rows in ([3], [5, 1], list(range(0, max_batch, 7))):
            sub = sub_problem(p, rows)
            wide = torch.zeros((len(rows), 4096), dtype=torch.int32, device=device())
            wide[:, :seen] = sub.block_table
            sub.block_table = wide
            assert torch.equal(run_gpu(sub, attn=attn).view(torch.int16),
                               got[rows].view(torch.int16)), rows
        if flags & B.RL_DA_CHECKED:
            assert attn.check_error() == 0
    print(check_close(bf16_to_f64(got), oracle_ref(p), "by length, many",
                      extra_abs=decode_extra(p, flags)))
    assert np.all(bf16_to_f64(got)[np.array(lengths) == 0] == 0)


@pytest.mark.parametrize("splits", [1, 2])
def test_merge_of_many_rows(splits):
    """Batches whose merge takes up to eight heads of a sequence a work-group, of
    one split each and of two or three, among them empty sequences."""
    rng = np.random.default_rng(splits)
    lengths = [int(x) for x in rng.integers(0, 100 if splits == 1 else 190, 513)]
    lengths[0], lengths[-1] = 0, 129
    p = problem(32, 2, lengths, seed=121 + splits, max_pages=12)
    got = run_gpu(p, split_tokens=64 if splits == 2 else 128)
    print(check_close(bf16_to_f64(got), oracle_ref(p), "merge rows", extra_abs=decode_extra(p, 0)))
    assert np.all(bf16_to_f64(got)[np.array(lengths) == 0] == 0)
    rows = [1, 300, 512]
    part = run_gpu(sub_problem(p, rows), split_tokens=64 if splits == 2 else 128)
    assert torch.equal(part.view(torch.int16), got[rows].view(torch.int16))
