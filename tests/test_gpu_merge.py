"""Parity of mdx_merge with the oracle.

mdx_merge partitions both tables, splits every partition into LDS-sized
sub-buckets and joins each sub-bucket in LDS; when a build sub-bucket is too
large for LDS (heavily repeated keys) the device switches to the global-table
join.  Both routes are compared with the oracle here, plus the 1E8 x 1E8
workload in the launch configuration the benchmark times, checked through
properties that hold at any size."""

import numpy as np
import pytest

import oracle
from tests.gpu_util import (announce, assert_join_equals_oracle, dev, host, require_gpu,
                            run_merge)
from tests.helpers import fmix64_np, part_np
from workloads import config_inputs, edge_tables, match_fraction_tables, uniform_tables, zipf_tables

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


def test_merge_plain_workload():
    announce("merge plain")
    kl, vl, kr, vr = config_inputs("plain")
    got = run_merge(kl, vl, kr, vr, 4)
    assert_join_equals_oracle(kl, vl, kr, vr, 4, got)


@pytest.mark.parametrize("scale", [0.02, 0.05])
def test_merge_paper_shape_reduced(scale):
    """The 1E8 workload's generator at 2E6 and 5E6 rows per side, P = 32
    (both split passes active)."""
    announce(f"merge paper x{scale}")
    kl, vl, kr, vr = config_inputs("paper", scale=scale)
    got = run_merge(kl, vl, kr, vr, 32)
    assert_join_equals_oracle(kl, vl, kr, vr, 32, got)


@pytest.mark.parametrize("P", [1, 3, 7, 64, 257, 4096])
def test_merge_partition_counts(P):
    announce(f"merge P={P}")
    kl, vl, kr, vr = match_fraction_tables(400_000, 300_001, 0.3, seed=P)
    got = run_merge(kl, vl, kr, vr, P)
    assert_join_equals_oracle(kl, vl, kr, vr, P, got)


@pytest.mark.parametrize("dtype", [np.int64, np.int32])
def test_merge_repeated_keys_radix(dtype):
    """Repeated keys whose sub-buckets still fit LDS: chains hold equal keys."""
    announce(f"merge repeated keys {np.dtype(dtype).name}")
    kl, vl, kr, vr = uniform_tables(200_000, 150_000, 60_000, seed=6, key_dtype=dtype)
    total = oracle.join(kl, vl, kr, vr, materialize=False)["total"]
    got = run_merge(kl, vl, kr, vr, 8, cap=total)
    assert_join_equals_oracle(kl, vl, kr, vr, 8, got)


@pytest.mark.parametrize("nl,nr,frac,P,dtype", [
    (3_000, 200_000, 0.5, 2, np.int64),   # small build side, large probe side
    (6_000, 8_000, 1.0, 1, np.int64),     # one sub-bucket, every probe row matches
    (6_000, 8_000, 1.0, 1, np.int32),
    (6_000, 6_400, 1.0, 1, np.int64),
])
def test_merge_join_routes(nl, nr, frac, P, dtype):
    """Uneven sides and sub-buckets where every probe row matches, against
    the oracle."""
    announce(f"merge routes {nl}x{nr} f={frac} P={P} {np.dtype(dtype).name}")
    kl, vl, kr, vr = match_fraction_tables(nl, nr, frac, seed=nl + nr, key_dtype=dtype)
    total = oracle.join(kl, vl, kr, vr, materialize=False)["total"]
    got = run_merge(kl, vl, kr, vr, P, cap=total)
    assert got["status"] == 0
    assert_join_equals_oracle(kl, vl, kr, vr, P, got)


def test_merge_probe_sub_bucket_spans_batches():
    """One probe key repeated 20000 times: its sub-bucket holds more probe
    rows than one 8192-row batch, so the join counts and then writes it
    batch by batch (sub-buckets are sized by the larger side, so only a
    repeated probe key gets there)."""
    announce("merge probe key x 20000")
    rng = np.random.default_rng(21)
    kl = rng.permutation(50_000).astype(np.int64)
    kr = np.concatenate([np.full(20_000, 777, np.int64), rng.integers(0, 100_000, 30_000)])
    kr = kr[rng.permutation(kr.size)]
    vl, vr = np.arange(kl.size, dtype=np.int64), np.arange(kr.size, dtype=np.int64)
    total = oracle.join(kl, vl, kr, vr, materialize=False)["total"]
    for P in (1, 4):
        got = run_merge(kl, vl, kr, vr, P, cap=total)
        assert got["status"] == 0
        assert_join_equals_oracle(kl, vl, kr, vr, P, got)


def test_merge_some_sub_buckets_repeat_keys():
    """20 build keys appear twice among 300000 distinct ones: only the
    sub-buckets holding them have probe rows with two matches."""
    announce("merge mixed routes")
    rng = np.random.default_rng(12)
    base = rng.permutation(300_000).astype(np.int64)
    kl = np.concatenate([base, base[rng.integers(0, base.size, 20)]])
    kl = kl[rng.permutation(kl.size)]
    kr = np.concatenate([base[rng.integers(0, base.size, 90_000)],
                         rng.integers(300_000, 600_000, 210_000)])
    kr = kr[rng.permutation(kr.size)]
    vl, vr = np.arange(kl.size, dtype=np.int64), np.arange(kr.size, dtype=np.int64)
    total = oracle.join(kl, vl, kr, vr, materialize=False)["total"]
    got = run_merge(kl, vl, kr, vr, 8, cap=total)
    assert got["status"] == 0
    assert_join_equals_oracle(kl, vl, kr, vr, 8, got)


def test_merge_int32_keys():
    announce("merge int32")
    kl, vl, kr, vr = match_fraction_tables(300_000, 250_000, 0.3, seed=4, key_dtype=np.int32)
    got = run_merge(kl, vl, kr, vr, 8)
    assert_join_equals_oracle(kl, vl, kr, vr, 8, got)


def test_merge_fallback_for_oversized_sub_bucket():
    """20000 build rows of one key: one sub-bucket exceeds the LDS table, so
    the device must take the global-table join."""
    announce("merge fallback (one key x 20000)")
    rng = np.random.default_rng(1)
    kl = np.concatenate([np.full(20_000, 5, np.int64), rng.integers(10, 10_000, 30_000)])
    kr = np.concatenate([np.full(50, 5, np.int64), rng.integers(10, 10_000, 20_000)])
    kl, kr = kl[rng.permutation(kl.size)], kr[rng.permutation(kr.size)]
    vl, vr = np.arange(kl.size, dtype=np.int64), np.arange(kr.size, dtype=np.int64)
    total = oracle.join(kl, vl, kr, vr, materialize=False)["total"]
    got = run_merge(kl, vl, kr, vr, 4, cap=total)
    assert_join_equals_oracle(kl, vl, kr, vr, 4, got)


@pytest.mark.parametrize("b", [3455, 3456, 3457, 3840, 3841])
@pytest.mark.parametrize("P", [1, 4])
def test_merge_one_key_at_table_size(b, P):
    """A build side of one key repeated b times, so one sub-bucket of b rows:
    at most 3456 (a merge's LDS table, and then the build side fits one
    table, so the global-table kernels are not even launched) it is joined
    in LDS, beyond it the device takes the global-table join.  The probe
    side has 3 matching rows and 500 misses."""
    announce(f"merge one key x {b}, P={P}")
    rng = np.random.default_rng(b + P)
    kl = np.full(b, 7, np.int64)
    kr = np.concatenate([np.full(3, 7, np.int64), rng.integers(100, 300, 500)])
    kr = kr[rng.permutation(kr.size)]
    vl, vr = np.arange(kl.size, dtype=np.int64), np.arange(kr.size, dtype=np.int64)
    total = oracle.join(kl, vl, kr, vr, materialize=False)["total"]
    got = run_merge(kl, vl, kr, vr, P, cap=total)
    assert_join_equals_oracle(kl, vl, kr, vr, P, got)


def test_merge_skewed_reduced():
    announce("merge zipf reduced")
    kl, vl, kr, vr = zipf_tables(15_000, 15_000, 1.1, 10_000, seed=0)
    total = oracle.join(kl, vl, kr, vr, materialize=False)["total"]
    got = run_merge(kl, vl, kr, vr, 16, cap=total)
    assert_join_equals_oracle(kl, vl, kr, vr, 16, got)


@pytest.mark.parametrize("name", ["empty_left", "empty_right", "both_empty", "all_equal", "extremes",
                                  "int32_negative", "int32_extremes"])
def test_merge_edge_tables(name):
    announce(f"merge edge {name}")
    kl, vl, kr, vr, _ = edge_tables(name)
    total = oracle.join(kl, vl, kr, vr, materialize=False)["total"]
    for P in [1, 5, 32]:
        got = run_merge(kl, vl, kr, vr, P, cap=max(total, 1))
        assert_join_equals_oracle(kl, vl, kr, vr, P, got)


def test_merge_capacity_overflow():
    announce("merge capacity overflow")
    import paper_2101_08878_amd as mdx
    kl, vl, kr, vr = match_fraction_tables(100_000, 100_000, 0.5, seed=2)
    got = run_merge(kl, vl, kr, vr, 8, cap=10_000)
    assert got["off"][-1] == 50_000
    assert got["status"] & mdx.MDX_DEV_OUTPUT_OVERFLOW


def assert_paper_merge(kl, kr, P, got):
    """Left keys are a permutation of [0, n), so a right row matches iff its
    key is below n, and then exactly once: the output must be exactly the
    right rows with key < n, each paired with the unique left row holding
    its key (payload = row index), and partition p's block must hold exactly
    the output keys with destination p.  This fixes the output up to the
    order of rows inside a partition."""
    n = kl.size
    assert got["status"] == 0
    off = got["off"]
    total = int(off[-1])
    key, lp, rp = got["key"][:total], got["lpay"][:total], got["rpay"][:total]
    # every output row is a genuine match
    assert np.array_equal(kl[lp], key)
    assert np.array_equal(kr[rp], key)
    # completeness and no duplicates: the right payloads are exactly the hits
    hits = np.flatnonzero(kr < n)
    assert hits.size == total
    assert np.array_equal(np.sort(rp), hits)
    # partition blocks
    dest = np.repeat(np.arange(P), np.diff(off))
    assert np.array_equal(part_np(key, P), dest)
    return total


@pytest.mark.parametrize("P", [1, 2, 3])
def test_merge_placement_by_partition(P):
    """1.3E7 x 1.3E7 (the 1E8 workload's generator): at P = 1 and 2 a
    partition holds 8192 or 4096 sub-buckets, at least 8 per workgroup of the
    join, so its output rows are placed by partition cursor and a chained scan
    over partitions; at P = 3 (2048) by the chained scan over sub-buckets."""
    announce(f"merge placement P={P}")
    kl, vl, kr, vr = config_inputs("paper", scale=0.13)
    got = run_merge(kl, vl, kr, vr, P)
    assert assert_paper_merge(kl, kr, P, got) == round(0.3 * kl.size)


@pytest.mark.parametrize("P", [32, 1])
def test_merge_paper_scale_properties(P):
    """1E8 x 1E8, P = 32 (what the benchmark times) and P = 1 (its secondary
    figure, output placed by partition cursor): |J| = 3E7, checked row by
    row as in assert_paper_merge."""
    announce(f"merge paper scale 1e8 P={P}")
    n = 100_000_000
    kl, vl, kr, vr = config_inputs("paper")
    got = run_merge(kl, vl, kr, vr, P, cap=n)
    assert assert_paper_merge(kl, kr, P, got) == 30_000_000


@pytest.mark.parametrize("hot", [4095, 4096, 4097, 8192, 8193, 40_961])
def test_merge_hot_probe_key_items(hot):
    """A probe key repeated around multiples of a probe batch (4096 rows): its
    sub-bucket is one join item up to a batch and one per batch beyond it.  A
    second hot key, absent from the build side, makes items without output."""
    announce(f"merge hot probe key x {hot}")
    rng = np.random.default_rng(hot)
    kl = rng.permutation(60_000).astype(np.int64)
    kr = np.concatenate([np.full(hot, 31, np.int64), np.full(9000, 70_000, np.int64),
                         rng.integers(0, 120_000, 30_000)])
    kr = kr[rng.permutation(kr.size)]
    vl, vr = np.arange(kl.size, dtype=np.int64), np.arange(kr.size, dtype=np.int64)
    total = oracle.join(kl, vl, kr, vr, materialize=False)["total"]
    for P in (1, 5):
        got = run_merge(kl, vl, kr, vr, P, cap=total)
        assert got["status"] == 0
        assert_join_equals_oracle(kl, vl, kr, vr, P, got)


@pytest.mark.parametrize("P", [1, 3])
def test_merge_hot_probe_key_many_sub_buckets(P):
    """The item list over more sub-buckets than one workgroup plans (8192 at
    P = 1, rows placed by partition; 6144 at P = 3, by sub-bucket), with a
    tenth of the probe rows on one key."""
    announce(f"merge hot probe key, many sub-buckets, P={P}")
    kl, vl, kr, vr = config_inputs("paper", scale=0.13)
    kr = kr.copy()
    kr[np.random.default_rng(P).integers(0, kr.size, kr.size // 10)] = 12_345
    got = run_merge(kl, vl, kr, vr, P)
    assert_paper_merge(kl, kr, P, got)


def test_merge_batch_chunked_hot_items():
    """A lane merge whose one sub-bucket has more build rows than a table and
    more probe rows than a batch: chunks and items together."""
    announce("lanes: hot build and probe key")
    import torch

    import paper_2101_08878_amd as mdx
    rng = np.random.default_rng(3)
    kl = np.concatenate([np.full(3600, 5, np.int64), rng.integers(10, 40_000, 20_000)])
    kr = np.concatenate([np.full(4200, 5, np.int64), rng.integers(10, 40_000, 10_000)])
    kl, kr = kl[rng.permutation(kl.size)], kr[rng.permutation(kr.size)]
    vl, vr = np.arange(kl.size, dtype=np.int64), np.arange(kr.size, dtype=np.int64)
    total = oracle.join(kl, vl, kr, vr, materialize=False)["total"]
    status = torch.zeros(1, dtype=torch.int32, device="cuda")
    job = mdx.MergeJob(dev(kl), dev(vl), dev(kr), dev(vr), 4, total, status=status)
    mdx.mdx_merge_batch([job], lanes=1)
    torch.cuda.synchronize()
    got = dict(key=host(job.out[0]), lpay=host(job.out[1]), rpay=host(job.out[2]),
               off=host(job.out_offsets), status=int(status.item()), cap=total)
    assert_join_equals_oracle(kl, vl, kr, vr, 4, got)


@pytest.mark.parametrize("n", [1_590_000, 1_600_000])
@pytest.mark.parametrize("dtype", [np.int64, np.int32])
def test_merge_one_and_two_passes(n, dtype):
    """512 sub-buckets (split by the first pass alone) and 1024 (two passes)."""
    announce(f"merge passes {n} {np.dtype(dtype).name}")
    kl, vl, kr, vr = match_fraction_tables(n, n // 2, 0.3, seed=n, key_dtype=dtype)
    got = run_merge(kl, vl, kr, vr, 1)
    assert_join_equals_oracle(kl, vl, kr, vr, 1, got)


@pytest.mark.parametrize("n,hot,P", [
    (3457, 3457, 1),           # smallest merge that launches it, one key
    (20_000, 5_000, 7),
    (140_000, 9_000, 300),     # a sampled build; more partitions than workgroups
    (1_000_000, 60_000, 8),
    (2_097_152 - 50_000, 4_000, 3),  # the most rows one launch takes
    (2_097_153 - 50_000, 4_000, 3),  # several launches
])
@pytest.mark.parametrize("dtype", [np.int64, np.int32])
def test_merge_global_join_launches(n, hot, P, dtype):
    """The global-table join as one launch and as several: one build key
    repeated `hot` times (more than an LDS table's rows), the other build keys
    twice each, 50000 probe rows, the hot key among them 5 times.  Run
    twice: the second call finds the first one's workspace contents."""
    announce(f"global-table join {n} rows, hot key x {hot}, P={P} {np.dtype(dtype).name}")
    import torch

    import paper_2101_08878_amd as mdx
    rng = np.random.default_rng(n + P)
    kl = np.concatenate([np.full(hot, -7), np.repeat(np.arange((n - hot + 1) // 2), 2)[:n - hot]])
    kl = kl[rng.permutation(n)].astype(dtype)
    kr = np.concatenate([np.full(5, -7), rng.integers(0, max(n, 2), 49_995)])
    kr = kr[rng.permutation(kr.size)].astype(dtype)
    vl, vr = np.arange(n, dtype=np.int64), np.arange(kr.size, dtype=np.int64)
    total = oracle.join(kl, vl, kr, vr, materialize=False)["total"]
    kt = mdx.MDX_KEY_I64 if dtype == np.int64 else mdx.MDX_KEY_I32
    ws = torch.full((mdx.mdx_merge_workspace_bytes(n, kr.size, P, kt),), 0xa5, dtype=torch.uint8,
                    device="cuda")
    status = torch.zeros(1, dtype=torch.int32, device="cuda")
    ins = [dev(a) for a in (kl, vl, kr, vr)]
    for _ in range(2):
        ok, ol, orr, off = mdx.mdx_merge(*ins, P, out_capacity=total, workspace=ws, status=status)
        torch.cuda.synchronize()
        got = dict(key=host(ok), lpay=host(ol), rpay=host(orr), off=host(off),
                   status=int(status.item()), cap=total)
        assert_join_equals_oracle(kl, vl, kr, vr, P, got)


def test_merge_count_beyond_2_to_40_rows():
    """Output offsets stay exact where one partition's rows, placed by cursor
    (P = 1), pass 2^40: one build key 3456 times (a full LDS table) against the
    same key in 3.182E8 of the probe rows and a key that is absent in 1000 more.
    No output is written (out_capacity 0)."""
    announce("merge of 1.1E12 output rows, counted only")
    import torch

    import paper_2101_08878_amd as mdx
    b, m = 3456, 318_200_000
    assert b * m > 1 << 40
    kl = torch.full((b,), 7, dtype=torch.int32, device="cuda")
    vl = torch.arange(b, dtype=torch.int64, device="cuda")
    kr = torch.full((m + 1000,), 7, dtype=torch.int32, device="cuda")
    kr[::318_000][:1000] = 9
    vr = torch.zeros(kr.numel(), dtype=torch.int64, device="cuda")
    status = torch.zeros(1, dtype=torch.int32, device="cuda")
    *_, off = mdx.mdx_merge(kl, vl, kr, vr, 1, out_capacity=0, status=status)
    torch.cuda.synchronize()
    assert host(off).tolist() == [0, b * m]
    assert int(status.item()) == mdx.MDX_DEV_OUTPUT_OVERFLOW


@pytest.mark.parametrize("nl,nr,P,bits", [
    (100_000, 50_000, 1, 6),         # split in one pass, as two would split it
    (1_500_000, 1_000_000, 8, 4),    # in one pass into 512: the probe rows split again
    (1_200_000, 1_200_000, 200, 0),  # likewise, a P that is no power of two
    (2_000_000, 1_500_000, 3, 5),    # in two passes, and one launch per step
])
@pytest.mark.parametrize("dtype", [np.int64, np.int32])
def test_merge_global_join_order(nl, nr, P, bits, dtype):
    """The global-table join's rows follow the probe rows by partition, then the
    top `bits` bits of the hash that a split into at most 128 has, then input
    order, whichever way the merge was split; more than 2^21 rows among them.
    A build key repeated 5000 times sends the merge there."""
    announce(f"global-table join order {nl}x{nr} P={P} {np.dtype(dtype).name}")
    rng = np.random.default_rng(nl + P)
    kl = np.concatenate([np.full(5000, -7), rng.permutation(nl - 5000)]).astype(dtype)
    kr = np.concatenate([np.full(3, -7), rng.integers(0, 2 * nl, nr - 3)]).astype(dtype)
    kl, kr = kl[rng.permutation(nl)], kr[rng.permutation(nr)]
    vl, vr = np.arange(nl, dtype=np.int64), np.arange(nr, dtype=np.int64)
    total = oracle.join(kl, vl, kr, vr, materialize=False)["total"]
    got = run_merge(kl, vl, kr, vr, P, cap=total)
    assert_join_equals_oracle(kl, vl, kr, vr, P, got)
    h = fmix64_np(kr)
    top = (h >> np.uint64(64 - bits)).astype(np.int64) if bits else np.zeros(nr, np.int64)
    order = np.lexsort((vr, top, part_np(kr, P)))
    matches = np.where(kr == -7, 5000, kr < nl - 5000)
    assert np.array_equal(got["rpay"][:total], np.repeat(vr[order], matches[order]))


@pytest.mark.parametrize("n,one", [(100_000, True), (2_200_000, False)])
def test_merge_global_join_is_traced(n, one):
    """mdx_trace_kernel brackets a merge's global-table join, as one kernel or as
    its steps, once each."""
    announce(f"traced global-table join, {n} rows")
    import torch

    import paper_2101_08878_amd as mdx
    names = ["tbl_init", "tbl_insert", "grp_count", "probe_chain", "probe_expand"]
    kl = np.concatenate([np.full(4000, -7), np.arange(n - 4000)])
    kr = np.arange(-10, 1000)
    traces = {k: mdx.KernelTrace(k, 4) for k in names + ["global_join"]}
    try:
        for t in traces.values():
            t.start()
        got = run_merge(kl, kl, kr, kr, 3, cap=10_000)
        mdx.KernelTrace.stop_all()
        assert got["off"][-1] == 4000 + 1000
        assert {k: t.launches() for k, t in traces.items()} == \
            {**dict.fromkeys(names, 0 if one else 1), "global_join": 1 if one else 0}
        assert all(d > 0 for t in traces.values() for d in t.durations_ms())
    finally:
        mdx.KernelTrace.stop_all()
        for t in traces.values():
            t.close()
