"""The records of split units and the rows of a merge, at the edges of the
waves and blocks that reduce them: against the oracle or a float64 reference,
and a fused step, whose merge combines the records itself, bit for bit against
its three calls."""
import numpy as np
import pytest

from kf_testlib import compare_all, host, run_gpu, run_oracle
from kf_workloads import make_instance, workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hq,hkv,lens,part", [
    (4, 1, [20000], 1 << 20),                 # 79 ranges: more records than lanes
    (5, 1, [16 * 16 * 64 + 1], 1 << 20),      # 65 pages past 64 ranges of 16
    (8, 2, [4096, 300, 0, 17], 2048),         # whole, split and empty routes in one launch
    (2, 1, [40 * 256], 512),                  # 20 rows of one sequence, 2 ranges each: a combine launch
    (16, 1, [300] * 3, 1 << 20),              # 16 heads, 2 ranges
])
def test_split_units_fused_equals_calls_and_oracle(gpu, hq, hkv, lens, part):
    wl = workload("llama8b_32k", num_seqs=len(lens), num_q_heads=hq, num_kv_heads=hkv,
                  part_tokens=part)
    for broken in (False, True):
        inst = make_instance(wl, seed=11, steps=1, seq_lens=lens)
        if broken:   # an inverted CSR row: its routes' partials are still written
            inst.seq_route_begin[0] = inst.seq_route_begin[1] + 1
        o = run_oracle(inst, 1)
        g, f = host(run_gpu(inst, 1)), host(run_gpu(inst, 1, fused=True))
        compare_all(g, o)
        for k in g:
            if g[k] is not None:
                assert np.array_equal(np.asarray(g[k]), np.asarray(f[k]), equal_nan=True), k


def _regroup(inst, n, orphans=0):
    """Sequence 0 takes the first n rows and the n - 1 sequences whose rows they
    were are left without any; the last `orphans` rows are in no CSR row."""
    inst.routes[:n, 0] = 0
    b = inst.seq_route_begin
    b[1:n] = n
    np.minimum(b, len(inst.routes) - orphans, out=b)
    inst.tail_route[:n] = -1
    inst.tail_route[0] = n - 1
    if orphans:
        inst.tail_route[-orphans:] = -1


@pytest.mark.parametrize("hq,hkv,fp8,lens,places", [
    # equal routes: 3 ranges each, some whole or empty
    (16, 1, False, [600] * 36 + [0, 5, 600, 590], 3),       # four waves per head
    (32, 2, False, [600] * 66 + [0, 5, 600, 590], 3),       # one wave per head
    # one KV head, few long routes: more ranges per row than a group of lanes
    (2, 1, False, [6000] * 18, 24),
    # spans: rows cut by workgroups beside whole ones
    (32, 8, False, [30, 900, 0, 2500, 17] * 8, 0),          # four waves
    (64, 8, False, [30, 900, 0, 2500, 17] * 8, 0),          # one wave
    (64, 8, True, [30, 1900, 0, 4500, 17] * 7, 0),
    (8, 2, False, [64000, 3, 40000] + [20] * 20, 0),        # rows of up to 200 records
])
@pytest.mark.parametrize("n,orphans", [(1, 6), (2, 0), (4, 6), (5, 0), (16, 6), (17, 0), (17, 6)])
def test_sequence_of_many_rows_combined_in_the_merge(gpu, hq, hkv, fp8, lens, places, n, orphans):
    """A sequence of n rows (up to four per group of rows, up to and past those
    kept in LDS) beside sequences of one row and of none, and rows with tokens
    that no sequence lists.  The merge of these fused steps (as many rows as
    sequences) combines the records itself: the bits of the three calls."""
    n = min(n, len(lens) - 1)
    wl = workload("llama8b_32k", num_seqs=len(lens), num_q_heads=hq, num_kv_heads=hkv,
                  part_tokens=1 << 20, permuted=True, kv_dtype="fp8" if fp8 else "bf16")
    inst = make_instance(wl, seed=12, steps=1, seq_lens=lens)
    assert len(inst.routes) == len(lens)
    _regroup(inst, n, orphans)
    from paper_2606_29207_amd import kf
    from paper_2606_29207_amd.step import DecodeState
    st = DecodeState.from_instance(inst)
    plan = kf.partial_attn_plan(st.shape, len(inst.routes), st.max_pages_per_route)
    assert places == 0 or plan[1] == places, plan
    del st
    o = run_oracle(inst, 1)
    g, f = host(run_gpu(inst, 1)), host(run_gpu(inst, 1, fused=True))
    compare_all(f, o)
    for k in g:
        if g[k] is not None:
            assert np.array_equal(np.asarray(g[k]), np.asarray(f[k]), equal_nan=True), k


@pytest.mark.parametrize("n", [1, 3, 4, 5, 8, 31, 32, 33, 63, 64, 65, 255, 256, 257, 600])
@pytest.mark.parametrize("seqs", [1, 40])
def test_merge_fan_in_edges(gpu, n, seqs):
    """Rows per sequence at the edges of a wave's and a workgroup's blocks of
    weights; 39 one-row sequences beside it bring the mean below the
    four-wave merge's threshold.  float32 sums of n rows: 1e-6 relative."""
    import torch
    from paper_2606_29207_amd import kf
    gen = torch.Generator(device="cuda").manual_seed(n)
    counts = [n] + [1] * (seqs - 1)
    begin = torch.tensor(np.concatenate([[0], np.cumsum(counts)]), dtype=torch.int32, device="cuda")
    R = sum(counts)
    o = torch.randn((R, 5, 128), generator=gen, device="cuda")
    l = 3.0 * torch.randn((R, 5), generator=gen, device="cuda")
    if n > 3:
        l[1, 2] = float("-inf")     # an empty route
        o[1, 2] = 0.0
    out, lse = torch.empty((seqs, 5, 128), device="cuda"), torch.empty((seqs, 5), device="cuda")
    err = torch.zeros(1, dtype=torch.int32, device="cuda")
    kf.merge_partials(seqs, o, l, begin, out, lse, err)
    ld, od = l.double(), o.double()
    for b in range(seqs):
        r0, r1 = int(begin[b]), int(begin[b + 1])
        t = torch.logsumexp(ld[r0:r1], 0)
        ref = (torch.exp(ld[r0:r1] - t)[:, :, None] * od[r0:r1]).sum(0)
        assert (lse[b] - t).abs().max() <= 4e-6
        assert (out[b] - ref).norm() <= 1e-6 * ref.norm()
