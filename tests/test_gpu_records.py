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
    (2, 1, [40 * 256], 512),                  # 20 rows per sequence, 2 ranges each: past the LDS rows
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
