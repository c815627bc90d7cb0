"""Span launches: a ragged batch's tiles, route after route, cut into equal
wave columns.  Each case is checked against the oracle and against the same
batch launched over an identity route list, which keeps the chunk plan, and
as a fused step bit for bit against its three calls and against the step that
uses the library's scratch array."""
import numpy as np
import pytest

from kf_testlib import compare_all, host, run_gpu, run_oracle
from kf_workloads import make_instance, workload

pytestmark = pytest.mark.gpu

# (q heads, KV heads, fp8, lengths, route length); lengths reach two tiles per
# wave: pages * KV heads >= 8192 (bf16, 2-page tiles) or 16384 (fp8, 4-page)
_RAGGED = [
    # ends at, before and past pages and tiles, one-token and empty sequences
    (32, 8, False, [1, 16, 17, 31, 32, 33, 48, 0, 2048, 5000, 7777, 1, 0, 1500], 65536),
    # one long route cut over most columns beside short ones
    (8, 2, False, [65000, 5, 900, 1, 33], 65536),
    # more routes than workgroup columns (record places by column), 16 KV heads
    (16, 16, False, [int(x) for x in np.random.default_rng(3).integers(1, 700, 60)], 65536),
    # 16 query heads per KV head, several routes per sequence
    (64, 4, False, [9000, 17000, 2100, 6001, 40], 4096),
    # one KV head and a group of 3
    (3, 1, False, [100000, 50000, 1000, 7], 65536),
    # fp8, groups of 8 and 1, tiles of 4 pages
    (64, 8, True, [3, 16, 4096, 64, 65, 12000, 63, 0, 18001, 33], 65536),
    (4, 4, True, [40000, 29000, 128, 8000, 1], 65536),
]


def _instance(case, steps, seed=5):
    hq, hkv, fp8, lens, part = case
    wl = workload("llama8b_32k", num_seqs=len(lens), num_q_heads=hq, num_kv_heads=hkv,
                  part_tokens=part, kv_dtype="fp8" if fp8 else "bf16", permuted=True)
    return make_instance(wl, seed=seed, steps=steps, seq_lens=lens)


def _is_span(inst):
    from paper_2606_29207_amd import kf
    s = kf.make_shape(inst.wl.num_seqs, inst.wl.num_q_heads, inst.wl.num_kv_heads,
                      kf.KV_BF16 if inst.k_scale is None else kf.KV_FP8_E4M3, inst.num_pages,
                      len(inst.page_ids), inst.scale)
    return kf.partial_attn_spans(s, len(inst.routes), inst.max_pages_per_route) > 0


@pytest.mark.parametrize("case", _RAGGED, ids=lambda c: f"{c[0]}q{c[1]}kv{'fp8' if c[2] else ''}")
def test_span_launch_matches_oracle_and_chunk_plan(gpu, case):
    import torch
    from paper_2606_29207_amd import kf
    inst = _instance(case, steps=2)
    assert _is_span(inst)
    o = run_oracle(inst, 2)
    st = run_gpu(inst, 2)
    g = host(st)
    compare_all(g, o)
    fused = host(run_gpu(inst, 2, fused=True))
    for k in g:
        if g[k] is None:
            continue
        assert np.array_equal(np.asarray(g[k]), np.asarray(fused[k]), equal_nan=True), k
    # the chunk plan on the same state: other sums, the same values to float32
    # rounding (a few hundred 2^-24 steps over sums of up to 65536 terms)
    o_part, lse_part = st.o_part.clone(), st.lse_part.clone()
    ident = torch.arange(len(inst.routes), dtype=torch.int32, device=st.device)
    kf.partial_attn(st.shape, st.q, st.k_pool, st.v_pool, st.routes, st.max_pages_per_route,
                    st.page_ids, st.o_part, st.lse_part, st.workspace, st.err_flags,
                    k_scale=st.k_scale, v_scale=st.v_scale, route_list=ident)
    torch.cuda.synchronize()
    err = (o_part - st.o_part).norm() / st.o_part.norm()
    assert err <= 2e-5, float(err)
    both = torch.isfinite(lse_part)
    assert torch.equal(both, torch.isfinite(st.lse_part))
    assert (lse_part[both] - st.lse_part[both]).abs().max() <= 2e-5


@pytest.mark.parametrize("case,bound", [
    # multi-head, columns of many short routes; long columns of one route
    ((32, 32, False, [65 + 23 * i for i in range(40)], 65536), 1.0),
    ((64, 4, False, [40000, 30000, 20000, 500, 12000], 65536), 1.0),
    # fp8: nearly all of the error is that of the split of p, the same in both
    ((16, 2, True, [60000, 45000, 31000, 700], 65536), 1.01),
], ids=["mha", "gqa16", "fp8"])
def test_span_error_is_no_larger_than_the_chunk_plans(gpu, case, bound):
    """A span wave sums runs several times as long as a chunk wave's in
    float32; the partials stay no further from float64 than the chunk plan's."""
    import torch
    from paper_2606_29207_amd import kf
    inst = _instance(case, steps=1, seed=9)
    assert _is_span(inst)
    o = run_oracle(inst, 1)
    st = run_gpu(inst, 1)
    ref = torch.from_numpy(o["o_part"]).to(st.device)
    ident = torch.arange(len(inst.routes), dtype=torch.int32, device=st.device)
    err = [float((st.o_part.double() - ref).norm() / ref.norm())]
    kf.partial_attn(st.shape, st.q, st.k_pool, st.v_pool, st.routes, st.max_pages_per_route,
                    st.page_ids, st.o_part, st.lse_part, st.workspace, st.err_flags,
                    k_scale=st.k_scale, v_scale=st.v_scale, route_list=ident)
    err.append(float((st.o_part.double() - ref).norm() / ref.norm()))
    print(f"[spans] error {err[0]:.3e}, chunk plan {err[1]:.3e}", flush=True)
    assert err[0] <= bound * err[1], err


def test_span_step_without_a_workspace_is_the_same(gpu):
    import torch
    from paper_2606_29207_amd.step import DecodeState
    inst = _instance(_RAGGED[0], steps=1, seed=6)
    a, b = DecodeState.from_instance(inst), DecodeState.from_instance(inst)
    tok = a.upload_new_tokens(*inst.new_tokens(0))
    a.step_fused(*tok)
    b.step_no_alloc(*tok)
    torch.cuda.synchronize()
    for n in ("o_part", "lse_part", "out", "lse", "routes", "k_pool", "v_pool"):
        x, y = getattr(a, n), getattr(b, n)   # bits: unused slots are NaN
        bits = torch.int16 if x.element_size() == 2 else torch.int32
        assert torch.equal(x.view(bits), y.view(bits)), n


def test_span_launch_with_bad_rows_and_pages(gpu):
    """A row of a wrong sequence, one that needs more pages than the launch
    allows, a page id outside the pool in the middle of a cut route, an
    inverted CSR row: NaN and flags as the oracle has them, other rows whole."""
    inst = _instance(_RAGGED[0], steps=1, seed=7)
    assert _is_span(inst)
    inst.routes[2, 0] = 99                     # no such sequence
    inst.routes[4, 3] = inst.routes[4, 2] - 3  # ends before it begins
    inst.page_ids[inst.routes[10, 4] + 150] = inst.num_pages + 5
    inst.seq_route_begin[9] = inst.seq_route_begin[8] - 1
    o = run_oracle(inst, 1)
    for fused in (False, True):
        g = host(run_gpu(inst, 1, fused=fused))
        compare_all(g, o)


@pytest.mark.parametrize("fp8", [False, True])
def test_span_launch_skips_runs_of_empty_routes(gpu, fp8):
    """More than a wave of empty routes before, between and behind those with
    tokens, as in a table of fixed size: waves step over them to their next
    tile and to their next token.  Two of the empty ones are tails and take a
    token (the first and the last row of a run), one is a bad row's."""
    lens = [0] * 70 + [14000 if fp8 else 7000, 17] + [0] * 130 + [33, 18000 if fp8 else 8500] + [0] * 66
    inst = _instance((64, 8, fp8, lens, 65536) if fp8 else (32, 8, fp8, lens, 65536), steps=2, seed=8)
    assert len(inst.routes) == len(lens) and _is_span(inst)
    tail = np.where(np.asarray(lens) > 0, inst.tail_route, -1)
    for b in (0, 201, 205, 269):
        tail[b] = inst.tail_route[b]
    inst.routes[205, 4] = len(inst.page_ids) + 3   # no such page list: bad, takes no token
    o = run_oracle(inst, 2, tail_route=tail)
    for fused in (False, True):
        compare_all(host(run_gpu(inst, 2, tail_route=tail, fused=fused)), o)
