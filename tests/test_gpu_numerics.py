"""Numerical corner cases of dora_decode_attn through the C ABI, against the
fp64 oracle and closed forms: a caller-set softmax scale, scores large enough
that all but a few weights underflow, a zero query (every weight equal, so
the output is the plain mean of the values), and the geometry's limits (a
very long sequence, the widest KV-head count, the largest block-table
stride)."""
import numpy as np
import pytest
import torch

import oracle
import workloads as wl
from gpu_util import (TOL, gpu_batch, max_abs_err, minus_infinity_pages, oracle_for,
                      run_decode)

pytestmark = pytest.mark.gpu

LENS = np.array([1, 17, 300, 2049, 0, 64, 5000, 33], np.int32)


def _w(d, P, dt, G=8, Hkv=2):
    pages = int(wl.pages_needed(LENS, P).sum()) * 2 + 8
    return wl.Workload("n", len(LENS), G * Hkv, Hkv, d, P, dt, pages, "uniform", lo=1, hi=1)


def _oracle(b, scale):
    s = wl.subset_for_oracle(b, list(range(b.w.num_seqs)))
    return oracle.decode(s["q"], s["k_pages"], s["v_pages"], s["block_table"], s["seq_lens"],
                         num_kv_heads=b.w.num_kv_heads, page_size=b.w.page_size,
                         kv_dtype=b.w.kv_dtype, scale=scale, k_scales=s["k_scales"],
                         v_scales=s["v_scales"], num_pages=s["num_pages"])


@pytest.mark.parametrize("dt,P", [(0, 16), (1, 32)])
@pytest.mark.parametrize("scale", [0.03, 1.0])
def test_caller_softmax_scale(dt, P, scale):
    print(f"[case] sm_scale {scale} dt={dt} P={P}", flush=True)
    b = gpu_batch(_w(128, P, dt), lengths=LENS, seed_index=300 + dt)
    out = run_decode(b, sm_scale=scale)
    err = max_abs_err(out, _oracle(b, scale))
    assert err <= TOL[dt], err


@pytest.mark.parametrize("dt,P", [(0, 16), (1, 32)])
def test_large_scores_underflow_safely(dt, P):
    """q scaled by 24: scores of a few hundred, so exp() of most tokens'
    scores relative to the maximum underflows to zero; the online softmax must
    still give the oracle's nearly one-hot mixture, with no NaN or infinity."""
    print(f"[case] large scores dt={dt} P={P}", flush=True)
    b = gpu_batch(_w(128, P, dt), lengths=LENS, seed_index=310 + dt)
    b.q.copy_((b.q.float() * 24).to(torch.bfloat16))
    out = run_decode(b)
    err = max_abs_err(out, oracle_for(b))
    assert err <= TOL[dt], err


@pytest.mark.parametrize("dt,P", [(0, 16), (1, 32)])
def test_zero_query_is_the_mean_of_values(dt, P):
    """With q = 0 every score is 0 and the output is the mean of the
    sequence's value rows: checked against a direct mean of the stored values,
    computed here from the page layout with no attention code."""
    print(f"[case] zero query dt={dt} P={P}", flush=True)
    w = _w(64, P, dt)
    b = gpu_batch(w, lengths=LENS, seed_index=320 + dt)
    b.q.zero_()
    out = run_decode(b).float().cpu().numpy()
    G = w.num_q_heads // w.num_kv_heads
    vp = b.v_pages.cpu()
    vp = (vp.view(torch.float8_e4m3fn).float() if dt == 1 else vp.float()).numpy()
    vs = b.v_scales.cpu().numpy() if dt == 1 else None
    bt = b.block_table_h
    for s, L in enumerate(LENS):
        for g in range(w.num_kv_heads):
            if L == 0:
                assert np.all(out[s, g * G:(g + 1) * G] == 0)
                continue
            rows = []
            for t in range(L):
                p = int(bt[s, t // P])
                v = vp[p, g, :, t % P] * (vs[p] if dt == 1 else 1.0)   # [d], V stored [d][P]
                rows.append(v)
            mean = np.mean(np.stack(rows), axis=0)
            for h in range(G):
                err = np.abs(out[s, g * G + h] - mean).max()
                assert err <= TOL[dt], (s, g, h, err)


@pytest.mark.parametrize("dt,P", [(0, 16), (1, 32)])
def test_one_sequence_of_half_a_million_tokens(dt, P):
    """The geometry's far corner: one sequence of 2^19 tokens (2^15 or 2^14
    pages in one block-table row) over the widest query group (G = 16) of a
    single KV head, by the default call (fp8: 1,024 chunks of 512 tokens) and by
    stream-K, which cuts the one segment across every wavefront, so that the
    combine merges about a thousand pieces either way.  A softmax
    scale of 1 keeps the output dominated by a few tokens (with 1/sqrt(d) the
    output of half a million random values would be near zero and say
    little).  The oracle takes about ten seconds per case."""
    print(f"[case] 2^19 tokens dt={dt} P={P}", flush=True)
    lens = np.array([1 << 19], np.int32)
    pages = int(wl.pages_needed(lens, P).sum()) + 8
    w = wl.Workload("m", 1, 16, 1, 64, P, dt, pages, "uniform", lo=1, hi=1)
    b = gpu_batch(w, lengths=lens, seed_index=330 + dt)
    ref = _oracle(b, 1.0)
    assert np.abs(ref).max() > 0.5, "the check needs outputs of order one"
    for cut in ({}, {"min_range_pages": 8}):
        err = max_abs_err(run_decode(b, sm_scale=1.0, **cut), ref)
        assert err <= TOL[dt], (cut, err)


def test_widest_kv_head_count():
    """127 KV heads (the descriptor's limit), one query head each."""
    print("[case] Hkv=127", flush=True)
    lens = np.array([1, 17, 300, 0, 2049], np.int32)
    pages = int(wl.pages_needed(lens, 16).sum()) * 2 + 8
    w = wl.Workload("h", len(lens), 127, 127, 64, 16, 0, pages, "uniform", lo=1, hi=1)
    b = gpu_batch(w, lengths=lens, seed_index=340)
    out = run_decode(b)
    err = max_abs_err(out, oracle_for(b))
    assert err <= TOL[0], err


def test_largest_block_table_stride():
    """Block-table rows of 2^19 - 1 entries (the descriptor's limit): row
    offsets past 2^21 bytes, the pages of each sequence at the row's start."""
    print("[case] stride 2^19-1", flush=True)
    lens = np.array([1, 500, 33], np.int32)
    pages = int(wl.pages_needed(lens, 16).sum()) * 2 + 8
    w = wl.Workload("s", len(lens), 8, 2, 64, 16, 0, pages, "uniform", lo=1, hi=1)
    b = wl.make_batch(w, device="cuda", seed_index=341, lengths=lens, stride=(1 << 19) - 1)
    assert b.block_table.shape[1] == (1 << 19) - 1
    out = run_decode(b)
    err = max_abs_err(out, oracle_for(b))
    assert err <= TOL[0], err


@pytest.mark.parametrize("d,P,dt", [(128, 16, 0), (64, 16, 0), (128, 32, 0), (128, 16, 1),
                                    (64, 32, 1)])
def test_pages_of_minus_infinity_scores(d, P, dt):
    """Pages whose scores are all -inf have no weight, wherever they lie: the
    first page of a sequence, of a wave, of a chunk, a whole chunk, all pages
    but the last.  Over the segment kernel (1,120 tokens: chunks of 256) and
    over the stream-K cut, whose ranges start anywhere."""
    print(f"[case] -inf pages d={d} P={P} dt={dt}", flush=True)
    n = 1120 // P
    runs = [(0, 1), (1, 2), (2, 3), (3, 5), (4, 5), (256 // P, 256 // P + 1),
            (256 // P, 512 // P), (0, 512 // P), (n - 1, n), (0, n - 1), (7, n - 2)]
    lens = np.full(len(runs), 1120, np.int32)
    w = wl.Workload("i", len(runs), 8, 2, d, P, dt, 2 * n * len(runs), "uniform", lo=1, hi=1)
    b = gpu_batch(w, lengths=lens, seed_index=350 + d + P + dt)
    minus_infinity_pages(b, [int(b.block_table_h[s, j]) for s, (lo, hi) in enumerate(runs)
                              for j in range(lo, hi)])
    ref = oracle_for(b)
    for cut in ({}, {"min_range_pages": 8}, {"num_waves": 50, "min_range_pages": 1}):
        err = max_abs_err(run_decode(b, **cut), ref)
        assert err <= TOL[dt], (cut, err)


@pytest.mark.parametrize("dt,P", [(0, 16), (1, 32)])
@pytest.mark.parametrize("case", ["scale", "large", "zero"])
def test_stream_k_scales_and_scores(dt, P, case):
    """A caller's softmax scale, scores of a few hundred and a zero query, by the
    stream-K cut (the default call runs these batches per segment)."""
    print(f"[case] stream-K {case} dt={dt} P={P}", flush=True)
    b = gpu_batch(_w(128, P, dt), lengths=LENS, seed_index=360 + dt)
    scale = 1.0 if case == "scale" else 0.0
    if case == "large":
        b.q.copy_((b.q.float() * 24).to(torch.bfloat16))
    elif case == "zero":
        b.q.zero_()
    ref = _oracle(b, scale)
    out = run_decode(b, sm_scale=scale, min_range_pages=8)
    assert max_abs_err(out, ref) <= TOL[dt]
    assert max_abs_err(run_decode(b, sm_scale=scale), ref) <= TOL[dt]
