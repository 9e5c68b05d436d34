"""GPU parity of dora_decode_attn (through the C ABI) against the fp64 oracle.

Bar: max-abs error <= 2e-2 on bf16-KV outputs and <= 5e-2 on fp8-KV outputs;
bitwise equality where the result is unique (length-1 sequences, page
permutation, migration, repeated runs).
"""
import numpy as np
import pytest
import torch

import workloads as wl
from gpu_util import (TOL, cut_segments, decode_waves, gpu_batch, lib, max_abs_err, oracle_for,
                      page_chunks, run_decode, segment_pages)

pytestmark = pytest.mark.gpu


def _w(name="t", B=8, Hq=8, Hkv=2, d=64, P=16, dt=0, pages=None, lens=None):
    pages = pages or max(64, int(wl.pages_needed(np.asarray(lens), P).sum()) * 2 + 8)
    return wl.Workload(name, B, Hq, Hkv, d, P, dt, pages, "uniform", lo=1, hi=1)


RAGGED = [0, 1, 2, 15, 16, 17, 31, 32, 33, 100, 257, 1000, 4097]


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("P", [16, 32])
@pytest.mark.parametrize("dt", [0, 1])
@pytest.mark.parametrize("G", [1, 4, 7, 16])
def test_shapes_ragged_lengths(d, P, dt, G):
    print(f"[case] shapes d={d} P={P} dt={dt} G={G}", flush=True)
    Hkv = 2
    lens = np.array(RAGGED, np.int32)
    w = _w(B=len(lens), Hq=G * Hkv, Hkv=Hkv, d=d, P=P, dt=dt, lens=lens)
    b = gpu_batch(w, lengths=lens, seed_index=100 + d + P + dt + G)
    out = run_decode(b)
    ref = oracle_for(b)
    err = max_abs_err(out, ref)
    assert err <= TOL[dt], err
    assert torch.all(out[0] == 0), "empty sequence must give zeros"


def test_tiny_workload_full_parity():
    w = wl.WORKLOADS[0]
    print(f"[case] {w.name}", flush=True)
    b = gpu_batch(w, seed_index=0)
    out = run_decode(b)
    err = max_abs_err(out, oracle_for(b))
    assert err <= TOL[0], err


@pytest.mark.parametrize("waves", [1, 2, 7, 64, 1000, 0])
def test_wave_count_invariance(waves):
    """Cutting the work among 1 ... 1000 wavefronts (ranges as small as one
    page-head, so segments are cut into many partials) agrees with the oracle
    and with the default cut."""
    print(f"[case] waves={waves}", flush=True)
    lens = np.array([5, 700, 1300, 33, 2048, 16, 0, 1], np.int32)
    w = _w(B=len(lens), Hq=16, Hkv=2, d=128, P=16, dt=0, lens=lens)
    b = gpu_batch(w, lengths=lens, seed_index=7)
    out = run_decode(b, num_waves=waves, min_range_pages=1)
    ref = oracle_for(b)
    assert max_abs_err(out, ref) <= TOL[0]
    base = run_decode(b)
    diff = (out.float() - base.float()).abs().max().item()
    assert diff <= TOL[0]


def test_wave_count_invariance_fp8_page32():
    lens = np.array([2000, 64, 4500, 1], np.int32)
    w = _w(B=len(lens), Hq=16, Hkv=2, d=128, P=32, dt=1, lens=lens)
    b = gpu_batch(w, lengths=lens, seed_index=8)
    ref = oracle_for(b)
    for waves in (1, 5, 300):
        out = run_decode(b, num_waves=waves, min_range_pages=1)
        assert max_abs_err(out, ref) <= TOL[1]


def test_deterministic_bitwise():
    lens = np.array([3000, 17, 900, 4000, 1], np.int32)
    w = _w(B=len(lens), Hq=28, Hkv=4, d=128, P=16, dt=0, lens=lens)
    b = gpu_batch(w, lengths=lens, seed_index=9)
    a = run_decode(b).clone()
    for _ in range(3):
        assert torch.equal(run_decode(b), a)


def test_length_one_is_value_row_bitwise():
    lens = np.ones(6, np.int32)
    w = _w(B=6, Hq=8, Hkv=2, d=128, P=16, dt=0, lens=lens)
    b = gpu_batch(w, lengths=lens, seed_index=10)
    out = run_decode(b)
    for s in range(6):
        pg = int(b.block_table_h[s, 0])
        for h in range(8):
            v = b.v_pages[pg, h // 4, :, 0]          # token slot 0, all head dims
            assert torch.equal(out[s, h], v)


def test_physical_page_permutation_bitwise():
    lens = np.array([300, 1, 77, 1024], np.int32)
    w = _w(B=4, Hq=8, Hkv=2, d=128, P=16, dt=0, lens=lens)
    b = gpu_batch(w, lengths=lens, seed_index=11)
    ref = run_decode(b).clone()
    perm = torch.randperm(w.num_pages, generator=torch.Generator().manual_seed(3)).cuda()
    k2 = torch.empty_like(b.k_pages)
    v2 = torch.empty_like(b.v_pages)
    k2[perm] = b.k_pages
    v2[perm] = b.v_pages
    bt2 = perm[b.block_table.long()].to(torch.int32)
    b.k_pages, b.v_pages, b.block_table = k2, v2, bt2.contiguous()
    assert torch.equal(run_decode(b), ref)


def test_batch_permutation():
    """Permuting the batch permutes the outputs.  The work cut moves with the
    order, so the match is to tolerance, not bitwise."""
    lens = np.array([300, 1, 77, 1024, 5000, 0], np.int32)
    w = _w(B=6, Hq=8, Hkv=2, d=128, P=16, dt=0, lens=lens)
    b = gpu_batch(w, lengths=lens, seed_index=12)
    ref = run_decode(b).clone()
    perm = torch.tensor([3, 5, 0, 4, 1, 2])
    b.q = b.q[perm.cuda()].contiguous()
    b.block_table = b.block_table[perm.cuda()].contiguous()
    b.seq_lens = b.seq_lens[perm.cuda()].contiguous()
    b.version_ids = b.version_ids[perm.cuda()].contiguous()
    diff = (run_decode(b).float() - ref[perm.cuda()].float()).abs().max().item()
    assert diff <= TOL[0]


def test_workspace_contents_ignored():
    lens = np.array([800, 2000, 3], np.int32)
    w = _w(B=3, Hq=8, Hkv=2, d=128, P=16, dt=0, lens=lens)
    b = gpu_batch(w, lengths=lens, seed_index=13)
    d = lib()
    ref = run_decode(b, num_waves=40, min_range_pages=1).clone()
    desc = d.make_decode_desc(num_seqs=3, num_q_heads=8, num_kv_heads=2, head_dim=128,
                              page_size=16, block_table_stride=b.stride,
                              num_pages=w.num_pages, num_waves=40, min_range_pages=1)
    ws = torch.full((d.dora_decode_workspace_bytes(desc) // 4,), float("nan"),
                    device="cuda").view(torch.uint8)
    out = torch.full_like(b.q, float("nan"))
    run_decode(b, out=out, num_waves=40, min_range_pages=1, workspace=ws)
    assert torch.equal(out, ref)


def test_batch_larger_than_one_launch():
    """More sequences than one decode launch takes (8192): the call is cut into
    launches; outputs of sequences in both launches match the oracle."""
    rng = np.random.default_rng(3)
    lens = rng.integers(0, 40, 9000).astype(np.int32)
    w = _w(B=len(lens), Hq=8, Hkv=2, d=64, P=16, dt=0, lens=lens)
    b = gpu_batch(w, lengths=lens, seed_index=14)
    out = run_decode(b)
    seqs = [0, 1, 8190, 8191, 8192, 8193, 8999] + [int(i) for i in rng.choice(9000, 20)]
    seqs = sorted(set(seqs))
    assert max_abs_err(out, oracle_for(b, seqs), seqs) <= TOL[0]


def test_validate_flag_accepts_good_and_rejects_bad_pages():
    w = wl.WORKLOADS[3].scaled(48, num_pages=8192)   # three versions in one pool
    b = gpu_batch(w, seed_index=3, lengths=np.random.default_rng(1).integers(1, 1500, 48)
                  .astype(np.int32))
    d = lib()
    run_decode(b, flags=d.DORA_FLAG_VALIDATE, page_owner=b.page_owner)
    # a page of another version in sequence 0's table
    other = int(np.nonzero(b.versions_h != b.versions_h[0])[0][0])
    bt = b.block_table.clone()
    bt[0, 0] = b.block_table[other, 0]
    b2 = b
    b2.block_table = bt
    with pytest.raises(d.DoraError) as e:
        run_decode(b2, flags=d.DORA_FLAG_VALIDATE, page_owner=b.page_owner)
    assert e.value.status == d.DORA_ERR_DEVICE_CHECK
    bt = bt.clone()
    bt[0, 0] = w.num_pages + 5
    b2.block_table = bt
    with pytest.raises(d.DoraError) as e:
        run_decode(b2, flags=d.DORA_FLAG_VALIDATE)
    assert e.value.status == d.DORA_ERR_DEVICE_CHECK



@pytest.mark.parametrize("bad", ["len_past_table", "len_negative", "page_negative"])
def test_validate_flag_rejects_bad_lengths_and_ids(bad):
    """DORA_FLAG_VALIDATE also rejects a length the block table cannot hold,
    a negative length and a negative page id, before any decode launch (the
    output keeps its sentinel), and a good call right after passes (the
    check's flag is cleared on every call)."""
    print(f"[case] validate {bad}", flush=True)
    lens = np.array([40, 300, 17, 129], np.int32)
    w = _w(B=len(lens), Hq=8, Hkv=2, d=64, P=16, dt=0, lens=lens)
    b = gpu_batch(w, lengths=lens, seed_index=9)
    d = lib()
    good_bt, good_lens = b.block_table.clone(), b.seq_lens.clone()
    stride = b.block_table.shape[1]
    if bad == "len_past_table":
        b.seq_lens[1] = stride * w.page_size + 1
    elif bad == "len_negative":
        b.seq_lens[2] = -1
    else:
        b.block_table[3, 2] = -3
    sentinel = torch.full_like(b.q, 7.0)
    out = sentinel.clone()
    with pytest.raises(d.DoraError) as e:
        run_decode(b, out=out, flags=d.DORA_FLAG_VALIDATE)
    assert e.value.status == d.DORA_ERR_DEVICE_CHECK
    assert torch.equal(out, sentinel)
    b.block_table, b.seq_lens = good_bt, good_lens
    out = run_decode(b, flags=d.DORA_FLAG_VALIDATE)
    assert max_abs_err(out, oracle_for(b)) <= TOL[0]

def test_empty_batch_is_a_no_op():
    d = lib()
    q = torch.empty((0, 8, 64), dtype=torch.bfloat16, device="cuda")
    kp = torch.zeros((4, 2, 8, 16, 8), dtype=torch.bfloat16, device="cuda")
    vp = torch.zeros((4, 2, 64, 16), dtype=torch.bfloat16, device="cuda")
    bt = torch.zeros((0, 1), dtype=torch.int32, device="cuda")
    z = torch.zeros(0, dtype=torch.int32, device="cuda")
    d.dora_decode_attn(q, kp, vp, bt, z, z, q.clone(), num_kv_heads=2, page_size=16)


# ---------------------------------------------------------------------------
# the long-tail workloads at full size, in the launch configuration the
# benchmark times: every output element of every sequence against the oracle
# (in runs of sequences, to bound the host copies).
# ---------------------------------------------------------------------------

@pytest.mark.parametrize("idx", [1, 2, 3, 4])
def test_full_size_workloads_every_sequence(idx):
    w = wl.WORKLOADS[idx]
    print(f"[case] full-size {w.name}", flush=True)
    b = gpu_batch(w, seed_index=idx)
    out = run_decode(b)
    assert torch.isfinite(out.float()).all()
    waves = decode_waves(b)
    cuts = cut_segments(b.lengths, w.page_size, b.stride, w.num_kv_heads, waves)
    # the default launch splits segments across wavefronts, so the combine runs
    assert cuts, "no segment is cut: the combine path would go untested"
    err, runs = 0.0, page_chunks(b.lengths, w.page_size, 24576)
    for seqs in runs:
        ref = oracle_for(b, seqs)
        err = max(err, max_abs_err(out, ref, seqs))
    print(f"[case] {w.name}: {w.num_seqs} seqs in {len(runs)} runs, {waves} waves, "
          f"{len(cuts)} cut segments in {len({c[0] for c in cuts})} seqs, "
          f"max-abs err {err:.3e}", flush=True)
    assert err <= TOL[w.kv_dtype], err
    del b, out
    torch.cuda.empty_cache()


def test_profiling_events_bracket_each_kernel():
    """The three events bracket the decode and the combine kernel: positive
    durations, and the call's result is unchanged."""
    lens = np.array([3000, 17, 900, 4000, 1], np.int32)
    w = _w(B=len(lens), Hq=28, Hkv=4, d=128, P=16, dt=0, lens=lens)
    b = gpu_batch(w, lengths=lens, seed_index=15)
    evs = [torch.cuda.Event(enable_timing=True) for _ in range(3)]
    for e in evs:
        e.record()
    torch.cuda.synchronize()
    ref = run_decode(b).clone()
    out = run_decode(b, events=[e.cuda_event for e in evs])
    assert torch.equal(out, ref)
    dec, comb = (evs[i].elapsed_time(evs[i + 1]) for i in range(2))
    assert 0 < dec < 1000 and 0 < comb < 1000, (dec, comb)


@pytest.mark.parametrize("dt,d,P,Hkv,G,stride", [
    (0, 128, 16, 1, 1, 1),        # one page a row
    (0, 64, 16, 2, 16, 63),       # 1,008 tokens: whole segments
    (0, 128, 16, 2, 7, 64),       # 1,024 tokens: chunks of 256
    (1, 128, 32, 4, 16, 33),      # fp8, chunks of 8 pages of 32
    (1, 64, 16, 8, 4, 96),        # 1,536 tokens, 11 x 8 segments: chunks of 256
    (0, 128, 16, 8, 16, 96),      # 16 query heads
    (0, 128, 16, 40, 1, 80),      # 440 segments: whole up to 1,280 tokens ...
    (0, 128, 16, 40, 1, 81),      # ... and stream-K past them
    (1, 128, 16, 40, 1, 96),      # fp8: whole up to 1,536, page by page
    (1, 128, 16, 2, 4, 31),       # fp8: in pairs of pages, an odd count
    (1, 64, 16, 40, 2, 128),      # head dim 64: whole up to 2,048 tokens, 32 pages a wave
    (0, 128, 32, 40, 2, 32),      # 32-token bf16 pages: whole up to 1,024
    (0, 128, 16, 9, 4, 189),      # chunks of 512 tokens: 99 segments of 3,024
    (1, 128, 32, 4, 8, 300),      # a last chunk that is not full
    (0, 128, 16, 14, 2, 81),      # past 1,280 tokens: 924 chunks of 256
    (0, 128, 16, 20, 1, 100),     # ... and stream-K past 1,024 of them
    (1, 128, 32, 20, 2, 80),      # fp8: 1,100 chunks of 512
    (1, 64, 16, 30, 1, 130),      # fp8, head dim 64: 1,650 chunks of 512
    (1, 64, 16, 40, 1, 129),      # ... and stream-K past 2,048 of them
])
def test_segment_kernel_edges(dt, d, P, Hkv, G, stride):
    """Batches the default call cuts per segment or chunk, at the lines of that
    rule and at the edges of pages, waves, chunks and rows (empty, one token,
    one chunk exactly, one page more, a full row), with table entries past a
    sequence's pages that name no page: against the oracle, and against the
    stream-K cut (num_waves set)."""
    print(f"[case] segments dt={dt} d={d} P={P} Hkv={Hkv} G={G} stride={stride}", flush=True)
    full = stride * P
    lens = np.minimum(np.array([0, 1, P, P + 1, 4 * P, 4 * P + 1, 256, 257, 512, 513 + P, full],
                               np.int32), full)
    w = _w(B=len(lens), Hq=G * Hkv, Hkv=Hkv, d=d, P=P, dt=dt, lens=lens)
    b = gpu_batch(w, lengths=lens, seed_index=300 + stride + G)
    n = torch.from_numpy(wl.pages_needed(lens, P)).cuda()
    past = torch.arange(b.stride, device="cuda")[None, :] >= n[:, None]
    b.block_table = torch.where(past, torch.full_like(b.block_table, 1 << 30), b.block_table)
    assert b.stride == stride
    out = run_decode(b, out=torch.full_like(b.q, float("nan")))
    assert max_abs_err(out, oracle_for(b)) <= TOL[dt]
    assert not out[0].float().abs().any()
    assert torch.equal(run_decode(b), out)
    cut = run_decode(b, num_waves=64)
    # both round the same sums once to bf16, in another order
    assert (out.float() - cut.float()).abs().max().item() <= TOL[dt] / 2


@pytest.mark.parametrize("dt,d,P,Hkv,G,lens", [
    (0, 128, 16, 1, 16, [20000, 48, 9000, 0, 300, 16]),      # 512 tasks, 79 chunks of 256
    (1, 128, 32, 8, 4, [14000, 700, 3000, 1]),               # four rows of 8 heads: rotated
    (1, 64, 16, 2, 1, [17000, 40]),                          # 16 tasks
    (0, 128, 32, 1, 6, [40000]),                             # one row, chunks of 512
    (0, 64, 32, 1, 8, [36000, 36000]),
    (0, 128, 16, 2, 7, [8000, 4100, 4096, 4097, 256, 257]),  # ends at chunks' edges
    (1, 128, 16, 4, 7, [9000, 100, 5000]),                   # an odd number of rows
])
def test_segment_kernel_many_chunks(dt, d, P, Hkv, G, lens):
    """Rows of many chunks: the combine shares a segment's tasks out, and an even
    number of rows is rotated from chunk to chunk.  Against the oracle and against
    stream-K; bitwise the same when repeated."""
    print(f"[case] chunks dt={dt} d={d} P={P} Hkv={Hkv} G={G} rows={lens}", flush=True)
    lens = np.array(lens, np.int32)
    w = _w(B=len(lens), Hq=G * Hkv, Hkv=Hkv, d=d, P=P, dt=dt, lens=lens)
    b = gpu_batch(w, lengths=lens, seed_index=400 + G)
    assert 0 < segment_pages(b) * 16 < b.stride
    out = run_decode(b, out=torch.full_like(b.q, float("nan")))
    assert max_abs_err(out, oracle_for(b)) <= TOL[dt]
    assert torch.equal(run_decode(b), out)
    cut = run_decode(b, min_range_pages=8)
    assert (out.float() - cut.float()).abs().max().item() <= TOL[dt] / 2


# ---------------------------------------------------------------------------
# the stream-K decode: the default call of small batches runs the segment kernel,
# so these name the default stream-K cut (min_range_pages = 8) themselves
# ---------------------------------------------------------------------------

STREAM_K = {"min_range_pages": 8}


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("P", [16, 32])
@pytest.mark.parametrize("dt", [0, 1])
@pytest.mark.parametrize("G", [1, 4, 7, 16])
def test_stream_k_ragged_lengths(d, P, dt, G):
    print(f"[case] stream-K shapes d={d} P={P} dt={dt} G={G}", flush=True)
    Hkv = 2
    lens = np.array(RAGGED, np.int32)
    w = _w(B=len(lens), Hq=G * Hkv, Hkv=Hkv, d=d, P=P, dt=dt, lens=lens)
    b = gpu_batch(w, lengths=lens, seed_index=100 + d + P + dt + G)
    assert segment_pages(b) > 0 and segment_pages(b, **STREAM_K) == 0
    out = run_decode(b, out=torch.full_like(b.q, float("nan")), **STREAM_K)
    assert max_abs_err(out, oracle_for(b)) <= TOL[dt]
    assert torch.all(out[0] == 0), "empty sequence must give zeros"
    assert torch.equal(run_decode(b, **STREAM_K), out)


def test_stream_k_cuts_are_deterministic_bitwise():
    lens = np.array([3000, 17, 900, 4000, 1], np.int32)
    w = _w(B=len(lens), Hq=28, Hkv=4, d=128, P=16, dt=0, lens=lens)
    b = gpu_batch(w, lengths=lens, seed_index=9)
    assert cut_segments(lens, 16, b.stride, 4, decode_waves(b, **STREAM_K))
    a = run_decode(b, **STREAM_K).clone()
    for _ in range(3):
        assert torch.equal(run_decode(b, **STREAM_K), a)
    assert max_abs_err(a, oracle_for(b)) <= TOL[0]


@pytest.mark.parametrize("long_row", [0, 20000])
def test_stream_k_batch_larger_than_one_launch(long_row):
    """More sequences than one launch takes (8192), by stream-K: cut records per
    wavefront, in both launches; with a long row in the second."""
    rng = np.random.default_rng(3)
    lens = rng.integers(0, 40, 9000).astype(np.int32)
    if long_row:
        lens[8500] = long_row
    w = _w(B=len(lens), Hq=8, Hkv=2, d=64, P=16, dt=0, lens=lens)
    b = gpu_batch(w, lengths=lens, seed_index=14)
    out = run_decode(b, out=torch.full_like(b.q, float("nan")), **STREAM_K)
    seqs = [0, 1, 8190, 8191, 8192, 8193, 8500, 8999] + [int(i) for i in rng.choice(9000, 20)]
    seqs = sorted(set(seqs))
    assert max_abs_err(out, oracle_for(b, seqs), seqs) <= TOL[0]
