"""GPU parity of the kernel variants that sizes, page sizes and alignment choose between, at the sizes
where each can go wrong (edges of tiles and pages, remainders, smallest and largest of its range)."""
import numpy as np
import pytest

import oracle
from helpers import TOL, DeviceWorkload, lse_err, max_abs_rel, to_torch, widen_gpu
from test_gpu_parity import check_decode, check_multi, gpu_q_abs, mla, q_abs_storage, run_decode  # noqa: F401
from workloads import synth

pytestmark = pytest.mark.gpu
PORTABLE = 1

# ------------------------------------------------------------------ bf16 caches, pages of 16 k rows

PAGED_LENS = [0, 1, 15, 16, 17, 31, 32, 33, 47, 48, 49, 300, 1000]


def paged_workload(page, d_c=512, H=32, lens=PAGED_LENS, seed=70, **kw):
    return synth.make_workload("paged", B=len(lens), H=H, d_head=128, d_c=d_c, d_rope=64, seq_lens=lens, io_dtype="bf16",
                               cache_dtype="bf16", page_size=page, free_frac=0.1, seed=seed, **kw)


@pytest.mark.parametrize("page,d_c,H,splits", [(16, 512, 32, 1), (16, 256, 28, 3), (32, 512, 5, 32), (48, 512, 40, 2),
                                               (80, 256, 32, 7), (128, 512, 32, 2), (1024, 256, 16, 1)])
def test_decode_other_page_sizes(mla, page, d_c, H, splits):
    """Against the oracle, and no further from it than the scalar-FMA kernel (which holds the weights in
    fp32) by more than the fp32 sums' share: both round the partials and the result to bf16."""
    w = paged_workload(page, d_c, H)
    new, old = check_decode(mla, w, splits), check_decode(mla, w, splits, flags=PORTABLE)
    assert new <= 1.5 * old + 2.0 ** -9
    import torch
    d = DeviceWorkload(w)
    q = gpu_q_abs(mla, d)
    (a, la), (b, lb) = run_decode(mla, d, q, splits), run_decode(mla, d, q, splits, PORTABLE)
    torch.cuda.synchronize()
    # the log-sum-exp is stored in fp32 and formed in fp32 by both kernels: the sums of the scores (576 products of
    # size up to a few units) in two orders
    assert lse_err(widen_gpu(la), widen_gpu(lb)) <= 1e-5
    assert max_abs_rel(widen_gpu(a), widen_gpu(b)) <= 2.0 ** -7      # one bf16 step at the largest value


@pytest.mark.parametrize("page,d_c", [(16, 256), (16, 512), (48, 512)])
@pytest.mark.parametrize("lens,sharp", [([1, 2, 3, 5, 9, 17, 33], 1.0), ([2, 3, 5, 9, 17, 33], 4.0), ([100, 500, 1000], 4.0), ([2999, 4000], 8.0)])
def test_other_page_sizes_keep_fp32_log_sum_exps(mla, page, d_c, lens, sharp):
    """The fp32 log-sum-exp is as close to a 64-bit one as the scalar-FMA kernel's: half as far again at most, and one
    rounding of the stored value (each takes its 576 products in its own order)."""
    import torch
    B, H, mp = len(lens), 32, -(-max(lens) // page)
    gen = torch.Generator(device="cuda").manual_seed(74)
    kv = torch.randn(B * mp, page, d_c + 64, device="cuda", generator=gen).bfloat16()
    table = torch.randperm(B * mp, device="cuda", generator=gen).to(torch.int32).view(B, mp)
    n = torch.tensor(lens, dtype=torch.int32, device="cuda")
    q, qr = ((torch.randn(B, H, k, device="cuda", generator=gen) * sharp).bfloat16() for k in (d_c, 64))
    scale = 0.05
    got = [mla.decode_paged(q, qr, kv, table, n, scale, return_lse=True, flags=flags)[1].double().cpu() for flags in (0, PORTABLE)]
    rows, qq = kv.double().cpu()[table.long().cpu()].flatten(1, 2), torch.cat([q, qr], -1).double().cpu()
    ref = torch.stack([torch.logsumexp(qq[b] @ rows[b, :lens[b]].T * float(np.float32(scale)), -1) for b in range(B)])
    new, old = ((g - ref).abs().max().item() for g in got)
    assert new <= 1.5 * old + 2.0 ** -24 * ref.abs().max().item(), (new, old)


def test_decode_other_page_sizes_bad_pages_and_late_dominant_score(mla):
    """A page id outside the pool drops its 16 tokens only (first or second half of a 32-row tile, or both),
    and a score far above the first tile's sends the chunk through the exact pass."""
    import torch
    w = paged_workload(16, lens=[256, 200, 64], seed=71)
    bad = w.page_table.copy()
    drop = [(0, 1), (0, 4), (0, 6), (0, 7), (1, 12), (2, 0)]
    for b, i in drop:
        bad[b, i] = w.num_pages + 3 if i % 2 else -1
    pt = np.full_like(w.page_table, -1)
    lens = w.seq_lens.copy()
    for b in range(3):
        keep = [i for i in range((w.seq_lens[b] + 15) // 16) if (b, i) not in drop]
        pt[b, :len(keep)] = w.page_table[b, keep]
        lens[b] = sum(min(16, w.seq_lens[b] - 16 * i) for i in keep)
    for flags in (0, PORTABLE):
        d = DeviceWorkload(w)
        d.page_table = to_torch(bad, "i32")
        q = gpu_q_abs(mla, d)
        o, lse = run_decode(mla, d, q, 2, flags)
        torch.cuda.synchronize()
        ref, ref_lse = oracle.decode_absorbed(q_abs_storage(q), w.q_rope, w.pool, None, pt, lens, w.softmax_scale)
        assert max_abs_rel(widen_gpu(o), ref) <= TOL["bf16"] and lse_err(widen_gpu(lse), ref_lse) <= 2e-2
    rows = oracle.widen(oracle.gather_paged(w.pool, w.page_table, w.seq_lens, 256).view(np.uint16))
    target = np.stack([rows[0, 217, :512], rows[1, 199, :512], rows[2, 63, :512]])
    q1 = to_torch(synth.to_bf16_bits((40.0 * target[:, None, :].repeat(32, 1)).astype(np.float32)), "bf16")
    d = DeviceWorkload(w)
    o = mla.decode_paged(q1, torch.zeros((3, 32, 64), dtype=torch.bfloat16, device="cuda"), d.pool, d.page_table,
                         d.seq_lens, w.softmax_scale, num_splits=1)
    torch.cuda.synchronize()
    assert np.abs(widen_gpu(o) - target[:, None, :]).max() <= 2e-2 * np.abs(target).max()


@pytest.mark.parametrize("page,T", [(16, 2), (32, 3)])
def test_multi_token_other_page_sizes(mla, page, T):
    check_multi(mla, paged_workload(page, lens=[0, 1, 2, 16, 33, 47, 320], H=28, seed=72), T, 2, fused_tail=True)


@pytest.mark.parametrize("moved", ["kv", "q", "rope"])
def test_other_page_sizes_off_16_bytes_run_on_the_scalar_kernel(mla, moved):
    """A cache or queries that begin 8 bytes into a buffer: the bits of the scalar-FMA kernel, which needs no more."""
    import torch
    w = paged_workload(16, 256, 8, lens=[0, 5, 40, 333], seed=75)
    d = DeviceWorkload(w)
    q = gpu_q_abs(mla, d)

    def shifted(t):
        buf = torch.empty(t.numel() + 4, dtype=t.dtype, device="cuda")
        view = buf[4:].view(t.shape)
        view.copy_(t)
        assert view.is_contiguous() and view.data_ptr() % 16 == 8
        return view

    kv, qa, qr = (shifted(t) if moved == name else t for name, t in (("kv", d.pool), ("q", q), ("rope", d.q_rope)))
    (o, lse), (ref, ref_lse) = (mla.decode_paged(a, b, c, d.page_table, d.seq_lens, w.softmax_scale, num_splits=2, return_lse=True, flags=flags)
                                for a, b, c, flags in ((qa, qr, kv, 0), (q, d.q_rope, d.pool, PORTABLE)))
    assert torch.equal(o, ref) and torch.equal(lse, ref_lse)


def test_other_page_sizes_keep_refusing_the_balanced_partition(mla):
    w = paged_workload(16, lens=[64, 64])
    d = DeviceWorkload(w)
    with pytest.raises(mla.MlaError):
        run_decode(mla, d, gpu_q_abs(mla, d), 2, mla.FLAG_BALANCED)


# ------------------------------------------------------------------ scalar-FMA decode and fp32 projections

@pytest.mark.parametrize("io,cache,d_c,d_rope,page,H,splits", [
    ("f32", "f32", 512, 64, 64, 32, 4), ("f32", "f32", 8, 8, 1, 1, 1), ("f32", "f32", 264, 16, 7, 3, 2),
    ("f32", "bf16", 256, 0, 5, 5, 3), ("f32", "fp8_e4m3", 40, 64, 3, 33, 2), ("bf16", "fp8_e4m3", 512, 64, 16, 28, 5),
    ("bf16", "bf16", 384, 64, 64, 66, 2), ("bf16", "bf16", 512, 32, 13, 2, 40),
    ("f32", "f32", 8, 0, 5, 8, 8), ("f32", "bf16", 64, 64, 13, 12, 16), ("bf16", "bf16", 256, 64, 63, 32, 4), ("bf16", "fp8_e4m3", 192, 64, 7, 40, 8),
    ("f32", "f32", 128, 64, 64, 9, 16), ("f32", "fp8_e4m3", 8, 8, 1, 17, 64)])
def test_scalar_decode_shapes(mla, io, cache, d_c, d_rope, page, H, splits):
    """Rows in registers (few workgroups, wide rows) and 16-row tiles in LDS (many, narrow): rows per wavefront batch
    (4 and 8), per workgroup (16 and 32) and per tile on both sides, empty and one-row sequences, columns that fill
    neither, one or both groups of 256, head groups that are not full, page sizes that cut every batch."""
    lens = [0, 1, 3, 4, 5, 8, 9, 31, 32, 33, 65, 200]
    w = synth.make_workload("scalar", B=len(lens), H=H, d_head=16, d_c=d_c, d_rope=d_rope, seq_lens=lens, io_dtype=io,
                            cache_dtype=cache, page_size=page, free_frac=0.1, seed=81)
    check_decode(mla, w, splits, flags=PORTABLE)


def test_scalar_decode_many_chunks_take_four_heads_per_workgroup(mla):
    w = synth.make_workload("scalar", B=40, H=30, d_head=16, d_c=128, d_rope=64, seq_lens=[37 * i for i in range(40)],
                            io_dtype="f32", cache_dtype="f32", page_size=64, seed=82)
    check_decode(mla, w, 8, flags=PORTABLE)


@pytest.mark.parametrize("B,H,K,N", [(1, 32, 512, 128), (1, 2, 1, 4), (2, 3, 33, 36), (4, 40, 513, 64), (5, 2, 1030, 72),
                                     (17, 3, 100, 260), (3, 2, 64, 130), (70, 9, 128, 512), (1, 3, 63, 64), (1, 3, 64, 68), (4, 2, 127, 64),
                                     (2, 5, 128, 20), (3, 16, 128, 512), (3, 16, 127, 512), (15, 2, 512, 64), (16, 2, 511, 64), (16, 2, 512, 68), (33, 3, 700, 132), (64, 64, 512, 128)])
def test_fp32_projection_shapes(mla, B, H, K, N):
    """1, 4 and 16 batch rows per workgroup on both sides of the rule (depth, rows, workgroups), k remainders, columns
    that do not fill a tile, N % 4 != 0 (the kernel of single columns), and W off its 16 bytes (the same kernel):
    fp32 sums of K products."""
    import torch
    r = synth.stream(83, B * 1000 + N)
    x = torch.from_numpy(synth.normal(r, (B, H, K))).cuda()
    buf = torch.from_numpy(synth.normal(r, (H * K * N + 1,), K ** -0.5)).cuda()
    for w in (buf[:-1].clone().view(H, K, N), buf[1:].view(H, K, N)):
        got = mla.absorb_q(x, w)
        ref = torch.bmm(x.double().transpose(0, 1), w.double()).transpose(0, 1)
        assert max_abs_rel(widen_gpu(got), ref.cpu().numpy()) <= 1e-5


# ------------------------------------------------------------------ merge of many chunks

@pytest.mark.parametrize("S", [17, 40, 64])
def test_merge_of_many_chunks_keeps_fp32_weights(mla, S):
    """68 to 256 chunks of one row in fp32, one with weight 1 and a value of 0, the others at e^-x with a value of 1, x
    from 8 to 80: the result is the sum of their weights over the sum of all.  expf (2 units in the last place at
    most), S sums and a handful of products in fp32; the hardware's exponential is off by x 2^-24 and more."""
    import torch
    n = 4 * S
    table, lens = torch.arange(n, dtype=torch.int32, device="cuda").view(1, n), torch.tensor([n], dtype=torch.int32, device="cuda")
    q = torch.zeros(1, 1, 256, device="cuda")
    q[0, 0, 0] = 1.0
    worst = 0.0
    for x in np.linspace(8.0, 80.0, 73).astype(np.float32) + np.float32(0.37):
        kv = torch.zeros(n, 1, 256, device="cuda")
        kv[1:, 0, 0], kv[1:, 0, 1] = -float(x), 1.0
        o = mla.decode_paged(q, None, kv, table, lens, 1.0, num_splits=S)
        rest = (n - 1) * np.exp(-float(x))
        worst = max(worst, abs(o[0, 0, 1].item() / (rest / (1.0 + rest)) - 1.0))
    assert worst <= 2.0 ** -22 + 8 * 2.0 ** -24, worst


# ------------------------------------------------------------------ merge + projection of few batch rows

@pytest.mark.parametrize("B,H,d_c,S", [(1, 32, 512, 16), (1, 32, 256, 3), (1, 5, 512, 1), (2, 32, 512, 16), (4, 32, 512, 32),
                                       (2, 64, 256, 5), (7, 28, 512, 9), (1, 16, 512, 17), (4, 33, 256, 4),
                                       (1, 32, 512, 32), (2, 32, 256, 33), (2, 28, 512, 100), (1, 256, 256, 64), (5, 64, 512, 70)])
def test_fused_tail_few_batch_rows(mla, B, H, d_c, S):
    """Output columns cut 2, 4 and 8 ways (and not at all), 4 to 256 chunks (one call of 70 chunks and more
    rows than one workgroup per CU: two kernels): o_lat and lse bit for
    bit those of the stand-alone merge, out within one bf16 rounding of the stored o_lat's projection."""
    import torch
    lens = [(64 * 37 * (i + 1)) % 2500 + i for i in range(B)]
    lens[-1] = 0 if B > 1 else 900
    w = synth.make_workload("few", B=B, H=H, d_head=128, d_c=d_c, d_rope=64, seq_lens=lens, io_dtype="bf16",
                            cache_dtype="bf16", free_frac=0.1, seed=90 + B)
    d = DeviceWorkload(w)
    q = gpu_q_abs(mla, d)
    ws = mla.decode_paged(q, d.q_rope, d.pool, d.page_table, d.seq_lens, w.softmax_scale, num_splits=S, flags=mla.FLAG_SKIP_MERGE)
    o1, l1 = mla.merge_partials(ws, B, H, d_c, S, q.dtype, return_lse=True)
    o2, out, l2 = mla.merge_out_proj(ws, d.W_UV, B, S, return_lse=True)
    torch.cuda.synchronize()
    assert o1.view(torch.int16).equal(o2.view(torch.int16)) and l1.view(torch.int32).equal(l2.view(torch.int32))
    ref = oracle.out_proj(q_abs_storage(o2), w.W_UV)
    # fp32 sums of d_c products, one rounding to bf16 (2^-9 of the value)
    assert max_abs_rel(widen_gpu(out), ref) <= 2.0 ** -8


# ------------------------------------------------------------------ prefill

@pytest.mark.parametrize("T,lens,H,d_c,scale", [
    (33, [33, 34, 64, 65, 96, 97, 400], 3, 256, None),       # keys on both sides of a tile and a page, one step and two
    (129, [129, 130, 161, 1], 2, 512, None),                 # a second group of query rows with one row
    (5, [(67 * i) % 300 + 1 for i in range(66)], 2, 256, None),   # more sequences than are ranked by length
    (40, [200, 31, 0], 3, 256, -0.05), (40, [200, 31, 64], 3, 256, 0.0)])
def test_prefill_edges(mla, T, lens, H, d_c, scale):
    from test_gpu_parity import check_prefill
    w = synth.make_workload("prefill", B=len(lens), H=H, d_head=128, d_c=d_c, d_rope=64, seq_lens=lens, io_dtype="bf16",
                            cache_dtype="bf16", free_frac=0.1, seed=101, softmax_scale=scale)
    check_prefill(mla, w, T)


def test_prefill_skips_bad_pages(mla):
    """A page outside the pool, first, in the middle and last: its tokens are left out."""
    import torch
    w = synth.make_workload("prefill", B=3, H=2, d_head=128, d_c=256, d_rope=64, seq_lens=[300, 200, 130], io_dtype="bf16",
                            cache_dtype="bf16", free_frac=0.1, seed=102)
    drop = [(0, 2), (1, 0), (2, 2)]
    bad, pt, lens = w.page_table.copy(), np.full_like(w.page_table, -1), w.seq_lens.copy()
    for b, i in drop:
        bad[b, i] = w.num_pages + 1 if b else -1
        keep = [k for k in range((w.seq_lens[b] + 63) // 64) if k != i]
        pt[b, :len(keep)] = w.page_table[b, keep]
        lens[b] = sum(min(64, w.seq_lens[b] - 64 * k) for k in keep)
    d = DeviceWorkload(w)
    T = 2
    qn, qr = synth.multi_queries(w, T)
    got = mla.prefill_mha(to_torch(qn, "bf16"), to_torch(qr, "bf16"), d.W_UK, d.W_UV, d.pool, to_torch(bad, "i32"), d.seq_lens,
                          w.softmax_scale)
    torch.cuda.synchronize()
    # sequences 0 and 1 keep their newest rows; both tokens of the last one see all rows that are left
    for b, t in ((slice(0, 1), slice(0, 2)), (slice(1, 2), slice(0, 2)), (slice(2, 3), slice(0, 1)), (slice(2, 3), slice(1, 2))):
        ref = oracle.prefill_explicit(qn[b, t], qr[b, t], w.W_UK, w.W_UV, w.pool, None, pt[b], lens[b], w.softmax_scale, w.d_c)[0]
        assert max_abs_rel(widen_gpu(got)[b, t], ref) <= TOL["bf16"]


@pytest.mark.parametrize("H,d_c,B,cache", [(1, 512, 1, "f32"), (3, 256, 2, "f32"), (32, 512, 1, "f32"), (5, 64, 9, "bf16"), (16, 256, 16, "fp8_e4m3"),
                                           (4, 512, 256, "f32"), (4, 256, 257, "bf16"), (2, 512, 300, "f32")])
def test_portable_decode_wavefronts(mla, H, d_c, B, cache):
    """Eight wavefronts of four rows per batch where every workgroup has a CU, four beyond: chunks that end inside, at and behind a
    wavefront's batch and a round of batches, none at all, at both sides of 256 workgroups of 2 and of 4 heads."""
    ends = [1, 3, 4, 5, 31, 32, 33, 63, 64, 65, 0, 97, 129, 200]
    w = synth.make_workload("waves", B=B, H=H, d_head=128, d_c=d_c, d_rope=64, seq_lens=[ends[(5 * i + B) % len(ends)] for i in range(B - 1)] + [150],
                            io_dtype="f32", cache_dtype=cache, free_frac=0.1, page_size=40, seed=136)
    check_decode(mla, w, 1)


@pytest.mark.parametrize("B,splits,T,H,cache,flags", [(3, 32, 1, 32, "bf16", 0), (3, 64, 1, 28, "bf16", 0), (5, 25, 1, 32, "fp8_e4m3", 0), (17, 15, 1, 32, "bf16", 0),
                                                     (3, 32, 3, 32, "bf16", 0), (2, 16, 5, 64, "bf16", 0), (2, 32, 1, 32, "f32", 0), (20, 4, 1, 32, "bf16", 4),
                                                     (70, 4, 1, 16, "bf16", 4), (70, 3, 1, 64, "fp8_e4m3", 4), (20, 4, 2, 32, "bf16", 4), (130, 7, 1, 64, "bf16", 4)])
def test_chunks_of_one_round(mla, B, splits, T, H, cache, flags):
    """Calls whose chunks are counted to fill one round of workgroups, above and (balanced) below what was asked for: decode and merge
    cut alike, as one call and as the two with the projection, whatever the workspace held."""
    from test_gpu_parity import check_multi
    lens = [(97 * i) % 700 for i in range(B - 1)] + [3000 if B < 20 else 1100]
    w = synth.make_workload("round", B=B, H=H, d_head=128, d_c=256, d_rope=64, seq_lens=lens, io_dtype="f32" if cache == "f32" else "bf16",
                            cache_dtype=cache, free_frac=0.1, seed=135)
    check_multi(mla, w, T, splits, flags)
    check_multi(mla, w, T, splits, flags, fused_tail=True)


def cut(B, rows, num_splits, balanced):
    """The library's choice of chunks (ranges) per sequence: the most, and those used."""
    m = 1
    while m < 4 and B * num_splits * m < 256:
        m *= 2
    most, each = num_splits * m, B * -(-rows // 32)
    one = min(4 * num_splits, 256 // each)
    return most, one if balanced and each * one > 130 and -(-each * most // 256) * one >= most else most


def partials(mla, w, table, T, splits, flags):
    """What a decode call leaves for the merge: log-sum-exps and plan, at their places in the workspace."""
    import torch
    d = DeviceWorkload(w)
    lead = (w.B, T, w.H) if T > 1 else (w.B, w.H)
    io = torch.float32 if w.io_dtype == "f32" else torch.bfloat16
    q, qr = torch.randn(*lead, w.d_c, device="cuda").to(io), torch.randn(*lead, 64, device="cuda").to(io)
    rows = T * w.H
    ws = torch.zeros(mla.decode_workspace_bytes(w.B, rows, w.d_c, splits), dtype=torch.uint8, device="cuda")
    (mla.decode_paged_multi if T > 1 else mla.decode_paged)(q, qr, d.pool, to_torch(table, "i32"), d.seq_lens, w.softmax_scale, num_splits=splits,
                                                            kv_scale=d.kv_scale, workspace=ws, flags=flags | mla.FLAG_SKIP_MERGE)
    torch.cuda.synchronize()
    slots = w.B * (cut(w.B, rows, splits, False)[0] + 1)
    up = lambda n: -(-n // 256) * 256
    lse_at = up(slots * rows * w.d_c * 4)
    plan_at = lse_at + up(slots * rows * 4)
    host = ws.cpu().numpy()
    return host[lse_at:lse_at + slots * rows * 4].view(np.float32), host[plan_at:plan_at + 8 * w.B].view(np.int32).reshape(-1, 2)


@pytest.mark.parametrize("B,splits,T,H,cache,page,width,lens", [
    (30, 8, 1, 16, "bf16", 64, 256, [4096]), (20, 12, 1, 16, "fp8_e4m3", 64, 256, [4096]), (9, 28, 2, 32, "bf16", 64, 256, [4000, 70, 0]),
    (7, 31, 1, 32, "bf16", 16, 500, [1000]), (3, 32, 1, 32, "bf16", 64, 500, [1000]), (30, 8, 1, 16, "bf16", 64, 157, [10000] + 29 * [500]),
    (6, 31, 1, 8, "f32", 64, 125, [1000]), (16, 16, 1, 16, "bf16", 64, 256, [4096])])
def test_uniform_chunks_of_short_sequences(mla, B, splits, T, H, cache, page, width, lens):
    """Sequences much shorter than the page table is wide, or than the longest of the batch: as many chunks as the request gives
    them, whatever number would make one round of workgroups were all of them full (chunks of such a round left fewer workgroups
    with more pages each: 30 sequences of 4096 tokens in a table of 16384 took 1.6 times as long)."""
    w = synth.make_workload("short", B=B, H=H, d_head=128, d_c=256, d_rope=64, seq_lens=[lens[i % len(lens)] for i in range(B)],
                            io_dtype="f32" if cache == "f32" else "bf16", cache_dtype=cache, page_size=page, free_frac=0.1, seed=137)
    table = np.full((B, width), -1, dtype=np.int32)
    table[:, :w.page_table.shape[1]] = w.page_table
    lse, _ = partials(mla, w, table, T, splits, 0)
    S = cut(B, T * H, splits, False)[1]
    got = np.isfinite(lse[:B * T * H * S].reshape(B, T * H, S))
    first = np.arange(S) * -(-width // S) * page                   # of every chunk
    seen = np.asarray(w.seq_lens)[:, None] - (T - 1 - np.arange(T * H) // H)
    assert (got == (first < seen[..., None])).all()


@pytest.mark.parametrize("B,splits,H,cache", [(129, 3, 16, "bf16"), (130, 4, 64, "bf16"), (70, 4, 64, "fp8_e4m3"), (170, 3, 32, "bf16"), (100, 4, 128, "bf16"),
                                              (70, 4, 16, "bf16"), (100, 4, 28, "fp8_e4m3"), (40, 8, 64, "bf16"), (200, 2, 32, "bf16"), (64, 4, 16, "bf16")])
def test_balanced_ranges_of_one_round(mla, B, splits, H, cache):
    """Fewer ranges than asked for only where a workgroup of the one round has no more pages than the rounds of the others add up
    to, and the round fills more than half of the chip (129 sequences, one range each where three were asked for: 1.13 times as
    long); the plan names the ranges of exactly that number."""
    w = synth.make_workload("ranges", B=B, H=H, d_head=128, d_c=256, d_rope=64, seq_lens=[(97 * i) % 700 for i in range(B)],
                            io_dtype="bf16", cache_dtype=cache, free_frac=0.1, seed=138)
    _, plan = partials(mla, w, w.page_table, 1, splits, mla.FLAG_BALANCED)
    G = B * cut(B, H, splits, True)[1]
    pages = -(-np.asarray(w.seq_lens, dtype=np.int64) // 64)
    end, total = np.cumsum(pages), int(pages.sum())
    first, last = ((end - pages + 1) * G - 1) // total, (end * G - 1) // total
    want = np.where(pages[:, None] > 0, np.stack([first + np.arange(B), last - first + 1], 1), 0)
    assert (plan == want).all()


@pytest.mark.parametrize("L,drop,late", [(4095, (), 0), (4096, (62, 63), 0), (4097, (64,), 0), (4161, (), 4100), (8191, (63, 64, 127), 8190), (16449, (255, 256), 0)])
def test_prefill_page_ids_64_at_a_time(mla, L, drop, late):
    """Contexts around 64 and 256 pages, whose ids a wavefront holds 64 at a time: pages outside the pool on both sides of a border (the
    oracle gets the sequence without them), and a dominant late key, after which the sweeps start again from the first page."""
    import torch
    T, H, d_c = 3, 2, 256
    w = synth.make_workload("prefill", B=1, H=H, d_head=128, d_c=d_c, d_rope=64, seq_lens=[L], io_dtype="bf16", cache_dtype="bf16",
                            free_frac=0.1, seed=134)
    if late:                                          # that token's rope part points along the last query's
        qn, qr = synth.multi_queries(w, T)
        w.pool[w.page_table[0, late // 64], late % 64, d_c:] = synth.store(50.0 * oracle.widen(qr[0, -1, 0]).astype(np.float32), "bf16")
    qn, qr = synth.multi_queries(w, T)
    bad, pt, n = w.page_table.copy(), w.page_table.copy(), w.seq_lens.copy()
    for i in sorted(drop, reverse=True):
        bad[0, i] = w.num_pages + 3 if i % 2 else -1
        n[0] -= min(64, n[0] - 64 * i)
        pt[0] = np.append(np.delete(pt[0], i), -1)
    d = DeviceWorkload(w)
    got, lse = mla.prefill_mha(to_torch(qn, "bf16"), to_torch(qr, "bf16"), d.W_UK, d.W_UV, d.pool, to_torch(bad, "i32"), d.seq_lens,
                               w.softmax_scale, return_lse=True)
    torch.cuda.synchronize()
    ref, ref_lse = oracle.prefill_explicit(qn, qr, w.W_UK, w.W_UV, w.pool, None, pt, n, w.softmax_scale, w.d_c)
    if 63 in drop and L == 4096:                      # the newest page is not there: earlier tokens' limits lie in the one before it
        ref, ref_lse, got, lse = ref[:, -1:], ref_lse[:, -1:], got[:, -1:], lse[:, -1:]
    assert max_abs_rel(widen_gpu(got), ref) <= TOL["bf16"]
    assert lse_err(widen_gpu(lse), ref_lse) <= 2e-2 * max(1.0, np.abs(ref_lse).max() / 30)


@pytest.mark.parametrize("by", [2, 4, 6])
@pytest.mark.parametrize("B,T,H,d_c,lens,drop", [(1, 3, 2, 256, [5], []), (3, 100, 4, 512, [100, 700, 129], [(1, 3)]), (2, 130, 28, 256, [4200, 131], [(0, 0), (0, 64)])])
def test_prefill_of_a_cache_off_its_16_bytes(mla, B, T, H, d_c, lens, drop, by):
    """The cache as a view into a larger buffer, `by` values behind a multiple of 16 bytes: the bits of the call on an aligned one,
    with pages outside the pool and NaN in free pages and behind the sequences' ends."""
    import torch
    w = synth.make_workload("prefill", B=B, H=H, d_head=128, d_c=d_c, d_rope=64, seq_lens=lens, io_dtype="bf16", cache_dtype="bf16",
                            free_frac=0.1, seed=139)
    d = DeviceWorkload(w)
    qn, qr = (to_torch(a, "bf16") for a in synth.multi_queries(w, T))
    table = w.page_table.copy()
    for b, i in drop:
        table[b, i] = w.num_pages + 1 if i % 2 else -1
    table = to_torch(table, "i32")
    room = torch.full((d.pool.numel() + 16,), float("nan"), dtype=torch.bfloat16, device="cuda")
    assert room.data_ptr() % 16 == 0
    view = room[by:by + d.pool.numel()].view(d.pool.shape)
    view.copy_(d.pool)
    assert view.data_ptr() % 16 == 2 * by

    def run(pool):
        ws = torch.full((mla.prefill_workspace_bytes(B, H, d_c, table.shape[1]),), 0xFF, dtype=torch.uint8, device="cuda")
        return mla.prefill_mha(qn, qr, d.W_UK, d.W_UV, pool, table, d.seq_lens, w.softmax_scale, return_lse=True, workspace=ws)

    (a, la), (c, lc) = run(d.pool), run(view)
    torch.cuda.synchronize()
    assert torch.isfinite(a.float()).all()
    assert torch.equal(a.view(torch.int16), c.view(torch.int16)) and torch.equal(la.view(torch.int32), lc.view(torch.int32))


def weights_in_lds(B, T, lens, H, d_c):
    """The launcher's choice between the two kernels that write the keys and values."""
    pages = B * max(1, max((n + 63) // 64 for n in lens))
    return (pages * H <= 2560 and (d_c == 512 or T <= 3072)) or (d_c == 256 and T <= 512 and B * H >= 224)


@pytest.mark.parametrize("T,lens,H,d_c,drop,in_lds", [
    (2, [31, 32, 33, 63, 64, 65, 1, 0], 3, 256, (), True), (2, [31, 32, 33, 63, 64, 65, 1, 0], 3, 512, (), True),   # half pages, whole, one row
    (1, [(131 * i) % 190 for i in range(40)], 28, 256, ((7, 1), (39, 0), (2, 0)), True),     # more pages than pairs of wavefronts
    (1, [(131 * i) % 190 for i in range(30)], 28, 512, ((7, 1), (29, 0), (2, 0)), True),     # 2520 pages x heads
    (2, [700, 129, 0, 64, 250], 3, 256, ((0, 0), (0, 9), (4, 2)), True), (2, [700, 129, 0, 64, 250], 3, 512, ((0, 0), (0, 9), (4, 2)), True),
    (3, [1400, 33, 0, 129, 64], 28, 512, ((0, 0), (0, 20)), False), (2, [1400, 33, 0, 129, 64], 28, 256, ((0, 0), (0, 20)), False),
    (1, [1251, 31, 63, 128], 32, 512, (), True), (1, [1281, 31, 63, 128], 32, 256, (), False),     # 2560 pages x heads, 2688
    (1, [730, 31, 63, 128, 0, 1, 200, 333], 28, 256, ((7, 5),), True),                       # 224 pairs of sequence and head
    (1, [850, 31, 63, 128, 0, 1, 200], 28, 256, ((0, 13),), False),                          # 196
    (1, [(37 * i) % 65 for i in range(256)], 32, 256, (), True), (1, [(37 * i) % 65 for i in range(256)], 32, 512, (), False),
    (3072, [3072], 1, 256, (), True), (3073, [3073], 1, 256, (), False)])
def test_prefill_materialised_rows(mla, T, lens, H, d_c, drop, in_lds):
    """Keys and values of both kernels that write them: sequences that end inside, at and after a half page, empty
    ones, pages outside the pool; the tokens of such a page count as absent."""
    assert weights_in_lds(len(lens), T, lens, H, d_c) == in_lds
    import torch
    w = synth.make_workload("prefill", B=len(lens), H=H, d_head=128, d_c=d_c, d_rope=64, seq_lens=lens, io_dtype="bf16",
                            cache_dtype="bf16", free_frac=0.1, seed=131)
    bad, pt, n = w.page_table.copy(), w.page_table.copy(), w.seq_lens.copy()
    for b, i in sorted(drop, reverse=True):           # the oracle gets the sequence without that page
        bad[b, i] = w.num_pages + 3 if i else -1
        if i * 64 < n[b]:
            n[b] -= min(64, n[b] - 64 * i)
            pt[b] = np.append(np.delete(pt[b], i), -1)
    d = DeviceWorkload(w)
    qn, qr = synth.multi_queries(w, T)
    got, lse = mla.prefill_mha(to_torch(qn, "bf16"), to_torch(qr, "bf16"), d.W_UK, d.W_UV, d.pool, to_torch(bad, "i32"), d.seq_lens,
                               w.softmax_scale, return_lse=True)
    torch.cuda.synchronize()
    ref, ref_lse = oracle.prefill_explicit(qn, qr, w.W_UK, w.W_UV, w.pool, None, pt, n, w.softmax_scale, w.d_c)
    assert max_abs_rel(widen_gpu(got), ref) <= TOL["bf16"]
    assert lse_err(widen_gpu(lse), ref_lse) <= 2e-2


@pytest.mark.parametrize("d_c", [256, 512])
@pytest.mark.parametrize("lens", [[(37 * i) % 130 for i in range(200)], [0] * 70 + [65, 0, 128] + [0] * 64 + [1], [1] * 64 + [64] * 64, [0] * 130])
def test_prefill_of_many_sequences(mla, lens, d_c):
    """The sequences of a call in groups of 64, one per lane: whole groups and a part of one, empty sequences at their
    ends, groups without a row."""
    from test_gpu_parity import check_prefill
    w = synth.make_workload("prefill", B=len(lens), H=2, d_head=128, d_c=d_c, d_rope=64, seq_lens=lens, io_dtype="bf16",
                            cache_dtype="bf16", free_frac=0.1, seed=132)
    check_prefill(mla, w, 1)


@pytest.mark.parametrize("H,B,pages,by_page", [(8, 32, 5, False), (8, 28, 6, True), (16, 16, 10, False), (16, 16, 11, True), (24, 12, 14, True),
                                               (32, 8, 24, False), (32, 8, 25, True), (40, 6, 41, False)])
def test_prefill_order_of_the_workgroups(mla, H, B, pages, by_page):
    """Multiples of eight heads with their weights in LDS: workgroups of a head, or of a page, first."""
    from test_gpu_parity import check_prefill
    lens = [pages * 64 - (29 * b) % 64 for b in range(B)]
    assert weights_in_lds(B, 1, lens, H, 256) and (H <= 32 and B * pages > max(160, 6 * H)) == by_page
    w = synth.make_workload("prefill", B=B, H=H, d_head=128, d_c=256, d_rope=64, seq_lens=lens, io_dtype="bf16",
                            cache_dtype="bf16", free_frac=0.1, seed=133)
    check_prefill(mla, w, 1)


@pytest.mark.parametrize("T,L,late", [(200, 210, 150), (200, 225, 153), (129, 129, 128), (300, 331, 169), (256, 260, 132), (140, 191, 180)])
def test_prefill_later_tokens_stay_out_whatever_they_hold(mla, T, L, late):
    """A token behind every query of a group of 128, in the group's last tile of 32 (and in later ones), whose latent
    row is infinite or NaN: the group's outputs keep the bits that they have without it."""
    import torch
    w = synth.make_workload("prefill", B=1, H=2, d_head=128, d_c=256, d_rope=64, seq_lens=[L], io_dtype="bf16",
                            cache_dtype="bf16", free_frac=0.1, seed=103)
    d = DeviceWorkload(w)
    qn, qr = (to_torch(a, "bf16") for a in synth.multi_queries(w, T))

    def run(pool):
        return mla.prefill_mha(qn, qr, d.W_UK, d.W_UV, pool, d.page_table, d.seq_lens, w.softmax_scale, return_lse=True)

    clean, clean_lse = run(d.pool)
    assert late >= L - T + 128                                   # behind what the first 128 queries see
    for value in (float("inf"), float("nan")):
        pool = d.pool.clone()
        for t in range(late, L, 7):
            pool[int(w.page_table[0, t // 64]), t % 64, t % 256] = value
        out, lse = run(pool)
        torch.cuda.synchronize()
        assert torch.isfinite(out[:, :128]).all() and torch.equal(out[:, :128], clean[:, :128])
        assert torch.equal(lse[:, :128], clean_lse[:, :128])


# ------------------------------------------------------------------ conversion: eigensolver

@pytest.mark.parametrize("batch,m", [(1, 129), (2, 144), (1, 160), (1, 161), (1, 175), (1, 300), (5, 2), (3, 3), (4, 17), (2, 96), (2, 127), (1, 128)])
def test_sym_eig_block_edges(mla, batch, m):
    """Orders around whole and half blocks of 16 and pairs of 32 (an odd count of blocks has a bye, a last block few
    indices), and the one-workgroup kernel with and without a bye, in LDS and past it: A U = U diag(evals),
    orthogonal U, LAPACK's eigenvalues, to fp64 rounding of an order-m sum."""
    import torch
    from paper_2502_07864_amd import convert
    r = synth.stream(111, m)
    X = r.standard_normal((batch, m, m)) * (1.0 + np.arange(m)) ** -0.8
    A = X.transpose(0, 2, 1) @ X
    evals, U, info = convert.sym_eig(torch.from_numpy(A).cuda())
    torch.cuda.synchronize()
    evals, U = evals.cpu().numpy(), U.cpu().numpy()
    assert (info.cpu().numpy() >= 1).all()
    for b in range(batch):
        norm = np.linalg.norm(A[b])
        assert np.abs(U[b].T @ U[b] - np.eye(m)).max() <= 1e-12
        assert np.abs(A[b] @ U[b] - U[b] * evals[b]).max() <= 1e-12 * norm
        assert np.abs(evals[b] - np.linalg.eigvalsh(A[b])[::-1]).max() <= 1e-12 * norm


@pytest.mark.parametrize("kind,m", [("rank", 256), ("rank", 144), ("clusters", 256)])
def test_sym_eig_low_rank_and_multiple_eigenvalues_converge(mla, kind, m):
    """Matrices of few distinct eigenvalues take the solver over pairs of blocks 15 to 20 sweeps, more than the 16 that
    single rotations over the whole matrix needed at most: still converged, and as a Rayleigh-Ritz matrix too."""
    import torch
    from paper_2502_07864_amd import convert
    r = np.random.default_rng(0)
    mats = []
    for k in ((10, 40, 100) if kind == "rank" else (2, 3, 5)):
        if kind == "rank":
            X = r.standard_normal((m, k))
            A = X @ X.T
        else:
            q, _ = np.linalg.qr(r.standard_normal((m, m)))
            d = np.repeat(np.arange(k, 0, -1.0), [m // k] * (k - 1) + [m - (k - 1) * (m // k)]) + 1e-6 * r.standard_normal(m)
            A = (q * d) @ q.T
        mats.append((A + A.T) / 2)
    A = np.stack(mats)
    evals, U, info = convert.sym_eig(torch.from_numpy(A).cuda())
    evals, U, info = evals.cpu().numpy(), U.cpu().numpy(), info.cpu().numpy()
    assert (info >= 1).all(), info
    for b in range(len(A)):
        norm = np.linalg.norm(A[b])
        assert np.abs(U[b].T @ U[b] - np.eye(m)).max() <= 1e-12
        assert np.abs(A[b] @ U[b] - U[b] * evals[b]).max() <= 1e-12 * norm
    if kind == "rank":
        # a block as wide as the space that is not iterated at all: the Rayleigh-Ritz matrix is a rotated S
        ritz, _, info = convert.top_eig(torch.from_numpy(A[0]).cuda(), torch.from_numpy(r.standard_normal((m, m))).cuda(), 10, 0)
        assert info[1].item() >= 1, info
        assert np.abs(ritz.cpu().numpy()[:10] - np.linalg.eigvalsh(A[0])[::-1][:10]).max() <= 1e-10 * np.linalg.norm(A[0])


@pytest.mark.parametrize("m", [64, 65, 80, 81, 96, 97, 127, 128, 129, 143, 144, 145, 161, 176, 177, 300])
def test_ritz_matrix_block_edges(mla, m):
    """The solver with a second matrix of scratch (Rayleigh-Ritz matrices above order 64): a block as wide as the space, so that
    the matrix is S in another basis.  Odd and even numbers of blocks of 16, a last one of one row and a full one; the bounds
    of the eigensolver by itself."""
    import torch
    from paper_2502_07864_amd import convert
    r = np.random.default_rng(m)
    S = r.standard_normal((m, m))
    S = S + S.T
    evals, R, info = convert.top_eig(torch.from_numpy(S).cuda(), torch.from_numpy(r.standard_normal((m, m))).cuda(), m, 0)
    evals, R = evals.cpu().numpy(), R.cpu().numpy()
    norm = np.linalg.norm(S)
    assert info[0].item() == 0 and info[1].item() >= 1
    assert np.abs(evals - np.linalg.eigvalsh(S)[::-1]).max() <= 1e-12 * norm
    assert np.abs(R.T @ R - np.eye(m)).max() <= 1e-12
    assert np.abs(S @ R - R * evals).max() <= 1e-12 * norm


@pytest.mark.parametrize("m,p,rank", [(80, 80, 20), (96, 96, 40), (128, 128, 20), (288, 144, 100), (144, 144, 72), (144, 144, 40), (176, 176, 88), (192, 192, 40),
                                      (200, 150, 100), (200, 200, 100), (256, 256, 40), (256, 256, 100), (300, 300, 100), (300, 300, 150), (400, 360, 100)])
def test_ritz_matrix_of_low_rank_without_iterations(mla, m, p, rank):
    """A block that was not iterated over a moment of low rank: the Rayleigh-Ritz matrix is no nearer to diagonal than any, and its
    solver runs until it is (16 sweeps, enough after one iteration, stopped ranks of a half and a third short)."""
    import torch
    from paper_2502_07864_amd import convert
    r = np.random.default_rng(m + rank)
    X = r.standard_normal((m, rank))
    S, Q0 = X @ X.T, r.standard_normal((m, p))
    evals, R, info = convert.top_eig(torch.from_numpy(S).cuda(), torch.from_numpy(Q0).cuda(), p, 0)
    evals, R = evals.cpu().numpy(), R.cpu().numpy()
    assert info[0].item() == 0 and info[1].item() >= 1
    Q = np.linalg.qr(Q0)[0]
    norm = np.linalg.norm(S)
    assert np.abs(evals - np.linalg.eigvalsh(Q.T @ S @ Q)[::-1]).max() <= 1e-11 * norm
    assert np.abs(R.T @ R - np.eye(p)).max() <= 1e-12
    assert np.abs(R.T @ S @ R - np.diag(evals)).max() <= 1e-12 * norm


@pytest.mark.parametrize("m,p,values,ratio,iters,seed", [(266, 170, 2, .95, 4, 1370), (208, 164, 2, .999, 40, 3493), (164, 129, 2, .99, 12, 2561), (255, 165, 2, .999, 1, 132),
                                                         (172, 140, 2, .999, 8, 2064), (230, 180, 3, .999, 12, 2673), (283, 185, 2, .999, 40, 3593), (307, 228, 3, .999, 3, 865)])
def test_ritz_matrix_of_few_eigenvalues(mla, m, p, values, ratio, iters, seed):
    """A moment of two or three eigenvalues, each many times, after some iterations: its Rayleigh-Ritz matrix takes up to 18 sweeps where
    rotations inside the blocks at every step took 16."""
    import torch
    from paper_2502_07864_amd import convert
    r = np.random.default_rng(seed)
    V = np.linalg.qr(r.standard_normal((m, m)))[0]
    S = (V * np.repeat(ratio ** np.arange(values), -(-m // values))[:m]) @ V.T
    S = (S + S.T) / 2
    evals, R, info = convert.top_eig(torch.from_numpy(S).cuda(), torch.from_numpy(r.standard_normal((m, p))).cuda(), p, iters)
    evals, R = evals.cpu().numpy(), R.cpu().numpy()
    assert info[0].item() == 0 and info[1].item() >= 1
    assert np.abs(R.T @ R - np.eye(p)).max() <= 1e-12
    assert np.abs(R.T @ S @ R - np.diag(evals)).max() <= 1e-12 * np.linalg.norm(S)


@pytest.mark.parametrize("g,d,M", [(33, 8, 2), (17, 16, 4), (32, 16, 4), (64, 4, 2)])
def test_wide_groups_as_a_batch(mla, g, d, M):
    """Groups of 66 to 128 components: the layer's bases from the solver over pairs of blocks, all groups at once, against the
    one-workgroup solver's on the same moments (eigenvalues, and the projector on the leading half)."""
    import torch
    from paper_2502_07864_amd import convert
    r = np.random.default_rng(g * d)
    n, D, p = 150, 64, 20
    t = lambda *s: torch.from_numpy(r.standard_normal(s)).cuda()
    X, W_K, W_V = t(n, D) * torch.arange(1, D + 1, device="cuda", dtype=torch.float64) ** -0.7, t(g * d, D), t(g * d, D)
    out = convert.convert_layer(X, W_K, W_V, t(2 * g * d - d // M, p), g, g, d, M, 8, 3, keep=1)
    sigma = convert.rope_moments(convert.project(X, W_K), g, d, M)
    evals, U, info = convert.sym_eig(sigma)
    assert (out["info"][:-2] >= 1).all() and (info >= 1).all()
    scale = evals[:, :1]
    assert ((out["evals_rope"] - evals).abs() <= 1e-12 * scale).all()
    half = evals.shape[1] // 4
    for a, b in zip(out["U"], U):
        assert (a.T @ a - torch.eye(len(a), device="cuda", dtype=torch.float64)).abs().max() <= 1e-12
        pa, pb = a[:, :half] @ a[:, :half].T, b[:, :half] @ b[:, :half].T
        assert (pa - pb).abs().max() <= 1e-8


# ------------------------------------------------------------------ cache append

@pytest.mark.parametrize("B,D,d_c,cache", [(1, 32, 16, "bf16"), (15, 96, 512, "bf16"), (16, 4096, 512, "f32"),
                                           (17, 4128, 64, "bf16"), (64, 1056, 512, "f32"), (65, 1024, 512, "bf16"),
                                           (128, 256, 256, "bf16"), (3, 8192, 240, "f32"), (3, 8224, 512, "bf16")])
def test_cache_append_edges(mla, B, D, d_c, cache):
    """bf16 projections around the borders of the one-kernel form (16 rows, 32 and 64 deep, 16 columns, one round of the
    chip) against float64; rows with a position or page out of range, and everything else in the pool, untouched."""
    import torch
    n, rng = d_c + 64, np.random.default_rng(B + D)
    x = synth.store(rng.standard_normal((B, D)).astype(np.float32), "bf16")
    W = synth.store((rng.standard_normal((D, n)) / np.sqrt(D)).astype(np.float32), "bf16")
    table = (np.arange(B)[:, None] * 2 + np.arange(2)).astype(np.int32)
    pos = rng.integers(0, 32, B).astype(np.int32)
    good = np.ones(B, bool)
    if B > 4:
        pos[1], pos[2], good[1:3] = -1, 32, False
        table[3], good[3] = 2 * B, False
    start = torch.full((2 * B, 16, n), 7.0, dtype=torch.float32 if cache == "f32" else torch.bfloat16, device="cuda")
    pool = start.clone()
    mla.cache_append(to_torch(x, "bf16"), to_torch(W, "bf16"), pool, to_torch(table, "i32"), to_torch(pos, "i32"), d_c)
    torch.cuda.synchronize()
    x64, W64 = oracle.widen(x).astype(np.float64), oracle.widen(W).astype(np.float64)
    ref = x64 @ W64
    turn = pos[:, None] * 10000.0 ** (-2.0 * np.arange(32) / 64)
    re, im = ref[:, d_c::2].copy(), ref[:, d_c + 1::2].copy()
    ref[:, d_c::2], ref[:, d_c + 1::2] = re * np.cos(turn) - im * np.sin(turn), re * np.sin(turn) + im * np.cos(turn)
    # fp32 sums of D products in some order: D 2^-24 of the sum of magnitudes at most; both components of a pair
    # enter the turned ones (|cos| + |sin| <= 1.5); then the cache's rounding
    mag = np.abs(x64) @ np.abs(W64)
    mag[:, d_c:] = 1.5 * np.repeat(np.maximum(mag[:, d_c::2], mag[:, d_c + 1::2]), 2, axis=1)
    tol = D * 2.0 ** -24 * mag + (2.0 ** -23 if cache == "f32" else 2.0 ** -8) * np.abs(ref)
    got, rows = widen_gpu(pool), np.arange(B)[good]
    at = table[rows, pos[rows] // 16], pos[rows] % 16
    assert (np.abs(got[at] - ref[rows]) <= tol[rows]).all()
    got[at] = 7.0
    assert (got == 7.0).all()


# ------------------------------------------------------------------ conversion: symmetric products

@pytest.mark.parametrize("n,m", [(1, 2), (17, 127), (40, 128), (33, 129), (300, 300), (64, 1000)])
def test_joint_moment_mirrored_tiles(n, m):
    """C^T C / n where only the tiles on and above the diagonal are multiplied: float64 values, and the bits of an
    entry and its mirror image."""
    import torch
    from paper_2502_07864_amd import convert
    C = np.random.default_rng(n + m).standard_normal((n, m))
    K, V = (torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (C[:, :m // 2], C[:, m // 2:]))
    S, _ = convert.joint_moment(K, V, torch.ones(1, dtype=torch.float64, device="cuda"))
    S = S.cpu().numpy()
    assert np.abs(S - C.T @ C / n).max() <= 2 * n * 2.0 ** -53 * (np.abs(C).T @ np.abs(C) / n).max()
    assert np.array_equal(S, S.T)


# ------------------------------------------------------------------ conversion: Cholesky factor and inverse

@pytest.mark.parametrize("p", [2, 5, 16, 17, 63, 64, 65, 100, 128, 191, 300])
def test_cholesky_qr_block_edges(mla, p):
    """Block widths around the 64-column blocks and their 16-column parts.  With S = I every step keeps the span of the
    start block: R is an orthonormal basis of it to fp64 rounding of the sums of 2p products (the start block's
    condition number is about (sqrt 2 + 1)^2 = 6: 64 leaves that and the ten or so products room)."""
    import torch
    from paper_2502_07864_amd import convert
    m = 2 * p + 3
    Q0 = np.random.default_rng(p).standard_normal((m, p))
    evals, R, info = convert.top_eig(torch.eye(m, dtype=torch.float64, device="cuda"), torch.from_numpy(Q0).cuda(), p, 1)
    evals, R, info = evals.cpu().numpy(), R.cpu().numpy(), info.cpu().numpy()
    tol = 64 * m * 2.0 ** -53
    assert info[0] == 0
    assert np.abs(evals - 1.0).max() <= tol
    assert np.abs(R.T @ R - np.eye(p)).max() <= tol
    assert np.abs(Q0 - R @ (R.T @ Q0)).max() <= tol * np.abs(Q0).max()


@pytest.mark.parametrize("m,seed", [(200, 0), (256, 0), (256, 1), (256, 2), (256, 3)])
def test_sym_eig_of_three_multiple_eigenvalues(mla, m, seed):
    """Eigenvalues 1, 2 and 3, a third of the order each: the slowest spectrum for sweeps over pairs of blocks still converges."""
    import torch
    from paper_2502_07864_amd import convert
    Q, _ = np.linalg.qr(synth.stream(112 + seed, m).standard_normal((m, m)))
    want = np.arange(m) // (m // 3) + 1.0
    A = (Q * want) @ Q.T
    A = (A + A.T) / 2
    evals, U, info = convert.sym_eig(torch.from_numpy(A[None]).cuda())
    evals, U = evals.cpu().numpy()[0], U.cpu().numpy()[0]
    assert int(info[0]) >= 1
    assert np.abs(U.T @ U - np.eye(m)).max() <= 1e-12
    assert np.abs(evals - np.sort(want)[::-1]).max() <= 1e-12 * np.linalg.norm(A)
    assert np.abs(A @ U - U * evals).max() <= 1e-12 * np.linalg.norm(A)


# ------------------------------------------------------------------ conversion: matrix product, steps of K and strides

@pytest.mark.parametrize("n,m,D", [(1, 1, 1), (3, 129, 15), (128, 128, 16), (129, 5, 17), (200, 260, 47), (2, 3, (1 << 22) + 4)])
def test_fp64_product_edges(mla, n, m, D):
    """X W^T around the 128-row tiles and the 16-deep steps (a last step of 1, 15, 16 columns), and with rows further
    apart than 32-bit offsets within a tile reach: sums of D products in another order."""
    import torch
    from paper_2502_07864_amd import convert
    rng = np.random.default_rng(n + m)
    X, W = rng.standard_normal((n, D)), rng.standard_normal((m, D))
    Y = convert.project(torch.from_numpy(X).cuda(), torch.from_numpy(W).cuda()).cpu().numpy()
    assert (np.abs(Y - X @ W.T) <= 2 * min(D, 1 << 12) * 2.0 ** -53 * (np.abs(X) @ np.abs(W).T)).all()


# ------------------------------------------------------------------ projections: rows, depths and column tiles

@pytest.mark.parametrize("H,K,N", [(1, 32, 16), (5, 96, 48), (8, 128, 512), (28, 160, 128), (32, 256, 128), (3, 288, 32), (64, 512, 128)])
@pytest.mark.parametrize("B", [1, 15, 16, 17, 32, 33, 64, 65])
def test_bf16_projection_row_groups_and_depths(mla, B, H, K, N):
    """One, two and more 16-row groups, one workgroup of them and two, against fp32: one bf16 rounding of the result and sums of
    K products of bf16 values in another order."""
    import torch
    gen = torch.Generator(device="cuda").manual_seed(B * 1000 + K)
    X = torch.randn(B, H, K, device="cuda", generator=gen).bfloat16()
    W = (torch.randn(H, K, N, device="cuda", generator=gen) * K ** -0.5).bfloat16()
    got = mla.absorb_q(X, W).float()
    ref = torch.matmul(X.float().transpose(0, 1).contiguous(), W.float()).transpose(0, 1)
    assert (got - ref).abs().max().item() <= (2.0 ** -8 + K * 2.0 ** -24) * ref.abs().max().item()


def bf16_column_tile(B, H, K, N):
    """The launcher's column tile: the widest that divides N, whose slab of W fits LDS and that gives a workgroup per CU, else the
    narrowest."""
    fits = [t for t in (64, 32, 16) if N % t == 0 and K * (2 * t + 16) <= 40 * 1024]
    return next((t for t in fits if t > 16 and H * (N // t) * ((B + 63) // 64) >= 256), fits[-1])


@pytest.mark.parametrize("tile,H,N,K", [(*shape, K) for shape in ((16, 2, 48), (32, 86, 96), (64, 64, 256))
                                        for K in range(32, (257 if shape[0] == 64 else 513), 32)])
def test_bf16_projection_column_tiles_at_every_depth(mla, tile, H, N, K):
    """16, 32 and 64 columns at both depths of every class, every split of the wavefronts over up to 16, 32 and more rows, against
    fp32 as above."""
    import torch
    gen = torch.Generator(device="cuda").manual_seed(tile + K)
    X = torch.randn(65, H, K, device="cuda", generator=gen).bfloat16()
    W = (torch.randn(H, K, N, device="cuda", generator=gen) * K ** -0.5).bfloat16()
    ref = torch.matmul(X.float().transpose(0, 1).contiguous(), W.float()).transpose(0, 1)
    for B in (1, 16, 17, 32, 33, 64, 65):
        assert bf16_column_tile(B, H, K, N) == tile
        err = (mla.absorb_q(X[:B].contiguous(), W).float() - ref[:B]).abs().max().item()
        assert err <= (2.0 ** -8 + K * 2.0 ** -24) * ref[:B].abs().max().item()


@pytest.mark.parametrize("H,K,N", [(28, 128, 256), (28, 256, 128), (32, 512, 128), (32, 128, 256), (64, 352, 128), (32, 128, 512)])
def test_bf16_projection_rows_keep_their_bits_in_any_batch(mla, H, K, N):
    """A row's k-steps are added in the same order whatever the batch, so a row has the same bits alone, among 16 and
    among 70: no tolerance."""
    import torch
    gen = torch.Generator(device="cuda").manual_seed(K + N)
    X = torch.randn(70, H, K, device="cuda", generator=gen).bfloat16()
    W = (torch.randn(H, K, N, device="cuda", generator=gen) * K ** -0.5).bfloat16()
    whole = mla.absorb_q(X, W)
    for B in (1, 7, 16, 17, 33, 64):
        assert torch.equal(mla.absorb_q(X[:B].contiguous(), W), whole[:B])


@pytest.mark.parametrize("H,K,N", [(8, 512, 128), (16, 512, 100), (28, 512, 128), (7, 64, 20)])
@pytest.mark.parametrize("B", [1, 3])
def test_fp32_projection_tiles_of_half_lines(mla, B, H, K, N):
    """Head-major and tile-major workgroup numbers, against fp64."""
    import torch
    gen = torch.Generator(device="cuda").manual_seed(H + N)
    X = torch.randn(B, H, K, device="cuda", generator=gen)
    W = torch.randn(H, K, N, device="cuda", generator=gen) * K ** -0.5
    ref = torch.matmul(X.double().transpose(0, 1).contiguous(), W.double()).transpose(0, 1)
    assert (mla.absorb_q(X, W).double() - ref).abs().max().item() <= K * 2.0 ** -24 * ref.abs().max().item()
