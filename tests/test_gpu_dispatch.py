"""GPU parity at the edges of the launch rules: sizes where a rule picks another kernel, another split
of the work list or another tile count. Oracle and tolerances as in test_gpu_parity (bf16 products with
fp32 sums; the bounds there cover any order of the sums)."""
import ctypes

import numpy as np
import pytest
import torch

import moc_inputs as mi
from paper_2508_21058_amd import binding as mb
from tests import bruteforce as bf
from tests.test_gpu_parity import check_close, run_case

pytestmark = pytest.mark.gpu


# heads that do not divide over the eight slices of the list, streams without captions, streams of
# captions almost alone, and token counts on both sides of a caption segment boundary (256, then N / 4)
@pytest.mark.parametrize("B,H,shots,text,frames,frame", [
    (1, 1, 1, 130, 2, 62),          # one head, two caption tiles, N = 254: one segment
    (1, 3, 2, 33, 2, 70),           # N = 346: two segments, caption tiles of 33 keys
    (3, 3, 1, 257, 1, 40),          # nine slices of the list; N = 297, almost all caption
    (1, 5, 3, 0, 3, 96),            # no caption at all
    (1, 2, 4, 40, 4, 240),          # N = 4000: four segments, the last one ragged
])
def test_key_stationary_work_split(B, H, shots, text, frames, frame):
    lay = mi.multishot_layout(shots, text, frames, frame, frame // 2, "frame") if text else _no_captions(shots, frames, frame)
    run_case(lay, B, H, 64, 2, torch.bfloat16, seed=31 + H)


# caption segments of a tile taken by one workgroup: all four where the call has 256 caption items or more, two
# of four from 171 on, each on its own below; the last segment ragged
@pytest.mark.parametrize("H,text,shots,video", [(64, 500, 1, 600), (70, 129, 2, 1000), (43, 500, 1, 1000), (42, 500, 1, 1000),
                                                (64, 130, 1, 301)])
def test_joined_caption_segments(H, text, shots, video):
    run_case(mi.stream_layout(shots, text, video, 50, "chunk"), 1, H, 64, 1, torch.bfloat16, seed=111 + H)


# video items: heads that every XCD takes whole, heads left over and dealt out two items at a time (up to three of
# them, or 256 items a head), with none, some and only incomplete turns (16 items) among them, heads left in slices
@pytest.mark.parametrize("H,chunks", [(1, 7), (1, 17), (2, 16), (3, 33), (4, 33), (7, 5), (8, 3), (11, 11), (13, 7), (16, 2),
                                      (5, 255), (5, 256)])
def test_video_items_over_the_xcds(H, chunks):
    run_case(mi.stream_layout(1, 9, 21 * chunks, 21, "chunk"), 1, H, 64, 2, torch.bfloat16, seed=81 + H)


def _no_captions(shots, frames, frame):
    offs = np.arange(0, shots * frames * frame + 1, 48, dtype=np.int32)
    C = len(offs) - 1
    per = C // shots
    return mi.Layout("no_captions", offs, (np.arange(C) // per).astype(np.int32), np.arange(C, dtype=np.int32),
                     np.zeros((0, 2), dtype=np.int32))


# a caption longer than the resident rows of the chunk-stationary kernels beside chunks that fit (288),
# and chunks of one key too many (a call this small takes the tiled kernels for both)
@pytest.mark.parametrize("chunk", [288, 289])
def test_routed_chunks_beside_a_long_caption(chunk):
    run_case(mi.multishot_layout(2, 300, 2, 2 * chunk, chunk, "frame"), 1, 2, 128, 2, torch.bfloat16, seed=41)


# routed items of many short chunks (ten keys), the last one of a head cut off
@pytest.mark.parametrize("H", [3, 8, 24])
def test_query_tiles_per_workgroup(H):
    run_case(mi.stream_layout(1, 37, 603, 10, "chunk"), 1, H, 64, 16, torch.bfloat16, seed=61 + H)


# fp32 storage through the same kernels as bf16: both head sizes, ragged last tiles; k = 0 leaves forced
# links alone
@pytest.mark.parametrize("d,chunk,topk", [(64, 33, 3), (128, 288, 2), (128, 300, 2), (64, 300, 1), (128, 65, 0)])
def test_fp32_storage(d, chunk, topk):
    run_case(mi.stream_layout(2, 37, 4 * chunk + 5, chunk, "chunk"), 1, 3, d, topk, torch.float32, seed=51 + chunk)


# fp32 storage without routed links: the forced-link items read the queries as they are stored
@pytest.mark.parametrize("d,chunk,captions", [(64, 33, 37), (64, 129, 0), (128, 257, 0), (128, 31, 140)])
def test_fp32_forced_links_alone(d, chunk, captions):
    run_case(mi.stream_layout(2, captions, 3 * chunk + 5, chunk, "chunk"), 1, 3, d, 0, torch.float32, seed=101 + chunk)


# epilogue of the forced-link items: rows of slots on both sides of the eight that are loaded together, in
# windows of a few queries, with rows of fewer candidates than slots
@pytest.mark.parametrize("topk", [7, 8, 9, 17, 32])
@pytest.mark.parametrize("d", [64, 128])
def test_merged_slots(topk, d):
    run_case(mi.stream_layout(1, 11, 300, 7, "chunk"), 1, 2, d, topk, torch.bfloat16, seed=91 + topk)


# list builder: 3,006 to 99,000 entries a head (one workgroup a head to the general way), rows whose
# slots fill 64 lanes exactly or leave some idle, more chunks than a workgroup has lanes
@pytest.mark.parametrize("N,chunk,topk", [(4096, 64, 8), (4097, 64, 8), (1000, 1, 5), (1002, 1, 3), (2340, 13, 14), (300, 7, 32),
                                          (12000, 9, 7), (9000, 60, 11)])
def test_list_builder_ranges(N, chunk, topk):
    check_lists(N, chunk, topk)


def check_lists(N, chunk, topk, H=3):
    """The lists of random selections against numpy's; -> how they were built: "head" (a workgroup a head), the queries a
    block of the two launches had, or "general". The tables tell: each way writes others."""
    offs = np.unique(np.r_[np.arange(0, N, chunk), N]).astype(np.int32)
    C = len(offs) - 1
    lay = mi.Layout("lists", offs, np.zeros(C, np.int32), np.arange(C, dtype=np.int32),
                    np.asarray([[0, offs[1]]], dtype=np.int32))
    meta = mb.chunk_meta(lay.offsets, lay.shot, lay.window, lay.text_spans)
    g = torch.Generator(device="cuda").manual_seed(N)
    q, k, v = (torch.randn(1, H, N, 64, generator=g, device="cuda").to(torch.bfloat16) for _ in range(3))
    # rows as a caller may write them: repeated, forced and out-of-range entries among them
    sel = torch.randint(-1, C + 1, (1, H, N, topk), generator=g, device="cuda", dtype=torch.int32)
    ws = mb.attn_workspace(meta, 1, H, 64, topk, torch.bfloat16, False)
    ws.fill_(0x7f)
    mb.attn_fwd(meta, q, k, v, sel, workspace=ws)
    torch.cuda.synchronize()
    # the workspace begins with chunk counts, list offsets and tile offsets; the lists come after tables
    # whose sizes follow from the shape (every part 256-byte aligned)
    at, parts = 0, {}
    for name, n in (("cnt", H * C), ("off", H * (C + 1)), ("tile", H * (C + 1)), ("vmask", H * N), ("gsum", H * 32 * C),
                    ("blk", H * -(-N // 256) * C), ("list", H * N * topk)):
        parts[name] = ws[at:at + 4 * n].view(torch.int32).cpu().numpy()
        at += -(-4 * n // 256) * 256
    chunk_of = np.repeat(np.arange(C), np.diff(offs))
    s = sel.cpu().numpy()[0]
    for h in range(H):
        first = np.ones((N, topk), bool)
        for r in range(1, topk):
            first[:, r] = (s[h][:, r:r + 1] != s[h][:, :r]).all(1)
        ok = first & (s[h] >= 1) & (s[h] < C) & (s[h] != chunk_of[:, None])      # chunk 0 is the caption
        assert np.array_equal(parts["vmask"].view(np.uint32)[h * N:(h + 1) * N], (ok.astype(np.uint64) << np.arange(topk, dtype=np.uint64)).sum(1).astype(np.uint32))
        qi, r = np.nonzero(ok)
        order = np.argsort(s[h][qi, r], kind="stable")
        cnt = np.bincount(s[h][qi, r], minlength=C)
        assert np.array_equal(parts["off"][h * (C + 1):(h + 1) * (C + 1)], np.r_[0, np.cumsum(cnt)])
        assert np.array_equal(parts["tile"][h * (C + 1):(h + 1) * (C + 1)], np.r_[0, np.cumsum(-(-cnt // 128))])
        assert np.array_equal(parts["list"][h * N * topk:h * N * topk + len(qi)], ((qi << 5) | r)[order])
    meta.close()
    # log-sum-exps and outputs of the slots follow, then the table of the two launches, where a call has one
    for n in (4 * H * N * (topk + 1), 2 * H * N * (topk + 1) * 64):
        at += -(-n // 256) * 256
    untouched = (parts["blk"] == 0x7f7f7f7f).all()
    if at == ws.numel() * ws.element_size():
        return "head" if untouched else "general"
    assert untouched
    table = ws[at:].view(torch.int32).cpu().numpy()
    rows = [r for r in (64, 128, 256) if -(-4 * H * -(-N // r) * C // 256) * 256 == 4 * len(table)]
    assert len(rows) == 1
    used = table[:H * -(-N // rows[0]) * C].reshape(H, -1, C)
    assert np.array_equal(used.sum(1), parts["off"].reshape(H, C + 1)[:, 1:] - parts["off"].reshape(H, C + 1)[:, :-1])
    return rows[0]


# selection at the list widths the kernel is built for (4, 8, 16, 32) and one past each, over eleven tiles
# of chunks, the last one ragged; scores of both signs, many exact ties (quarter-integer keys,
# one-hot queries), zeros of both signs. Scores are exact in fp32 here, so the order is pinned: higher
# score first, lower chunk on a tie.
@pytest.mark.parametrize("topk", [1, 3, 4, 5, 8, 9, 16, 17, 32])
@pytest.mark.parametrize("levels,dtype", [(1, torch.bfloat16), (3, torch.bfloat16), (200, torch.float32)])
def test_selection_order_and_ties(topk, levels, dtype):
    C, per, H, d = 330, 4, 2, 64
    N = C * per
    rng = np.random.default_rng(topk * 7 + levels)
    kbar = rng.integers(-levels, levels + 1, (H, C, d)) / 4.0
    kbar[:, ::5] *= np.where(rng.random((H, 66, 1)) < 0.5, -0.0, 1.0)
    k = np.repeat(kbar, per, axis=1)[None]
    q = np.zeros((1, H, N, d))
    q[0, np.arange(H)[:, None], np.arange(N)[None], rng.integers(0, d, (H, N))] = rng.choice([-1.0, 1.0], (H, N))
    offs = np.arange(0, N + 1, per, dtype=np.int32)
    meta = mb.chunk_meta(offs, np.zeros(C, np.int32), np.arange(C, dtype=np.int32), None)
    qd, kd = (torch.from_numpy(x).to("cuda").to(dtype).contiguous() for x in (q, k))
    _, sel = mb.route(meta, qd, kd, topk, False)
    sel = sel.cpu().numpy()[0]
    for h in range(H):
        s = q[0, h] @ kbar[h].T
        s[np.arange(N), np.arange(N) // per] = -np.inf                # the own chunk is a forced link
        want = np.argsort(-s, axis=1, kind="stable")[:, :topk]
        assert np.array_equal(sel[h], want)
    meta.close()


# scores that differ only in the products added last: pooled keys whose three bf16 planes are all in use
# and differ only in the third (one-hot queries), and queries whose first two planes cancel and whose third
# meets integer keys. Every product and sum is exact in fp32, so the order is pinned. 21 distinct scores
# among 330 chunks: ties throughout.
@pytest.mark.parametrize("topk", [2, 8, 16, 32])
@pytest.mark.parametrize("where,dtype", [("keys", torch.bfloat16), ("keys", torch.float32), ("queries", torch.float32)])
def test_selection_by_the_last_products(topk, where, dtype):
    C, per, H, d = 330, 4, 2, 128
    N = C * per
    rng = np.random.default_rng(topk)
    t = rng.integers(1, 22, (H, C))
    hi, mid, lo = 1.0, 3 * 2.0 ** -10, 2.0 ** -23
    q, k = np.zeros((1, H, N, d)), np.zeros((1, H, N, d))
    if where == "keys":          # mean of (4 hi, 4 mid, 4 t lo, 0) in every feature; bf16 holds each of them
        rows = np.stack([np.full((H, C), 4 * hi), np.full((H, C), 4 * mid), 4 * t * lo, np.zeros((H, C))], axis=2)
        k[0] = rows.reshape(H, N)[..., None]
        q[0, np.arange(H)[:, None], np.arange(N)[None], rng.integers(0, d, (H, N))] = rng.choice([-1.0, 1.0], (H, N))
    else:                        # features x and y hold the same integer: score = t * lo
        x = rng.permutation(d)[:2]
        k[0, :, :, x] = np.repeat(t, per, axis=1)
        q[0, :, :, x[0]], q[0, :, :, x[1]] = hi + mid + 5 * lo, -(hi + mid)
    offs = np.arange(0, N + 1, per, dtype=np.int32)
    meta = mb.chunk_meta(offs, np.zeros(C, np.int32), np.arange(C, dtype=np.int32), None)
    qd, kd = (torch.from_numpy(a).to("cuda").to(dtype).contiguous() for a in (q, k))
    assert torch.equal(qd.double().cpu(), torch.from_numpy(q)) and torch.equal(kd.double().cpu(), torch.from_numpy(k))
    _, sel = mb.route(meta, qd, kd, topk, False)
    sel = sel.cpu().numpy()[0]
    kbar = k[0].reshape(H, C, per, d).mean(2)
    for h in range(H):
        s = q[0, h] @ kbar[h].T
        s[np.arange(N), np.arange(N) // per] = -np.inf
        assert len(np.unique(s[0])) == 22
        assert np.array_equal(sel[h], np.argsort(-s, axis=1, kind="stable")[:, :topk])
    meta.close()


# a NaN score is no candidate: the chunk never appears, a query of NaN selects nothing
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_nan_scores_are_no_candidates(dtype):
    C, per, d, topk = 70, 4, 64, 5
    N = C * per
    g = torch.Generator().manual_seed(3)
    q, k = (torch.randn(1, 1, N, d, generator=g).to(torch.bfloat16).float() for _ in range(2))
    q[0, 0, 9, 3] = float("nan")
    for c, v in ((2, float("nan")), (40, float("inf")), (69, float("-inf"))):
        k[0, 0, c * per, 5] = v
    offs = np.arange(0, N + 1, per, dtype=np.int32)
    meta = mb.chunk_meta(offs, np.zeros(C, np.int32), np.arange(C, dtype=np.int32), None)
    _, sel = mb.route(meta, q.cuda().to(dtype).contiguous(), k.cuda().to(dtype).contiguous(), topk, False)
    sel = sel.cpu().numpy()[0, 0]
    kbar = k[0, 0].double().numpy().reshape(C, per, d).mean(1)
    s = q[0, 0].double().numpy() @ np.nan_to_num(kbar, nan=0.0, posinf=0.0, neginf=0.0).T
    s[:, [2, 40, 69]] = -np.inf
    s[np.arange(N), np.arange(N) // per] = -np.inf
    want = np.argsort(-s, axis=1, kind="stable")[:, :topk]
    want[9] = -1
    assert np.array_equal(sel, want)
    meta.close()


# routed chunks on both sides of the key tiles, in calls small enough for the tiled kernels
@pytest.mark.parametrize("chunk", [1, 16, 17, 32, 33, 64, 65, 80, 81, 96, 97, 128, 257, 273, 288])
@pytest.mark.parametrize("d", [64, 128])
def test_routed_tile_edges(chunk, d):
    run_case(mi.stream_layout(2, 20, 5 * chunk + (chunk + 1) // 2, chunk, "chunk"), 1, 2, d, 3, torch.bfloat16, seed=71 + chunk)


# The chunk-stationary kernels, which take the routed items from 92 query tiles (of 128 entries) per compute
# unit on: the same edges (64-key tiles, a tail of at most 32 keys, one or two 16-key steps of V), reached by
# many short heads; with one head less the tiled kernels run. Three heads are checked against dense float64.
@pytest.mark.parametrize("chunk,caption,less", [(1, 20, 0), (16, 20, 0), (17, 300, 0), (32, 20, 0), (33, 20, 0), (64, 20, 0),
                                                (65, 20, 1), (80, 20, 0), (96, 20, 0), (97, 20, 0), (128, 300, 1),
                                                (257, 300, 0), (273, 20, 0), (288, 20, 0), (289, 20, 0)])
@pytest.mark.parametrize("d,dtype", [(64, torch.bfloat16), (128, torch.bfloat16), (128, torch.float32)])
def test_routed_items_of_many_heads(chunk, caption, less, d, dtype):
    topk = 4
    lay = mi.stream_layout(1, caption, max(5 * chunk, 500) + (chunk + 1) // 2, chunk, "chunk")
    N = lay.N
    H = -(-92 * 256 * 128 // (N * topk)) - less
    g = torch.Generator(device="cuda").manual_seed(chunk + d)
    q, k, v, d_o = (torch.randn(1, H, N, d, generator=g, device="cuda").bfloat16().to(dtype) for _ in range(4))
    meta = mb.chunk_meta(lay.offsets, lay.shot, lay.window, lay.text_spans)
    _, sel = mb.route(meta, q, k, topk)
    ws = mb.attn_workspace(meta, 1, H, d, topk, dtype, True)
    o, lse = mb.attn_fwd(meta, q, k, v, sel, workspace=ws)
    dq, dk, dv = mb.attn_bwd(meta, q, k, v, o, lse, d_o, sel, workspace=ws, after_fwd=True)
    for h in (0, H // 2, H - 1):
        qn, kn, vn, dn = (x[0, h].double().cpu().numpy() for x in (q, k, v, d_o))
        ref = bf.dense_masked_attention(qn, kn, vn, bf.token_mask(lay, sel[0, h].cpu().numpy()), dn)
        for name, x in (("o", o), ("lse", lse), ("dq", dq), ("dk", dk), ("dv", dv)):
            check_close(name, x[0, h].double().cpu().numpy(), ref[name])
    meta.close()


def _workspace_bytes(meta, H, topk, dtype, with_bwd=True):
    n = ctypes.c_size_t()
    assert mb.lib().moc_attn_workspace_bytes(meta.handle, 1, H, 128, topk, int(dtype == torch.float32), int(with_bwd), ctypes.byref(n)) == 0
    return n.value


def _first_wide_heads(meta, topk, dtype):
    """The number of heads from which the library takes the wide key tiles: there the statistics become records of twice the
    size, for all heads at once, and the workspace grows by more than one head's share. None: never."""
    steps = np.diff([_workspace_bytes(meta, H, topk, dtype) for H in range(1, 1500)])
    jumps = np.nonzero(steps > 1.5 * np.median(steps))[0]
    assert len(jumps) <= 1
    return int(jumps[0]) + 2 if len(jumps) else None


# The key-stationary kernel of wide tiles (256 keys, or the last 160 to 255 of a chunk): tiles on both sides of the least size, of
# three and four filled waves, with a rest and without, captions as such tiles, lists and windows of whole, partly filled and of few
# stages of 16 queries, at the least number of heads it takes a call of; with one head less the other kernel takes all. Two heads
# are checked against dense float64.
@pytest.mark.parametrize("chunk,caption,topk,less", [(159, 300, 2, 0), (160, 20, 2, 0), (192, 512, 1, 0), (193, 256, 3, 0), (256, 256, 2, 0),
                                                     (256, 512, 2, 1), (257, 161, 2, 0), (415, 20, 1, 0), (416, 300, 2, 0),
                                                     (416, 416, 1, 0), (512, 256, 0, 0), (700, 40, 3, 0), (700, 40, 3, 1)])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_wide_key_tiles(chunk, caption, topk, less, dtype):
    lay = mi.stream_layout(1, caption, 4 * chunk, chunk, "chunk")
    N = lay.N
    meta = mb.chunk_meta(lay.offsets, lay.shot, lay.window, lay.text_spans)
    H = _first_wide_heads(meta, topk, dtype) - less
    g = torch.Generator(device="cuda").manual_seed(chunk)
    q, k, v, d_o = (torch.randn(1, H, N, 128, generator=g, device="cuda").bfloat16().to(dtype) for _ in range(4))
    _, sel = mb.route(meta, q, k, topk)
    ws = mb.attn_workspace(meta, 1, H, 128, topk, dtype, True)
    o, lse = mb.attn_fwd(meta, q, k, v, sel, workspace=ws)
    dq, dk, dv = mb.attn_bwd(meta, q, k, v, o, lse, d_o, sel, workspace=ws, after_fwd=True)
    for h in (0, H - 1):
        qn, kn, vn, dn = (x[0, h].double().cpu().numpy() for x in (q, k, v, d_o))
        rows = sel[0, h].cpu().numpy() if topk else np.zeros((N, 0), dtype=np.int32)
        ref = bf.dense_masked_attention(qn, kn, vn, bf.token_mask(lay, rows), dn)
        for name, x in (("o", o), ("lse", lse), ("dq", dq), ("dk", dk), ("dv", dv)):
            check_close(name, x[0, h].double().cpu().numpy(), ref[name])
    again = mb.attn_bwd(meta, q, k, v, o, lse, d_o, sel, workspace=ws)
    assert all(torch.equal(x, y) for x, y in zip((dq, dk, dv), again))
    meta.close()


# Tiles of 160 to 192 keys fill three of the kernel's four waves: it takes a call only if fuller ones, or half of their own lists, stream as many
# queries as their windows have (a caption's is the stream of N = 4 * chunk + caption queries; the lists have N * topk in all).
@pytest.mark.parametrize("chunk,caption,topk,wide", [(160, 160, 0, False), (192, 192, 2, False), (160, 20, 1, False), (160, 20, 2, True),
                                                     (192, 20, 1, False), (192, 20, 2, True), (193, 20, 0, True), (20, 192, 2, False),
                                                     (20, 193, 2, True), (159, 416, 2, True), (192, 256, 0, True), (416, 20, 3, True),
                                                     (256, 192, 0, False), (256, 192, 1, True), (193, 192, 0, False), (193, 192, 1, True)])
def test_three_filled_waves_beside_four(chunk, caption, topk, wide):
    lay = mi.stream_layout(1, caption, 4 * chunk, chunk, "chunk")
    meta = mb.chunk_meta(lay.offsets, lay.shot, lay.window, lay.text_spans)
    assert (_first_wide_heads(meta, topk, torch.bfloat16) is not None) == wide
    meta.close()


# A head of 4 GiB of rows and more: the wide tiles' copies of Q and dO take 64-bit offsets. The last chunk's queries choose the
# first chunk and the one before the last in turn; the three, whose keys nobody else attends, are checked against dense float64.
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_wide_key_tiles_of_a_long_head(dtype):
    lens = [512] + [4096] * 4096 + [512, 512]
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    C, N = len(lens), int(off[-1])
    assert int(off[-3]) * 256 >= 1 << 32
    chunks = np.arange(C, dtype=np.int32)
    meta = mb.chunk_meta(off, np.zeros(C, np.int32), chunks, None)
    # wide: a delta and two records of four words a query (and, with fp32 storage, its dO in bf16)
    assert _workspace_bytes(meta, 1, 1, dtype) - _workspace_bytes(meta, 1, 1, dtype, False) >= N * (36 + 256 * (dtype == torch.float32))
    g = torch.Generator(device="cuda").manual_seed(3)
    q, k, v, d_o = (torch.randn(1, 1, N, 128, generator=g, device="cuda", dtype=torch.bfloat16).to(dtype) for _ in range(4))
    sel = torch.full((1, 1, N, 1), -1, dtype=torch.int32, device="cuda")
    sel[0, 0, off[-2]::2, 0] = 0
    sel[0, 0, off[-2] + 1::2, 0] = C - 2
    ws = mb.attn_workspace(meta, 1, 1, 128, 1, dtype, True)
    o, lse = mb.attn_fwd(meta, q, k, v, sel, workspace=ws)
    dq, dk, dv = mb.attn_bwd(meta, q, k, v, o, lse, d_o, sel, workspace=ws, after_fwd=True)

    def pick(x):
        return torch.cat([x[0, 0, :512], x[0, 0, off[-3]:]]).double().cpu().numpy()

    lay = mi.Layout("three", np.arange(4, dtype=np.int32) * 512, np.zeros(3, np.int32), np.arange(3, dtype=np.int32), np.zeros((0, 2), np.int32))
    rows = np.full((3 * 512, 1), -1, np.int32)
    rows[1024::2], rows[1025::2] = 0, 1
    ref = bf.dense_masked_attention(*(pick(x) for x in (q, k, v)), bf.token_mask(lay, rows), pick(d_o))
    for name, x in (("o", o), ("lse", lse), ("dq", dq), ("dk", dk), ("dv", dv)):
        check_close(name, pick(x), ref[name])
    meta.close()
    del q, k, v, d_o, ws, o, lse, dq, dk, dv
    torch.cuda.empty_cache()


# Padding rows of the wide tiles (the rest of the last stage of a window or a list, and the stages up to a whole turn of the ring):
# a NaN or an infinity in one query's q or dO reaches the keys which that query attends and no others. The first query of the
# stream is a caption's, so it attends the caption alone.
@pytest.mark.parametrize("chunk", [256, 250])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_non_finite_rows_stay_with_their_keys(chunk, dtype):
    lay = mi.stream_layout(1, 256, 4 * chunk, chunk, "chunk")
    H, N, topk = 180, lay.N, 2             # eight wide tiles a head (four of them of the caption), no rest
    g = torch.Generator(device="cuda").manual_seed(chunk)
    q, k, v, d_o = (torch.randn(1, H, N, 128, generator=g, device="cuda").bfloat16().to(dtype) for _ in range(4))
    meta = mb.chunk_meta(lay.offsets, lay.shot, lay.window, lay.text_spans)
    _, sel = mb.route(meta, q, k, topk)
    assert (sel[:, :, 0] == -1).all()

    def grads(q, d_o):
        o, lse = mb.attn_fwd(meta, q, k, v, sel)
        return mb.attn_bwd(meta, q, k, v, o, lse, d_o, sel)[1:]

    clean = grads(q, d_o)
    for value in (float("nan"), float("inf")):
        for which in (0, 1):
            bad = [q.clone(), d_o.clone()]
            bad[which][:, :, 0, 5] = value
            for name, x, y in zip(("dk", "dv"), grads(*bad), clean):
                assert torch.equal(x[:, :, 256:], y[:, :, 256:]), (name, value, which)
                assert not torch.isfinite(x[:, :, :256]).all()
    meta.close()


# regularised rows at the widths the kernel's lists are sized for (8 + 4, 16 + 4, 32) and one past each,
# no routed chunk at all, nothing added, more requested than there are candidates
@pytest.mark.parametrize("topk,max_in", [(8, 4), (8, 5), (7, 5), (16, 4), (16, 5), (0, 3), (20, 12), (32, 0), (1, 31)])
def test_regularised_row_widths(topk, max_in):
    from tests.test_gpu_perturb import _case
    lay = mi.random_layout(90 + topk, n_chunks=45, max_len=31, n_shots=3)
    _case(lay, H=2, d=64, topk=topk, causal=True, p_max=1.0, lam=6.0, max_in=max_in, seed=topk, dtype=torch.bfloat16)


# row gather: tables that travel with the launch (up to 64 ranges) and larger ones, rows of one 16-byte
# word, of an odd number of them and of more than a workgroup moves, several planes, single-row ranges
@pytest.mark.parametrize("n_ranges", [1, 12, 64, 65, 300])
@pytest.mark.parametrize("words", [1, 3, 16, 2500])
def test_gather_table_sizes(n_ranges, words):
    N, outer = 1500, 3
    rng = np.random.default_rng(n_ranges + words)
    src = torch.randint(0, 1 << 15, (outer, N, words * 8), device="cuda", dtype=torch.int16).view(torch.bfloat16)
    ranges = [(int(a), int(rng.integers(0, 14 if n_ranges > 12 else 400))) for a in rng.integers(0, N - 400, n_ranges)]
    rows = np.concatenate([np.arange(a, a + n) for a, n in ranges])
    if rows.size == 0:
        ranges[0], rows = (5, 1), np.array([5])
    got = mb.gather_rows(src, ranges)
    assert torch.equal(got.view(torch.int16), src.view(torch.int16)[:, torch.from_numpy(rows).cuda()])


# many short ranges under one workgroup's words: tables on both sides of a round of the 64-wide search (64, 4096
# entries), more ranges than are walked, one huge range beside single rows; two and eight words a lane
@pytest.mark.parametrize("n_ranges", [65, 4096, 4097, 9000])
@pytest.mark.parametrize("words,outer", [(1, 1), (3, 2), (8, 3), (96, 1)])
def test_gather_of_short_ranges(n_ranges, words, outer):
    N = 7000
    rng = np.random.default_rng(n_ranges + words)
    src = torch.randint(0, 1 << 15, (outer, N, words * 8), device="cuda", dtype=torch.int16).view(torch.bfloat16)
    ranges = [(int(a), 1 + int(rng.random() < 0.1)) for a in rng.integers(0, N - 2, n_ranges)]
    ranges[n_ranges // 2] = (5, N - 5)
    rows = np.concatenate([np.arange(a, a + n) for a, n in ranges])
    got = mb.gather_rows(src, ranges)
    assert torch.equal(got.view(torch.int16), src.view(torch.int16)[:, torch.from_numpy(rows).cuda()])


# The forced-link part of a query among its routed partials, for d = 64 and fp32 storage: rounded to bf16 first, then
# weighted and added last, like the partials in the workspace. These and the log-sum-exps give o back. The log-sum-exps
# are fp32 numbers below 16 (half an ulp 5e-7), so weights and o are good to about 1e-6; a part rounded after its weight
# is 1e-3 off. In bf16 storage an error of 1e-6 crosses a rounding boundary (3e-3 apart) in one value of a thousand.
@pytest.mark.parametrize("d,dtype", [(64, torch.bfloat16), (64, torch.float32), (128, torch.float32)])
@pytest.mark.parametrize("topk", [1, 8, 18])
def test_forced_part_is_rounded_before_its_weight(d, dtype, topk):
    lay, H = mi.stream_layout(2, 37, 900, 33, "chunk"), 3
    N, C = lay.N, lay.C
    meta = mb.chunk_meta(lay.offsets, lay.shot, lay.window, lay.text_spans)
    g = torch.Generator(device="cuda").manual_seed(topk)
    q, k, v = (torch.randn(1, H, N, d, generator=g, device="cuda").to(dtype) for _ in range(3))
    _, sel = mb.route(meta, q, k, topk, True)
    ws = mb.attn_workspace(meta, 1, H, d, topk, dtype, False)
    o, lse = mb.attn_fwd(meta, q, k, v, sel, workspace=ws)
    forced, flse = mb.attn_fwd(meta, q, k, v, sel[..., :0].contiguous())
    at, slots = 0, topk + 1
    for n in (H * C, H * (C + 1), H * (C + 1), H * N, H * 32 * C, H * -(-N // 256) * C, H * N * topk):
        at += -(-4 * n // 256) * 256
    plse = ws[at:at + 4 * H * N * slots].view(torch.float32).view(H, N, slots)[..., :topk].double()
    at += -(-4 * H * N * slots // 256) * 256
    po = ws[at:at + 2 * H * N * slots * d].view(torch.bfloat16).view(H, N, slots, d)[..., :topk, :].double()
    used = (sel[0] >= 0)[..., None]
    parts = torch.where(used, po * torch.exp(plse - lse[0].double()[..., None])[..., None], 0.0).sum(2)
    want = parts + forced[0].double().bfloat16().double() * torch.exp(flse[0].double() - lse[0].double())[..., None]
    got = o[0].double()
    if dtype == torch.float32:
        assert float((got - want).norm() / want.norm()) < 1e-5
    else:
        assert float((got != want.bfloat16().double()).double().mean()) < 5e-3
    meta.close()


# routing in one launch right after another on other keys, with nothing between the launches: the workspace, which the
# allocator hands back each time, still holds the planes of the keys before when the pooling workgroups rewrite it. More
# workgroups than are resident, a list width each.
@pytest.mark.parametrize("d,topk", [(128, 3), (64, 8), (128, 16), (64, 32)])
def test_fused_routing_of_other_keys_back_to_back(d, topk):
    lay, H = mi.stream_layout(2, 40, 3000, 21, "chunk"), 24
    meta = mb.chunk_meta(lay.offsets, lay.shot, lay.window, lay.text_spans)
    g = torch.Generator(device="cuda").manual_seed(d + topk)
    q, *keys = (torch.randn(1, H, lay.N, d, generator=g, device="cuda").bfloat16() for _ in range(4))
    want = [mb.route(meta, q, k, topk) for k in keys]
    order = [0, 1, 2, 1, 0, 2, 0]
    torch.cuda.synchronize()
    got = [mb.route_fused(meta, q, keys[i], topk) for i in order]
    for i, (pooled, sel) in zip(order, got):
        assert torch.equal(pooled, want[i][0]) and torch.equal(sel, want[i][1])
    assert not mb.route_fused_timed_out()
    meta.close()


# the list builder's ways on both sides of each edge: 8,192 entries; two chunks; 880 chunks and a table of 49,152 words,
# filled to its last word, with blocks of 64, 128 and 256 queries (a last workgroup of one block among them); k = 8 with
# blocks of 256 queries, 16 with 24 heads; one workgroup a head where two launches are out of reach; many heads
@pytest.mark.parametrize("N,chunk,topk,H,way", [
    (2048, 20, 4, 3, "head"), (2049, 20, 4, 3, 64), (4100, 2050, 3, 3, 64),
    (880, 1, 10, 3, 64), (881, 1, 10, 3, "head"), (1000, 1, 10, 3, "head"), (1001, 1, 10, 3, "general"), (65 * 64 + 1, 70, 2, 3, 64),
    (32768, 256, 1, 3, 128), (49152, 192, 1, 3, 256), (49153, 192, 1, 3, "general"), (32768, 256, 17, 3, 128),
    (8192, 10, 8, 3, 256), (8192, 10, 9, 3, "general"), (8192, 10, 16, 24, 256), (8192, 10, 17, 24, "general"),
    (16384, 17, 1, 3, "head"), (16385, 17, 1, 3, "general"), (16385, 17, 1, 48, "head"), (16500, 17, 2, 48, "general"),
    (1300, 163, 8, 191, 64), (1300, 163, 8, 192, "head"), (1300, 60, 8, 192, 64)])
def test_list_builder_ways(N, chunk, topk, H, way):
    assert check_lists(N, chunk, topk, H) == way


# two groups of 32 queries a wave, taken from 4,096 workgroups of 256 queries up (bf16, d = 128, k <= 8) where few or many
# chunks go with them: without the causal mask to 96 chunks and from 161 on, under it from 32,768 tokens on, to 64 and from 384.
# The selections of some heads are those of a call of these heads alone, which takes one group a wave (and which the oracle
# checks); the last workgroup holds one query, one group, one query past a group, or all; one tile of chunks, two, and many
# with text in them; the first six but the fourth stay with one group
@pytest.mark.parametrize("N,chunk,text,topk,causal", [(2049, 100, 0, 8, True), (2080, 33, 60, 3, True), (2209, 17, 90, 8, False),
                                                      (2304, 70, 0, 5, False), (2303, 70, 300, 4, True), (2050, 7, 20, 8, True),
                                                      (2209, 12, 90, 8, False), (2080, 33, 60, 3, False), (32769, 600, 0, 8, True),
                                                      (32800, 80, 60, 3, True), (33025, 85, 300, 4, True), (33024, 1100, 90, 8, True),
                                                      (80001, 800, 20, 8, True)])
def test_route_pair_of_query_groups(N, chunk, text, topk, causal):
    lay = mi.stream_layout(1, text, N - text, chunk, "chunk")
    BH = 4096 // ((N + 255) // 256) + 1
    g = torch.Generator(device="cuda")
    g.manual_seed(N)
    q = torch.randn(1, BH, lay.N, 128, generator=g, device="cuda").to(torch.bfloat16)
    k = torch.randn(1, BH, lay.N, 128, generator=g, device="cuda").to(torch.bfloat16)
    k[0, :, text:text + 4 * chunk] = k[0, :, text + 4 * chunk:text + 8 * chunk]     # equal means: ties go to the lower chunk
    meta = mb.chunk_meta(lay.offsets, lay.shot, lay.window, lay.text_spans)
    pooled, sel = mb.route(meta, q, k, topk, causal)
    few = min(100, BH // 2)
    for heads in (slice(0, few), slice(BH - few, BH)):
        want_pooled, want = mb.route(meta, q[:, heads].contiguous(), k[:, heads].contiguous(), topk, causal)
        assert torch.equal(pooled[:, heads], want_pooled) and torch.equal(sel[:, heads], want)
    # rows wider than the list, with nothing drawn; scratch of the library's own, where it suffices
    _, wide = mb.route_perturbed(meta, q, k, topk, causal, 0.0, 0.0, 3, 1)
    assert torch.equal(wide[..., :topk], sel) and bool((wide[..., topk:] == -1).all())
    if BH * 3 * -(-lay.C // 32) * 32 * 128 * 2 <= 16 << 20:
        assert torch.equal(mb.route_static(meta, q, k, topk, causal)[1], sel)
    meta.close()


# fp32 storage, conversions that ride with the count of the two launches and of the general way (fewer entries, as in the
# cases above, take one workgroup a head)
@pytest.mark.parametrize("video,chunk,topk", [(1380, 5, 8), (1010, 1, 32)])
def test_fp32_storage_beside_the_count(video, chunk, topk):
    run_case(mi.stream_layout(1, 20, video, chunk, "chunk"), 1, 2, 64, topk, torch.float32, seed=121 + chunk)


# fp32 storage of more than 1,024 chunks: the conversions go out in a launch of their own, a record of its own beside
# that of the lists
def test_fp32_storage_of_many_chunks():
    lay = mi.stream_layout(1, 20, 1100, 1, "chunk")
    assert lay.C == 1101
    run_case(lay, 1, 2, 64, 8, torch.float32, seed=131)
    meta = mb.chunk_meta(lay.offsets, lay.shot, lay.window, lay.text_spans)
    q, k, v = (torch.randn(1, 2, lay.N, 64, device="cuda") for _ in range(3))
    _, sel = mb.route(meta, q, k, 8)
    mb.prof_enable(True)
    for _ in range(3):
        mb.attn_fwd(meta, q, k, v, sel)
    torch.cuda.synchronize()
    rec = mb.prof_read()
    mb.prof_enable(False)
    assert {"to_bf16", "build_lists"} <= set(rec)
    assert all(n == 3 and 0 < ms < 1000 for n, ms in rec.values())
    meta.close()


# more than 10 million selections: the same, in the forward of fp32 storage; the first heads are those of a call of their own,
# whose conversions ride with the lists
def test_fp32_storage_of_many_selections():
    lay = mi.stream_layout(1, 30, 16000, 200, "chunk")
    H, topk, few = 40, 16, 2
    assert H * lay.N * topk > 10000000
    meta = mb.chunk_meta(lay.offsets, lay.shot, lay.window, lay.text_spans)
    g = torch.Generator(device="cuda").manual_seed(17)
    q, k, v = (torch.randn(1, H, lay.N, 64, generator=g, device="cuda") for _ in range(3))
    _, sel = mb.route(meta, q, k, topk)
    mb.prof_enable(True)
    o, lse = mb.attn_fwd(meta, q, k, v, sel)
    torch.cuda.synchronize()
    large = set(mb.prof_read())
    mb.prof_enable(True)
    o2, lse2 = mb.attn_fwd(meta, *(x[:, :few].contiguous() for x in (q, k, v, sel)))
    torch.cuda.synchronize()
    small = set(mb.prof_read())
    mb.prof_enable(False)
    assert "to_bf16" in large and "to_bf16" not in small
    check_close("o", o[:, :few].cpu().numpy(), o2.cpu().numpy())
    check_close("lse", lse[:, :few].cpu().numpy(), lse2.cpu().numpy())
    meta.close()
