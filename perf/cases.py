"""Performance cases of the Mixture-of-Contexts attention layer: the passes a user of the library
runs, through its public calls, from a sequence of a thousand tokens to the 181,760-token stream.

A case is a plain dict:
  path     "train"    route -> attention forward -> backward (the backward reuses the forward's lists)
           "forward"  route -> attention forward (sampling, validation)
           "regularised_route"  routing with drop-off / drop-in, as the training recipe routes
           "outer_forward"      outer-loop selection of shots, gather of the reduced stream, chunk
                                tables of that stream, then the inner layer's forward on it
  layout   "multishot" per shot a caption and frames of `frame` tokens cut into chunks of `chunk`
           "stream"    per shot a caption and `video` tokens cut every `chunk` tokens, ragged tail
           "mixed"     the same with the training schedule's four chunk sizes side by side
           "ragged"    content-aligned chunks: lengths drawn between 1 and 2 * `chunk`, frames of a
                       few chunks, captions of odd lengths
  shots, text, frames, frame, video, chunk, window, B, H, d, k, dtype, causal, inputs.
`inputs` is "iid" (standard normal, selections of neighbouring queries unrelated) or "coherent"
(tokens of a chunk share a component, queries are correlated with one earlier chunk, as retrieval
in a trained layer is). Values are rounded to the storage type.
"""
from __future__ import annotations

import numpy as np
import torch

import moc_inputs as mi
from paper_2508_21058_amd import binding as mb

_SCHEDULE = (10240, 5120, 2560, 1280)      # chunk sizes of the multi-shot training schedule


def _case(name, path, layout, **kw):
    case = dict(path=path, layout=layout, shots=1, text=256, frames=9, frame=1560, video=0, chunk=260,
                window="frame", B=1, H=24, d=128, k=8, dtype="bf16", causal=True, inputs="iid", lseed=0)
    case.update(kw)
    if name:
        case["name"] = name
    return case


def listed():
    return [
        # the smallest configuration of the repository: fp32 storage, two heads, about a thousand tokens; latency
        _case("tiny_train_f32", "train", "multishot", text=64, frames=4, frame=256, chunk=64, window="chunk", H=2, d=64,
              k=2, dtype="f32"),
        # single-shot training set-up (8 s clip): no causal mask, own-chunk window, a ragged last chunk
        _case("short_train", "train", "stream", video=6000, chunk=256, window="chunk", k=3, causal=False),
        # the same clip in the sampling loop of the finished model: forward only
        _case("short_forward", "forward", "stream", video=6000, chunk=256, window="chunk", k=3, causal=False),
        # single-shot DiT layer of 33k tokens, forward only, iid inputs
        _case("single_forward", "forward", "multishot", text=512, frames=21, k=5),
        # the same layer in training, on chunk-coherent inputs
        _case("single_train", "train", "multishot", text=512, frames=21, k=5, inputs="coherent"),
        # content-aligned chunks of unequal, odd lengths, the smaller head size, two samples in a batch
        _case("ragged_train_d64", "train", "ragged", shots=3, text=77, frames=10, chunk=170, B=2, H=8, d=64, k=6, lseed=3),
        # fp32 storage at the model's head size (master-precision activations), ragged chunks
        _case("ragged_train_f32", "train", "ragged", shots=2, text=120, frames=8, chunk=200, H=6, d=128, k=5, dtype="f32",
              lseed=4),
        # the benchmark workload: eight shots, 114k tokens, frame window, k = 8
        _case("eight_train", "train", "multishot", shots=8),
        # its routing with the training-time regularisers: rows widened by four drop-in slots
        _case("eight_regularised_route", "regularised_route", "multishot", shots=8),
        # one shot generated against its three best earlier shots: outer routing, reduced stream, inner forward
        _case("eight_outer_forward", "outer_forward", "multishot", shots=8, H=12),
        # minute-scale stream (32 shots, 457k tokens) on the heads one of four head shards holds, smallest chunk, widest k
        _case("sweep_train_head_shard", "train", "multishot", shots=32, chunk=130, H=6, k=16),
        # the 181,760-token stream: shot window, the schedule's chunk sizes 1280 .. 10240 mixed in one stream
        _case("long_train", "train", "mixed", shots=8, video=22464, window="shot", k=5),
    ]


def draw(rng):
    """One more case of the listed ranges; never more work than a third of the largest case."""
    def log_int(lo, hi):
        return int(round(lo * (hi / lo) ** rng.random()))

    limit = work(listed()[-1])["flops"] / 3
    while True:
        path = rng.choice(["train", "train", "train", "forward", "forward", "regularised_route", "outer_forward"])
        dtype = "f32" if rng.random() < 0.2 else "bf16"
        layout = rng.choice(["multishot", "stream", "mixed", "ragged", "ragged"])
        kw = dict(dtype=dtype, d=128 if rng.random() < 0.75 else 64, H=rng.choice([1, 2, 3, 6, 8, 12, 16, 24]),
                  B=2 if rng.random() < 0.2 else 1, k=rng.choice([1, 2, 3, 4, 5, 6, 8, 8, 11, 16]),
                  causal=rng.random() < 0.8, text=log_int(30, 520), shots=rng.choice([1, 1, 2, 3, 4, 6, 8, 16]),
                  inputs=rng.choice(["iid", "iid", "coherent"]), lseed=rng.randrange(1 << 20))
        if layout == "multishot":
            chunk = log_int(48, 520)
            kw.update(chunk=chunk, frame=chunk * rng.randint(1, 12), frames=rng.randint(2, 21),
                      window=rng.choice(["chunk", "frame", "frame", "shot"]))
        elif layout == "stream":
            kw.update(video=log_int(900, 23000), chunk=log_int(64, 10240), window=rng.choice(["chunk", "shot"]))
        elif layout == "mixed":
            kw.update(video=log_int(12000, 23000), window="shot")
        else:
            kw.update(chunk=log_int(40, 400), frames=rng.randint(3, 16), window=rng.choice(["chunk", "frame", "shot"]))
        if path == "outer_forward":
            kw.update(shots=rng.choice([3, 4, 6, 8, 16]), B=1)
        case = _case(None, path, layout, **kw)
        n = _layout(case).N
        cells = case["B"] * case["H"] * n * case["d"] * (4 if dtype == "f32" else 2)
        if 900 <= n <= 460000 and cells <= 1.5e9 and work(case)["flops"] <= limit:
            return case


# ---- layouts ------------------------------------------------------------------------------------------------------

def _layout(case):
    if case["layout"] == "multishot":
        return mi.multishot_layout(case["shots"], case["text"], case["frames"], case["frame"], case["chunk"], case["window"])
    if case["layout"] == "stream":
        return mi.stream_layout(case["shots"], case["text"], case["video"], case["chunk"], case["window"])
    if case["layout"] == "mixed":
        return mi.mixed_stream_layout(case["shots"], case["text"], case["video"], _SCHEDULE, case["window"])
    rng = np.random.default_rng(case["lseed"])
    offs, shot, win, spans, wid = [0], [], [], [], 0

    def add(length, s):
        offs.append(offs[-1] + int(length))
        shot.append(s)
        win.append(wid)

    for s in range(case["shots"]):
        start = offs[-1]
        add(case["text"] + rng.integers(0, 9), s)
        spans.append((start, offs[-1]))
        wid += case["window"] != "shot"
        for _ in range(case["frames"]):
            for _ in range(int(rng.integers(1, 6))):
                add(rng.integers(1, 2 * case["chunk"] + 1), s)
                wid += case["window"] == "chunk"
            wid += case["window"] == "frame"
        wid += case["window"] == "shot"
    return mi.Layout("ragged", *(np.asarray(x, dtype=np.int32) for x in (offs, shot, win)),
                     np.asarray(spans, dtype=np.int32).reshape(-1, 2))


# ---- inputs -------------------------------------------------------------------------------------------------------

def _tensors(case, lay, seed, count):
    """q, k, v, dO (the first `count`) on the GPU, made from the seed alone."""
    B, H, N, d = case["B"], case["H"], lay.N, case["d"]
    dtype = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))

    def normal(*shape):
        return torch.randn(*shape, generator=g, device="cuda", dtype=torch.float32)

    out = []
    if case["inputs"] == "coherent":
        C = lay.C
        chunk_of = torch.repeat_interleave(torch.arange(C, device="cuda"),
                                           torch.from_numpy(np.diff(lay.offsets).astype(np.int64)).cuda())
        uk = normal(B, H, C, d)
        target = (torch.rand(C, generator=g, device="cuda") * torch.arange(C, device="cuda")).long()
        uq = 0.5 * uk[:, :, target] + 0.75 ** 0.5 * normal(B, H, C, d)
        for u in (uq, uk):
            out.append((0.9 ** 0.5 * u[:, :, chunk_of] + 0.1 ** 0.5 * normal(B, H, N, d)).to(dtype).contiguous())
    while len(out) < count:
        out.append(normal(B, H, N, d).to(dtype))
    return out


def prepare(case, seed):
    """The tensors of one layer call and what a program keeps across calls: the chunk tables of the layout, the
    attention workspace and, in training, the output tensors."""
    lay = _layout(case)
    st = dict(case=case, lay=lay)
    train = case["path"] == "train"
    t = _tensors(case, lay, seed, 4 if train else 2 if case["path"] == "regularised_route" else 3)
    st["q"], st["k"] = t[0], t[1]
    if len(t) > 2:
        st["v"] = t[2]
    if case["path"] == "outer_forward":
        B, H, N, d = t[0].shape
        st["features"] = t[1][0].permute(1, 0, 2).reshape(N, H * d).contiguous()
        st["segments"], st["captions"] = mb.outer_segments(lay.offsets, lay.shot, lay.text_spans)
        return st
    st["meta"] = mb.chunk_meta(lay.offsets, lay.shot, lay.window, lay.text_spans)
    if case["path"] == "regularised_route":
        st["seed"] = seed
        return st
    B, H, N, d = t[0].shape
    st["ws"] = mb.attn_workspace(st["meta"], B, H, d, case["k"], t[0].dtype, train)
    if train:
        st["dO"] = t[3]
        st["out"] = (torch.empty_like(t[0]), torch.empty(B, H, N, dtype=torch.float32, device="cuda"))
        st["grads"] = tuple(torch.empty_like(t[0]) for _ in range(3))
    return st


def run(st):
    case, q, k = st["case"], st["q"], st["k"]
    if case["path"] == "regularised_route":
        width = min(4, mb.MOC_MAX_TOPK - case["k"])
        pooled, sel = mb.route_perturbed(st["meta"], q, k, case["k"], case["causal"], 0.5, 1.0, width, st["seed"])
        return dict(pooled=pooled, sel=sel)
    if case["path"] == "outer_forward":
        lay, seg = st["lay"], st["segments"]
        mean, scores, best, kept = mb.outer_route(st["features"], seg, st["captions"], len(seg) - 2, min(3, case["shots"] - 1),
                                                  case["causal"])
        off, shot, win, spans, ranges = mb.reduce_layout(lay.offsets, lay.shot, lay.window, lay.text_spans, seg, kept)
        qr, kr, vr = (mb.gather_rows(x, ranges) for x in (q, k, st["v"]))
        st["meta"] = meta = mb.chunk_meta(off, shot, win, spans)
        pooled, sel = mb.route(meta, qr, kr, case["k"], case["causal"])
        o, lse = mb.attn_fwd(meta, qr, kr, vr, sel)
        return dict(mean=mean, scores=scores, best=best, q=qr, k=kr, v=vr, pooled=pooled, sel=sel, o=o, lse=lse)
    meta, v = st["meta"], st["v"]
    pooled, sel = mb.route(meta, q, k, case["k"], case["causal"])
    if case["path"] == "forward":
        o, lse = mb.attn_fwd(meta, q, k, v, sel, workspace=st["ws"])
        return dict(pooled=pooled, sel=sel, o=o, lse=lse)
    o, lse = mb.attn_fwd(meta, q, k, v, sel, workspace=st["ws"], out=st["out"])
    dq, dk, dv = mb.attn_bwd(meta, q, k, v, o, lse, st["dO"], sel, workspace=st["ws"], out=st["grads"], after_fwd=True)
    return dict(pooled=pooled, sel=sel, o=o, lse=lse, dq=dq, dk=dk, dv=dv)


# ---- work and tolerance -------------------------------------------------------------------------------------------

def _pairs(lay, k, causal):
    """Per head: attended (query, key) pairs and scored (query, chunk) pairs. The routed share counts the mean length
    of a query's candidate chunks: which ones it takes depends on the data."""
    off = lay.offsets.astype(np.int64)
    lens = np.diff(off)
    text = np.zeros(lay.C, bool)
    for s, e in lay.text_spans.reshape(-1, 2):
        text |= (off[:-1] >= s) & (off[1:] <= e)
    _, win = np.unique(lay.window, return_inverse=True)
    vid = (~text).astype(np.int64)
    win_n, win_len = np.bincount(win, weights=vid), np.bincount(win, weights=vid * lens)
    forced = lens[text].sum() + win_len[win]
    if causal:          # earlier video chunks, without those of the own window
        n_before, len_before = np.cumsum(vid) - vid, np.cumsum(vid * lens) - vid * lens
        first = np.searchsorted(win, np.arange(win.max() + 1))
        cand, cand_len = n_before[first][win], len_before[first][win]
    else:
        cand, cand_len = vid.sum() - win_n[win], (vid * lens).sum() - win_len[win]
    routed = np.minimum(k, cand) * cand_len / np.maximum(cand, 1)
    return float((lens * (forced + routed)).sum()), float((lens * cand).sum())


def work(case):
    lay = _layout(case)
    BH, d, k, C = case["B"] * case["H"], case["d"], case["k"], lay.C
    esz = 4 if case["dtype"] == "f32" else 2
    n, extra = lay.N, 0.0
    if case["path"] == "outer_forward":
        seg, cap = mb.outer_segments(lay.offsets, lay.shot, lay.text_spans)
        g, m = len(seg) - 2, min(3, case["shots"] - 1)
        open_ = [j for j in range(len(seg) - 1) if not cap[j] and j != g]
        kept = sorted([j for j in range(len(seg) - 1) if cap[j]] + open_[:m] + [g])
        off, shot, win, spans, _ = mb.reduce_layout(lay.offsets, lay.shot, lay.window, lay.text_spans, seg, kept)
        lay = mi.Layout("reduced", off, shot, win, spans)
        extra = BH * d * esz * (n + 3.0 * lay.N)             # the features read, the reduced q, k, v written
        n, C = lay.N, lay.C
    pairs, scored = _pairs(lay, k, case["causal"])
    row = float(BH) * n * d * esz                            # one [B, H, N, d] tensor
    pooled = BH * C * d * 4.0
    score_flops = 2.0 * d * scored * BH
    if case["path"] == "regularised_route":
        width = k + min(4, mb.MOC_MAX_TOPK - k)
        return {"bytes": 2 * row + pooled + BH * n * width * 4.0, "flops": score_flops}
    bytes_ = pooled + BH * n * (k + 1) * 4.0
    if case["path"] == "train":
        return {"bytes": 8 * row + bytes_, "flops": score_flops + 14.0 * d * pairs * BH}
    return {"bytes": 4 * row + bytes_ + extra, "flops": score_flops + 4.0 * d * pairs * BH}


def tolerance(case):
    # Contractions on bf16 operands with fp32 accumulation and bf16 partials, against float64 on the same selections
    # (worst tensor is dq): 2.9e-3 with bf16 storage, 4.6e-3 with fp32 storage (its values are rounded to bf16 on entry),
    # 7.8e-3 on coherent inputs, whose peaked softmax makes dq nearly cancel. Pooled keys, which the regularised routing
    # returns alone, stay at 1e-7. A query whose k-th and next scores agree to fp32 rounding may take either chunk.
    if case["path"] == "regularised_route":
        return {"rel": 1e-6, "differ": 1e-4}
    rel = 1.2e-2 if case["dtype"] == "bf16" else 1.8e-2
    return {"rel": 3e-2 if case["inputs"] == "coherent" else rel, "differ": 1e-4}
