"""GPU parity at the edges of the launch rules: sizes where a rule picks another kernel, another split
of the work list or another tile count. Oracle and tolerances as in test_gpu_parity (bf16 products with
fp32 sums; the bounds there cover any order of the sums)."""
import numpy as np
import pytest
import torch

import moc_inputs as mi
from tests.test_gpu_parity import run_case

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


def _no_captions(shots, frames, frame):
    offs = np.arange(0, shots * frames * frame + 1, 48, dtype=np.int32)
    C = len(offs) - 1
    per = C // shots
    return mi.Layout("no_captions", offs, (np.arange(C) // per).astype(np.int32), np.arange(C, dtype=np.int32),
                     np.zeros((0, 2), dtype=np.int32))


# a caption longer than the resident rows of the chunk-stationary kernels beside chunks that fit (288),
# and chunks of one key too many
@pytest.mark.parametrize("chunk", [288, 289])
def test_routed_chunks_beside_a_long_caption(chunk):
    run_case(mi.multishot_layout(2, 300, 2, 2 * chunk, chunk, "frame"), 1, 2, 128, 2, torch.bfloat16, seed=41)


# fp32 storage through the same kernels as bf16: both head sizes, the chunk-stationary and the tiled
# routed items, one group per workgroup (small calls) and ragged last tiles; k = 0 leaves forced links alone
@pytest.mark.parametrize("d,chunk,topk", [(64, 33, 3), (128, 288, 2), (128, 300, 2), (64, 300, 1), (128, 65, 0)])
def test_fp32_storage(d, chunk, topk):
    run_case(mi.stream_layout(2, 37, 4 * chunk + 5, chunk, "chunk"), 1, 3, d, topk, torch.float32, seed=51 + chunk)
