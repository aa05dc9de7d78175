"""head_dim 64: the kernel's records are 128 query rows, half a block of the block-granular band, and two workgroups
share a compute unit.  Parity at the sizes where that can go wrong: token counts around one and two records, a text part
that ends inside either half of a block, windows around half a block; exact and block-granular band, both token orders."""
import numpy as np
import pytest
import torch

from paper_2503_22796_amd import workloads as W
from util import ARROW, CACHE, FULL, check_against_oracle, gpu_joint_attention

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_text,n_img", [(0, 127), (1, 127), (1, 128), (100, 155), (130, 126), (127, 130), (200, 600), (333, 1100)])
@pytest.mark.parametrize("flags", [0, 1, 2, 3])
def test_records_of_half_a_block(n_text, n_img, flags):
    from paper_2503_22796_amd import binding as B
    hp = np.asarray([FULL, ARROW, ARROW, CACHE, ARROW, ARROW], np.int32)
    win = np.asarray([0, 0, 63, 0, 64, 129], np.int32)
    wl = W.Workload("rows64", 2, 6, 64, n_text, n_img, hp, win, seed=700 + n_text)
    q, k, v = W.make_qkv(wl)
    cache = W.make_cache(wl)
    if flags & B.DIFA_FLAG_IMAGE_FIRST:
        rot = list(range(n_text, wl.N)) + list(range(n_text))
        q, k, v, cache = (t[:, :, rot].contiguous() for t in (q, k, v, cache))
    print(f"rows64 n_text={n_text} n_img={n_img} flags={flags}", flush=True)
    out = gpu_joint_attention(q, k, v, cache, hp, win, n_text, n_img, flags=flags)
    check_against_oracle(out, q, k, v, cache, hp, win, n_text, n_img, image_first=bool(flags & B.DIFA_FLAG_IMAGE_FIRST),
                         block=B.difa_tile_shape(64) if flags & B.DIFA_FLAG_BLOCK_BAND else None)
