"""head_dim 128: a layer that is small, has short records or gains by shorter ones runs in records of 128 query rows, two
workgroups to a compute unit and LDS rings of half tiles; another in records of 256.  Parity of the short form at the sizes where it can go
wrong (as for head_dim 64: around one and two records, one and several key tiles, a text part that ends inside either half of a
band block), and of both forms on layers just below and above the line between them."""
import numpy as np
import pytest
import torch

from paper_2503_22796_amd import workloads as W
from util import ARROW, CACHE, FULL, boundary_rows, check_against_oracle, gpu_joint_attention

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_text,n_img", [(0, 1), (0, 64), (1, 127), (100, 93), (130, 126), (127, 130), (200, 600), (77, 1300)])
@pytest.mark.parametrize("flags", [0, 1, 2, 3])
def test_short_records(n_text, n_img, flags):
    from paper_2503_22796_amd import binding as B
    hp = np.asarray([FULL, ARROW, ARROW, CACHE, ARROW, ARROW], np.int32)
    win = np.asarray([0, 0, 63, 0, 64, 129], np.int32)
    wl = W.Workload("rows128", 1, 6, 128, n_text, n_img, hp, win, seed=800 + n_text)
    q, k, v = W.make_qkv(wl)
    cache = W.make_cache(wl)
    if flags & B.DIFA_FLAG_IMAGE_FIRST:
        rot = list(range(n_text, wl.N)) + list(range(n_text))
        q, k, v, cache = (t[:, :, rot].contiguous() for t in (q, k, v, cache))
    print(f"rows128 n_text={n_text} n_img={n_img} flags={flags}", flush=True)
    out = gpu_joint_attention(q, k, v, cache, hp, win, n_text, n_img, flags=flags)
    check_against_oracle(out, q, k, v, cache, hp, win, n_text, n_img, image_first=bool(flags & B.DIFA_FLAG_IMAGE_FIRST),
                         block=B.difa_tile_shape(128) if flags & B.DIFA_FLAG_BLOCK_BAND else None)


@pytest.mark.parametrize("full,rows_per_record", [(4, 128), (12, 256)])   # the shorter records save 1.8 % or 0.6 % of the key tiles
def test_both_sides_of_the_line(full, rows_per_record):
    from paper_2503_22796_amd import binding as B
    import internal as I
    hp = np.asarray([FULL] * full + [ARROW] * (18 - full) + [CACHE] * 6, np.int32)
    wl = W.Workload("line", 1, 24, 128, 256, 16384, hp, np.where(hp == ARROW, 1056, 0).astype(np.int32), seed=860)
    q, k, v = W.make_qkv(wl)
    cache = W.make_cache(wl)
    plan = B.difa_plan_create(1, 24, 128, max_tokens=wl.N)
    try:
        out = gpu_joint_attention(q, k, v, cache, hp, wl.window, wl.n_text, wl.n_img, plan=plan)
        assert I.last_call(plan)["rows"] == rows_per_record
    finally:
        B.difa_plan_destroy(plan)
    rows = boundary_rows(wl.n_text, wl.n_img, [1056], extra=24, seed=full)
    check_against_oracle(out, q, k, v, cache, hp, wl.window, wl.n_text, wl.n_img, rows=rows)
