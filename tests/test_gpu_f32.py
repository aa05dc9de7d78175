"""The fp32 path's blocks are 16 query rows, its key tiles 16 keys dealt to eight wavefronts: parity at token counts around
one tile and one round of tiles, bands that start and end inside a tile, a text part that ends inside a row block; both
head_dims, both token orders, cached and residual-sharing heads in the one launch."""
import numpy as np
import pytest
import torch

from paper_2503_22796_amd import workloads as W
from util import ARROW, CACHE, FULL, TOL_F32

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("n_text,n_img,image_first", [(0, 1, False), (1, 15, False), (3, 14, True), (16, 112, False),
                                                      (17, 111, True), (40, 250, False), (77, 331, True), (0, 129, False)])
def test_fp32_tile_edges(D, n_text, n_img, image_first):
    from oracle import residual_oracle as R
    from paper_2503_22796_amd import binding as B
    dev = torch.device("cuda:0")
    hp = np.asarray([FULL, ARROW, ARROW, CACHE, 3, ARROW], np.int32)
    win = np.asarray([0, 0, 7, 0, 16, 100], np.int32)
    wl = W.Workload("f32", 2, 6, D, n_text, n_img, hp, win, seed=900 + n_img)
    q, k, v = W.make_qkv(wl, dtype=torch.float32)
    cache, residual = W.make_cache(wl, dtype=torch.float32), 0.25 * W.make_cache(wl, step=3, dtype=torch.float32)
    print(f"f32 D={D} n_text={n_text} n_img={n_img} image_first={image_first}", flush=True)
    out = torch.full_like(q, float("nan")).to(dev)
    plan = B.difa_plan_create(2, 6, D, dtype=B.DIFA_DTYPE_F32, max_tokens=wl.N, flags=B.DIFA_FLAG_IMAGE_FIRST if image_first else 0)
    try:
        B.difa_joint_attention_residual(plan, q.to(dev), k.to(dev), v.to(dev), out, cache.to(dev), residual.to(dev), hp, n_text, n_img, win)
        torch.cuda.synchronize()
    finally:
        B.difa_plan_destroy(plan)
    got = out.cpu()
    ref, raw = R.joint_attention(q, k, v, cache, residual, hp, win, n_text, n_img, image_first=image_first)
    for h in range(6):
        if hp[h] == CACHE:
            assert torch.equal(got[:, h].view(torch.int32), raw[:, h].contiguous().view(torch.int32))
        else:
            assert float((got[:, h].double() - ref[:, h]).abs().max()) <= TOL_F32, f"head {h}"
