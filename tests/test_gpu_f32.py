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


def _run_f32(q, k, v, hp, win, n_text, n_img, scale=0.0, image_first=False):
    from paper_2503_22796_amd import binding as B
    dev = torch.device("cuda:0")
    b, heads, n, d = q.shape
    out = torch.full_like(q, float("nan")).to(dev)
    plan = B.difa_plan_create(b, heads, d, dtype=B.DIFA_DTYPE_F32, max_tokens=n, softmax_scale=scale,
                              flags=B.DIFA_FLAG_IMAGE_FIRST if image_first else 0)
    try:
        B.difa_joint_attention(plan, q.to(dev), k.to(dev), v.to(dev), out, None, hp, n_text, n_img, win)
        torch.cuda.synchronize()
    finally:
        B.difa_plan_destroy(plan)
    return out.cpu()


def _logits(kind, D, N, seed):
    """Q and K whose scores are of a stated magnitude.  Every entry is an integer and the softmax scale a power of two, so
    that the scores (below 2^53) and their differences are the same numbers in any order of summation, and what is
    compared is the softmax alone."""
    g = torch.Generator().manual_seed(seed)
    q, k = (torch.randint(-3, 4, (1, 2, N, D), generator=g).float() for _ in range(2))
    if kind == "all below -1e30":                       # the small entries vanish beside 2^110: two levels of scores
        q[..., 0], k[..., 0] = 2.0 ** 60, -2.0 ** 50
        k[:, :, ::3, 0] = -2.0 ** 51
    elif kind == "beyond fp32":
        q[..., 0], k[..., 0] = 2.0 ** 75, 2.0 ** 60
        k[:, :, ::3, 0] = 2.0 ** 59
    else:                                               # a common part of the stated size under differences of a few units
        q[..., 0], k[..., 0] = kind[0], kind[1]
    return q, k


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("kind", [(2.0 ** 12, 2.0 ** 11), (2.0 ** 20, 2.0 ** 20), (2.0 ** 24, -2.0 ** 24), "all below -1e30", "beyond fp32"])
def test_fp32_logits_of_any_finite_magnitude(D, kind):
    """Nothing limits the magnitude of finite fp32 inputs: rows whose scores are 2^20, 2^37, -2^45, all below -1e30, or beyond
    fp32's own range.  The bar is the path's own 1e-5: relative to the scores' differences the weights are exact."""
    from oracle import difa_oracle as O
    n_text, n_img = 21, 250
    hp, win = np.asarray([FULL, ARROW], np.int32), np.asarray([0, 40], np.int32)
    q, k = _logits(kind, D, n_text + n_img, seed=17)
    v = torch.randn(1, 2, n_text + n_img, D, generator=torch.Generator().manual_seed(18))
    scale = 2.0 ** -5
    print(f"f32 logits {kind} D={D}", flush=True)
    got = _run_f32(q, k, v, hp, win, n_text, n_img, scale=scale)
    ref, _, _ = O.joint_attention(q, k, v, None, hp, win, n_text, n_img, scale=scale)
    assert torch.isfinite(got).all()
    assert float((got.double() - ref).abs().max()) <= TOL_F32


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("image_first", [False, True])
@pytest.mark.parametrize("bad", [float("inf"), float("-inf"), float("nan")])
def test_fp32_a_key_that_is_not_finite_stays_with_the_rows_that_see_it(D, image_first, bad):
    """Non-finite inputs make the rows that see them undefined and no others: a masked key takes part in the matrix products
    of its tile with weight 0, which is not enough against an infinity in V."""
    from oracle import difa_oracle as O
    n_text, n_img, w = 21, 250, 19
    N, img0 = n_text + n_img, 0 if image_first else n_text
    hp, win = np.asarray([ARROW, ARROW, ARROW], np.int32), np.asarray([w, 0, 30], np.int32)
    g = torch.Generator().manual_seed(23)
    q, k, v = (torch.randn(1, 3, N, D, generator=g) for _ in range(3))
    ref, _, _ = O.joint_attention(q, k, v, None, hp, win, n_text, n_img, image_first=image_first)
    keys = [img0 + 3, img0 + 117, img0 + 118, img0 + n_img - 1]
    v[:, :, keys[0], D // 2] = bad
    v[:, :, keys[1]] = bad
    k[:, :, keys[2], 1] = bad
    v[:, :, keys[3], D - 1] = bad
    print(f"f32 not finite: {bad} D={D} image_first={image_first}", flush=True)
    got = _run_f32(q, k, v, hp, win, n_text, n_img, image_first=image_first)
    rows = torch.arange(N)
    image = (rows >= img0) & (rows < img0 + n_img)
    for h in range(3):
        blind = image & torch.stack([(rows - j).abs() > int(win[h]) for j in keys]).all(0)
        assert int(blind.sum()) >= 20
        assert float((got[:, h, blind].double() - ref[:, h, blind]).abs().max()) <= TOL_F32, f"head {h}"
    rest = (got[:, 0, img0 + 3, :D // 2].double() - ref[:, 0, img0 + 3, :D // 2]).abs().max()
    assert float(rest) <= TOL_F32                         # features of V that are finite are not touched either


@pytest.mark.parametrize("D", [64, 128])
def test_fp32_tensors_need_no_more_than_element_alignment(D):
    """Tensors that begin one float into an allocation: the kernel reads and writes four floats at a time."""
    from oracle import difa_oracle as O
    from paper_2503_22796_amd import binding as B
    dev = torch.device("cuda:0")
    hp, win = np.asarray([FULL, ARROW, CACHE], np.int32), np.asarray([0, 12, 0], np.int32)
    wl = W.Workload("f32a", 1, 3, D, 21, 150, hp, win, seed=930)
    q, k, v = W.make_qkv(wl, dtype=torch.float32)
    cache = W.make_cache(wl, dtype=torch.float32)

    def shifted(t):
        buf = torch.full((t.numel() + 1,), float("nan"), device=dev)
        view = buf[1:].view(t.shape)
        view.copy_(t.to(dev))
        return buf, view

    (_, qd), (_, kd), (_, vd), (_, cd), (whole, out) = (shifted(t) for t in (q, k, v, cache, torch.zeros_like(q)))
    print(f"f32 element alignment D={D}", flush=True)
    plan = B.difa_plan_create(1, 3, D, dtype=B.DIFA_DTYPE_F32, max_tokens=wl.N)
    try:
        B.difa_joint_attention(plan, qd, kd, vd, out, cd, hp, wl.n_text, wl.n_img, win)
        torch.cuda.synchronize()
    finally:
        B.difa_plan_destroy(plan)
    assert bool(torch.isnan(whole[0]))                    # nothing is written before the tensor
    got = out.cpu()
    ref, raw, _ = O.joint_attention(q, k, v, cache, hp, win, wl.n_text, wl.n_img)
    assert float((got[:, :2].double() - ref[:, :2]).abs().max()) <= TOL_F32
    assert torch.equal(got[:, 2].view(torch.int32), raw[:, 2].contiguous().view(torch.int32))


@pytest.mark.parametrize("n_tokens", [2, 18])
def test_token_rows_of_hundreds_of_megabytes(n_tokens):
    # 2^19 heads of 64 in [batch, token, head, feature] order: 16 token rows span 2 GiB, more than a 32-bit byte offset reaches
    from paper_2503_22796_amd import binding as B
    heads, D, dev = 1 << 19, 64, torch.device("cuda:0")
    g = torch.Generator(device=dev)
    g.manual_seed(n_tokens)
    q, k, v = (torch.randn((1, n_tokens, heads, D), device=dev, generator=g) for _ in range(3))
    out = torch.full_like(q, float("nan"))
    plan = B.difa_plan_create(1, heads, D, dtype=B.DIFA_DTYPE_F32, layout=B.DIFA_LAYOUT_BNHD, max_tokens=n_tokens)
    try:
        B.difa_joint_attention(plan, q, k, v, out, None, np.zeros(heads, np.int32), 0, n_tokens, np.zeros(heads, np.int32))
        torch.cuda.synchronize()
    finally:
        B.difa_plan_destroy(plan)
    for h0 in (0, 12345, heads - 64):                            # 64 heads at a time, in fp64 on the host
        qh, kh, vh = (t[0, :, h0:h0 + 64].transpose(0, 1).cpu().double().contiguous() for t in (q, k, v))
        ref = torch.matmul(torch.softmax(torch.matmul(qh, kh.transpose(1, 2).contiguous()) / 8.0, dim=2), vh)
        got = out[0, :, h0:h0 + 64].transpose(0, 1).cpu().double()
        assert float((got - ref).abs().max()) <= TOL_F32
