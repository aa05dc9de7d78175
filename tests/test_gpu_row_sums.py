"""Rows whose logits leap: the reference a row's weights are expressed against moves only when a block's row sum outgrows
2^40, and the sums of rows 16 apart come out of one matrix product, an infinite weight of one row meeting a zero coefficient
of the other.  Each row of a wavefront leaps in a block of its own choice, or not at all, alone or together with its partner,
by a finite weight or an infinite one, once or twice.  A row of Q that is not finite makes its own output so and no other."""
import numpy as np
import pytest
import torch

from paper_2503_22796_amd import workloads as W
from util import ARROW, FULL, TOL_BF16, check_against_oracle, gpu_joint_attention
import internal as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,rows", [(64, 128), (128, 128), (128, 256)])
@pytest.mark.parametrize("step", [30.0, 60.0, 400.0])          # leap in the log2 domain: below 2^40, above it, beyond fp32
def test_leaping_rows(D, rows, step):
    from paper_2503_22796_amd import binding as B
    n_text, n_img = 40, 360
    hp, win = np.asarray([FULL, ARROW], np.int32), np.asarray([0, 90], np.int32)
    wl = W.Workload("leap", 1, 2, D, n_text, n_img, hp, win, seed=900 + D, positional=False)
    q, k, v = (t.clone() for t in W.make_qkv(wl))
    # feature f carries the leap at key[f]: only rows that have something there see it
    keys = [2, 35, 70, 101, 150, 399]
    q[..., :len(keys)] = 0
    k[..., :len(keys)] = 0
    unit = step * np.log(2.0) * D ** 0.5 / 16
    for f, j in enumerate(keys):
        k[:, :, j, f] = 16.0
    for i in range(wl.N):
        leaps = {0: [], 1: [2], 2: [1, 4], 3: [3], 4: [0, 5], 5: [4], 6: [2, 3]}[(i * 5 + i // 16) % 7]
        for n, f in enumerate(leaps):
            q[:, :, i, f] = unit * (n + 1)                      # a second leap starts from the first
    print(f"leap D={D} rows={rows} step={step}", flush=True)
    plan = B.difa_plan_create(1, 2, D, max_tokens=wl.N)
    try:
        I.force_rows(plan, rows)
        out = gpu_joint_attention(q, k, v, None, hp, win, n_text, n_img, plan=plan)
    finally:
        B.difa_plan_destroy(plan)
    check_against_oracle(out, q, k, v, None, hp, win, n_text, n_img)


@pytest.mark.parametrize("D,rows", [(64, 128), (128, 128), (128, 256)])
@pytest.mark.parametrize("value", [float("nan"), float("inf")])
def test_query_rows_that_are_not_finite_stay_alone(D, rows, value):
    from paper_2503_22796_amd import binding as B
    n_text, n_img = 40, 360
    hp, win = np.asarray([FULL, ARROW], np.int32), np.asarray([0, 90], np.int32)
    wl = W.Workload("alone", 1, 2, D, n_text, n_img, hp, win, seed=950 + D, positional=False)
    q, k, v = W.make_qkv(wl)
    bad = [0, 21, 39, 50, 130, 255, 399]                        # text and image rows of either half of 32, none 16 from another
    broken = q.clone()
    broken[:, :, bad, 3] = value
    print(f"not finite D={D} rows={rows} value={value}", flush=True)
    plan = B.difa_plan_create(1, 2, D, max_tokens=wl.N)
    try:
        I.force_rows(plan, rows)
        clean = gpu_joint_attention(q, k, v, None, hp, win, n_text, n_img, plan=plan)
        out = gpu_joint_attention(broken, k, v, None, hp, win, n_text, n_img, plan=plan)
    finally:
        B.difa_plan_destroy(plan)
    assert not bool(torch.isfinite(out[:, :, bad].float()).any())
    out[:, :, bad] = clean[:, :, bad]
    check_against_oracle(out, q, k, v, None, hp, win, n_text, n_img)


@pytest.mark.parametrize("D,rows", [(64, 128), (128, 128), (128, 256)])
@pytest.mark.parametrize("key", [50, 200])                      # in the records' first block, and in a later one
@pytest.mark.parametrize("value", [float("nan"), float("inf")])
def test_keys_that_are_not_finite_reach_only_the_rows_that_see_them(D, rows, key, value):
    # The band's edge lies inside a block of 32 rows: of rows 16 apart one sees the key and the other does not.  An infinite
    # feature makes the key's score +inf or -inf by the sign of the row's own feature: no result, or weight 0.
    from paper_2503_22796_amd import binding as B
    n_text, n_img, w = 40, 360, 90
    hp, win = np.asarray([FULL, ARROW], np.int32), np.asarray([0, w], np.int32)
    wl = W.Workload("keys", 1, 2, D, n_text, n_img, hp, win, seed=970 + D, positional=False)
    q, k, v = (t.clone() for t in W.make_qkv(wl))
    k[:, :, key, 3] = value
    i = torch.arange(wl.N)
    far = (i[:, None] >= n_text) & (i[None, :] >= n_text) & ((i[:, None] - i[None, :]).abs() > w)
    s = torch.stack([torch.mm(q[0, h].double(), k[0, h].double().t()) / D ** 0.5 for h in range(2)])
    s[1].masked_fill_(far, float("-inf"))
    ref = torch.stack([torch.mm(torch.softmax(s[h], dim=1), v[0, h].double()) for h in range(2)])
    finite = torch.isfinite(ref)
    assert any(bool(finite[1, r].all()) and not bool(finite[1, r + 16].any()) or bool(finite[1, r + 16].all()) and not bool(finite[1, r].any())
               for r in range(n_text, wl.N - 16) if r % 32 < 16)
    print(f"keys D={D} rows={rows} key={key} value={value}", flush=True)
    plan = B.difa_plan_create(1, 2, D, max_tokens=wl.N)
    try:
        I.force_rows(plan, rows)
        out = gpu_joint_attention(q, k, v, None, hp, win, n_text, n_img, plan=plan)[0].double()
    finally:
        B.difa_plan_destroy(plan)
    assert torch.equal(torch.isfinite(out), finite)
    assert float((out - ref)[finite].abs().max()) <= TOL_BF16


@pytest.mark.parametrize("D,rows", [(64, 128), (128, 128), (128, 256)])
def test_query_rows_that_are_not_finite_may_be_16_apart(D, rows):
    from paper_2503_22796_amd import binding as B
    n_text, n_img = 40, 360
    hp, win = np.asarray([FULL, ARROW], np.int32), np.asarray([0, 90], np.int32)
    wl = W.Workload("pairs", 1, 2, D, n_text, n_img, hp, win, seed=990 + D, positional=False)
    q, k, v = W.make_qkv(wl)
    bad = [5, 21, 130, 146, 300]                                # two pairs that share a matrix product, and one row
    broken = q.clone()
    broken[:, :, bad, 3] = float("nan")
    print(f"pairs D={D} rows={rows}", flush=True)
    plan = B.difa_plan_create(1, 2, D, max_tokens=wl.N)
    try:
        I.force_rows(plan, rows)
        clean = gpu_joint_attention(q, k, v, None, hp, win, n_text, n_img, plan=plan)
        out = gpu_joint_attention(broken, k, v, None, hp, win, n_text, n_img, plan=plan)
    finally:
        B.difa_plan_destroy(plan)
    assert not bool(torch.isfinite(out[:, :, bad].float()).any())
    out[:, :, bad] = clean[:, :, bad]
    check_against_oracle(out, q, k, v, None, hp, win, n_text, n_img)
