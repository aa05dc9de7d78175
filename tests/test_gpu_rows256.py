"""head_dim 128, records of 256 query rows (one workgroup of eight wavefronts to a compute unit): which layers run in this
form is a rule on their work, and most layers of a test's size do not.  Here the form is chosen by hand, at the sizes where
it can go wrong: a text part and bands that end inside a record, a wavefront's rows or a key tile, a ragged tail, both token
orders, both layouts, the block-granular band, cached and residual-sharing heads, cut records; and both forms in turn on one
plan object, which share the scratch for cut records, the tickets and the run-time reports."""
import numpy as np
import pytest
import torch

import internal as I
from paper_2503_22796_amd import workloads as W
from util import ARROW, CACHE, FULL, TOL_BF16, boundary_rows, check_against_oracle

pytestmark = pytest.mark.gpu
RES = 3


def _tensors(wl, image_first):
    q, k, v = W.make_qkv(wl)
    cache = W.make_cache(wl)
    if image_first:
        rot = list(range(wl.n_text, wl.N)) + list(range(wl.n_text))
        q, k, v, cache = (t[:, :, rot].contiguous() for t in (q, k, v, cache))
    return q, k, v, cache


def _call(plan, q, k, v, cache, wl, layout="bhnd", residual=None):
    from paper_2503_22796_amd import binding as B
    dev = torch.device("cuda:0")
    put = lambda t: (t.transpose(1, 2).contiguous() if layout == "bnhd" else t).to(dev)
    out = put(torch.full_like(q, float("nan")))
    B.difa_joint_attention_residual(plan, put(q), put(k), put(v), out, put(cache), put(residual) if residual is not None else None,
                                    wl.head_plan, wl.n_text, wl.n_img, wl.window)
    torch.cuda.synchronize()
    return (out.transpose(1, 2) if layout == "bnhd" else out).contiguous().cpu()


@pytest.mark.parametrize("n_text,n_img", [(0, 1), (0, 64), (1, 127), (100, 155), (130, 126), (255, 258), (200, 600), (77, 1300)])
@pytest.mark.parametrize("flags", [0, 1, 2, 3])
@pytest.mark.parametrize("layout", ["bhnd", "bnhd"])
def test_long_records(n_text, n_img, flags, layout):
    from paper_2503_22796_amd import binding as B
    wl = W.Workload("rows256", 2, 6, 128, n_text, n_img, np.asarray([FULL, ARROW, ARROW, CACHE, ARROW, ARROW], np.int32),
                    np.asarray([0, 0, 63, 0, 64, 300], np.int32), seed=840 + n_text)
    image_first = bool(flags & B.DIFA_FLAG_IMAGE_FIRST)
    q, k, v, cache = _tensors(wl, image_first)
    print(f"rows256 n_text={n_text} n_img={n_img} flags={flags} {layout}", flush=True)
    plan = B.difa_plan_create(2, 6, 128, max_tokens=wl.N, flags=flags, layout=B.DIFA_LAYOUT_BNHD if layout == "bnhd" else B.DIFA_LAYOUT_BHND)
    try:
        I.force_rows(plan, 256)
        out = _call(plan, q, k, v, cache, wl, layout)
        assert I.last_call(plan)["rows"] == 256
    finally:
        B.difa_plan_destroy(plan)
    check_against_oracle(out, q, k, v, cache, wl.head_plan, wl.window, n_text, n_img, image_first=image_first,
                         block=B.difa_tile_shape(128) if flags & B.DIFA_FLAG_BLOCK_BAND else None)


@pytest.mark.parametrize("image_first", [False, True])
def test_long_records_with_residual_sharing(image_first):
    from oracle import residual_oracle as R
    from paper_2503_22796_amd import binding as B
    wl = W.Workload("rows256r", 1, 5, 128, 77, 900, np.asarray([RES, FULL, RES, CACHE, RES], np.int32),
                    np.asarray([40, 0, 300, 0, 5000], np.int32), seed=870)
    q, k, v, cache = _tensors(wl, image_first)
    residual = (0.25 * W.make_cache(wl, step=3, dtype=torch.float32)).to(torch.bfloat16)
    plan = B.difa_plan_create(1, 5, 128, max_tokens=wl.N, flags=B.DIFA_FLAG_IMAGE_FIRST if image_first else 0)
    try:
        I.force_rows(plan, 256)
        out = _call(plan, q, k, v, cache, wl, residual=residual)
    finally:
        B.difa_plan_destroy(plan)
    ref, raw = R.joint_attention(q, k, v, cache, residual, wl.head_plan, wl.window, wl.n_text, wl.n_img, image_first=image_first)
    for h in range(5):
        if wl.head_plan[h] == CACHE:
            assert torch.equal(out[:, h].view(torch.int16), raw[:, h].contiguous().view(torch.int16))
        else:
            assert float((out[:, h].double() - ref[:, h]).abs().max()) <= TOL_BF16, f"head {h}"


def test_a_layer_above_the_line_with_bands_a_ragged_tail_and_cut_records():
    from paper_2503_22796_amd import binding as B
    # a CFG pair of a 2K plan, 21 M pairs for each of 256 compute units; 333 text and 16367 image tokens are multiples of nothing
    hp = np.asarray(([FULL] * 8 + [ARROW] * 10 + [CACHE] * 6), np.int32)
    win = np.asarray([0] * 8 + [512, 1024, 2048] * 3 + [777] + [0] * 6, np.int32)
    wl = W.Workload("above", 2, 24, 128, 333, 16367, hp, win, seed=880, grid=(1, 16367))
    q, k, v, cache = _tensors(wl, False)
    plan = B.difa_plan_create(2, 24, 128, max_tokens=wl.N)
    try:
        out = _call(plan, q, k, v, cache, wl)
        last = I.last_call(plan)
        assert last["rows"] == 256 and last["n_pieces"] > 0, last
    finally:
        B.difa_plan_destroy(plan)
    rows = boundary_rows(wl.n_text, wl.n_img, [512, 777, 1024, 2048], bm=256, extra=24, seed=5)
    check_against_oracle(out, q, k, v, cache, hp, win, wl.n_text, wl.n_img, rows=rows, flat_below=4.0)


def test_both_forms_in_turn_on_one_plan_object():
    from paper_2503_22796_amd import binding as B
    modes = np.asarray([FULL, ARROW, ARROW, CACHE, FULL, ARROW, ARROW, FULL, CACHE, ARROW, FULL, ARROW], np.int32)
    wins = np.asarray([0, 64, 300, 0, 0, 128, 1000, 0, 0, 17, 0, 512], np.int32)
    layers = [W.Workload("turn", 1, 12, 128, nt, ni, modes, wins, seed=890 + nt) for nt, ni in ((512, 4096), (77, 2048))]
    data = [_tensors(wl, False) for wl in layers]
    refs = {}
    plan = B.difa_plan_create(1, 12, 128, max_tokens=layers[0].N)
    try:
        for turn, (rows, n) in enumerate([(256, 0), (128, 1), (256, 1), (128, 0), (256, 0), (128, 1)]):
            wl = layers[n]
            I.force_rows(plan, rows)
            print(f"both forms: turn {turn}, {rows} rows, {wl.N} tokens", flush=True)
            out = _call(plan, *data[n], wl)
            last = I.last_call(plan)
            assert last["rows"] == rows and last["n_pieces"] > 0, last
            key = (n, "ref")
            if key not in refs:
                check_against_oracle(out, *data[n], wl.head_plan, wl.window, wl.n_text, wl.n_img, flat_below=4.0)
                refs[key] = out
            diff = (out.double() - refs[key].double()).abs()
            assert torch.isfinite(out.float()).all() and float(diff.max()) <= 2 * TOL_BF16 + 2.0 ** -7 * float(out.abs().max())
    finally:
        B.difa_plan_destroy(plan)
