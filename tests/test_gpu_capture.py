"""A layer captured into a HIP graph while its schedule is still being corrected: the graph goes on launching the schedule it
was captured with, whatever the plan object does afterwards."""
import pytest
import torch

import internal as I
from paper_2503_22796_amd import workloads as W
from util import same_result_bf16

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("warm_up", [1, 4, 10])
@pytest.mark.parametrize("static", [True, False])
def test_a_captured_layer_keeps_its_schedule(warm_up, static):
    from paper_2503_22796_amd import binding as B
    wl = W.flux_1k()
    dev = torch.device("cuda:0")
    q, k, v = (t.to(dev) for t in W.make_qkv(wl))
    cache = W.make_cache(wl).to(dev)
    call = B.difa_joint_attention_static if static else B.difa_joint_attention
    plan = B.difa_plan_create(wl.B, wl.H, wl.D, max_tokens=wl.N)
    stream = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    eager, captured = torch.empty_like(q), torch.empty_like(q)
    print(f"capture: warm_up={warm_up} static={static}", flush=True)
    try:
        stream.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(stream):
            for _ in range(warm_up):
                call(plan, q, k, v, eager, cache, wl.head_plan, wl.n_text, wl.n_img, wl.window)
                stream.synchronize()
            first = eager.clone()
            before = B.difa_plan_die_speeds(plan)[2]
            with torch.cuda.graph(graph, stream=stream):
                call(plan, q, k, v, captured, cache, wl.head_plan, wl.n_text, wl.n_img, wl.window)
            pieces = I.last_call(plan)["n_pieces"]
            assert pieces > 0
            for turn in range(4):
                captured.fill_(float("nan"))
                graph.replay()
                stream.synchronize()
                # (not bit for bit: which piece of a cut record finishes last, and folds the others in, is a matter of time)
                same = same_result_bf16(captured.cpu(), first.cpu())
                assert same, f"replay {turn}"
                for _ in range(20):              # as many eager calls as three corrections take
                    eager.fill_(float("nan"))
                    call(plan, q, k, v, eager, cache, wl.head_plan, wl.n_text, wl.n_img, wl.window)
                    stream.synchronize()
                same = same_result_bf16(eager.cpu(), first.cpu())
                assert same, f"eager calls behind replay {turn}"
            assert B.difa_plan_die_speeds(plan)[2] == before and I.last_call(plan)["n_pieces"] == pieces
    finally:
        torch.cuda.synchronize()
        del graph
        B.difa_plan_destroy(plan)


def test_a_graph_whose_schedule_has_given_way_writes_nothing_and_harms_nothing():
    """The schedule's place is taken by one for the other record length; the graph was captured for 256 rows on 256 workgroups."""
    from paper_2503_22796_amd import binding as B
    wl = W.flux_1k()
    dev = torch.device("cuda:0")
    q, k, v = (t.to(dev) for t in W.make_qkv(wl))
    cache = W.make_cache(wl).to(dev)
    plan = B.difa_plan_create(wl.B, wl.H, wl.D, max_tokens=wl.N)
    stream, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    eager, captured = torch.empty_like(q), torch.empty_like(q)

    def call(out):
        B.difa_joint_attention(plan, q, k, v, out, cache, wl.head_plan, wl.n_text, wl.n_img, wl.window)

    print("capture: a schedule that has given way", flush=True)
    try:
        stream.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(stream):
            I.force_rows(plan, 256)
            call(eager)
            stream.synchronize()
            first = eager.clone()
            with torch.cuda.graph(graph, stream=stream):
                call(captured)
            captured.fill_(float("nan"))
            graph.replay()
            stream.synchronize()
            same = same_result_bf16(captured.cpu(), first.cpu())
            assert same
            I.force_rows(plan, 128)               # the plan object forgets its schedules: the next one takes the first place
            for _ in range(3):
                eager.fill_(float("nan"))
                call(eager)
                captured.fill_(float("nan"))
                graph.replay()
                stream.synchronize()
                assert I.last_call(plan)["rows"] == 128 and I.last_call(plan)["n_pieces"] > 0
                same = same_result_bf16(eager.cpu(), first.cpu())
                untouched = bool(torch.isnan(captured).all())
                assert same and untouched
    finally:
        torch.cuda.synchronize()
        del graph
        B.difa_plan_destroy(plan)
