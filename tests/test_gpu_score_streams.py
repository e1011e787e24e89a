"""A context's small scoring calls, whose few records are reduced by the pass that writes them, after launches that overlapped: those
share the records and may spoil each other's scores (one context per stream), but no later call's.  And calls on several streams in turn,
with captured ones between."""
import pytest

pytestmark = pytest.mark.gpu

import paper_2603_03592_amd as sv
import stage_inputs as si

ARGS = dict(metrics=("rel_l2", "l1", "zl2", "sfr"), tau={"rel_l2": 0.5, "l1": 0.5, "zl2": 0.5, "sfr": 0.2})
SHAPES = [(1, 256, 512), (1, 31, 64), (16, 16, 128), (3, 77, 960)]


def _inputs(n, T, D, scale):
    import torch
    ref = torch.randn(n, T, D, device="cuda")
    return (ref + scale * torch.randn(n, T, D, device="cuda")).bfloat16(), ref


def _score(ver, x):
    import torch
    got = ver.score_and_flag(*x, **ARGS)["result"].view(torch.uint8).reshape(-1)
    return got


def _want(x):
    import torch
    return sv.score_and_flag_noalloc(*x, torch.zeros(x[0].shape[0], 32, dtype=torch.uint8, device="cuda"), **ARGS).reshape(-1)


def _verifier():
    return sv.Verifier(si.StageDesc(1, 128, 4, 4, 512, mlp="gelu", norm="ln", rope=False, dtype="f32"), 64, 64)


def test_launches_that_overlapped_spoil_no_later_call():
    import torch
    torch.manual_seed(5)
    ver = _verifier()
    ins = [_inputs(*s, 0.1 + i) for i, s in enumerate(SHAPES)]
    wants = [_want(x) for x in ins]
    side = [torch.cuda.Stream() for _ in range(3)]
    torch.cuda.synchronize()
    kept = []
    for rep in range(20):
        for i, s in enumerate(side):
            with torch.cuda.stream(s):
                kept.append(_score(ver, ins[(rep + i) % len(ins)]))
    torch.cuda.synchronize()
    for s in [torch.cuda.current_stream()] + side:
        for x, want in zip(ins, wants):
            with torch.cuda.stream(s):
                got = _score(ver, x)
            s.synchronize()
            assert torch.equal(got, want)
    ver.close()


def test_streams_in_turn_with_captured_calls_between():
    import torch
    torch.manual_seed(6)
    ver = _verifier()
    ins = [_inputs(*s, 0.1 + i) for i, s in enumerate(SHAPES)]
    wants = [_want(x) for x in ins]
    for x, want in zip(ins, wants):
        assert torch.equal(_score(ver, x), want)
    torch.cuda.synchronize()
    graph, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    static = [t.clone() for t in ins[0]]
    with torch.cuda.graph(graph, stream=torch.cuda.Stream()):
        out = _score(ver, static)
    for rep in range(4):
        x, want = ins[0], wants[0]
        if rep % 2:
            x = _inputs(*SHAPES[0], 0.1 * rep)
            want = _want(x)
        for a, b in zip(static, x):
            a.copy_(b)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want), rep
        with torch.cuda.stream(side):
            got = [_score(ver, x) for x in ins]
        side.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(got, wants))
    del graph
    ver.close()
