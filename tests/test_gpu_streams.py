"""GPU tests of the launch contract: everything is enqueued on the caller's stream, nothing is
allocated or synchronised inside the library, so a call can run on a side stream and can be
captured into a HIP graph and replayed."""
import numpy as np
import pytest
import torch

import paper_2605_02568_amd as P

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def _problem(seed, S, T, k, H=64, D=128, B=1):
    g = torch.Generator(device="cpu").manual_seed(seed)
    q = torch.randn((B, S, H, D), generator=g).to(torch.bfloat16).to(DEV)
    K = torch.randn((B, T, D), generator=g).to(torch.bfloat16).to(DEV)
    w = (torch.randn((B, S, H), generator=g) / np.sqrt(H)).to(DEV)
    return q, K, w


def _outputs(S, k, B=1):
    return (torch.full((B, S, k), -7, dtype=torch.int32, device=DEV),
            torch.full((B, S, k), 123.0, dtype=torch.float32, device=DEV))


def _same(a, b):
    return torch.equal(a[0], b[0]) and torch.equal(a[1].view(torch.int32), b[1].view(torch.int32))


@pytest.mark.parametrize("schedule", ["tiled", "single_pass", "single_pass_wide", "static"])
@pytest.mark.parametrize("S,T,m,k", [(2048, 512, 4, 64), (1536, 1536, 1, 1024)])
def test_side_stream_and_graph_replay(S, T, m, k, schedule):
    print(f"streams S={S} T={T} m={m} k={k} {schedule}", flush=True)
    q, K, w = _problem(11, S, T, k)
    c_S, c_T = 512, 384
    if schedule == "tiled":
        ws = torch.empty(P.si_workspace_bytes(1, S, 64, 128, T, k, c_S, c_T), dtype=torch.uint8, device=DEV)
        call = lambda oi, os_, stream=None: P.si_indexer_topk_tiled(  # noqa: E731
            q, K, w, m, k, P.SI_MASK_CAUSAL_BLOCK, c_S, c_T, oi, os_, ws, stream=stream)
    elif schedule == "static":  # scratch inside the library; its address is looked up by the eager call below
        ws = torch.empty(256, dtype=torch.uint8, device=DEV)
        call = lambda oi, os_, stream=None: P.si_indexer_topk_static(  # noqa: E731
            q, K, w, m, k, P.SI_MASK_CAUSAL_BLOCK, oi, os_, stream=stream)
    else:  # the library's choice of workgroup shape (narrow at these key ranges), or the wide one
        shape = 8 if schedule == "single_pass_wide" else 0
        ws = torch.empty(P.si_fused_workspace_bytes(1, S, 64, 128, T, k, c_S), dtype=torch.uint8, device=DEV)
        call = lambda oi, os_, stream=None: P.si_indexer_topk_fused_shape(  # noqa: E731
            q, K, w, m, k, P.SI_MASK_CAUSAL_BLOCK, c_S, shape, oi, os_, ws, stream=stream)

    eager = _outputs(S, k)
    call(eager[0], eager[1])
    torch.cuda.synchronize()

    # a side stream (default priority): the result is there once that stream is synchronised
    side = torch.cuda.Stream()
    on_side = _outputs(S, k)
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        call(on_side[0], on_side[1], stream=side)
    side.synchronize()
    assert _same(eager, on_side)

    # graph capture of the whole call; every replay is checked, with eager work and
    # synchronisations of the program's own in between
    captured = _outputs(S, k)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call(captured[0], captured[1])
    for replay in range(3):
        captured[0].fill_(-9)
        captured[1].fill_(-1.0)
        ws.random_(0, 255)  # the workspace carries nothing from call to call
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert _same(eager, captured), f"replay {replay}"
        again = _outputs(S, k)
        call(again[0], again[1])
        torch.cuda.synchronize()
        assert _same(eager, again)


def _replays(call, outputs, ws):
    """call(outputs, stream) eagerly, on a side stream and captured; every replay checked, with eager work and
    synchronisations of the program's own in between."""
    def fresh():
        return [torch.full_like(o, -9) for o in outputs]

    def same(a, b):
        return all(torch.equal(x.view(torch.int32), y.view(torch.int32)) for x, y in zip(a, b))

    eager, on_side, captured = fresh(), fresh(), fresh()
    call(eager, None)
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        call(on_side, side)
    side.synchronize()
    assert same(eager, on_side)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call(captured, None)
    for replay in range(3):
        for o in captured:
            o.fill_(-9)
        ws.random_(0, 255)  # the workspace carries nothing from call to call
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert same(eager, captured), f"replay {replay}"
        again = fresh()
        call(again, None)
        torch.cuda.synchronize()
        assert same(eager, again)


@pytest.mark.parametrize("B,S,H,D,T,m,k,mask,kernels", [
    (1, 2, 64, 128, 40000, 1, 512, 0, 2),    # one wave per query, several workgroups per row (counters in the workspace)
    (1, 16, 64, 128, 40000, 1, 512, 0, 3),   # shared keys, maxima in a kernel of their own
    (1800, 1, 64, 32, 1000, 1, 100, 0, 2),   # rows selected by one wave
    (1, 9000, 64, 128, 2500, 4, 100, 1, 2),  # causal, by two waves
    (1, 2500, 64, 128, 2500, 4, 100, 1, 1),  # scores and selection in one kernel
])
def test_dense_schedule_on_a_side_stream_and_replayed(B, S, H, D, T, m, k, mask, kernels):
    print(f"streams dense B={B} S={S} H={H} D={D} T={T} k={k}", flush=True)
    q, K, w = _problem(14, S, T, k, H, D, B)
    ws = torch.empty(B * S * T * 4 + (32 << 20), dtype=torch.uint8, device=DEV)
    P.si_profile_reset()
    P.si_profile_enable(True)
    P.si_indexer_topk(q, K, w, m, k, mask, *_outputs(S, k, B), ws)
    prof = P.si_profile_read()
    P.si_profile_enable(False)
    assert prof["score_tile"][1] == 1 and prof["finalize"][1] == int(kernels > 1) and prof["init"][1] == int(kernels > 2)
    assert sum(n for _, n in prof.values()) == kernels
    _replays(lambda o, stream: P.si_indexer_topk(q, K, w, m, k, mask, o[0], o[1], ws, stream=stream), _outputs(S, k, B), ws)


@pytest.mark.parametrize("R,n,k", [(2, 140000, 512), (3, 300, 16), (2000, 1000, 512)])
def test_selection_on_a_side_stream_and_replayed(R, n, k):
    print(f"streams selection R={R} n={n} k={k}", flush=True)
    x = torch.randn((R, n), generator=torch.Generator().manual_seed(n)).to(DEV)
    ws = torch.empty(P.si_workspace_bytes(1, R, 1, 32, n, k, R, 8192), dtype=torch.uint8, device=DEV)
    outputs = (torch.empty((R, k), dtype=torch.int32, device=DEV), torch.empty((R, k), device=DEV))
    _replays(lambda o, stream: P.si_topk_from_scores(x, None, k, 8192, o[0], o[1], ws, stream=stream), outputs, ws)


def test_few_queries_of_the_consumer_on_a_side_stream_and_replayed():
    B, H, D, T, k = 5, 64, 128, 700, 300
    g = torch.Generator().manual_seed(15)
    qa = torch.randn((B, 1, H, D), generator=g).to(torch.bfloat16).to(DEV)
    K = torch.randn((B, T, D), generator=g).to(torch.bfloat16).to(DEV)
    idx = torch.stack([torch.randperm(T, generator=g)[:k] for _ in range(B)]).to(torch.int32).view(B, 1, k).to(DEV)
    _replays(lambda o, stream: P.si_sparse_attention(qa, K, idx, 1, 0, 17, 0.1, o[0], stream=stream),
             (torch.empty((B, 1, H, D), device=DEV),), torch.empty(16, dtype=torch.uint8, device=DEV))


def test_consumer_under_graph_replay():
    """si_sparse_attention launches one kernel and allocates nothing: capture and replay."""
    S, T, m, k, H, D = 512, 128, 4, 32, 64, 128
    q, K, w = _problem(12, S, T, k)
    g = torch.Generator(device="cpu").manual_seed(13)
    qa = torch.randn((1, S, H, D), generator=g).to(torch.bfloat16).to(DEV)
    idx, score = _outputs(S, k)
    ws = torch.empty(P.si_fused_workspace_bytes(1, S, H, D, T, k), dtype=torch.uint8, device=DEV)
    P.si_indexer_topk(q, K, w, m, k, P.SI_MASK_CAUSAL_BLOCK, idx, score, ws)
    eager = torch.empty((1, S, H, D), dtype=torch.float32, device=DEV)
    P.si_sparse_attention(qa, K, idx, m, P.SI_MASK_CAUSAL_BLOCK, 8, 0.1, eager)
    torch.cuda.synchronize()
    captured = torch.empty_like(eager)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        P.si_sparse_attention(qa, K, idx, m, P.SI_MASK_CAUSAL_BLOCK, 8, 0.1, captured)
    for replay in range(3):
        captured.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(eager.view(torch.int32), captured.view(torch.int32)), f"replay {replay}"
