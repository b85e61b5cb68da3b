"""dX of a small layer: the scratch that it can use belongs to the call, not to what the calls of a stream share."""
import threading

import pytest
import torch

import paper_2409_09708_amd as nm
from paper_2409_09708_amd import binding


def test_small_layers_leave_the_shared_scratch_alone(monkeypatch):
    asked = []

    class Library:
        nm_backward_input_workspace_bytes = staticmethod(lambda O, K, T: 0 if O <= 3072 else 4096)
        nm_backward_input_scratch_bytes = staticmethod(lambda O, K, T: 0 if O == 32 else 8192)
        nm_linear_backward_input = staticmethod(lambda *a: asked.append(("required", a[11])) or 0)
        nm_linear_backward_input_scratch = staticmethod(lambda *a: asked.append(("scratch", a[11])) or 0)

    class Calls:
        backward_input = staticmethod(lambda *a: NotImplemented)

    own = lambda nbytes, stream=None: asked.append("own") or torch.empty(nbytes, dtype=torch.uint8)
    shared = lambda nbytes, device, stream=None: asked.append("shared") or torch.empty(nbytes, dtype=torch.uint8)
    for name, value in (("_CALLS", Calls), ("load_library", lambda: Library), ("_need", lambda *a: None), ("_own_scratch", own),
                        ("_workspace", shared), ("_stream_handle", lambda stream: 0)):
        monkeypatch.setattr(binding, name, value)
    for O, want in ((3072, ["own", ("scratch", 8192)]), (4096, ["shared", ("required", 4096)]), (32, [("required", 0)])):
        asked.clear()
        nm.nm_linear_backward_input(torch.zeros(O, 64, dtype=torch.bfloat16), torch.zeros(5, O, dtype=torch.bfloat16))
        assert asked == want


def layer(T, K, O, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    draw = lambda r, c: torch.empty(r, c, dtype=torch.bfloat16, device="cuda").normal_(generator=g)
    assert nm.nm_backward_input_workspace_bytes(O, K, T) == 0 < binding.load_library().nm_backward_input_scratch_bytes(O, K, T)
    return draw(O, K), draw(T, O)


@pytest.mark.gpu
@pytest.mark.parametrize("explicit", [False, True])
def test_a_recorded_product_outlives_larger_calls_on_its_stream(explicit):
    W, dY = layer(197, 768, 3072, 1)
    side = torch.cuda.Stream()
    kept = dict(binding._WORKSPACES)
    out = torch.zeros(197, 768, device="cuda")
    graph = torch.cuda.CUDAGraph()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.graph(graph, stream=side):
        nm.nm_linear_backward_input(W, dY, out=out, stream=side if explicit else None)
    assert binding._WORKSPACES == kept
    large = torch.zeros(12608, 2304, dtype=torch.bfloat16, device="cuda")
    Wl = torch.zeros(2304, 768, dtype=torch.bfloat16, device="cuda")
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        nm.nm_linear_backward_input(Wl, large)  # grows the scratch that the stream's calls share
        others = [torch.full((1 << 20,), 3, dtype=torch.uint8, device="cuda") for _ in range(24)]
    torch.cuda.synchronize()
    for seed in (2, 3, 4):
        Wn, dYn = layer(197, 768, 3072, seed)
        W.copy_(Wn), dY.copy_(dYn)
        want = nm.nm_linear_backward_input(W, dY)
        out.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want)
        assert all(bool((o == 3).all()) for o in others)


@pytest.mark.gpu
@pytest.mark.parametrize("named", [False, True])
def test_two_threads_on_one_stream(named):
    stream = torch.cuda.Stream() if named else None  # (not the current stream: the scratch is that stream's all the same)
    layers = [layer(197, 768, 3072, 10), layer(65, 768, 2304, 11)]
    want = [nm.nm_linear_backward_input(W, dY, workspace=torch.empty(8, dtype=torch.uint8, device="cuda")) for W, dY in layers]
    assert binding._CALLS.backward_input(*layers[0], None, None, None, stream) is not NotImplemented
    torch.cuda.synchronize()
    wrong, start = [], threading.Barrier(2)

    def work(n):
        W, dY = layers[n]
        start.wait()
        got = [nm.nm_linear_backward_input(W, dY, stream=stream) for _ in range(300)]
        torch.cuda.synchronize()
        wrong.append(sum(not torch.equal(y, want[n]) for y in got))

    threads = [threading.Thread(target=work, args=(n,)) for n in (0, 1)]
    [t.start() for t in threads], [t.join() for t in threads]
    assert wrong == [0, 0]


def test_when_the_scratch_is_worth_bringing():
    lib = binding.load_library()
    for T, O, K, f32, bf16 in ((197, 3072, 768, 1, 1), (4, 256, 256, 0, 0), (64, 256, 64, 0, 0), (65, 256, 64, 1, 0), (788, 256, 768, 1, 0),
                               (1, 384, 64, 1, 1), (12608, 2304, 768, 1, 1), (1576, 768, 2048, 0, 0), (4, 32, 64, 0, 0), (0, 256, 256, 0, 0)):
        assert [lib.nm_backward_input_scratch_pays(O, K, T, dtype, None) for dtype in (0, 1)] == [f32, bf16], (T, O, K)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("T,K,O,alone", [(4, 256, 256, 0), (64, 64, 256, 0), (197, 768, 3072, 1)])
def test_launches_of_a_call_and_of_a_recorded_one(T, K, O, alone, dtype):
    W, dY = layer(T, K, O, 20)
    out, recorded = (torch.zeros(T, K, dtype=dtype, device="cuda") for _ in range(2))
    call = lambda y: nm.nm_linear_backward_input(W, dY, out=y)
    call(out)
    allocations = lambda: torch.cuda.memory_stats()["allocation.all.allocated"]
    before = allocations()
    call(out)
    assert allocations() - before == alone  # the copy's scratch: two launches
    side, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.graph(graph, stream=side):
        before = allocations()
        call(recorded)
        assert allocations() - before == 1
    for _ in range(3):
        recorded.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(recorded, out)
