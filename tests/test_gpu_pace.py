"""Calls whose time must not depend on what a neighbouring call's does not: the two are timed in turn, in one process, as captured
graphs of several calls.  The bounds lie about half way between the two readings of a slow and a sound kernel."""
import pytest
import torch

from paper_2510_08055_amd import inputs

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
CALLS, ROUNDS = 20, 15


def captured(fn):
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        fn()
    torch.cuda.current_stream().wait_stream(side)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        for _ in range(CALLS):
            fn()
    graph.replay()
    torch.cuda.synchronize()
    return graph


def times(*fns):
    """The shortest of several rounds of each, us a call."""
    graphs = [captured(f) for f in fns]
    best = [float("inf")] * len(fns)
    for _ in range(ROUNDS):
        for i, g in enumerate(graphs):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            g.replay()
            b.record()
            torch.cuda.synchronize()
            best[i] = min(best[i], a.elapsed_time(b) * 1000 / CALLS)
    return best


# A token's rows are in flight eight at a time whatever divides their number: 29 rows take no longer than 32 (measured, us, one by
# one / by eights and the rest: fp32, 256 tokens 11.1 / 6.6 where 32 take 7; bf16 15.4 / 9)
@pytest.mark.parametrize("dtype,H", [("f32", 1024), ("bf16", 2048)])
@pytest.mark.parametrize("few,many", [(29, 32), (13, 16)])
def test_combine_of_any_number_of_rows(gpu_lib, dtype, H, few, many):
    T, dt = 256, inputs.torch_dtype(dtype)

    def call(K):
        ctx = gpu_lib.Context(H, 64, K, 64, dt, max_tokens=T, device=DEV)
        y = torch.ones((T * K, H), dtype=dt, device=DEV)
        inv = torch.randperm(T * K, generator=torch.Generator().manual_seed(K)).to(torch.int32).to(DEV)
        w, x = torch.ones((T, K), device=DEV), torch.ones((T, H), dtype=dt, device=DEV)
        out = torch.empty_like(x)
        return lambda: ctx.moe_combine(y, inv, w, residual=x, out=out)

    a, b = times(call(few), call(many))
    assert a <= 1.2 * b, (a, b)


# Counting the assignments of one popular expert takes no turns of all lanes at one counter (12288 to one of 128 experts, us, one counter /
# eight: 22.9 / 6.9, evenly routed 6.7 / 6.3)
@pytest.mark.parametrize("E,A", [(128, 12288), (16, 12288), (16, 8192), (512, 4096)])
def test_permutation_of_skewed_routing(gpu_lib, E, A):
    ctx = gpu_lib.Context(64, E, 1, 64, torch.bfloat16, max_tokens=A, device=DEV)
    x = torch.ones((A, 64), dtype=torch.bfloat16, device=DEV)
    even = (torch.randperm(A, generator=torch.Generator().manual_seed(A)) % E).to(torch.int32).view(A, 1).to(DEV)
    one = torch.full((A, 1), E // 2, dtype=torch.int32, device=DEV)
    a, b = times(lambda: ctx.moe_permute(x, one, want_x_perm=False), lambda: ctx.moe_permute(x, even, want_x_perm=False))
    assert a <= 1.35 * b, (a, b)


# The one-launch routing of 256 tokens is 16 tiles of what 16 tokens are, side by side (256 experts, H = 4096, us, kernel trace: a tile's
# sums formed by four waves 36.6 / 17.0, by sixteen 24.1 / 16.2)
def test_one_launch_routing_of_many_tokens(gpu_lib):
    H, E, K, I = 4096, 256, 8, 8
    w = inputs.Workload("pace", H=H, E=E, K=K, I=I, n_layers=1, D=256, P=0, dtype="bf16", seed=5)
    L = inputs.make_layer(w, 0, device=DEV)
    best = {}
    for T in (16, 256):
        ctx = gpu_lib.Context(H, E, K, I, torch.bfloat16, max_tokens=T, device=DEV)
        x = inputs.randn((T, H), 1.0, T, "x", 0, "bf16", DEV)
        ms = []
        for _ in range(ROUNDS):
            ctx.moe_kernel_timing(["router_logits"])
            ctx.moe_group_forward([L], x, None)
            ms.append(ctx.moe_read_kernel_timing("router_logits")[0])
        best[T] = 1000 * min(ms)
    assert best[256] <= 1.65 * best[16], best
