"""Each grouped-GEMM and routing kernel at the sizes where its tiling can go wrong (edges of tiles, remainders, the
smallest and largest sizes of its range), against the fp64 oracle with the tolerance of tests/parity.py."""
import numpy as np
import pytest
import torch

import oracle
from paper_2510_08055_amd import inputs
from parity import assert_close

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def dense_ffn(x_perm, offsets, L, dtype, E):
    """The grouped FFN as each expert's dense SwiGLU FFN in the oracle (a one-expert layer with weight 1)."""
    ref = np.zeros(tuple(x_perm.shape))
    for e in range(E):
        lo, hi = int(offsets[e]), int(offsets[e + 1])
        if hi > lo:
            ones = inputs.to_numpy(torch.ones((1, x_perm.shape[1]), dtype=inputs.torch_dtype(dtype)))
            ref[lo:hi], _, _ = oracle.moe_layer(inputs.to_numpy(x_perm[lo:hi]), ones, None,
                                                inputs.to_numpy(L["w_gate_up"][e:e + 1]),
                                                inputs.to_numpy(L["w_down"][e:e + 1]), 1)
    return ref


# fp32: tiles of 32 rows x 16 columns, 16-wide k-chunks split over 4 waves
@pytest.mark.parametrize("H,I,rows", [
    (8, 8, [1]),                          # half a chunk, half a column tile
    (16, 24, [31, 0, 33]),                # one chunk: three of the four waves have no work; a ragged second column tile
    (72, 40, [32, 1, 64, 17]),            # 4.5 chunks: a ragged last chunk in the first wave
    (264, 136, [0, 15, 100]),
])
def test_f32_grouped_ffn(gpu_lib, H, I, rows):
    E, A = len(rows), sum(rows)
    w = inputs.Workload("f32", H=H, E=E, K=1, I=I, n_layers=1, D=0, P=A, dtype="f32", seed=21)
    L = inputs.make_layer(w, 0)
    x_perm = inputs.randn((A, H), 1.0, 21, "x_perm", 0, "f32")
    offsets = torch.tensor(np.concatenate([[0], np.cumsum(rows)]), dtype=torch.int32)
    ctx = gpu_lib.Context(H, E, 1, I, torch.float32, max_tokens=A, device=DEV)
    y = ctx.moe_grouped_ffn(x_perm.to(DEV), offsets.to(DEV), L["w_gate_up"].to(DEV), L["w_down"].to(DEV))
    assert_close(y, dense_ffn(x_perm, offsets, L, "f32", E), "f32", "fp32 grouped_ffn")


# one-launch routing of small batches (at most 256 tokens, 256 experts, top-16): 16-token tiles, 64-token words of the
# choice bitmask; the same layer through the step calls (three-launch routing) must give the same bits
@pytest.mark.parametrize("E,K", [(8, 2), (128, 8), (40, 16), (256, 5), (257, 3)])
@pytest.mark.parametrize("T", [1, 16, 17, 64, 65, 255, 256, 257])
def test_one_launch_routing_equals_the_steps(gpu_lib, T, E, K):
    H, I = 72, 64
    w = inputs.Workload("small", H=H, E=E, K=K, I=I, n_layers=1, D=T, P=0, dtype="bf16", seed=100 * T + E)
    L = {k: (v.to(DEV) if v is not None else None) for k, v in inputs.make_layer(w, 0).items()}
    x = inputs.randn((T, H), 1.0, w.seed, "x", 0, "bf16").to(DEV)
    for renorm in (True, False):
        ctx = gpu_lib.Context(H, E, K, I, torch.bfloat16, max_tokens=T, renormalize=renorm, residual=False, device=DEV)
        idx, wt = ctx.moe_router_topk(x, L["w_router"])
        counts, offsets, perm, inv, x_perm = ctx.moe_permute(x, idx)
        y_steps = ctx.moe_combine(ctx.moe_grouped_ffn(x_perm, offsets, L["w_gate_up"], L["w_down"]), inv, wt)
        for _ in range(2):       # a second launch finds the ticket counters at zero again
            y, _ = ctx.moe_group_forward([L], x, None)
            assert torch.equal(y, y_steps)
        assert ctx.moe_read_counters().active_experts_total == 2 * int((counts > 0).sum())


# The same at hidden sizes whose rows are long enough for the ring of asynchronous loads (16 waves take 32-wide chunks in turn:
# four chunks per wave and more from H = 1568 on): the ring once, with a tail and a partial chunk, twice; both types; a bias;
# rows from two buffers
@pytest.mark.parametrize("H,dtype", [(2048, "bf16"), (2888, "bf16"), (4096, "bf16"), (2048, "f32"), (2888, "f32")])
@pytest.mark.parametrize("T", [1, 40, 256])
def test_one_launch_routing_of_long_rows(gpu_lib, H, dtype, T):
    E, K, I = 72, 4, 64
    w = inputs.Workload("long", H=H, E=E, K=K, I=I, n_layers=1, D=T // 2, P=T - T // 2, dtype=dtype, seed=H + T)
    L = {k: (v.to(DEV) if v is not None else None) for k, v in inputs.make_layer(w, 0).items()}
    L["router_bias"] = inputs.randn((E,), 0.3, w.seed, "bias", 0, "f32").to(DEV)
    xd, xp = inputs.make_hidden(w, device=DEV)
    x = torch.cat([xd, xp])
    ctx = gpu_lib.Context(H, E, K, I, inputs.torch_dtype(dtype), max_tokens=T, residual=False, device=DEV)
    idx, wt = ctx.moe_router_topk(x, L["w_router"], L["router_bias"])
    o_idx, _ = oracle.router_topk(inputs.to_numpy(x), inputs.to_numpy(L["w_router"]), inputs.to_numpy(L["router_bias"]), K)
    assert (idx.cpu().numpy() == o_idx).all()
    _, offsets, _, inv, x_perm = ctx.moe_permute(x, idx)
    y_steps = ctx.moe_combine(ctx.moe_grouped_ffn(x_perm, offsets, L["w_gate_up"], L["w_down"]), inv, wt)
    for _ in range(2):
        yd, yp = ctx.moe_group_forward([L], xd if w.D else None, xp)
        assert torch.equal(torch.cat([yd, yp]), y_steps)


# Routing of larger batches through exact integer sums: 32-token tiles, 32-expert groups (1, 2 and 4 of them; up to and above one
# block per compute unit), 64-value steps (a ragged last one), and rows that the 32-bit fixed point holds with one rest, with
# three, not at all (four rests; no fp32 scale), of zeros.  Indices are exact; a weight is one rounding to fp32 of a quotient of
# fp64 values: 2^-23 relative.
@pytest.mark.parametrize("H,E,K,T", [(2056, 128, 8, 2290), (4104, 17, 5, 4580), (4096, 32, 1, 8225), (8, 128, 16, 586000),
                                     (16384, 64, 9, 577), (2048, 33, 3, 9190), (2048, 97, 16, 8193), (2056, 128, 8, 4690),
                                     (4104, 49, 5, 8705), (512, 96, 1, 8225)])
@pytest.mark.parametrize("renorm", [True, False])
def test_exact_routing(gpu_lib, H, E, K, T, renorm):
    if H == 8 and not renorm:
        pytest.skip("one pass over the long batch is enough")
    w = inputs.Workload("exact", H=H, E=E, K=K, I=8, n_layers=1, D=T, P=0, dtype="bf16", seed=T)
    x = inputs.randn((T, H), 1.0, w.seed, "x", 0, "bf16").float()
    wr = inputs.randn((E, H), 0.02, w.seed, "w_router", 0, "bf16").float()
    some = [0, 1, 31, 32, T - 33, T - 2, T - 1]
    for i, t in enumerate(some):
        top = float(x[t].abs().max())
        for j in range([1, 3, 4, 1, 0, 2, 1][i]):         # values far below the row's largest, with bits to the last
            x[t, (7 * j + 3 * i) % H] = (-1) ** j * top * 2.0 ** (-23 - 2 * j) * 1.3
    x[5] = 0
    x[6] *= 2.0 ** 40
    x[7] *= 2.0 ** -110
    wr[2, 1] = float(wr[2].abs().max()) * 2.0 ** -25 * 1.7
    wr[3, :4] = wr[3].abs().max() * 2.0 ** -26 * 1.9
    wr[min(11, E - 1)] = 0
    wr[min(12, E - 1)] = wr[min(14, E - 1)]               # equal logits: the lower index first
    x, wr = x.bfloat16(), wr.bfloat16()
    bias = inputs.randn((E,), 0.1, w.seed, "bias", 0, "f32")
    bias[min(12, E - 1)] = bias[min(14, E - 1)]
    ctx = gpu_lib.Context(H, E, K, 8, torch.bfloat16, max_tokens=T, renormalize=renorm, device=DEV)
    idx, wt = ctx.moe_router_topk(x.to(DEV), wr.to(DEV), bias.to(DEV))
    rows = np.unique(np.concatenate([np.arange(min(T, 64)), np.arange(T - 64, T), np.random.default_rng(1).integers(0, T, 2000)]))
    o_idx, o_w = oracle.router_topk(inputs.to_numpy(x[rows]), inputs.to_numpy(wr), bias.numpy(), K, renorm)[:2]
    assert (idx.cpu().numpy()[rows] == o_idx).all()
    np.testing.assert_allclose(wt.cpu().numpy()[rows], o_w, rtol=2.0 ** -23, atol=0)


# ... and the same bits as the fp64 pass, which smaller batches take: experts and weights of a token do not depend on its batch.
# (moe_router_topk_noalloc always takes the fp64 pass.)  Rows and experts for which that is decided by the rounding of a sum, rows
# and experts that the fixed point cannot hold, values that are not finite, biases that mask experts.
def _hard_routing(kind, T, H, E, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    x = torch.randn((T, H), generator=g, device=DEV)
    wr = torch.randn((E, H), generator=g, device=DEV) * 0.02
    bias = torch.randn((E,), generator=g, device=DEV) * 0.1
    rows = torch.randint(0, T, (T // 50,), generator=g, device=DEV)
    if kind == "ties":            # equal sums of the same products in another order, in a tenth of the rows
        # (over exponents so wide that the fp64 sums round)
        x *= 2.0 ** -torch.randint(0, 16, (T, H), generator=g, device=DEV).float()
        wr *= 2.0 ** -torch.randint(0, 16, (E, H), generator=g, device=DEV).float()
        rows = torch.randint(0, T, (T // 10,), generator=g, device=DEV)
        x[rows, H // 2:] = x[rows, :H // 2]
        for e in range(0, E - 1, 2):
            wr[e + 1] = wr[e].roll(H // 2)
            bias[e + 1] = bias[e]
    elif kind == "outliers":      # one value 10^4 times the others in some rows, 10^6 times in others: none to dozens of rests
        x[rows, rows % H] = 1e4
        x[(rows + 1) % T, rows % H] = 1e6
    elif kind == "all_outliers":  # ... and in every row
        x[:, 3] = 2e6
    elif kind == "not_finite":
        x[rows, rows % H] = torch.tensor([float("nan"), float("inf"), -float("inf")], device=DEV)[rows % 3]
        x[(rows + 1) % T] = 0
        x[(rows + 2) % T] *= 2.0 ** 60
        x[(rows + 3) % T] *= 2.0 ** -60
    elif kind == "masked":        # fewer finite logits than K in the second half of the experts' order, and zero rows: all logits tie
        bias[E // 2:] = -float("inf")
        x[rows] = 0
        bias[:E // 2] = bias[:E // 2].round(decimals=1)
    elif kind == "strays":        # experts with as many rests as are listed, and one fewer
        wr[2, :4] = wr[2].abs().max() * 2.0 ** -25 * 1.7
        wr[E - 1, H - 3:] = wr[E - 1].abs().max() * -(2.0 ** -27) * 1.9
    elif kind == "lost_expert":   # with one more; infinite
        wr[1, :5] = wr[1].abs().max() * 2.0 ** -25 * 1.7
    elif kind == "infinite_expert":
        wr[E - 2, 5] = float("inf")
    elif kind == "wide":          # values over 14 powers of two: sums that are rounded in some places, in all, in none
        x *= 2.0 ** -torch.randint(0, 15, (T, H), generator=g, device=DEV).float()
        wr[::2] *= 2.0 ** -torch.randint(0, 15, (E, H), generator=g, device=DEV).float()[::2]
    elif kind == "zero_router":
        wr.zero_()
    return x.bfloat16(), wr.bfloat16(), bias


@pytest.mark.parametrize("kind", ["normal", "ties", "outliers", "all_outliers", "not_finite", "masked", "strays", "lost_expert",
                                  "infinite_expert", "zero_router", "wide"])
@pytest.mark.parametrize("H,E,K,T,renorm", [(2048, 128, 8, 6000, True), (2056, 100, 16, 16421, False), (2880, 64, 4, 17000, True),
                                            (3080, 50, 3, 12345, False), (1096, 64, 6, 24000, True), (16376, 97, 9, 4800, False)])
def test_exact_routing_is_the_fp64_pass(gpu_lib, kind, H, E, K, T, renorm):
    x, wr, bias = _hard_routing(kind, T, H, E, 7 * T + H)
    ctx = gpu_lib.Context(H, E, K, 8, torch.bfloat16, max_tokens=T, renormalize=renorm, device=DEV)
    step = (1 << 19) // E
    for b in (bias, None):
        want = [gpu_lib.moe_router_topk_noalloc(x[t:t + step], wr, b, K, renormalize=renorm) for t in range(0, T, step)]
        want_idx, want_w = torch.cat([i for i, _ in want]), torch.cat([w for _, w in want])
        for _ in range(2):
            idx, w = ctx.moe_router_topk(x, wr, b)
            assert torch.equal(idx, want_idx)
            assert torch.equal(w.view(torch.int32), want_w.view(torch.int32)) or (
                torch.equal(w.isnan(), want_w.isnan()) and torch.equal(w.nan_to_num(), want_w.nan_to_num()))


@pytest.mark.parametrize("kind", ["ties", "outliers", "not_finite", "lost_expert"])
@pytest.mark.parametrize("H,E,K,T", [(2048, 128, 8, 6000), (2880, 64, 4, 17000)])
def test_hard_routing_in_a_group(gpu_lib, kind, H, E, K, T):
    """The histograms behind the permutation hold listed tokens too; a token's outputs are those of a small batch."""
    I = 64
    x, wr, bias = _hard_routing(kind, T, H, E, T + H)
    w = inputs.Workload("hard", H=H, E=E, K=K, I=I, n_layers=1, D=0, P=T, dtype="bf16", seed=9)
    L = {k: (v.to(DEV) if v is not None else None) for k, v in inputs.make_layer(w, 0).items()}
    L["w_router"], L["router_bias"] = wr, bias
    ctx = gpu_lib.Context(H, E, K, I, torch.bfloat16, max_tokens=T, residual=False, device=DEV)
    for _ in range(2):
        _, y = ctx.moe_group_forward([L], None, x, "layered")
        _, part = ctx.moe_group_forward([L], None, x, "chunked", 1000)
        assert torch.equal(y.view(torch.int16), part.view(torch.int16))
    idx, wt = ctx.moe_router_topk(x, wr, bias)
    counts, offsets, perm, inv, x_perm = ctx.moe_permute(x, idx)
    z = ctx.moe_combine(ctx.moe_grouped_ffn(x_perm, offsets, L["w_gate_up"], L["w_down"]), inv, wt)
    assert torch.equal(y.view(torch.int16), z.view(torch.int16))
    packed, out, want = ctx.pack_layers([L]), torch.empty_like(y), y.clone()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        ctx.moe_group_forward([L], None, x, "layered", packed=packed, y_prefill=out)
    for _ in range(3):               # every replay finds the list empty
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out.view(torch.int16), want.view(torch.int16))
        ctx.moe_group_forward([L], None, x.roll(1, 0), "layered")


# Which batches take them: a number of logits, whatever the length of the rows (the top-k then has no launch of its own).
@pytest.mark.parametrize("H,E,T,exact", [(16384, 64, 577, False), (16384, 128, 300, False), (4096, 128, 1200, False),
                                         (2880, 48, 17000, False), (2048, 128, 3583, False), (2048, 128, 3584, True),
                                         (2048, 64, 7167, False), (2048, 64, 7168, True), (256, 50, 10751, False),
                                         (256, 50, 10752, True)])
def test_exact_routing_rule(gpu_lib, H, E, T, exact):
    w = inputs.Workload("rule", H=H, E=E, K=2, I=8, n_layers=1, D=0, P=T, dtype="bf16", seed=3)
    L = {k: (v.to(DEV) if v is not None else None) for k, v in inputs.make_layer(w, 0).items()}
    x = torch.randn((T, H), dtype=torch.bfloat16, device=DEV)
    ctx = gpu_lib.Context(H, E, 2, 8, torch.bfloat16, max_tokens=T, device=DEV)
    ctx.moe_kernel_timing(["topk"])
    ctx.moe_group_forward([L], None, x, "layered")
    assert ctx.moe_read_kernel_timing("topk")[1] == (0 if exact else 1)


# What the timing interface counts in such a pass: one launch a layer for each kernel, the digits with the first layer's logits
def test_timed_launches_of_a_large_batch(gpu_lib):
    H, E, K, I, T, n = 2048, 128, 8, 8, 4700, 10
    w = inputs.Workload("timed", H=H, E=E, K=K, I=I, n_layers=n, D=0, P=T, dtype="bf16", seed=5)
    layers = [{k: (v.to(DEV) if v is not None else None) for k, v in inputs.make_layer(w, l).items()} for l in range(n)]
    x = inputs.randn((T, H), 1.0, 5, "x", 0, "bf16").to(DEV)
    ctx = gpu_lib.Context(H, E, K, I, torch.bfloat16, max_tokens=T, device=DEV)
    ctx.moe_kernel_timing(list(gpu_lib.KERNELS))
    ctx.moe_group_forward(layers, None, x)
    assert [ctx.moe_read_kernel_timing(k)[1] for k in gpu_lib.KERNELS] == [n, 0, n, n, n, n]


# ... as part of a pass: the digits of ten layers come in two launches, and the top-k counts the permutation's histograms
@pytest.mark.parametrize("T", [2300, 4700])
def test_exact_routing_in_a_group(gpu_lib, T):
    H, E, K, I, n = 2048, 128, 8, 64, 10
    w = inputs.Workload("exact", H=H, E=E, K=K, I=I, n_layers=n, D=0, P=T, dtype="bf16", seed=5)
    layers = [{k: (v.to(DEV) if v is not None else None) for k, v in inputs.make_layer(w, l).items()} for l in range(n)]
    x = inputs.randn((T, H), 1.0, 5, "x", 0, "bf16").to(DEV)
    ctx = gpu_lib.Context(H, E, K, I, torch.bfloat16, max_tokens=T, device=DEV)
    for _ in range(2):
        _, y = ctx.moe_group_forward(layers, None, x, "layered")
        z = x
        for L in layers:
            idx, wt = ctx.moe_router_topk(z, L["w_router"])
            counts, offsets, perm, inv, x_perm = ctx.moe_permute(z, idx)
            z = ctx.moe_combine(ctx.moe_grouped_ffn(x_perm, offsets, L["w_gate_up"], L["w_down"]), inv, wt, residual=z)
        assert torch.equal(y, z)


# Many permutation tiles: from 2^25 histogram words read in all (tiles squared times experts), the tiles' running sums come from
# a pass of their own; one tile to either side of the border, 64-expert groups that are not whole
@pytest.mark.parametrize("T,K,E", [(65536, 8, 512), (65537, 8, 512), (300000, 5, 65), (1 << 20, 8, 3)])
def test_permute_many_tiles(gpu_lib, T, K, E):
    gen = torch.Generator(device=DEV).manual_seed(T + E)
    idx = torch.randint(0, E, (T, K), generator=gen, dtype=torch.int32, device=DEV)
    idx = torch.minimum(idx, torch.randint(0, E, (T, K), generator=gen, dtype=torch.int32, device=DEV))      # skewed
    ctx = gpu_lib.Context(8, E, min(K, E), 8, torch.bfloat16, max_tokens=T * K // min(K, E) + 1, device=DEV)
    flat = idx.reshape(-1)[:T * K // ctx.K * ctx.K].reshape(-1, ctx.K)
    counts, offsets, perm, inv, _ = ctx.moe_permute(None, flat, want_x_perm=False)
    order = torch.sort(flat.reshape(-1).long(), stable=True)
    assert torch.equal(perm.long(), order.indices)
    assert torch.equal(flat.reshape(-1)[perm.long()].long(), order.values)
    assert torch.equal(inv[perm.long()].long(), torch.arange(perm.numel(), device=DEV))
    want = torch.bincount(flat.reshape(-1).long(), minlength=E)
    assert torch.equal(counts.long(), want)
    assert torch.equal(offsets.long(), torch.cat([torch.zeros(1, dtype=torch.long, device=DEV), want.cumsum(0)]))


def test_layer_of_many_permutation_tiles(gpu_lib):
    """The same with the histograms counted by the top-k kernel: a layer against its steps."""
    T, K, E, H, I = 65600, 8, 512, 8, 8
    w = inputs.Workload("tiles", H=H, E=E, K=K, I=I, n_layers=1, D=0, P=T, dtype="bf16", seed=81, residual=False)
    L = inputs.make_layer(w, 0, device=DEV)
    x = inputs.randn((T, H), 1.0, 81, "x", 0, "bf16", DEV)
    ctx = gpu_lib.Context(H, E, K, I, torch.bfloat16, max_tokens=T, residual=False, device=DEV)
    idx, wt = ctx.moe_router_topk(x, L["w_router"])
    _, offsets, _, inv, x_perm = ctx.moe_permute(x, idx)
    y = ctx.moe_combine(ctx.moe_grouped_ffn(x_perm, offsets, L["w_gate_up"], L["w_down"]), inv, wt)
    for _ in range(2):
        assert torch.equal(ctx.moe_group_forward([L], None, x)[1], y)


# Fewer than K finite logits: a removed expert and one at -infinity compare equal, so a token may list an expert twice (the
# second time with weight 0); NaN compares with nothing.  The permutation stays one, on either routing path.
@pytest.mark.parametrize("E,K,T", [(8, 3, 5), (40, 16, 16), (128, 8, 70), (256, 5, 256), (257, 3, 256), (128, 8, 300)])
@pytest.mark.parametrize("kind", ["bias", "nan"])
def test_routing_of_logits_that_are_not_finite(gpu_lib, E, K, T, kind):
    H, I = 72, 64
    w = inputs.Workload("odd", H=H, E=E, K=K, I=I, n_layers=1, D=T, P=0, dtype="bf16", seed=T + E)
    L = {k: (v.to(DEV) if v is not None else None) for k, v in inputs.make_layer(w, 0).items()}
    x = inputs.randn((T, H), 1.0, w.seed, "x", 0, "bf16").to(DEV)
    if kind == "bias":
        L["router_bias"] = torch.full((E,), float("-inf"), device=DEV)
        L["router_bias"][[1, E - 1]] = 0.25                     # two experts are left
    else:
        x[::3, 5] = float("nan")
        x[1::3] = x[1::3].abs()                                 # and rows whose logit of expert 2 is infinite
        L["w_router"][2] = float("inf")
    ctx = gpu_lib.Context(H, E, K, I, torch.bfloat16, max_tokens=T, residual=False, device=DEV)
    idx, wt = ctx.moe_router_topk(x, L["w_router"], L["router_bias"])
    assert int(idx.min()) >= 0 and int(idx.max()) < E
    counts, offsets, perm, inv, x_perm = ctx.moe_permute(x, idx)
    y_steps = ctx.moe_combine(ctx.moe_grouped_ffn(x_perm, offsets, L["w_gate_up"], L["w_down"]), inv, wt)
    fresh = gpu_lib.Context(H, E, K, I, torch.bfloat16, max_tokens=T, residual=False, device=DEV)
    fresh.workspace[256:].fill_(0xA5)                           # behind the counters: whatever a pass does not write shows
    y, _ = fresh.moe_group_forward([L], x, None)
    assert torch.equal(y.view(torch.int16), y_steps.view(torch.int16))
    # the permutation the pass used, in the context's workspace (slices of whole 256 bytes: counters, logits, indices,
    # weights, counts, offsets, perm, inverse)
    at = (fresh.workspace.data_ptr() + 255) // 256 * 256 - fresh.workspace.data_ptr() + 256
    sizes = [T * E * 8, T * K * 4, T * K * 4, E * 4, (E + 1) * 4]
    at += sum((n + 255) // 256 * 256 for n in sizes)
    got = fresh.workspace[at:at + T * K * 4].view(torch.int32)
    assert torch.equal(got, perm)
    assert torch.equal(torch.sort(perm).values, torch.arange(T * K, dtype=torch.int32, device=DEV))


# The two streaming shapes: 64 x 128 tiles (four waves, a ring of three stages) and, taken when the launch has few tiles, 32 x 64
# (two waves, five stages).  k-extents around the length of the ring, row and column edges, a plain and a split
# intermediate.  Against the register-staged kernel bit for bit (the order of a sum is the same in every shape) and against
# the oracle.
@pytest.mark.parametrize("H,I,rows", [
    (64, 128, [1]),                        # one and two stages
    (192, 256, [31, 32, 33]),              # three and four stages (the ring's look-ahead)
    (320, 384, [0, 5, 0, 64, 65]),         # five and six
    (448, 72 * 8, [1, 0, 2]),              # seven and nine
    (1280, 64, [3] * 9),                   # 20 stages and one
])
def test_few_tiles_grouped_ffn(gpu_lib, H, I, rows):
    E, A = len(rows), sum(rows)
    w = inputs.Workload("few", H=H, E=E, K=1, I=I, n_layers=1, D=0, P=A, dtype="bf16", seed=51)
    L = inputs.make_layer(w, 0)
    x_perm = inputs.randn((A, H), 1.0, 51, "x_perm", 0, "bf16")
    offsets = torch.tensor(np.concatenate([[0], np.cumsum(rows)]), dtype=torch.int32)
    args = (x_perm.to(DEV), offsets.to(DEV), L["w_gate_up"].to(DEV), L["w_down"].to(DEV))
    for fmt in ({}, {"y_perm_f32": True}, {"y_perm_f32": True, "act_split": True}):
        ctx = gpu_lib.Context(H, E, 1, I, torch.bfloat16, max_tokens=A, device=DEV, **fmt)
        ctx.moe_set_ffn_variant("tile128")
        ref = ctx.moe_grouped_ffn(*args)
        for shape in ("few", "small", "few"):
            ctx.moe_set_ffn_variant(shape)
            assert torch.equal(ctx.moe_grouped_ffn(*args), ref), (shape, fmt)
    ctx = gpu_lib.Context(H, E, 1, I, torch.bfloat16, max_tokens=A, device=DEV)
    ctx.moe_set_ffn_variant("few")
    assert_close(ctx.moe_grouped_ffn(*args), dense_ffn(x_perm, offsets, L, "bf16", E), "bf16", "few tiles")


# 256 x 256 tiles with a block each (short rows): one to three stages on either GEMM, and longer rows when pinned; row blocks per
# wave from none to four, ragged columns, both output formats and the split intermediate
@pytest.mark.parametrize("H,I,rows", [
    (64, 192, [1, 0, 33]),
    (128, 128, [255, 256, 257, 31, 0, 95, 160]),
    (192, 64, [300] + [0] * 70 + [7]),
    (192, 320, [129, 64]),
    (8 * 41, 128, [200, 97]),                                   # gate_up takes another kernel, down has 328 columns
])
def test_wide_tiles_grouped_ffn(gpu_lib, H, I, rows):
    E, A = len(rows), sum(rows)
    w = inputs.Workload("wide", H=H, E=E, K=1, I=I, n_layers=1, D=0, P=A, dtype="bf16", seed=61)
    L = inputs.make_layer(w, 0)
    x_perm = inputs.randn((A, H), 1.0, 61, "x_perm", 0, "bf16")
    offsets = torch.tensor(np.concatenate([[0], np.cumsum(rows)]), dtype=torch.int32)
    args = (x_perm.to(DEV), offsets.to(DEV), L["w_gate_up"].to(DEV), L["w_down"].to(DEV))
    for fmt in ({}, {"y_perm_f32": True}, {"y_perm_f32": True, "act_split": True}):
        ctx = gpu_lib.Context(H, E, 1, I, torch.bfloat16, max_tokens=A, device=DEV, **fmt)
        ctx.moe_set_ffn_variant("tile128")
        ref = ctx.moe_grouped_ffn(*args)
        ctx.moe_set_ffn_variant("wide")
        for _ in range(2):
            assert torch.equal(ctx.moe_grouped_ffn(*args), ref), fmt
        if not fmt:
            assert_close(ref, dense_ffn(x_perm, offsets, L, "bf16", E), "bf16", "wide tiles")


# Weight tiles that one block alone reads are loaded as a stream: all experts in one m-tile, some, none, by the shape's tile height
@pytest.mark.parametrize("shape,H,I,rows", [
    ("few", 448, 392, [32, 1, 0, 20]), ("few", 384, 64, [33, 32, 5]), ("small", 512, 448, [64, 0, 1, 40]),
    ("small", 256, 328, [65, 64, 200]), ("big", 512, 328, [256, 1, 0, 130]), ("big", 320, 448, [100] * 17 + [257]),
    ("big", 320, 448, [257, 256, 90]),
])
@pytest.mark.parametrize("fmt", [{}, {"y_perm_f32": True, "act_split": True}])
def test_streamed_weight_tiles(gpu_lib, shape, H, I, rows, fmt):
    E, A = len(rows), sum(rows)
    w = inputs.Workload("stream", H=H, E=E, K=1, I=I, n_layers=1, D=0, P=A, dtype="bf16", seed=A)
    L = {k: (v.to(DEV) if v is not None else None) for k, v in inputs.make_layer(w, 0).items()}
    x_perm = inputs.randn((A, H), 1.0, A, "x_perm", 0, "bf16").to(DEV)
    offsets = torch.tensor(np.concatenate([[0], np.cumsum(rows)]), dtype=torch.int32).to(DEV)
    ctx = gpu_lib.Context(H, E, 1, I, torch.bfloat16, max_tokens=A, device=DEV, **fmt)
    ctx.moe_set_ffn_variant("tile128")
    want = ctx.moe_grouped_ffn(x_perm, offsets, L["w_gate_up"], L["w_down"]).clone()
    ctx.moe_set_ffn_variant(shape)
    assert torch.equal(ctx.moe_grouped_ffn(x_perm, offsets, L["w_gate_up"], L["w_down"]), want)


# ... unless the weights do not start on a 128-byte line (16 bytes are enough for the library): the same bits from there
@pytest.mark.parametrize("shape,H,I,rows", [("few", 384, 64, [32, 1, 0, 20]), ("small", 512, 448, [64, 0, 1, 40]),
                                            ("big", 512, 320, [256, 1, 0, 130])])
@pytest.mark.parametrize("off", [8, 32, 64])
def test_streamed_weight_tiles_inside_a_line(gpu_lib, shape, H, I, rows, off):
    E, A = len(rows), sum(rows)
    w = inputs.Workload("stream", H=H, E=E, K=1, I=I, n_layers=1, D=0, P=A, dtype="bf16", seed=A)
    L = {k: (v.to(DEV) if v is not None else None) for k, v in inputs.make_layer(w, 0).items()}
    x_perm = inputs.randn((A, H), 1.0, A, "x_perm", 0, "bf16").to(DEV)
    offsets = torch.tensor(np.concatenate([[0], np.cumsum(rows)]), dtype=torch.int32).to(DEV)
    ctx = gpu_lib.Context(H, E, 1, I, torch.bfloat16, max_tokens=A, device=DEV)
    ctx.moe_set_ffn_variant(shape)
    want = ctx.moe_grouped_ffn(x_perm, offsets, L["w_gate_up"], L["w_down"]).clone()

    def moved(t):
        buf = torch.empty(t.numel() + 128, dtype=t.dtype, device=DEV)
        at = (-buf.data_ptr() % 128) // 2 + off
        return buf[at:at + t.numel()].view(t.shape).copy_(t)

    assert torch.equal(ctx.moe_grouped_ffn(x_perm, offsets, moved(L["w_gate_up"]), moved(L["w_down"])), want)


# Expert outputs whose rows are not whole lines are read as a stream from 160 MiB on: the same bits as in pieces below that, and as
# from a copy inside a line for those whose rows are
@pytest.mark.parametrize("H,K,T,dtype", [(2048, 8, 517, "bf16"), (1160, 7, 10330, "bf16"), (1160, 7, 10331, "bf16"), (2056, 3, 7000, "f32"),
                                         (96, 3, 77, "f32")])
def test_streamed_combine(gpu_lib, H, K, T, dtype):
    dt = inputs.torch_dtype(dtype)
    g = torch.Generator(device=DEV).manual_seed(T)
    y_perm, x = (torch.randn((n, H), generator=g, device=DEV).to(dt) for n in (T * K, T))
    w = torch.rand((T, K), generator=g, device=DEV)
    cut = [0, T // 3, T // 2, T]
    local = [torch.randperm((b - a) * K, generator=g, device=DEV).to(torch.int32).view(-1, K) for a, b in zip(cut, cut[1:])]
    ctx = gpu_lib.Context(H, 16, K, 8, dt, max_tokens=T, device=DEV)
    inv = torch.cat([l + a * K for l, a in zip(local, cut)])
    y = ctx.moe_combine(y_perm, inv, w, residual=x)
    for l, a, b in zip(local, cut, cut[1:]):
        part = ctx.moe_combine(y_perm[a * K:b * K], l, w[a:b], residual=x[a:b])
        assert torch.equal(y[a:b], part)
    inside = torch.empty(T * K * H + 8, dtype=dt, device=DEV)[8:].view(T * K, H).copy_(y_perm)
    assert torch.equal(ctx.moe_combine(inside, inv, w, residual=x), y)
    want = (y_perm[inv.long().view(-1)].view(T, K, H).float() * w[:, :, None]).sum(1) + x.float()
    bound = 2.0 ** -8 if dtype == "bf16" else 2.0 ** -20      # one rounding; K + 1 fp32 sums of values up to 2^3
    assert ((y.float() - want).abs() <= bound * (want.abs() + 8)).all()


# The shape a launch takes is the one moe_ffn_variant names: pinned, or by the rule.  By the rule: a streaming shape up to 56
# rows per expert, and beyond as long as its tiles are one round (two per compute unit, 512 on 256 units); narrow tiles while
# these are less than one round.
FEW, SMALL, BIG, WIDE = "<1,64,1,5,1,2,", "<2,128,2,3,2,4,", "big", "<8,256,2,2,2,8,"


@pytest.mark.parametrize("H,E,K,I,T,want", [
    (2048, 128, 8, 768, 1, FEW),           # 8 experts x 24 narrow tiles
    (2048, 128, 8, 768, 2, FEW),           # 384
    (2048, 128, 8, 768, 3, SMALL),         # 576
    (2048, 128, 8, 768, 896, SMALL),       # 56 rows per expert
    (2048, 128, 8, 768, 897, BIG),
    (512, 4, 1, 512, 60 * 4, FEW),         # few experts of many rows: (7 + 2) x 16 narrow tiles
    (512, 4, 1, 512, 4 * 500, SMALL),      # (62 + 2) x 16 narrow tiles, (31 + 2) x 8 of 64 x 128
    (1024, 8, 2, 1024, 4 * 56, SMALL),     # (14 + 4) x 32 narrow tiles
    (1024, 8, 2, 1024, 4 * 224, SMALL),    # (28 + 4) x 16 tiles: one round
    (1024, 8, 2, 1024, 4 * 232, BIG),      # (29 + 4) x 16
    (512, 2, 1, 512, 8192, BIG),           # 129 x 8
    (192, 64, 1, 2048, 64 * 64, SMALL),    # short rows: 256 x 256 tiles above 64 rows per expert
    (192, 64, 1, 2048, 64 * 64 + 1, WIDE),
    (192, 2, 1, 512, 2 * 900, SMALL),      # (28 + 1) x 8
])
def test_shape_rule_and_names(gpu_lib, H, E, K, I, T, want):
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the rule counts compute units")
    ctx = gpu_lib.Context(H, E, K, I, torch.bfloat16, max_tokens=2, device=DEV)
    assert want in ctx.moe_ffn_variant(T)
    for pin, name in (("few", FEW), ("small", SMALL), ("wide", WIDE), ("big", BIG if H >= 256 else want), ("tile128", "<128,128,")):
        ctx.moe_set_ffn_variant(pin)
        assert name in ctx.moe_ffn_variant(T)


# The persistent 256 x 256 kernel: tiles of 128 to 256 rows cut from experts of any size, at least four k-stages, next
# tile's loads issued during the current one.  Checked against the oracle and, bit for bit, against the streaming shape.
@pytest.mark.parametrize("H,I,rows", [
    (256, 256, [1]),                                       # one row, four stages, one tile for the whole chip
    (256, 264, [255, 256, 257, 0, 31, 32, 33]),            # tile edges; a ragged column tile in gate_up (K = 264 keeps down off)
    (320, 512, [0] * 70 + [300] + [0] * 60 + [513]),       # experts in the second and third group of 64, the rest empty
    (264 * 8, 320, [40, 700, 1]),                          # 33 stages, a wide ragged output
    (256, 1024, [7 * i % 97 for i in range(130)]),         # many small experts: several tiles per block
])
def test_big_tiles_grouped_ffn(gpu_lib, H, I, rows):
    E, A = len(rows), sum(rows)
    w = inputs.Workload("big", H=H, E=E, K=1, I=I, n_layers=1, D=0, P=A, dtype="bf16", seed=31)
    L = inputs.make_layer(w, 0)
    x_perm = inputs.randn((A, H), 1.0, 31, "x_perm", 0, "bf16")
    offsets = torch.tensor(np.concatenate([[0], np.cumsum(rows)]), dtype=torch.int32)
    ctx = gpu_lib.Context(H, E, 1, I, torch.bfloat16, max_tokens=A, device=DEV)
    args = (x_perm.to(DEV), offsets.to(DEV), L["w_gate_up"].to(DEV), L["w_down"].to(DEV))
    ctx.moe_set_ffn_variant("small")
    small = ctx.moe_grouped_ffn(*args)
    ctx.moe_set_ffn_variant("big")
    for _ in range(2):
        assert torch.equal(ctx.moe_grouped_ffn(*args), small)
    assert_close(small, dense_ffn(x_perm, offsets, L, "bf16", E), "bf16", "big tiles")


# Columns that are a multiple of 8 only in the down GEMM (H = 328: K = 328 keeps gate_up off the pipelined kernels), in every
# output format: the last 32-column block of a tile is stored in part
@pytest.mark.parametrize("fmt", [{}, {"y_perm_f32": True}, {"y_perm_f32": True, "act_split": True}])
@pytest.mark.parametrize("H,rows", [(328, [255, 0, 257, 40]), (264, [1, 300]), (8 * 67, [128] * 3)])
def test_big_tiles_ragged_columns(gpu_lib, H, rows, fmt):
    I, E, A = 512, len(rows), sum(rows)
    w = inputs.Workload("ragged", H=H, E=E, K=1, I=I, n_layers=1, D=0, P=A, dtype="bf16", seed=33)
    L = inputs.make_layer(w, 0)
    x_perm = inputs.randn((A, H), 1.0, 33, "x_perm", 0, "bf16")
    offsets = torch.tensor(np.concatenate([[0], np.cumsum(rows)]), dtype=torch.int32)
    args = (x_perm.to(DEV), offsets.to(DEV), L["w_gate_up"].to(DEV), L["w_down"].to(DEV))
    ctx = gpu_lib.Context(H, E, 1, I, torch.bfloat16, max_tokens=A, device=DEV, **fmt)
    ctx.moe_set_ffn_variant("tile128")
    ref = ctx.moe_grouped_ffn(*args)
    ctx.moe_set_ffn_variant("big")
    assert torch.equal(ctx.moe_grouped_ffn(*args), ref)
    assert_close(ref, dense_ffn(x_perm, offsets, L, "bf16", E), "bf16", "ragged columns")


@pytest.mark.parametrize("T,E,K,fmt", [(300, 5, 1, {}), (517, 9, 3, {}), (700, 65, 7, {"y_perm_f32": True}),
                                       (259, 3, 3, {"y_perm_f32": True, "act_split": True})])
def test_big_tiles_with_gathered_rows(gpu_lib, T, E, K, fmt):
    """The rows come through the permutation (divided by K on the device), from two input buffers."""
    H, I = 512, 384
    w = inputs.Workload("bigmap", H=H, E=E, K=K, I=I, n_layers=1, D=T // 3, P=T - T // 3, dtype="bf16", seed=T)
    L = {k: (v.to(DEV) if v is not None else None) for k, v in inputs.make_layer(w, 0).items()}
    xd, xp = inputs.make_hidden(w, device=DEV)
    ctx = gpu_lib.Context(H, E, K, I, torch.bfloat16, max_tokens=T, device=DEV, **fmt)
    out = {}
    for v in ("small", "big"):
        ctx.moe_set_ffn_variant(v)
        out[v] = [y.clone() for y in ctx.moe_group_forward([L], xd, xp)]
    assert all(torch.equal(a, b) for a, b in zip(out["small"], out["big"]))


# MXFP4, compute-bound shape: double stages of codes (rows of an odd or even number of stages), chunks of 8 stages of
# scale bytes (the row's last chunk starts early), 256 x 256 tiles.  Checked against the 64-row shape bit for bit (it is
# checked against the oracle elsewhere), and against the oracle once.
@pytest.mark.parametrize("H,I,rows", [
    (512, 512, [1]),                                        # the smallest K: eight stages, one chunk of scales
    (576, 640, [33, 0, 255, 257, 96]),                      # 9 and 10 stages; ragged column tiles
    (1024 + 64, 960, [300, 7, 128]),                        # 17 stages: the last scale chunk holds one stage
    (2880, 576, [0] * 66 + [140, 3] + [0] * 3 + [511]),     # 45 stages, rows of 90 scale bytes
    (512, 1536, [40 + 3 * i % 50 for i in range(90)]),      # several tiles per block
])
def test_w4_big_tiles(gpu_lib, H, I, rows):
    E, A = len(rows), sum(rows)
    w = inputs.Workload("w4big", H=H, E=E, K=1, I=I, n_layers=1, D=0, P=A, dtype="bf16", seed=41, weight_format="mxfp4")
    L = {k: (v.to(DEV) if v is not None else None) for k, v in inputs.make_layer(w, 0).items()}
    L["s_gate_up"][0, 0, 0] = 0                             # 2^-127: the one scale byte that is not an exponent field
    x_perm = inputs.randn((A, H), 1.0, 41, "x_perm", 0, "bf16").to(DEV)
    offsets = torch.tensor(np.concatenate([[0], np.cumsum(rows)]), dtype=torch.int32).to(DEV)
    for f32 in (False, True):
        ctx = gpu_lib.Context(H, E, 1, I, torch.bfloat16, max_tokens=A, device=DEV, weight_format="mxfp4", y_perm_f32=f32)
        out = {}
        for v in ("w4_tile64", "w4_big", "w4_big"):
            ctx.moe_set_ffn_variant(v)
            y = ctx.moe_grouped_ffn_mxfp4(x_perm, offsets, L["w_gate_up"], L["s_gate_up"], L["w_down"], L["s_down"])
            assert torch.equal(out.setdefault("y", y), y), v
    # rows through the permutation, from two buffers
    T, K = 150, min(3, E)
    ctx = gpu_lib.Context(H, E, K, I, torch.bfloat16, max_tokens=T, device=DEV, weight_format="mxfp4")
    xd, xp = (inputs.randn((n, H), 1.0, 42, s, 0, "bf16").to(DEV) for n, s in ((50, "d"), (100, "p")))
    ys = {}
    for v in ("w4_tile64", "w4_big"):
        ctx.moe_set_ffn_variant(v)
        ys[v] = [y.clone() for y in ctx.moe_group_forward([L], xd, xp)]
    assert all(torch.equal(a, b) for a, b in zip(ys["w4_tile64"], ys["w4_big"]))


# The MXFP4 rule: streaming up to 48 rows per expert, and beyond up to one of its tiles per compute unit (256 units); then 64-row
# tiles up to one per unit (from 64 rows per expert; two for rows of up to eleven stages) and for rows under 512 values; else the big ones
STREAM4, TILE4, BIG4 = "w4_stream", "w4_kernel", "w4_big"


@pytest.mark.parametrize("H,E,I,T,want", [
    (2880, 32, 2880, 32 * 48, STREAM4),
    (2880, 32, 2880, 32 * 48 + 1, BIG4),
    (1024, 8, 1024, 8 * 112, STREAM4),         # (28 + 4) x 8 streaming tiles
    (1024, 8, 1024, 8 * 116, TILE4),           # (29 + 4) x 8
    (1024, 8, 1024, 8 * 224, TILE4),           # (28 + 4) x 8 tiles of 64 rows
    (1024, 8, 1024, 8 * 232, BIG4),
    (512, 4, 512, 4 * 500, STREAM4),           # (62 + 2) x 4 streaming tiles
    (512, 8, 512, 8 * 900, TILE4),             # (112 + 4) x 4
    (512, 8, 512, 8 * 1100, BIG4),             # (137 + 4) x 4
    (1024, 32, 640, 32 * 60, BIG4),            # (30 + 16) x 5, but an expert's rows fit one tile
    (256, 8, 2048, 8 * 60, TILE4),             # short rows
])
def test_w4_shape_rule_and_names(gpu_lib, H, E, I, T, want):
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the rule counts compute units")
    ctx = gpu_lib.Context(H, E, 1, I, torch.bfloat16, max_tokens=2, device=DEV, weight_format="mxfp4")
    assert want in ctx.moe_ffn_variant(T)
    for pin, name in (("w4_stream", STREAM4), ("w4_tile64", TILE4), ("w4_big", BIG4 if H >= 512 else TILE4)):
        ctx.moe_set_ffn_variant(pin)
        assert name in ctx.moe_ffn_variant(T)


def test_w4_big_tiles_against_the_oracle(gpu_lib):
    H, I, E, K, T = 640, 576, 4, 2, 300
    w = inputs.Workload("w4o", H=H, E=E, K=K, I=I, n_layers=1, D=0, P=T, dtype="bf16", seed=43, residual=False,
                        weight_format="mxfp4")
    L = inputs.make_layer(w, 0)
    _, x = inputs.make_hidden(w)
    ctx = gpu_lib.Context(H, E, K, I, torch.bfloat16, max_tokens=T, residual=False, device=DEV, weight_format="mxfp4")
    ctx.moe_set_ffn_variant("w4_big")
    _, y = ctx.moe_group_forward([{k: (v.to(DEV) if v is not None else None) for k, v in L.items()}], None, x.to(DEV))
    n = inputs.layer_to_numpy(L)
    ref, _, _ = oracle.moe_layer(inputs.to_numpy(x), n["w_router"], None, n["w_gate_up"], n["w_down"], K, residual=False,
                                 s_gate_up=n["s_gate_up"], s_down=n["s_down"])
    assert_close(y, ref, "bf16", "w4 big tiles")


# The one-launch routing: the four sums of a logit in four blocks, in two, in one (by the number of 16 x 16 tiles; 256 compute
# units), rows shorter and longer than a wave's stage, with a partial chunk and without, against the separate launches
@pytest.mark.parametrize("dtype,E,K,H,T", [
    ("bf16", 16, 4, 40, 1), ("bf16", 128, 8, 2048, 17), ("bf16", 130, 3, 32 * 16 * 6 + 40, 96), ("bf16", 200, 5, 520, 100),
    ("bf16", 256, 16, 72, 256), ("bf16", 32, 16, 32 * 16 * 12, 15), ("f32", 64, 4, 32 * 16 * 3 + 8, 33), ("f32", 250, 2, 200, 250),
])
def test_one_launch_routing_in_one_to_four_blocks(gpu_lib, dtype, E, K, H, T):
    w = inputs.Workload("one", H=H, E=E, K=K, I=64, n_layers=1, D=T, P=0, dtype=dtype, seed=H + T)
    L = inputs.make_layer(w, 0, device=DEV)
    L["router_bias"] = inputs.randn((E,), 0.5, w.seed, "bias", 0, "f32", DEV)
    dt = inputs.torch_dtype(dtype)
    for s in range(2):
        x = inputs.randn((T, H), 1.0, w.seed + s, "x", 0, dtype, DEV)
        ctx = gpu_lib.Context(H, E, K, 64, dt, max_tokens=T, residual=False, device=DEV, renormalize=bool(s))
        idx, wt = ctx.moe_router_topk(x, L["w_router"], L["router_bias"])
        _, offsets, _, inv, x_perm = ctx.moe_permute(x, idx)
        want = ctx.moe_combine(ctx.moe_grouped_ffn(x_perm, offsets, L["w_gate_up"], L["w_down"]), inv, wt)
        for _ in range(2):
            assert torch.equal(ctx.moe_group_forward([L], x, None)[0], want)


# The search for a block's tile: two experts to a lane and eight, experts without rows at the ends and between, one m-tile and
# several of each height.  Through the gather of the layer (row map, divided by K) and without.
@pytest.mark.parametrize("shape", ["small", "few", "tile128"])
@pytest.mark.parametrize("E,big", [(1, [0]), (2, [1]), (128, [0, 63, 127]), (129, [128]), (130, [1, 64]), (512, [7, 8, 511])])
def test_tile_search(gpu_lib, shape, E, big):
    H, I = 64, 72
    rows = [(e * 7 + 1) % 3 if e % 5 else 0 for e in range(E)]
    for e in big:
        rows[e] = 150 + e % 3
    A = sum(rows)
    w = inputs.Workload("search", H=H, E=E, K=1, I=I, n_layers=1, D=0, P=A, dtype="bf16", seed=E)
    L = inputs.make_layer(w, 0)
    x_perm = inputs.randn((A, H), 1.0, E, "x_perm", 0, "bf16")
    offsets = torch.tensor(np.concatenate([[0], np.cumsum(rows)]), dtype=torch.int32)
    ctx = gpu_lib.Context(H, E, 1, I, torch.bfloat16, max_tokens=A, device=DEV)
    ctx.moe_set_ffn_variant(shape)
    got = ctx.moe_grouped_ffn(x_perm.to(DEV), offsets.to(DEV), L["w_gate_up"].to(DEV), L["w_down"].to(DEV))
    assert_close(got, dense_ffn(x_perm, offsets, L, "bf16", E), "bf16", f"search {E} {shape}")


@pytest.mark.parametrize("K", [1, 3, 8, 13])
def test_row_map_division(gpu_lib, K):
    """The layer's gather (entry / K of the permutation) against rows gathered by the permutation's own call."""
    E, H, I, T = 16, 64, 64, 300
    w = inputs.Workload("map", H=H, E=E, K=K, I=I, n_layers=1, D=T, P=0, dtype="bf16", seed=K)
    L = inputs.make_layer(w, 0, device=DEV)
    x = inputs.randn((T, H), 1.0, K, "x", 0, "bf16", DEV)
    ctx = gpu_lib.Context(H, E, K, I, torch.bfloat16, max_tokens=T, residual=False, device=DEV)
    idx, wt = ctx.moe_router_topk(x, L["w_router"])
    _, offsets, _, inv, x_perm = ctx.moe_permute(x, idx)
    for shape in ("small", "few", "tile128"):
        ctx.moe_set_ffn_variant(shape)
        want = ctx.moe_combine(ctx.moe_grouped_ffn(x_perm, offsets, L["w_gate_up"], L["w_down"]), inv, wt)
        assert torch.equal(ctx.moe_group_forward([L], x, None)[0], want)


# Narrow tiles: 8 rows and fewer load less, waves have 16 output columns of a gated GEMM (ragged column tiles of both kinds)
@pytest.mark.parametrize("H,I,rows", [(64, 64, [8, 9, 0, 7, 1, 16]), (320, 64 + 40, [8, 32]), (448, 64 + 16, [9, 3]), (2880, 8, [1])])
@pytest.mark.parametrize("fmt", [{}, {"y_perm_f32": True}, {"y_perm_f32": True, "act_split": True}])
def test_narrow_tiles_of_two_waves(gpu_lib, H, I, rows, fmt):
    E, A = len(rows), sum(rows)
    w = inputs.Workload("narrow", H=H, E=E, K=1, I=I, n_layers=1, D=0, P=A, dtype="bf16", seed=A)
    L = inputs.make_layer(w, 0, device=DEV)
    x_perm = inputs.randn((A, H), 1.0, A, "x_perm", 0, "bf16", DEV)
    offsets = torch.tensor(np.concatenate([[0], np.cumsum(rows)]), dtype=torch.int32, device=DEV)
    ctx = gpu_lib.Context(H, E, 1, I, torch.bfloat16, max_tokens=A, device=DEV, **fmt)
    ctx.moe_set_ffn_variant("tile128")
    want = ctx.moe_grouped_ffn(x_perm, offsets, L["w_gate_up"], L["w_down"]).clone()
    ctx.moe_set_ffn_variant("few")
    for _ in range(2):
        assert torch.equal(ctx.moe_grouped_ffn(x_perm, offsets, L["w_gate_up"], L["w_down"]), want)


# The combine asks for up to 8 rows at once, for up to 16 in two equal groups, for others in eights and the rest; plain and streamed rows, one
# and two pieces per output
@pytest.mark.parametrize("K", [1, 2, 3, 4, 5, 6, 7, 8, 9, 11, 12, 14, 16, 64])
@pytest.mark.parametrize("dtype,H,fmt", [("bf16", 64, {}), ("bf16", 2056, {}), ("bf16", 72, {"y_perm_f32": True}), ("f32", 1064, {})])
def test_combine_rows_at_once(gpu_lib, K, dtype, H, fmt):
    T, E = 37, 64
    dt = inputs.torch_dtype(dtype)
    ctx = gpu_lib.Context(H, E, K, 8 if not fmt else 64, dt, max_tokens=T, device=DEV, **fmt)
    y_perm = inputs.randn((T * K, H), 1.0, K, "y", 0, "f32" if fmt else dtype, DEV)
    inv = torch.randperm(T * K, generator=torch.Generator().manual_seed(K)).to(torch.int32).to(DEV)
    wt = torch.rand((T, K), generator=torch.Generator().manual_seed(K + 1)).to(DEV) / K
    x = inputs.randn((T, H), 1.0, K, "x", 0, dtype, DEV)
    terms = wt.double()[:, :, None] * y_perm.double()[inv.long()].view(T, K, H)
    # K + 1 roundings of fp32 sums no larger than the terms' magnitudes, and the output's own rounding
    bound = (K + 1) * 2.0 ** -24 * (terms.abs().sum(1) + x.double().abs())
    for res in (None, x):
        want = terms.sum(1) + (0 if res is None else res.double())
        got = ctx.moe_combine(y_perm, inv, wt, residual=res).double()
        assert ((got - want).abs() <= bound + want.abs() * (2.0 ** -8 if dtype == "bf16" else 2.0 ** -23)).all()


@pytest.mark.parametrize("K", [10, 13, 15, 17, 18, 20, 21, 22, 23, 63])
@pytest.mark.parametrize("dtype,H,fmt", [("bf16", 2056, {}), ("bf16", 72, {"y_perm_f32": True}), ("f32", 1064, {})])
def test_combine_eights_and_the_rest(gpu_lib, K, dtype, H, fmt):
    test_combine_rows_at_once(gpu_lib, K, dtype, H, fmt)


# The permutation by itself counts up to 12288 assignments in every block of the scatter, in a pass up to 8192; beyond, a pass of its
# own or the top-k's histograms.  Against a stable sort, and as part of a layer.
@pytest.mark.parametrize("E,T,K", [(15, 512, 4), (15, 683, 3), (16, 2049, 1), (128, 1536, 8), (128, 1537, 8), (512, 4096, 3), (300, 12289, 1)])
def test_permutation_counts(gpu_lib, E, T, K):
    H, I, A = 64, 64, T * K
    w = inputs.Workload("count", H=H, E=E, K=K, I=I, n_layers=1, D=0, P=T, dtype="bf16", seed=A, residual=False)
    L = inputs.make_layer(w, 0, device=DEV)
    x = inputs.randn((T, H), 1.0, A, "x", 0, "bf16", DEV)
    ctx = gpu_lib.Context(H, E, K, I, torch.bfloat16, max_tokens=T, residual=False, device=DEV)
    idx, wt = ctx.moe_router_topk(x, L["w_router"])
    counts, offsets, perm, inv, x_perm = ctx.moe_permute(x, idx)
    flat = idx.view(-1).long()
    want = torch.sort(flat, stable=True).indices.to(torch.int32)
    assert torch.equal(perm.view(-1), want)
    assert torch.equal(counts.long(), torch.bincount(flat, minlength=E))
    assert torch.equal(offsets[1:].long(), torch.cumsum(counts.long(), 0)) and int(offsets[0]) == 0
    assert torch.equal(inv.view(-1)[want.long()], torch.arange(A, dtype=torch.int32, device=DEV))
    y = ctx.moe_combine(ctx.moe_grouped_ffn(x_perm, offsets, L["w_gate_up"], L["w_down"]), inv, wt)
    for _ in range(2):
        assert torch.equal(ctx.moe_group_forward([L], None, x)[1], y)


# A split intermediate: a weight stage serves a step of hi and a step of lo values; the shortest rows the persistent kernel takes, an
# odd number of weight stages, row blocks per wave from none to four, blocks with one tile (12 on 256 units), two (280, and 400 or 500 by the
# height of the tiles) and up to four (800 of four and of five weight stages: the ring of three slots goes on where the tile before left it)
@pytest.mark.parametrize("H,I,rows", [(512, 256, [35] * 140), (264, 320, [40, 1, 300] * 50), (768, 448, [256, 129, 0, 64]),
                                      (264, 256, [9, 40] * 200), (264, 320, [33] * 400)])
def test_split_weight_stages(gpu_lib, H, I, rows):
    E, A = len(rows), sum(rows)
    w = inputs.Workload("pairs", H=H, E=E, K=1, I=I, n_layers=1, D=0, P=A, dtype="bf16", seed=A)
    L = inputs.make_layer(w, 0, device=DEV)
    x_perm = inputs.randn((A, H), 1.0, A, "x_perm", 0, "bf16", DEV)
    offsets = torch.tensor(np.concatenate([[0], np.cumsum(rows)]), dtype=torch.int32, device=DEV)
    ctx = gpu_lib.Context(H, E, 1, I, torch.bfloat16, max_tokens=A, device=DEV, y_perm_f32=True, act_split=True)
    ctx.moe_set_ffn_variant("tile128")
    want = ctx.moe_grouped_ffn(x_perm, offsets, L["w_gate_up"], L["w_down"]).clone()
    for shape in ("big", "small", "wide", "big"):
        ctx.moe_set_ffn_variant(shape)
        assert torch.equal(ctx.moe_grouped_ffn(x_perm, offsets, L["w_gate_up"], L["w_down"]), want), shape


# The counters of the scatter under skewed routing, eight of each expert with the assignments in front of a tile in their upper halves: the last
# assignment and the first of a tile, all of one expert and of two, the fewest experts and the most
@pytest.mark.parametrize("A", [1, 2047, 2049, 8192, 12287, 12288, 12289])
@pytest.mark.parametrize("E,kind", [(1, "one"), (2, "two"), (15, "one"), (16, "last"), (100, "zipf"), (512, "one"), (512, "two")])
def test_permutation_of_skewed_choices(gpu_lib, E, kind, A):
    g = torch.Generator().manual_seed(A + E)
    f = torch.arange(A)
    flat = {"one": torch.full((A,), E // 2), "last": torch.full((A,), E - 1), "two": torch.where(f % 3 == 0, 0, E - 1),
            "zipf": (torch.rand(A, generator=g) ** 4 * E).long().clamp(max=E - 1)}[kind]
    ctx = gpu_lib.Context(64, E, 1, 64, torch.bfloat16, max_tokens=A, device=DEV)
    x = torch.zeros((A, 64), dtype=torch.bfloat16, device=DEV)
    counts, offsets, perm, inv, _ = ctx.moe_permute(x, flat.to(torch.int32).view(A, 1).to(DEV), want_x_perm=False)
    want = torch.sort(flat, stable=True).indices
    assert torch.equal(perm.cpu().long(), want)
    assert torch.equal(inv.cpu().long()[want], f)
    assert torch.equal(counts.cpu().long(), torch.bincount(flat, minlength=E))
    assert torch.equal(offsets.cpu().long(), torch.cat([torch.zeros(1, dtype=torch.int64), torch.cumsum(counts.cpu().long(), 0)]))


# Behind a top-k up to 8192 assignments are counted by the scatter, whatever the number of experts, more by the top-k
@pytest.mark.parametrize("E,T,K", [(2, 8192, 1), (2, 8193, 1), (15, 2048, 4), (15, 2049, 4), (128, 1024, 8), (128, 1025, 8)])
def test_who_counts_behind_a_topk(gpu_lib, E, T, K):
    H, I = 64, 64
    w = inputs.Workload("counts", H=H, E=E, K=K, I=I, n_layers=1, D=0, P=T, dtype="bf16", seed=T, residual=False)
    L = inputs.make_layer(w, 0, device=DEV)
    L["router_bias"] = -1.2 * torch.log(torch.arange(1, E + 1, dtype=torch.float32, device=DEV))
    x = inputs.randn((T, H), 1.0, T, "x", 0, "bf16", DEV)
    ctx = gpu_lib.Context(H, E, K, I, torch.bfloat16, max_tokens=T, residual=False, device=DEV)
    idx, wt = ctx.moe_router_topk(x, L["w_router"], L["router_bias"])
    _, offsets, _, inv, x_perm = ctx.moe_permute(x, idx)
    y = ctx.moe_combine(ctx.moe_grouped_ffn(x_perm, offsets, L["w_gate_up"], L["w_down"]), inv, wt)
    for _ in range(2):
        assert torch.equal(ctx.moe_group_forward([L], None, x)[1], y)


# The one-launch routing: a tile's sums in four blocks, in two (fp32) or whole in one.  Both sides of the line (the last length of the one shape,
# the first of the other), the most tiles of either, ragged rows; against the separate launches
@pytest.mark.parametrize("dtype,E,K,T,H", [
    ("bf16", 16, 2, 16, 600), ("bf16", 16, 2, 16, 608),            # 1 tile
    ("bf16", 128, 8, 1, 752), ("bf16", 128, 8, 1, 760),
    ("bf16", 256, 16, 64, 2488), ("bf16", 256, 8, 64, 2496),       # 64 tiles: 256 blocks
    ("bf16", 256, 8, 65, 4096), ("bf16", 130, 3, 256, 4104),       # 80 and 144
    ("f32", 128, 8, 200, 1144), ("f32", 128, 8, 200, 1152),        # 104 tiles, two classes to a block
    ("f32", 32, 16, 33, 1000), ("f32", 250, 5, 256, 520),
])
def test_one_launch_routing_whole_and_cut_tiles(gpu_lib, dtype, E, K, T, H):
    w = inputs.Workload("cut", H=H, E=E, K=K, I=64, n_layers=1, D=T, P=0, dtype=dtype, seed=H + T)
    L = inputs.make_layer(w, 0, device=DEV)
    L["router_bias"] = inputs.randn((E,), 0.5, w.seed, "bias", 0, "f32", DEV)
    for s in range(2):
        x = inputs.randn((T, H), 1.0, w.seed + s, "x", 0, dtype, DEV)
        ctx = gpu_lib.Context(H, E, K, 64, inputs.torch_dtype(dtype), max_tokens=T, residual=False, device=DEV, renormalize=bool(s))
        idx, wt = ctx.moe_router_topk(x, L["w_router"], L["router_bias"])
        _, offsets, _, inv, x_perm = ctx.moe_permute(x, idx)
        want = ctx.moe_combine(ctx.moe_grouped_ffn(x_perm, offsets, L["w_gate_up"], L["w_down"]), inv, wt)
        for _ in range(2):
            assert torch.equal(ctx.moe_group_forward([L], x, None)[0], want)


@pytest.mark.parametrize("dtype,E,K,T,H", [("bf16", 40, 16, 16, 1024), ("bf16", 128, 8, 70, 2048), ("f32", 128, 8, 200, 1152)])
def test_cut_tiles_of_logits_that_are_not_finite(gpu_lib, dtype, E, K, T, H):
    w = inputs.Workload("odd", H=H, E=E, K=K, I=64, n_layers=1, D=T, P=0, dtype=dtype, seed=T + E)
    L = inputs.make_layer(w, 0, device=DEV)
    x = inputs.randn((T, H), 1.0, w.seed, "x", 0, dtype, DEV)
    x[::3, 5] = float("nan")
    x[1::3] = x[1::3].abs()
    L["w_router"][2] = float("inf")
    L["router_bias"] = torch.full((E,), float("-inf"), device=DEV)
    L["router_bias"][[1, 2, E - 1]] = 0.25
    ctx = gpu_lib.Context(H, E, K, 64, inputs.torch_dtype(dtype), max_tokens=T, residual=False, device=DEV)
    idx, wt = ctx.moe_router_topk(x, L["w_router"], L["router_bias"])
    _, offsets, _, inv, x_perm = ctx.moe_permute(x, idx)
    want = ctx.moe_combine(ctx.moe_grouped_ffn(x_perm, offsets, L["w_gate_up"], L["w_down"]), inv, wt)
    bits = torch.int16 if dtype == "bf16" else torch.int32
    assert torch.equal(ctx.moe_group_forward([L], x, None)[0].view(bits), want.view(bits))
