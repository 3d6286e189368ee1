"""GPU parity of the matrix-core gate/down kernels for many tokens per expert (wide groups): every number of token tiles,
one and several groups, row counts off every tile edge, several pieces per group, h beyond the range of fp16."""
import numpy as np
import pytest
import torch

import floe_synth as S
import oracle as O
from test_gpu_layer import _run_layer_case, _threads  # noqa: F401  (the fixture sets the oracle's threads)

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _wide():
    import paper_2505_05950_amd as F
    F.load()
    F.floe_tuning(F.TUNE_UNION_KERNELS, 1)
    F.floe_tuning(F.TUNE_FUSED_TASKS, 1)
    yield
    F.floe_tuning(F.TUNE_UNION_KERNELS, 0)
    F.floe_tuning(F.TUNE_FUSED_TASKS, 0)


@pytest.mark.parametrize("d,f,bits,group,n,n_shared,top_k,T,pct", [
    (512, 33, 4, 64, 0, 1, 0, 16, 40),      # one tile of tokens, one pair of row tiles and one row
    (1024, 700, 2, 64, 0, 1, 0, 17, 80),    # two token tiles, the second with one token
    (1536, 95, 4, 128, 0, 1, 0, 33, 50),    # three
    (512, 1031, 8, 64, 0, 1, 0, 64, 95),    # four, full
    (1024, 515, 3, 32, 0, 1, 0, 80, 0),     # five, full; every channel selected
    (512, 3000, 2, 64, 0, 1, 0, 81, 97),    # ten
    (512, 261, 4, 32, 0, 2, 0, 161, 60),    # several groups of an expert, two experts
    (5120, 77, 2, 64, 3, 1, 2, 9, 70),      # more column blocks than rows fill
    (1024, 64, 2, 64, 12, 0, 2, 20, 70),    # many small groups
])
def test_wide_groups(d, f, bits, group, n, n_shared, top_k, T, pct):
    _run_layer_case(70 + T, 5, d, f, bits, group, n, n_shared, top_k, False, T, pct, gap=f * (100 - pct) >= 6400)


@pytest.mark.parametrize("d,f,bits,group,n,n_shared,top_k,T,pct", [
    (4096, 49, 2, 64, 0, 1, 0, 32, 50),      # eight waves that take turns; two full token tiles; one channel in the last block
    (4096, 130, 4, 32, 3, 0, 2, 25, 60),     # groups of one and of two token tiles beside each other
    (3584, 37, 3, 64, 0, 1, 0, 17, 0),       # seven waves
    (2560, 16, 3, 32, 2, 0, 1, 9, 50),       # five; half a mask word
    (1536, 95, 4, 64, 0, 2, 0, 31, 60),      # three waves, two workgroups per compute unit; two experts on the same tokens
    (512, 50, 4, 64, 70, 2, 8, 20, 50),      # one wave; more groups than a wave scans at a time
    (1024, 300, 4, 64, 2, 0, 1, 70, 60),     # three token tiles: groups of one and of two parts
    (2048, 90, 3, 32, 0, 1, 0, 49, 50),      # four: the second part holds one tile and one token
])
def test_up_projection_split_over_columns(d, f, bits, group, n, n_shared, top_k, T, pct):
    _run_layer_case(170 + T, 7, d, f, bits, group, n, n_shared, top_k, False, T, pct, gap=f * (100 - pct) >= 6400)


@pytest.mark.parametrize("d,f,bits,group,n,n_shared,top_k,T,pct", [
    (512, 33, 2, 64, 0, 1, 0, 160, 50),      # ten token tiles: two parts of five; one channel in the second block
    (1024, 290, 2, 64, 0, 1, 0, 112, 60),    # seven tiles in the body of seven; fewer blocks than waves in a pass
    (8192, 64, 2, 64, 0, 1, 0, 40, 60),      # more units than lanes of a wave
    (1536, 700, 3, 32, 0, 1, 0, 150, 60),    # ten tiles in two parts of five
    (1024, 400, 4, 64, 3, 1, 2, 200, 70),    # groups of different sizes, a shared expert
    (4608, 96, 4, 32, 0, 1, 0, 20, 50),      # a width that the columns are not split for
    (512, 64, 2, 64, 40, 4, 6, 300, 60),     # more parts than a wave scans
    (512, 8193, 2, 64, 0, 1, 0, 150, 85),    # blocks enough for eight waves of every compute unit: ten tiles in two parts of five
    (512, 13001, 4, 64, 0, 1, 0, 150, 90),   # the same for the wider codes
    (512, 6500, 3, 32, 0, 2, 0, 130, 90),    # two experts, nine tiles: parts of five and four
    (1024, 5003, 2, 64, 4, 0, 2, 80, 85),    # groups of three tiles, of two and of one
])
def test_up_projection_of_many_tokens(d, f, bits, group, n, n_shared, top_k, T, pct):
    _run_layer_case(370 + T, 11, d, f, bits, group, n, n_shared, top_k, False, T, pct, gap=f * (100 - pct) >= 6400)


@pytest.mark.parametrize("d,f,n,n_shared,top_k,T,pct", [
    (512, 300, 0, 1, 0, 140, 60),    # nine of ten token tiles; eight column slices on three ring slots: two behind the loop
    (1024, 291, 0, 1, 0, 160, 99),   # ten; one behind the loop; rows so far apart that v is gathered
    (1536, 64, 0, 1, 0, 75, 90),     # five tiles, no slice behind the loop; one span of v is the whole row
    (2048, 63, 3, 0, 2, 30, 10),     # fewer channels than a span
    (1024, 1100, 4, 0, 2, 120, 50),  # groups of different sizes: live tiles at and below what the launch is built for
])
def test_gate_rows_and_activations_through_lds(d, f, n, n_shared, top_k, T, pct):
    _run_layer_case(270 + T, 9, d, f, 2, 64, n, n_shared, top_k, False, T, pct, gap=f * (100 - pct) >= 6400)


@pytest.mark.parametrize("d,f,bits,group,n,n_shared,top_k,T,pct", [
    (512, 40, 2, 64, 600, 0, 8, 100, 50),    # more groups than workgroups: pieces that hold several segments
    (512, 2100, 2, 64, 0, 1, 0, 20, 60),     # pieces of 32 or 40 channels, the last eight of them half there
    (512, 3001, 4, 64, 44, 0, 4, 200, 40),   # pieces of 512 channels and more, several passes each; groups by the activations' kernel
    (512, 70, 2, 64, 20, 0, 8, 257, 50),     # one task more than that kernel groups: the grouping kernel in front
    (512, 70, 8, 64, 20, 0, 8, 40, 50),      # an up projection that keeps v and the masks by task
    (8192, 45, 4, 64, 5, 1, 2, 12, 50),      # two waves group the tasks
])
def test_segments_and_groups(d, f, bits, group, n, n_shared, top_k, T, pct):
    _run_layer_case(470 + T, 13, d, f, bits, group, n, n_shared, top_k, False, T, pct, gap=f * (100 - pct) >= 6400)


@pytest.mark.parametrize("d,f,bits,group,n,n_shared,top_k,T,elsewhere", [
    (512, 1408, 4, 64, 6, 0, 1, 16, 0),      # one group where six were expected: 176 pieces of eight channels, 256 workgroups
    (4096, 900, 3, 32, 8, 1, 1, 80, 0),      # two groups of nine
    (4096, 900, 3, 32, 8, 1, 1, 80, 1),      # and a token of its own beside them
    (512, 960, 8, 64, 8, 1, 1, 80, 2),       # the same where v and the masks are kept by task
    (1024, 384, 2, 64, 16, 2, 2, 70, 3),     # four crowded experts of eighteen
    (512, 161, 4, 64, 24, 1, 1, 16, 16),     # a shared expert beside groups of a token or two
])
def test_routing_that_fills_few_of_the_groups(d, f, bits, group, n, n_shared, top_k, T, elsewhere):
    """Equal or padding tokens, a collapsed router: all but `elsewhere` tokens go to the first top_k experts."""
    import gpu_common as G
    import paper_2505_05950_amd as F
    experts = [G.make_expert(*S.expert_weights(570, 13, d, f, 0, e), bits, group) for e in range(n + n_shared)]
    wr = S.router_weights(570, 13, n, d)
    x = S.tokens(570, 13, T, d)
    wr[:, 0] = 0.0
    wr[:top_k, 0] = 1.0 + 0.25 * np.arange(top_k, 0, -1)     # (the order among them is no near-tie either)
    x[:, 0] = 8.0
    x[T - elsewhere:, 0] = -8.0
    routed = np.argsort(-(x.astype(np.float64) @ wr.astype(np.float64).T), axis=1)[:, :top_k]
    slots = np.concatenate([routed, np.tile(n + np.arange(n_shared), (T, 1))], axis=1)
    tau, size = np.zeros((T, n + n_shared), np.float32), np.zeros(slots.shape, np.int32)
    for t in range(T):
        for s, e in enumerate(slots[t]):
            v = O.up_gemv(*experts[e][0][:3], d, bits, group, x[t])
            tau[t, e] = G.tau_in_widest_gap(v, 70, window=min(64, f // 8))[0]
            size[t, s] = O.select(v, float(tau[t, e])).size
    ref = O.moe_layer([e[0] for e in experts], n_shared, top_k, False, wr, x, tau, bits, group)
    L = F.Layer([e[1] for e in experts], n_shared, top_k, False, G.dev(wr), G.dev(tau), True)
    L.workspace(T).fill_(255)
    stats = torch.zeros((T, top_k + n_shared, 4), dtype=torch.int32, device=G.DEV)
    y = F.floe_moe_layer_decode(L, G.dev(x), stats=stats).cpu().numpy().astype(np.float64)
    st = stats.cpu().numpy()
    assert np.array_equal(st[:, :, 0], slots) and np.array_equal(st[:, :, 1], size)
    for t in range(T):
        assert G.rel_err(y[t], ref["y"][t]) <= G.Y_TIGHT, (t, G.rel_err(y[t], ref["y"][t]))


@pytest.mark.parametrize("n,top_k", [(8, 2), (70, 4)])   # picked by a wave, by one lane
def test_tokens_that_are_not_numbers_leave_the_others_alone(n, top_k):
    """Their logits are NaN: the router still picks experts of the table, and every task stands in a group."""
    import gpu_common as G
    import paper_2505_05950_amd as F
    d, f, bits, group, T = 512, 130, 4, 64, 40
    experts = [G.make_expert(*S.expert_weights(590, 13, d, f, 0, e), bits, group) for e in range(n)]
    wr, x = S.router_weights(590, 13, n, d), S.tokens(590, 13, T + 20, d)
    top = -np.sort(-(x.astype(np.float64) @ wr.astype(np.float64).T), axis=1)
    x = x[top[:, top_k - 1] - top[:, top_k] > 1e-3][:T]
    tau = np.full((T, n), -1.0, np.float32)
    ref = O.moe_layer([e[0] for e in experts], 0, top_k, True, wr, x, tau, bits, group)
    x = x.copy()
    x[[0, 17, T - 1]] = np.nan
    L = F.Layer([e[1] for e in experts], 0, top_k, True, G.dev(wr), G.dev(tau), True)
    L.workspace(T).fill_(255)
    stats = torch.zeros((T, top_k, 4), dtype=torch.int32, device=G.DEV)
    y = F.floe_moe_layer_decode(L, G.dev(x), stats=stats).cpu().numpy().astype(np.float64)
    ids = stats.cpu().numpy()[:, :, 0]
    assert ids.min() >= 0 and ids.max() < n
    for t in range(T):
        if t not in (0, 17, T - 1):
            assert G.rel_err(y[t], ref["y"][t]) <= G.Y_TIGHT, (t, G.rel_err(y[t], ref["y"][t]))


def test_a_layer_of_thousands_of_groups():
    """1024 + 48 experts, 64 slots, 3712 tokens: about 4000 groups and 256 pieces.  Experts share four sets of weights, and select every
    channel or none, so that a token's result is the weighted sum of four."""
    import gpu_common as G
    import paper_2505_05950_amd as F
    d, f, bits, group, n, n_shared, top_k, T = 512, 64, 4, 64, 1024, 48, 16, 3712
    kinds = [G.make_expert(*S.expert_weights(580, 13, d, f, 0, e), bits, group) for e in range(4)]
    x = S.tokens(580, 13, T, d)
    out = []
    for ex_np, _ in kinds:
        w_up = O.dequantize(*ex_np[:3], d, bits, group).astype(np.float64)
        v, g = x.astype(np.float64) @ w_up.T, x.astype(np.float64) @ ex_np[3][:, 0].astype(np.float64).T
        out.append((g / (1.0 + np.exp(-g)) * v) @ ex_np[3][:, 1].astype(np.float64))
    tau = np.where(np.arange(n + n_shared) % 3 == 2, 1e30, -1.0).astype(np.float32)
    L = F.Layer([kinds[e % 4][1] for e in range(n + n_shared)], n_shared, top_k, False, G.dev(S.router_weights(580, 13, n, d)), G.dev(tau), False)
    F.floe_tuning(F.TUNE_UNION_KERNELS, 0)
    stats = torch.zeros((T, top_k + n_shared, 4), dtype=torch.int32, device=G.DEV)
    y = F.floe_moe_layer_decode(L, G.dev(x), stats=stats).cpu().numpy().astype(np.float64)
    st = stats.cpu().numpy().view(F.SLOT_STAT_DTYPE).reshape(T, top_k + n_shared)
    assert np.array_equal(st["count"], np.where(tau[st["expert"]] > 0, 0, f))
    ref = np.zeros((T, d))
    for e in range(4):
        ref += np.where((st["expert"] % 4 == e) & (tau[st["expert"]] < 0), st["weight"], 0.0).sum(axis=1)[:, None] * out[e]
    worst = max(range(T), key=lambda t: G.rel_err(y[t], ref[t]))
    assert G.rel_err(y[worst], ref[worst]) <= G.Y_TIGHT, (worst, G.rel_err(y[worst], ref[worst]))


@pytest.mark.parametrize("d,f,n,n_shared,top_k,T,pct", [
    (1024, 300, 3, 1, 1, 150, 60),   # ten tiles, of which the routed experts fill two to four; an odd number of pairs
    (512, 97, 2, 1, 1, 155, 30),     # five to six; one row in the last pair
    (512, 260, 5, 0, 2, 130, 50),    # groups of three to five tiles
])
def test_down_products_of_live_tiles_only(d, f, n, n_shared, top_k, T, pct):
    _run_layer_case(300 + T, 9, d, f, 2, 64, n, n_shared, top_k, False, T, pct, gap=f * (100 - pct) >= 6400)


def test_h_beyond_fp16():
    """Large activations: |h| far beyond 65504 for some (row, token), ordinary for the others of the same group."""
    import gpu_common as G
    import paper_2505_05950_amd as F
    d, f, bits, group, T, pct = 512, 1500, 4, 64, 40, 80
    ex_np, ex_dev = G.make_expert(*S.expert_weights(91, 3, d, f), bits, group)
    x = S.tokens(91, 3, T, d).astype(np.float32)
    x[::3] *= 300.0                        # h ~ 2e4 typical, 1e5 and more at the tail
    x = x.astype(np.float16)
    tau = np.zeros((T, 1), np.float32)
    peak = 0.0
    for t in range(T):
        v = O.up_gemv(*ex_np[:3], d, bits, group, x[t])
        tau[t, 0], _ = G.tau_in_widest_gap(v, pct)
        h = O.sparse_ffn(ex_np[3], x[t], v, O.select(v, float(tau[t, 0])))[0]
        peak = max(peak, float(np.abs(h).max()))
    assert peak > 2 * 65504
    ref = O.moe_layer([ex_np], 1, 0, False, None, x, tau, bits, group)
    assert np.abs(ref["y"]).max() < 60000
    L = F.Layer([ex_dev], 1, 0, False, None, G.dev(tau), True)
    y = F.floe_moe_layer_decode(L, G.dev(x)).cpu().numpy().astype(np.float64)
    for t in range(T):
        assert G.rel_err(y[t], ref["y"][t]) <= G.Y_TIGHT, (t, G.rel_err(y[t], ref["y"][t]))


def test_groups_without_rows():
    """Experts whose thresholds nobody passes leave nothing behind, also next to experts that select everything."""
    import gpu_common as G
    import paper_2505_05950_amd as F
    d, f, bits, group, n, T = 512, 200, 4, 64, 3, 24
    experts = [G.make_expert(*S.expert_weights(92, 3, d, f, 0, e), bits, group) for e in range(n)]
    x = S.tokens(92, 3, T, d)
    for silent in ((0,), (1,), (0, 2), (0, 1, 2)):
        tau = np.zeros((T, n), np.float32)
        tau[:, list(silent)] = 1e9
        ref = O.moe_layer([e[0] for e in experts], n, 0, False, None, x, tau, bits, group)
        L = F.Layer([e[1] for e in experts], n, 0, False, None, G.dev(tau), True)
        stats = torch.zeros((T, n, 4), dtype=torch.int32, device=G.DEV)
        y = F.floe_moe_layer_decode(L, G.dev(x), stats=stats).cpu().numpy().astype(np.float64)
        assert np.array_equal(stats.cpu().numpy()[:, :, 1], np.where(tau > 0, 0, f))
        if len(silent) == n:
            assert not y.any()
        else:
            assert max(G.rel_err(y[t], ref["y"][t]) for t in range(T)) <= G.Y_TIGHT


@pytest.mark.parametrize("d,f,bits,group,T", [
    (1024, 700, 2, 64, 20), (512, 333, 4, 32, 40), (1536, 515, 3, 64, 33), (2048, 300, 4, 128, 18), (512, 97, 3, 32, 65),
    (1024, 130, 8, 64, 17),
])
def test_one_expert_many_tokens(d, f, bits, group, T):
    """floe_expert_ffn_sparse beyond the one-kernel batch: with the list, without it, and y accumulated."""
    import test_gpu_steps as steps
    steps.test_expert_ffn_sparse_matches_oracle(d, f, bits, group, T, [(80, 0, 95, 50)[t % 4] for t in range(T)])
    steps.test_expert_ffn_without_a_list_gives_the_same_result(d, f, bits, group, T)


def test_one_expert_scales_with_their_own_alignment_only():
    import gpu_common as G
    import paper_2505_05950_amd as F
    d, f, bits, group, T = 1024, 200, 2, 64, 24
    ex_np, ex_dev = G.make_expert(*S.expert_weights(93, 3, d, f), bits, group)
    x, tau = G.dev(S.tokens(93, 3, T, d)), G.dev(np.full((T,), 1.0, np.float32))
    y = F.floe_expert_ffn_sparse(ex_dev, x, tau, None, torch.zeros((T, d), dtype=torch.float32, device=G.DEV))[0]

    def moved(t):  # the same values two bytes off a 16-byte boundary
        buf = torch.empty((t.numel() + 8,), dtype=t.dtype, device=t.device)
        off = ((-buf.data_ptr()) % 16) // 2 + 1
        buf[off: off + t.numel()] = t.flatten()
        return buf[off: off + t.numel()]

    odd = F.Expert(d, f, bits, group, ex_dev.up_codes, moved(ex_dev.up_scale), moved(ex_dev.up_zero), ex_dev.gd)
    y2 = F.floe_expert_ffn_sparse(odd, x, tau, None, torch.zeros((T, d), dtype=torch.float32, device=G.DEV))[0]
    assert G.rel_err(y2.cpu().numpy(), y.cpu().numpy()) <= 1e-4   # another kernel's order of summation


@pytest.mark.parametrize("T", [40, 200])   # grouped up projection, one and four groups of 16 tokens per expert
def test_replayed_from_a_hip_graph(T):
    import test_gpu_layer as layer
    layer.test_layer_decode_replayed_from_a_hip_graph_matches_eager(T)


@pytest.mark.parametrize("d,f,bits,group,n,T", [(1536, 700, 3, 64, 4, 40), (1024, 5120, 2, 64, 8, 160)])   # no grouped kernel; many channels
def test_wide_up_projection_replayed_from_a_hip_graph(d, f, bits, group, n, T):
    """Replays, with eager work and synchronisations between them, reproduce the eager result bit for bit."""
    import gpu_common as G
    import paper_2505_05950_amd as F
    experts = [G.make_expert(*S.expert_weights(101, 3, d, f, 0, e), bits, group)[1] for e in range(n)]
    L = F.Layer(experts, 0, 2, True, G.dev(S.router_weights(101, 3, n, d)), G.dev(np.full((n,), 1.0, np.float32)), False)
    xs = [G.dev(S.tokens(101, 3, T, d, layer=i)) for i in range(3)]
    eager = [F.floe_moe_layer_decode(L, x).clone() for x in xs]
    x_in, y = xs[0].clone(), torch.empty((T, d), dtype=torch.float16, device=G.DEV)
    stream, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        F.floe_moe_layer_decode(L, x_in, y)
        stream.synchronize()
        with torch.cuda.graph(graph, stream=stream):
            F.floe_moe_layer_decode(L, x_in, y)
        for i in (0, 1, 2, 1, 0):
            torch.add(xs[i], 0.0, out=x_in)     # (a kernel on the same stream writes the input)
            y.fill_(float("nan"))
            graph.replay()
            stream.synchronize()
            assert torch.equal(y, eager[i]), i
            assert torch.equal(F.floe_moe_layer_decode(L, x_in), eager[i]), i


def test_one_pass_per_task_stays_a_choice():
    """FLOE_TUNE_GROUPED_GEMV = 2 keeps the up projection to one pass per (token, slot), also for large groups: no prepared
    activations in the workspace, the same masks."""
    import gpu_common as G
    import paper_2505_05950_amd as F
    d, f, n, T = 1024, 512, 2, 64
    experts = [G.make_expert(*S.expert_weights(94, 3, d, f, 0, e), 2, 64)[1] for e in range(n)]
    x = G.dev(S.tokens(94, 3, T, d))
    L = F.Layer(experts, n, 0, False, None, G.dev(np.full((n,), 1.0, np.float32)), False)
    stats, y, size = [], [], []
    try:
        for mode in (0, 2):
            F.floe_tuning(F.TUNE_GROUPED_GEMV, mode)
            size.append(F.floe_layer_workspace_bytes(L, T))
            stats.append(torch.zeros((T, n, 4), dtype=torch.int32, device=G.DEV))
            y.append(F.floe_moe_layer_decode(L, x, stats=stats[-1]).cpu().numpy())
    finally:
        F.floe_tuning(F.TUNE_GROUPED_GEMV, 0)
    assert size[1] < size[0]
    assert (stats[0][:, :, 1] - stats[1][:, :, 1]).abs().max() <= 1      # (a channel at the threshold)
    assert G.rel_err(y[1], y[0]) <= 5e-3


def _one_expert(seed, d, f, bits, group, x, pct, out_scale, ex=None):
    """floe_expert_ffn_sparse on x and its value in 64 bits -> (y [T][d] fp32, reference, expert)."""
    import gpu_common as G
    import paper_2505_05950_amd as F
    ex_np, ex_dev = ex if ex is not None else G.make_expert(*S.expert_weights(seed, 3, d, f), bits, group)
    T = x.shape[0]
    tau, ref = np.zeros((T,), np.float32), np.zeros((T, d))
    for t in range(T):
        v = O.up_gemv(*ex_np[:3], d, bits, group, x[t])
        tau[t], _ = G.tau_in_widest_gap(v, pct)
        ref[t] = float(out_scale[t]) * O.sparse_ffn(ex_np[3], x[t], v, O.select(v, float(tau[t])))[1]
    y = F.floe_expert_ffn_sparse(ex_dev, G.dev(x), G.dev(tau), G.dev(out_scale), torch.zeros((T, d), dtype=torch.float32, device=G.DEV),
                                 want_list=False)[0]
    return y.cpu().numpy().astype(np.float64), ref, (ex_np, ex_dev)


# y is fp32 and so is everything it is made of: sums of about d products for v and the gate, of a few hundred for y, 2^-24 a
# step, which adds up to about 1e-6 of y whatever its size.  Four times that.
FP32_BAR = 5e-6


@pytest.mark.parametrize("x_scale,out_scale", [(1.0, 1.0), (1.0, 1e-3), (1e-3, 1.0), (1.0, 1e-6), (1e-3, 1e-6), (1e-6, 1.0), (100.0, 1e5)])
@pytest.mark.parametrize("d,f,bits,group,T", [(1024, 1500, 2, 64, 17), (512, 900, 4, 64, 130)])   # two token tiles, ten
def test_small_and_large_results_keep_fp32_precision(d, f, bits, group, T, x_scale, out_scale):
    import gpu_common as G
    x = (S.tokens(95, 3, T, d).astype(np.float32) * x_scale).astype(np.float16)
    scale = (out_scale * np.linspace(0.5, 1.5, T)).astype(np.float32)
    y, ref, _ = _one_expert(95, d, f, bits, group, x, 70, scale)
    err = max(G.rel_err(y[t], ref[t]) for t in range(T))
    assert err <= FP32_BAR, err


@pytest.mark.parametrize("d,f,bits,group,T", [(1024, 1500, 2, 64, 20), (512, 900, 4, 64, 130)])
def test_a_token_with_huge_activations_costs_the_others_nothing(d, f, bits, group, T):
    import gpu_common as G
    x = S.tokens(96, 3, T, d).astype(np.float32)
    x[3] *= 2e4 / np.abs(x[3]).max()       # |h| ~ 1e7
    scale = np.ones((T,), np.float32)
    scale[3] = 1e4
    y, ref, _ = _one_expert(96, d, f, bits, group, x.astype(np.float16), 70, scale)
    err = [G.rel_err(y[t], ref[t]) for t in range(T)]
    assert max(err) <= FP32_BAR, (int(np.argmax(err)), max(err))


@pytest.mark.parametrize("d,f,bits,group,T", [(1024, 700, 2, 64, 20), (512, 900, 4, 64, 130)])
def test_a_weight_that_is_not_finite_reaches_only_the_tokens_that_select_its_row(d, f, bits, group, T):
    """Rows that a token did not select meet it as h = 0 in the matrix product, and rows past the end of a pair repeat the last
    one: 0 times infinity must not show."""
    import gpu_common as G
    w_up, gd = S.expert_weights(97, 3, d, f)
    gd = gd.copy()
    gd[f - 1, 1, 5] = np.inf               # the last row (of the last pair, where some token selects it)
    gd[f // 2, 1, :] = -np.inf
    gd[f // 3, 1, d - 1] = np.nan
    gd[7, 0, 3] = np.inf                   # a gate column: the channel's own h only
    ex = G.make_expert(w_up, gd, bits, group)
    x = S.tokens(97, 3, T, d)
    with np.errstate(invalid="ignore"):
        y, ref, _ = _one_expert(97, d, f, bits, group, x, 70, np.ones((T,), np.float32), ex=ex)
    clean = np.isfinite(ref).all(axis=1)
    assert 2 <= clean.sum() <= T - 2
    for t in range(T):
        fin = np.isfinite(ref[t])
        wrong = np.flatnonzero((np.isfinite(y[t]) != fin) | (np.isnan(y[t]) != np.isnan(ref[t])) | (np.isinf(ref[t]) & (y[t] != ref[t])))
        assert wrong.size == 0, (t, wrong.size, wrong[:8])
        if fin.any():
            assert G.rel_err(y[t][fin], ref[t][fin]) <= FP32_BAR, t


def test_gate_down_on_existing_lists_needs_no_wide_workspace():
    """floe_gate_down_sparse runs the one-token kernels at every batch size: their workspace is enough."""
    import gpu_common as G
    import paper_2505_05950_amd as F
    d, f, bits, group, T = 1024, 700, 2, 64, 130
    _, ex = G.make_expert(*S.expert_weights(98, 3, d, f), bits, group)
    x = G.dev(S.tokens(98, 3, T, d))
    wide = F.floe_expert_workspace_bytes(d, f, bits, group, T)
    F.floe_tuning(F.TUNE_UNION_KERNELS, 3)
    small = F.floe_expert_workspace_bytes(d, f, bits, group, T)
    F.floe_tuning(F.TUNE_UNION_KERNELS, 1)
    assert small < wide
    v = F.floe_up_gemv(ex.up_codes, ex.up_scale, ex.up_zero, x, d, bits, group)
    idx, count = F.floe_select_channels(v, torch.full((T,), 1.0, device=G.DEV))
    y = []
    for size in (wide, small):
        buf = torch.empty((size + 256,), dtype=torch.uint8, device=G.DEV)
        off = (-buf.data_ptr()) % 256
        y.append(F.floe_gate_down_sparse(ex, x, v, idx, count, None, torch.zeros((T, d), dtype=torch.float32, device=G.DEV),
                                         workspace=buf[off: off + size]))
    assert torch.equal(y[0], y[1])


def test_one_workspace_serves_every_batch_and_a_smaller_one_other_kernels():
    """Batches of every group size with the workspace of the largest one, and with what the one-token kernels need."""
    import gpu_common as G
    import paper_2505_05950_amd as F
    d, f, bits, group, top = 1024, 500, 2, 64, 165
    _, ex = G.make_expert(*S.expert_weights(99, 3, d, f), bits, group)
    L = F.Layer([ex], 1, 0, False, None, G.dev(np.full((1,), 1.0, np.float32)), False)
    x = G.dev(S.tokens(99, 3, top, d))
    size_l, size_e = F.floe_layer_workspace_bytes(L, top), F.floe_expert_workspace_bytes(d, f, bits, group, top)

    def cut(size):
        buf = torch.full((size + 256,), 255, dtype=torch.uint8, device=G.DEV)
        off = (-buf.data_ptr()) % 256
        return buf[off: off + size]

    def expert(T, ws):
        y = torch.zeros((T, d), dtype=torch.float32, device=G.DEV)
        return F.floe_expert_ffn_sparse(ex, x[:T], torch.full((T,), 1.0, device=G.DEV), None, y, workspace=ws, want_list=False)[0]

    for T in (17, 40, 81, 140, 160, 161, top):
        own = F.floe_moe_layer_decode(L, x[:T])
        L._ws[T] = cut(size_l)
        assert torch.equal(F.floe_moe_layer_decode(L, x[:T]), own), T
        y = expert(T, None)
        assert torch.equal(expert(T, cut(size_e)), y), T
        F.floe_tuning(F.TUNE_UNION_KERNELS, 3)
        small_l, small_e = F.floe_layer_workspace_bytes(L, T), F.floe_expert_workspace_bytes(d, f, bits, group, T)
        F.floe_tuning(F.TUNE_UNION_KERNELS, 0)
        L._ws[T] = cut(small_l)
        assert G.rel_err(F.floe_moe_layer_decode(L, x[:T]).float().cpu().numpy(), own.float().cpu().numpy()) <= 2.0 ** -10, T
        assert G.rel_err(expert(T, cut(small_e)).cpu().numpy(), y.cpu().numpy()) <= FP32_BAR, T
        F.floe_tuning(F.TUNE_UNION_KERNELS, 1)


def test_profiling_the_selection_sees_the_launch_that_carries_the_list():
    """A one-expert call of up to 16 tokens cuts its list beside the sums: events armed for either are recorded."""
    import gpu_common as G
    import paper_2505_05950_amd as F
    d, f, bits, group, T = 1024, 700, 2, 64, 2
    _, ex = G.make_expert(*S.expert_weights(100, 3, d, f), bits, group)
    x, tau = G.dev(S.tokens(100, 3, T, d)), torch.full((T,), 1.0, device=G.DEV)
    for name in ("select", "combine"):
        start, stop, before = (torch.cuda.Event(enable_timing=True) for _ in range(3))
        start.record(), stop.record(), before.record()
        F.floe_profile_kernel(name, start, stop)
        try:
            F.floe_expert_ffn_sparse(ex, x, tau, None, torch.zeros((T, d), dtype=torch.float32, device=G.DEV))
        finally:
            F.floe_profile_kernel("none")
        torch.cuda.synchronize()
        assert before.elapsed_time(start) > 0 and start.elapsed_time(stop) > 0, name
