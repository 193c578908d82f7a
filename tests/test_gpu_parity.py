"""GPU parity: every C-ABI entry point against the CPU oracle on the same seeded inputs.
Index outputs must be bit-exact; bf16 attention outputs within max-abs 2e-2 / mean-abs 2e-3."""
import math

import numpy as np
import pytest
import torch

import focus_inputs as fi
from oracle import focus_oracle as fo
from paper_2602_02159_amd import binding as fb

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def G(gpu_device):
    from tests import gpu_util
    return gpu_util


def _rand_bf16(seed, *shape, scale=1.0):
    g = torch.Generator().manual_seed(seed)
    return (torch.randn(*shape, generator=g) * scale).to(torch.bfloat16)


# ------------------------------------------------------------------------------------------------ stage 1
@pytest.mark.parametrize("n_gen,k,window", [(32, 8, 0), (64, 16, 0), (64, 16, 8), (64, 16, 9), (200, 7, 3), (256, 256, 0),
                                            (1000, 100, 2), (1024, 5, 1), (1500, 300, 4), (5000, 1, 0), (16384, 4000, 8)])
def test_select_queries(G, n_gen, k, window):
    rng = np.random.default_rng(n_gen * 31 + k)
    conf = rng.random(n_gen).astype(np.float32)
    conf[rng.integers(0, n_gen, n_gen // 4)] = 0.5          # plenty of exact ties
    masked = (rng.random(n_gen) < 0.8).astype(np.uint8)
    for m in (None, masked):
        for lo, hi in ((0, n_gen), (n_gen // 5, n_gen - n_gen // 7)):
            focus, active, counts = G.gpu_select(conf, m, k, window, lo, hi)
            ref_f = fo.select_focus(conf, m, k)
            ref_a = fo.expand_window(ref_f, window, lo, hi)
            c = counts.cpu().tolist()
            assert c == [len(ref_f), len(ref_a)]
            assert focus.cpu().tolist() == ref_f.tolist() + [-1] * (k - len(ref_f))
            assert active.cpu().tolist()[:len(ref_a)] == ref_a.tolist()
            assert set(active.cpu().tolist()[len(ref_a):]) <= {-1}


def test_select_queries_special_values(G):
    conf = np.array([np.nan, -np.inf, -0.0, 0.0, np.inf, 1.0, np.nan, 0.0], dtype=np.float32)
    for k in range(1, 9):
        focus, _, counts = G.gpu_select(conf, None, k, 0, 0, 8)
        assert focus.cpu().tolist()[:k] == fo.select_focus(conf, None, k).tolist()
    focus, active, counts = G.gpu_select(np.zeros(64, np.float32), np.zeros(64, np.uint8), 16, 8, 0, 64)
    assert counts.cpu().tolist() == [0, 0] and set(focus.cpu().tolist()) == {-1} and set(active.cpu().tolist()) == {-1}


@pytest.mark.parametrize("name", ["tiny", "ctx8k", "ctx32k"])
def test_select_queries_on_workloads(G, name):
    w = fi.WORKLOADS[name]
    conf = fi.confidence(w).numpy()
    focus, active, counts = G.gpu_select(conf, fi.masked_all(w).numpy(), w.k_focus, w.window, 0, w.n_gen)
    ref = fo.select_focus(conf, None, w.k_focus)
    assert focus.cpu().tolist() == ref.tolist() and active.cpu().tolist() == ref.tolist()
    assert counts.cpu().tolist() == [w.k_focus, w.k_focus]


# ------------------------------------------------------------------------------------------------ stage 2a
@pytest.mark.parametrize("H,M,N,d,B", [(2, 100, 7, 64, 16), (3, 1000, 40, 128, 128), (4, 1024, 32, 64, 64),
                                       (2, 777, 0, 128, 50), (1, 5, 3, 128, 128)])
def test_block_means(G, H, M, N, d, B):
    k = _rand_bf16(1, H, M + N, d).to(G.DEV)
    kbar = G.gpu_block_means(k, M, B)
    ref = fo.block_means(G.to_np(k), M, B)
    assert np.allclose(kbar.cpu().numpy(), ref, rtol=0, atol=2e-6 * math.sqrt(B))


def test_block_means_strided_layout(G):
    # K stored as [L, H, d] and viewed as [H, L, d]: head stride d, row stride H*d
    H, M, N, d, B = 4, 300, 20, 128, 64
    k = _rand_bf16(2, M + N, H, d).to(G.DEV).permute(1, 0, 2)
    assert not k.is_contiguous()
    ref = fo.block_means(G.to_np(k), M, B)
    assert np.allclose(G.gpu_block_means(k, M, B).cpu().numpy(), ref, atol=2e-5)


def test_block_scores_and_top_c(G):
    H, M, N, d, B, n_gen = 8, 2000, 24, 128, 64, 48
    q, k = _rand_bf16(3, H, n_gen, d).to(G.DEV), _rand_bf16(4, H, M + N, d).to(G.DEV)
    focus = [1, 5, 9, 20, 47]
    n_b = -(-M // B)
    Rref = fo.block_relevance(G.to_np(q), focus, fo.block_means(G.to_np(k), M, B))
    for n_keep in (0, 1, 5, n_b):
        fidx = G.i32(focus + [-1, -1, -1])
        counts = G.i32([len(focus), 0])
        scores, kept = G.gpu_block_scores(q, fidx, counts, k, None, M, B, n_keep)          # scans K
        assert np.allclose(scores.cpu().numpy(), Rref, atol=1e-5)
        assert kept.cpu().tolist() == fo.select_blocks(Rref, n_keep).tolist()
        kbar = G.gpu_block_means(k, M, B)
        scores2, kept2 = G.gpu_block_scores(q, fidx, counts, None, kbar, M, B, n_keep)     # cached means
        assert torch.equal(scores, scores2) and torch.equal(kept, kept2)
    # counts = NULL: every slot of focus_idx is used
    scores3, _ = G.gpu_block_scores(q, G.i32(focus), None, k, None, M, B, 3)
    assert np.allclose(scores3.cpu().numpy(), Rref, atol=1e-5)


@pytest.mark.parametrize("H,M,N,d,B,n_gen", [(8, 2000, 24, 128, 64, 48), (5, 1111, 0, 64, 128, 300), (3, 640, 8, 64, 32, 16)])
def test_block_partials_then_top_blocks(G, H, M, N, d, B, n_gen):
    """The two halves of block scoring: per-head partials match the oracle's per-head term of Eq. 7, the K-scanning and
    cached-means variants agree bit for bit, and ranking the partials reproduces focus_block_scores exactly."""
    q, k = _rand_bf16(31, H, n_gen, d).to(G.DEV), _rand_bf16(32, H, M + N, d).to(G.DEV)
    rng = np.random.default_rng(33)
    focus = sorted(rng.choice(n_gen, size=min(n_gen, 11), replace=False).tolist())
    if n_gen == 300:
        focus = sorted(rng.choice(n_gen, size=280, replace=False).tolist())   # more focus rows than one pass of the workgroup holds
    n_b = -(-M // B)
    fidx, counts = G.i32(focus + [-1, -1]), G.i32([len(focus), 0])
    s = fb.make_shape(q, k, None, M, B)
    part = torch.full((H, n_b), float("nan"), dtype=torch.float32, device=G.DEV)
    fb.block_partials(q, fidx, counts, k, None, s, part)
    kbar = G.gpu_block_means(k, M, B)
    part2 = torch.full_like(part, float("nan"))
    fb.block_partials(q, fidx, counts, None, kbar, s, part2)
    torch.cuda.synchronize()
    assert torch.equal(part, part2)
    kb_ref = fo.block_means(G.to_np(k), M, B)
    qsum = G.to_np(q).astype(np.float64)[:, focus].sum(axis=1)                       # [H, d]
    ref = np.einsum("hbd,hd->hb", kb_ref, qsum)
    assert np.allclose(part.cpu().numpy(), ref, rtol=0, atol=1e-4)
    for n_keep in (0, 3, n_b):
        scores = torch.full((n_b,), float("nan"), dtype=torch.float32, device=G.DEV)
        kept = G.i32(None, max(n_keep, 1))
        fb.top_blocks(part, counts, fidx.numel(), n_keep, scores, kept)
        scores_b, kept_b = G.gpu_block_scores(q, fidx, counts, k, None, M, B, n_keep)
        assert torch.equal(scores, scores_b) and torch.equal(kept[:n_keep], kept_b)
        Rref = fo.block_relevance(G.to_np(q), focus, kb_ref)
        assert np.allclose(scores.cpu().numpy(), Rref, atol=1e-5)


def test_top_c_ties_go_to_the_lower_block(G):
    # integer-valued kbar and a one-hot query make R exact, so ties are exact ties
    H, d, B, n_b, n_gen = 2, 64, 32, 300, 4
    M = n_b * B
    vals = np.random.default_rng(5).integers(0, 5, n_b).astype(np.float32)
    k = torch.zeros(H, M + 8, d)
    k[:, :M, 0] = torch.from_numpy(np.repeat(vals, B))
    q = torch.zeros(H, n_gen, d)
    q[:, :, 0] = 1.0
    q, k = q.to(torch.bfloat16).to(G.DEV), k.to(torch.bfloat16).to(G.DEV)
    for n_keep in (1, 7, 150, 299, 300):
        scores, kept = G.gpu_block_scores(q, G.i32([0, 2]), None, k, None, M, B, n_keep)
        assert np.array_equal(scores.cpu().numpy(), vals)
        assert kept.cpu().tolist() == fo.top_indices(vals, n_keep).tolist()


# ------------------------------------------------------------------------------------------------ stage 2b
@pytest.mark.parametrize("H,M,N,d,n_gen,n_act,n_sink", [(2, 300, 20, 64, 16, 5, 3), (4, 1000, 40, 128, 40, 16, 10),
                                                        (3, 2050, 33, 128, 80, 72, 20), (2, 4096, 0, 64, 32, 17, 41),
                                                        (5, 1003, 9, 128, 90, 62, 7),      # two query groups, the second past the count
                                                        (2, 3001, 10, 64, 140, 129, 20),   # ... three, the last with one query
                                                        (40, 2100, 5, 128, 40, 29, 5), (4, 70, 0, 128, 64, 33, 3),
                                                        (2, 32768, 64, 64, 32, 16, 327),   # the paper's 1 % rule at 32K
                                                        (2, 20000, 10, 64, 64, 28, 200),   # ragged last group, two passes
                                                        (1, 4096, 0, 64, 16, 4, 44),       # 1.4 per 128-key group: the most the bound-then-select path takes
                                                        (1, 4096, 0, 64, 16, 4, 45)])      # one more: radix select
def test_find_sinks(G, H, M, N, d, n_gen, n_act, n_sink):
    q, k = _rand_bf16(6, H, n_gen, d).to(G.DEV), _rand_bf16(7, H, M + N, d).to(G.DEV)
    act = np.sort(np.random.default_rng(8).choice(n_gen, n_act, replace=False))
    Sref = fo.sink_scores(G.to_np(q), act, G.to_np(k))
    cap = n_act + 3
    active = G.i32(list(act) + [-1] * (cap - n_act))
    col, sinks = G.gpu_find_sinks(q, active, G.i32([0, n_act]), k, M, 64, n_sink)
    S = col.cpu().numpy().astype(np.float64)
    assert np.allclose(S, Sref, rtol=2e-4, atol=1e-9)
    assert S.sum() == pytest.approx(1.0, abs=1e-4)
    margin = fo.decision_margin(Sref, n_sink, np.arange(M + N) < M)
    assert margin > 1e-5, "test inputs produce a near-tie; pick another seed"
    assert sinks.cpu().tolist() == fo.select_sinks(Sref, M, n_sink).tolist()
    assert sinks.cpu().tolist() == fo.select_sinks(S, M, n_sink).tolist()     # the selection itself, on the device's own values
    # counts = NULL with an exact-size list gives the same answer
    col2, sinks2 = G.gpu_find_sinks(q, G.i32(list(act)), None, k, M, 64, n_sink)
    assert torch.equal(sinks, sinks2) and np.allclose(col2.cpu().numpy(), S, rtol=1e-6)


@pytest.mark.parametrize("H,M,N,d,n_act", [
    (1, 32, 0, 64, 3),          # one split of one sub-tile
    (1, 8192, 64, 128, 16),     # one head: 65 splits, added up by eight threads per row in the column-mass kernel
    (3, 2049, 0, 64, 16),       # 17 splits: one more than two per thread
    (3, 2048, 0, 64, 16),       # 16
    (4, 3000, 7, 64, 9),        # four heads, all in flight
    (2, 3000, 7, 64, 16),       # two, with four in flight
    (5, 3000, 7, 64, 16),       # five, with eight; four threads per row
    (7, 3000, 7, 128, 16),
    (8, 3000, 7, 64, 5),        # eight
    (9, 3000, 7, 64, 16),       # nine, with sixteen; two threads per row
    (31, 600, 3, 64, 7),        # 496 rows: one thread each
    (33, 600, 3, 64, 16),       # 528 rows: two turns
    (64, 1100, 0, 64, 16),      # 1024 rows, the most; four splits
    (65, 1100, 0, 64, 16),      # one head more: the launch
    (1, 25216, 0, 64, 16),      # 197 splits, 4.97 MB of statistics read by all workgroups together
    (1, 25217, 0, 64, 16),      # 198 splits, 5.02 MB: a launch of its own adds the splits up
    (2, 131072, 0, 64, 16),     # 256 splits
    (8, 19456, 0, 64, 16),      # 32 splits of eight heads, 4.98 MB
    (8, 33000, 0, 64, 16),      # 64 splits, 17 MB
    (8, 45000, 0, 64, 16),      # 96 splits: three batches per thread of the launch
    (32, 8200, 56, 64, 16),     # 65 rounds in 16 splits, one of them with a fifth
    (32, 16400, 0, 64, 16),     # 129 rounds: two each
    (1, 32768, 64, 64, 30),     # two passes, 65 splits: eight threads per row in the second pass
    (8, 33000, 0, 64, 20),      # 65 splits
    (1, 131072, 64, 64, 17),    # 257 splits: the first that need the launch
    (1, 16000, 0, 64, 50),      # two query tiles, 125 splits, four threads per row
    (1, 16500, 0, 128, 50),     # 129 splits: the first that need the launch
    (3, 40, 0, 128, 100)])      # two query groups, one split
def test_find_sinks_statistics_of_the_key_splits(G, H, M, N, d, n_act):
    q, k = _rand_bf16(16, H, n_act, d).to(G.DEV), _rand_bf16(17, H, M + N, d).to(G.DEV)
    act = np.arange(n_act)
    col, _ = G.gpu_find_sinks(q, G.i32(act), None, k, M, 64, 1)
    S, Sref = col.cpu().numpy().astype(np.float64), fo.sink_scores(G.to_np(q), act, G.to_np(k))
    assert np.allclose(S, Sref, rtol=2e-4, atol=1e-9) and S.sum() == pytest.approx(1.0, abs=1e-4)


@pytest.mark.parametrize("H,L,d", [
    (32, 4096, 128),     # four rounds per wavefront everywhere: the fewest that take two stages
    (32, 4095, 128),     # ... the last sub-tile ragged
    (32, 4064, 128),     # ... and a sub-tile less: wavefronts of three rounds
    (32, 4097, 64),      # five rounds in one split, one row in the last
    (1, 131105, 128),    # 256 splits
    (600, 9001, 64),     # twelve rounds in 3600 workgroups
    (33, 8230, 128),     # 462 workgroups; splits of four and of five rounds
])
def test_find_sinks_in_two_stages(G, H, L, d):
    q, k = _rand_bf16(18, H, 16, d).to(G.DEV), _rand_bf16(19, H, L, d).to(G.DEV)
    col, top = G.gpu_find_sinks(q, G.i32(np.arange(13)), None, k, L - 3, 64, 4)
    mass = torch.zeros(L, dtype=torch.float64, device=G.DEV)
    for h in range(H):
        mass += torch.softmax(q[h, :13].double() @ k[h].double().t() / d ** 0.5, -1).mean(0)
    assert torch.allclose(col.double(), mass / H, rtol=2e-4, atol=1e-9)      # the bar of test_find_sinks
    assert top.cpu().tolist() == fo.select_sinks(col.cpu().numpy().astype(np.float64), L - 3, 4).tolist()


@pytest.mark.parametrize("n_gen,k,window,lo,hi,cap", [
    (64, 16, 0, 0, 64, 16), (64, 4, 8, 0, 64, 36), (63, 5, 9, 3, 60, 57), (64, 64, 0, 0, 64, 64), (64, 1, 300, 0, 64, 64),
    (1, 1, 0, 0, 1, 1), (33, 8, 2, 10, 11, 8), (65, 4, 2, 0, 65, 12), (200, 30, 3, 0, 200, 90), (64, 3, 200, 63, 64, 20)])
def test_select_and_find_sinks_equals_the_two_calls(G, n_gen, k, window, lo, hi, cap):
    H, M, N, d, n_sink = 3, 1500, 40, 64, 5
    g = torch.Generator().manual_seed(n_gen + k)
    conf = torch.rand(n_gen, generator=g)
    conf[:n_gen // 3] = 0.5  # ties
    masked = (torch.rand(n_gen, generator=g) < 0.7).to(torch.uint8)
    q, kk = _rand_bf16(61, H, n_gen, d).to(G.DEV), _rand_bf16(62, H, M + N, d).to(G.DEV)
    s = fb.make_shape(q, kk, None, M, 64)
    ws = G.ws(fb.workspace_bytes(fb.FN_FIND_SINKS, s, cap))
    for mask in (None, masked.to(G.DEV)):
        res = []
        for fused in (False, True):
            focus, active, counts, sinks = (torch.full((n,), -7, dtype=torch.int32, device=G.DEV) for n in (k, cap, 2, n_sink))
            col = torch.zeros(M + N, device=G.DEV)
            if fused:
                fb.select_and_find_sinks(conf.to(G.DEV), mask, k, window, lo, hi, focus, active, counts, q, kk, s, n_sink, col, sinks, ws)
            else:
                fb.select_queries(conf.to(G.DEV), mask, k, window, lo, hi, focus, active, counts)
                fb.find_sinks(q, active, counts, kk, s, n_sink, col, sinks, ws)
            torch.cuda.synchronize()
            res.append((focus, active, counts, col, sinks))
        assert all(torch.equal(a, b) for a, b in zip(*res))


@pytest.mark.parametrize("H,d", [(32, 64), (32, 128), (33, 64), (40, 128)])   # whole batches of sixteen heads, and not
def test_select_and_find_sinks_with_logits_past_the_memory_side_cache(G, H, d):
    """More than 200 MB of spilled logits, read back non-temporally from the last head on, with the selection in the same launch: the two
    calls' results bit for bit, and column masses that agree with fp64."""
    M, N, n_gen, k, n_sink = (200 << 20) // (64 * H) + 100, 37, 48, 13, 5
    L = M + N
    assert H * L * 64 > 200 << 20
    g = torch.Generator(device=G.DEV).manual_seed(330 + d)
    q, kk = (torch.randn(H, r, d, generator=g, device=G.DEV).to(torch.bfloat16) for r in (n_gen, L))
    planted = torch.tensor([0, 31, 50001, 77777, M - 1], device=G.DEV)   # clear winners among the masses
    kk[:, planted] += 3.0 * q.float().mean(1, keepdim=True).to(torch.bfloat16) * torch.arange(5, 10, device=G.DEV).view(1, 5, 1)
    conf = torch.rand(n_gen, generator=g, device=G.DEV)
    masked = (torch.rand(n_gen, generator=g, device=G.DEV) < 0.7).to(torch.uint8)
    s = fb.make_shape(q, kk, None, M, 128)
    res = []
    for fused in (False, True):
        focus, active, counts, sinks = G.i32(None, k), G.i32(None, k), G.i32(None, 2), G.i32(None, n_sink)
        col = torch.full((L,), float("nan"), device=G.DEV)
        w = G.ws(fb.workspace_bytes(fb.FN_FIND_SINKS, s, k))
        if fused:
            fb.select_and_find_sinks(conf, masked, k, 0, 0, n_gen, focus, active, counts, q, kk, s, n_sink, col, sinks, w)
        else:
            fb.select_queries(conf, masked, k, 0, 0, n_gen, focus, active, counts)
            fb.find_sinks(q, active, counts, kk, s, n_sink, col, sinks, w)
        torch.cuda.synchronize()
        res.append((focus, active, counts, col, sinks))
    assert all(torch.equal(a, b) for a, b in zip(*res))
    _, active, counts, col, sinks = res[0]
    rows = active[:int(counts[1])].long()
    S = torch.zeros(L, dtype=torch.float64, device=G.DEV)
    for h in range(H):
        z = torch.matmul(q[h, rows].double(), kk[h].double().T.contiguous()) / math.sqrt(d)
        S += torch.softmax(z, -1).mean(0) / H
    assert torch.allclose(col.double(), S, rtol=2e-4, atol=1e-9)
    assert fo.decision_margin(S.cpu().numpy(), n_sink, np.arange(L) < M) > 1e-5
    assert sinks.cpu().tolist() == fo.select_sinks(S.cpu().numpy(), M, n_sink).tolist()


def test_probe_layer_with_logits_past_the_memory_side_cache(G):
    """The same way back for logits that the probe layer's attention has kept, with a last batch of one head."""
    H, M, N, d, n_gen, n_act, n_sink = 33, 99400, 37, 64, 16, 13, 5
    L = M + N
    assert H * L * 64 > 200 << 20
    g = torch.Generator(device=G.DEV).manual_seed(340)
    q, k, v = (torch.randn(H, r, d, generator=g, device=G.DEV).to(torch.bfloat16) for r in (n_gen, L, L))
    planted = torch.tensor([0, 31, 50001, 77777, M - 1], device=G.DEV)
    k[:, planted] += 3.0 * q.float().mean(1, keepdim=True).to(torch.bfloat16) * torch.arange(5, 10, device=G.DEV).view(1, 5, 1)
    out, _, col, sinks = G.gpu_probe_layer(q, G.i32(np.arange(n_gen)), G.i32([0, n_act]), k, v, M, 128, n_sink)
    S, ref = torch.zeros(L, dtype=torch.float64, device=G.DEV), []
    for h in range(H):
        p = torch.softmax(torch.matmul(q[h, :n_act].double(), k[h].double().T.contiguous()) / math.sqrt(d), -1)
        S += p.mean(0) / H
        ref.append(torch.matmul(p, v[h].double()))
    G.assert_attention_close(out[:, :n_act], torch.stack(ref).cpu().numpy())
    assert torch.allclose(col.double(), S, rtol=2e-4, atol=1e-9)
    assert fo.decision_margin(S.cpu().numpy(), n_sink, np.arange(L) < M) > 1e-5
    assert sinks.cpu().tolist() == fo.select_sinks(S.cpu().numpy(), M, n_sink).tolist()


def test_find_sinks_with_the_workspace_of_one_key_split_less(G):
    """32 heads, 257 rounds: 129 splits, and 128 where their statistics do not fit; a byte less is refused."""
    H, M, N, d, n_act = 32, 32768, 64, 64, 16
    q, k = _rand_bf16(26, H, n_act, d).to(G.DEV), _rand_bf16(27, H, M + N, d).to(G.DEV)
    active, s = G.i32(np.arange(n_act)), fb.make_shape(q, k, None, M, 64)
    full = fb.workspace_bytes(fb.FN_FIND_SINKS, s, n_act)
    least = full - H * n_act * 8
    col, sinks = G.gpu_find_sinks(q, active, None, k, M, 64, 3)
    col2, sinks2, buf = torch.empty_like(col), torch.empty_like(sinks), torch.full((full,), 0x5B, dtype=torch.uint8, device=G.DEV)
    fb.find_sinks(q, active, None, k, s, 3, col2, sinks2, buf[:least])
    torch.cuda.synchronize()
    assert bool((buf[least:] == 0x5B).all()) and torch.equal(sinks, sinks2)
    assert torch.allclose(col, col2, rtol=1e-5, atol=1e-12)
    with pytest.raises(fb.FocusError):
        fb.find_sinks(q, active, None, k, s, 3, col2, sinks2, buf[:least - 1])


@pytest.mark.parametrize("H,M,N,d", [(3, 700, 5, 64), (2, 4100, 30, 128), (18, 900, 1, 128)])
@pytest.mark.parametrize("cap,n_act", [(1, 1), (3, 2), (8, 8), (9, 7), (15, 15), (16, 5)])
def test_logits_of_fewer_than_sixteen_queries(G, H, M, N, d, cap, n_act):
    """The slots past the capacity are neither written nor read: scratch memory that is NaN before changes nothing."""
    q, k, v = (_rand_bf16(161 + i, H, r, d).to(G.DEV) for i, r in enumerate((16, M + N, M + N)))
    rows = np.sort(np.random.default_rng(cap).choice(16, cap, replace=False))
    active, counts = G.i32(rows), G.i32([1, n_act])
    logits = torch.matmul(q[:, rows[:n_act]].float(), k.float().transpose(1, 2).contiguous()) / d ** 0.5
    mass = torch.softmax(logits, -1).mean((0, 1))
    out = torch.empty((H, cap, d), dtype=torch.bfloat16, device=G.DEV)
    s = fb.make_shape(q, k, v, M, 64, out)
    for probe in (False, True):
        nbytes = fb.workspace_bytes(fb.FN_PROBE_LAYER if probe else fb.FN_FIND_SINKS, s, cap)
        buf = torch.full((nbytes,), 0xFF, dtype=torch.uint8, device=G.DEV)   # NaN wherever it is read as floats
        col, sinks = torch.empty(M + N, device=G.DEV), G.i32(np.zeros(4))
        if probe:
            fb.probe_layer(q, active, counts, k, v, s, 4, out, None, col, sinks, buf)
        else:
            fb.find_sinks(q, active, counts, k, s, 4, col, sinks, buf)
        torch.cuda.synchronize()
        assert torch.allclose(col, mass, rtol=2e-4, atol=1e-9)   # the bar of test_find_sinks
        assert sinks.cpu().tolist() == fo.select_sinks(col.cpu().numpy().astype(np.float64), M, 4).tolist()


def test_find_sinks_equal_keys_fall_back_to_lowest_positions(G):
    H, M, N, d = 2, 500, 12, 64
    k = _rand_bf16(9, 1, 1, d).expand(H, M + N, d).contiguous().to(G.DEV)
    q = _rand_bf16(10, H, 16, d).to(G.DEV)
    col, sinks = G.gpu_find_sinks(q, G.i32([0, 3, 8]), None, k, M, 64, 5)
    assert np.allclose(col.cpu().numpy(), 1.0 / (M + N), rtol=1e-5)
    # all column masses are equal only up to rounding on the device, so check the tie rule on the device's own values
    assert len(set(sinks.cpu().tolist())) == 5
    assert sinks.cpu().tolist() == fo.select_sinks(col.cpu().numpy().astype(np.float64), M, 5).tolist()


@pytest.mark.parametrize("M,N,n_sink", [(32768, 64, 16), (32800, 0, 16), (16448, 0, 16), (4100, 30, 1), (4100, 30, 17), (9000, 8, 7),
                                        (32768, 64, 327), (32768, 0, 358), (32768, 0, 512), (20000, 10, 200), (32800, 0, 327)])
def test_find_sinks_selection_is_exact_with_many_exact_ties(G, M, N, n_sink):
    """Keys repeat with period 37, so column masses tie exactly across the whole prompt (and across the groups of the
    tournament that serves small N_sink, at and just past its size limits; for large N_sink thousands of positions
    clear the nominees' bound, so the bound-then-select path has to fall back to the radix select): the sinks must be
    the oracle's selection applied to the device's own masses, ties to the lower position."""
    H, d, n_gen = 2, 64, 16
    base = _rand_bf16(40, H, 37, d)
    k = base[:, torch.arange(M + N) % 37].contiguous().to(G.DEV)
    q = _rand_bf16(41, H, n_gen, d).to(G.DEV)
    col, sinks = G.gpu_find_sinks(q, G.i32([1, 4, 9, 15]), None, k, M, 64, n_sink)
    S = col.cpu().numpy().astype(np.float64)
    assert len(np.unique(S)) <= 37 * 4                      # ties really are exact (a few rounding classes at most)
    assert sinks.cpu().tolist() == fo.select_sinks(S, M, n_sink).tolist()
    Sref = fo.sink_scores(G.to_np(q), [1, 4, 9, 15], G.to_np(k))
    assert np.allclose(S, Sref, rtol=2e-4, atol=1e-9)


@pytest.mark.parametrize("M,N,n_sink,n_cluster", [
    (20000, 10, 200, 0),       # nominees of the 128-key groups suffice
    (20000, 10, 200, 16),      # one group has exactly as many as it may nominate
    (20000, 10, 200, 60),      # ... and many more: all positions that clear the bound
    (32768, 64, 1000, 900),    # seven whole groups
    (40000, 0, 1250, 1200),    # more than a workgroup ranks at once: radix select
    (131072, 0, 16, 16),       # few sinks, too many groups for the tournament
    (70001, 3, 700, 100),      # past 32768 positions, a ragged last group
    (131072, 0, 1310, 3),
    (300, 20, 9, 9),           # three groups
])
def test_find_sinks_that_cluster(G, M, N, n_sink, n_cluster):
    """Sinks side by side fill the nominees of their 128-key groups; the answer must not depend on where they sit."""
    H, d, n_gen = 2, 64, 16
    q, k = _rand_bf16(51, H, n_gen, d), _rand_bf16(52, H, M + N, d)
    u = q.float().mean(1, keepdim=True)
    first = (M // 2 // 128) * 128 if M > 4096 else 100
    k[:, first:first + n_cluster] += (6.0 * u / u.norm(dim=-1, keepdim=True)).to(torch.bfloat16)
    col, sinks = G.gpu_find_sinks(q.to(G.DEV), G.i32([0, 2, 7]), None, k.to(G.DEV), M, 64, n_sink)
    assert sinks.cpu().tolist() == fo.select_sinks(col.cpu().numpy().astype(np.float64), M, n_sink).tolist()


def test_find_sinks_many_sinks_with_an_unaligned_score_buffer(G):
    """The bound-then-select path reads the column masses with 16-byte loads; a caller's score buffer that is only
    4-byte aligned takes the radix select instead and must give the same sinks."""
    H, M, N, d, n_gen, n_sink = 2, 8192, 32, 64, 16, 80
    q, k = _rand_bf16(181, H, n_gen, d).to(G.DEV), _rand_bf16(182, H, M + N, d).to(G.DEV)
    active = G.i32([0, 3, 5, 9])
    col, sinks = G.gpu_find_sinks(q, active, None, k, M, 64, n_sink)
    s = fb.make_shape(q, k, None, M, 64)
    buf = torch.empty(M + N + 1, dtype=torch.float32, device=G.DEV)
    col2, sinks2 = buf[1:], G.i32(None, n_sink)
    assert col2.data_ptr() % 16 == 4
    fb.find_sinks(q, active, None, k, s, n_sink, col2, sinks2, G.ws(fb.workspace_bytes(fb.FN_FIND_SINKS, s, active.numel())))
    torch.cuda.synchronize()
    assert torch.equal(col, col2) and torch.equal(sinks, sinks2)
    assert sinks.cpu().tolist() == fo.select_sinks(col.cpu().numpy().astype(np.float64), M, n_sink).tolist()


# ------------------------------------------------------------------------------------------------ stage 3
def _attn_case(G, H, M, N, d, B, n_gen, active, kept, sinks, seed=11, counts=None, cap=None):
    q, k, v = (_rand_bf16(seed + i, H, r, d).to(G.DEV) for i, r in enumerate((n_gen, M + N, M + N)))
    cap = cap or len(active)
    a_dev = G.i32(list(active) + [-1] * (cap - len(active)))
    out, lse = G.gpu_sparse_attn(q, a_dev, counts, k, v, M, B, G.i32(kept) if len(kept) else None,
                                 G.i32(sinks) if len(sinks) else None)
    I_p = fo.attention_index_set(sinks, kept, M, B)
    ref, ref_lse = fo.sparse_attention(G.to_np(q), active, G.to_np(k), G.to_np(v), I_p, M)
    return out, lse, ref, ref_lse


@pytest.mark.parametrize("H,M,N,d,B,n_gen,n_act,n_keep,n_sink", [
    (4, 1024, 32, 64, 64, 32, 8, 4, 2),        # the tiny configuration's shape
    (2, 1000, 37, 128, 48, 40, 16, 5, 3),      # ragged everything: M % B, B % 32, N % 32
    (3, 2048, 64, 128, 128, 64, 16, 6, 4),
    (2, 4096, 96, 128, 64, 128, 72, 20, 41),   # five query tiles (window-expanded queries), many sinks
    (2, 600, 0, 64, 100, 24, 24, 2, 0),        # no response rows, no sinks
    (1, 512, 16, 128, 128, 16, 1, 0, 1),       # a single query, no blocks
    (5, 300, 5, 64, 7, 33, 33, 11, 9),         # tiny blocks
])
def test_sparse_attn(G, H, M, N, d, B, n_gen, n_act, n_keep, n_sink):
    rng = np.random.default_rng(H * 1000 + M)
    n_b = -(-M // B)
    active = np.sort(rng.choice(n_gen, n_act, replace=False))
    kept = rng.choice(n_b, n_keep, replace=False)        # unsorted on purpose
    sinks = rng.choice(M, n_sink, replace=False)
    out, lse, ref, ref_lse = _attn_case(G, H, M, N, d, B, n_gen, active, kept, sinks)
    G.assert_attention_close(out, ref)
    assert np.allclose(lse.cpu().numpy(), ref_lse, atol=2e-3)


@pytest.mark.parametrize("H,M,N,d,cap,live", [
    (32, 2177, 40, 128, 17, 17),   # one 32-query tile, several rounds per slot, ragged last sub-tile
    (32, 2300, 31, 128, 32, 3),    # most query slots past the device-side count
    (32, 4200, 64, 64, 32, 32),    # d = 64; an odd number of rounds
    (32, 2177, 40, 128, 33, 33),   # two tiles that share a slot, one query in the second
    (32, 2240, 64, 128, 64, 32),   # ... and none
    (32, 4200, 64, 64, 64, 64),
    (16, 2400, 10, 128, 65, 65),   # query groups: the last one holds one query
    (16, 2400, 10, 64, 130, 97),   # ... and one group is empty
    (32, 900, 20, 128, 48, 40),    # one sub-tile per slot
    (32, 300, 20, 64, 100, 70),    # ... with query groups
    (1, 16500, 33, 128, 16, 16),   # one head: more than a hundred key splits to merge
    (1, 16500, 33, 64, 40, 40),
])
def test_sparse_attn_query_tiles_and_key_splits(G, H, M, N, d, cap, live):
    rng = np.random.default_rng(H * M + cap)
    B, n_gen = 64, cap + 9
    active = np.sort(rng.choice(n_gen, live, replace=False))
    n_b = -(-M // B)
    kept = np.sort(rng.choice(n_b, n_b - 3, replace=False))
    out, lse, ref, ref_lse = _attn_case(G, H, M, N, d, B, n_gen, active, kept, np.sort(rng.choice(M, 45, replace=False)),
                                        counts=G.i32([1, live]), cap=cap)
    G.assert_attention_close(out[:, :live], ref)
    assert np.allclose(lse.cpu().numpy()[:, :live], ref_lse, atol=2e-3)
    assert torch.isnan(out[:, live:]).all()  # rows past the count are not written


@pytest.mark.parametrize("H,M,N", [
    (32, 4096, 0),      # 128 sub-tiles of 32 heads: the most with one per wavefront, 32 splits
    (32, 4096, 5),      # one more: a key loop in 16 splits
    (16, 8192, 0), (16, 8192, 1),      # 64 splits, and 32
    (15, 4500, 3),      # fewer heads would take more than 64 splits
    (8, 8000, 30)])
def test_sparse_attn_few_queries_of_64_columns(G, H, M, N):
    q, k, v = (_rand_bf16(75 + i, H, r, 64).to(G.DEV) for i, r in enumerate((16, M + N, M + N)))
    kept = np.arange(-(-M // 32))
    out, lse = G.gpu_sparse_attn(q, G.i32(np.arange(16)), G.i32([0, 11]), k, v, M, 32, G.i32(kept), None)
    ref, ref_lse = fo.sparse_attention(G.to_np(q), np.arange(11), G.to_np(k), G.to_np(v), np.arange(M), M)
    G.assert_attention_close(out[:, :11], ref)
    assert np.allclose(lse[:, :11].cpu().numpy(), ref_lse, atol=2e-3)


@pytest.mark.parametrize("n_act", [16, 30, 50])
@pytest.mark.parametrize("H,M,N,d", [
    (5, 20001, 30, 64),                        # 51 splits of two or three rounds, the last one ragged
    (64, 1300, 5, 128),                        # four splits of 64 heads: every starting place several times
    (300, 700, 9, 64),                         # more heads than rounds, one split
    (1, 40000, 64, 128),
])
def test_sparse_attn_heads_begin_at_different_places(G, H, M, N, d, n_act):
    q, k, v = (_rand_bf16(65 + i, H, r, d).to(G.DEV) for i, r in enumerate((n_act, M + N, M + N)))
    act = np.arange(n_act)
    out, lse = G.gpu_sparse_attn(q, G.i32(act), None, k, v, M, 64, G.i32(np.arange(-(-M // 64))), None)
    ref, ref_lse = fo.sparse_attention(G.to_np(q), act, G.to_np(k), G.to_np(v), np.arange(M), M)
    G.assert_attention_close(out, ref)
    assert np.allclose(lse.cpu().numpy(), ref_lse, atol=2e-3)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("n_act,M", [
    (16, 8180), (30, 8180),     # 64 rounds per slot, the last one ragged
    (16, 8200), (30, 8200),     # 65: the table of the sub-tiles is made twice
])
def test_key_loop_of_many_rounds(G, d, n_act, M):
    """One key split of four slots, with block ids outside the prompt in between (rounds in which a slot has nothing to do), responses and
    more sinks than one sub-tile holds; the probe layer, which writes its logits on the way, over the same rows."""
    H, N, B = 257, 3, 32
    q, k, v = (_rand_bf16(85 + i, H, r, d).to(G.DEV) for i, r in enumerate((n_act, M + N, M + N)))
    act, n_b = np.arange(n_act), -(-M // B)
    kept = np.arange(n_b)
    skipped = np.concatenate([np.arange(3, n_b, 41), np.arange(100, 104)])
    listed = kept.copy()
    listed[skipped] = np.where(np.arange(len(skipped)) % 2, -1, n_b + 5)
    sinks = np.sort(np.concatenate([skipped * B + 1, np.arange(0, M, 300)]))
    out, lse = G.gpu_sparse_attn(q, G.i32(act), None, k, v, M, B, G.i32(listed), G.i32(sinks))
    some = [0, 1, 128, 256]
    I_p = fo.attention_index_set(sinks, np.setdiff1d(kept, skipped), M, B)
    ref, ref_lse = fo.sparse_attention(G.to_np(q[some]), act, G.to_np(k[some]), G.to_np(v[some]), I_p, M)
    G.assert_attention_close(out[some], ref)
    assert np.allclose(lse[some].cpu().numpy(), ref_lse, atol=2e-3)
    out, lse, col, top = G.gpu_probe_layer(q, G.i32(act), None, k, v, M, B, 4)
    ref, ref_lse = fo.sparse_attention(G.to_np(q[some]), act, G.to_np(k[some]), G.to_np(v[some]), np.arange(M), M)
    G.assert_attention_close(out[some], ref)
    assert np.allclose(lse[some].cpu().numpy(), ref_lse, atol=2e-3)
    logits = torch.matmul(q.float(), k.float().transpose(1, 2).contiguous()) / d ** 0.5
    mass = torch.softmax(logits, -1).mean((0, 1))
    assert torch.allclose(col, mass, rtol=2e-4, atol=1e-9)   # the bar of test_find_sinks
    assert top.cpu().tolist() == fo.select_sinks(col.cpu().numpy().astype(np.float64), M, 4).tolist()


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("H,M,N,B,n_act,n_keep,n_sink", [
    (3, 700, 0, 32, 16, 5, 0),       # five sub-tiles: one more than the wavefronts of a split
    (2, 701, 33, 32, 11, 4, 32),     # seven, the last rows of the prompt, of the responses and a full list of sinks
    (2, 512, 1, 2, 1, 6, 3),         # eight, the most at d = 128; 256 blocks, the most
    (2, 514, 1, 2, 1, 6, 3),         # 257
    (33, 1000, 30, 64, 16, 3, 40),   # nine; sinks in two sub-tiles, against the bitmap of the kept blocks
    (2, 1000, 30, 64, 7, 4, 60),     # eleven
    (2, 4000, 64, 16, 16, 10, 7),    # thirteen
    (256, 300, 20, 16, 5, 15, 0),    # sixteen, the most at d = 64, with the most heads that get four key splits else
    (512, 150, 20, 16, 5, 7, 0),     # eight, with the most heads that get two
    (600, 300, 20, 16, 5, 15, 0),    # sixteen for more heads than that: a key loop
    (2, 4000, 20, 16, 5, 16, 0),     # seventeen
])
def test_sparse_attn_of_few_sub_tiles(G, d, H, M, N, B, n_act, n_keep, n_sink):
    """One workgroup per head or a plan of key splits: attention alone and the whole layer, per head and head-averaged relevances, with
    ids outside the prompt, padding of the active list and rows past it left alone."""
    rng, n_gen = np.random.default_rng(n_sink + M), 20
    q, k, v = (_rand_bf16(141 + i, H, r, d).to(G.DEV) for i, r in enumerate((n_gen, M + N, M + N)))
    k[:, 3 * B:4 * B] = k[:, 7 * B:8 * B]                   # equal relevances: ties go to the lower block
    some = list(range(0, H, max(1, H // 4)))
    act = np.sort(rng.choice(n_gen, n_act, replace=False))
    focus, active = G.i32(np.arange(3)), G.i32(np.concatenate([act, [0] * (16 - n_act)]))
    counts, sinks = G.i32([3, n_act]), G.i32(rng.choice(M, n_sink, replace=False)) if n_sink else None
    sink_rows = sinks.cpu().numpy() if n_sink else []
    kbar = G.gpu_block_means(k, M, B)
    scores, kept = G.gpu_block_scores(q, focus, counts, k, kbar, M, B, n_keep)
    out = torch.empty((H, 16, d), dtype=torch.bfloat16, device=G.DEV)
    lse, s2, k2 = torch.empty((H, 16), device=G.DEV), torch.empty_like(scores), torch.empty_like(kept)
    s = fb.make_shape(q, k, v, M, B, out)

    def check(blocks):
        rows = fo.attention_index_set(sink_rows, blocks, M, B)
        ref, ref_lse = fo.sparse_attention(G.to_np(q[some]), act, G.to_np(k[some]), G.to_np(v[some]), rows, M)
        G.assert_attention_close(out[some, :n_act], ref)
        assert np.allclose(lse[some, :n_act].cpu().numpy(), ref_lse, atol=2e-3)
        assert bool((out[:, n_act:] == 7).all()) and bool((lse[:, n_act:] == 9).all())

    listed = kept.clone()
    listed[-1] = -1
    listed[0] = -(-M // B)
    buf = G.ws(fb.workspace_bytes(fb.FN_SPARSE_ATTN, s, 16, n_keep, n_sink))
    out.fill_(7.0), lse.fill_(9.0)
    fb.sparse_attn(q, active, counts, k, v, s, listed, n_keep, sinks, n_sink, out, lse, buf)
    check(kept.cpu().numpy()[1:-1])
    for mean_k in (kbar, None):
        out.fill_(7.0), lse.fill_(9.0)
        fb.sparse_layer(q, focus, active, counts, k, v, mean_k, s, n_keep, sinks, n_sink, s2, k2, out, lse,
                        G.ws(fb.workspace_bytes(fb.FN_SPARSE_LAYER, s, 16, n_keep, n_sink)))
        assert torch.equal(k2, kept) and (mean_k is None or torch.equal(s2, scores))
        check(kept.cpu().numpy())


@pytest.mark.parametrize("H,M,d,B,n_keep,n_sink,n_focus,over", [
    (8, 256, 128, 16, 7, 3, 16, False),      # eight wavefronts, eight heads of sixteen blocks
    (4, 1024, 128, 32, 6, 2, 70, False),     # ... of two times sixteen, more focus rows than lanes
    (4, 1056, 128, 32, 6, 2, 1, False),      # ... of three times: relevances by a launch
    (9, 256, 128, 16, 7, 0, 9, False),       # nine heads: by a launch
    (12, 200, 64, 16, 10, 5, 33, False),     # twelve wavefronts, three groups of heads; a ragged last block
    (5, 700, 64, 16, 13, 5, 40, False),      # sixteen, for fifteen sub-tiles; two groups, one with one head
    (16, 100, 64, 8, 13, 40, 5, False),      # four groups
    (1, 4096, 64, 16, 15, 0, 80, False),     # one head, 256 blocks
    (8, 256, 128, 16, 7, 3, 16, True),       # the output lies over the queries: key splits, relevances by a launch
])
def test_relevance_in_the_attention_kernel(G, H, M, d, B, n_keep, n_sink, n_focus, over):
    """Short key lists of few heads: scores, blocks and output of the whole layer are bit for bit those of the separate calls."""
    rng, n_gen, N, n_act = np.random.default_rng(M + n_focus), 80, 32, 16
    q, k, v = (_rand_bf16(151 + i, H, r, d).to(G.DEV) for i, r in enumerate((n_gen, M + N, M + N)))
    k[:, 3 * B:4 * B] = k[:, 7 * B:8 * B]                   # equal relevances: ties go to the lower block
    focus = np.sort(rng.choice(n_gen, n_focus, replace=False))
    focus[n_focus // 2] = n_gen if n_focus > 1 else focus[0]   # an entry past the block adds nothing
    focus, active = G.i32(focus), G.i32(np.arange(n_act))
    counts = G.i32([max(1, n_focus - 1), n_act])
    sinks = G.i32(rng.choice(M, n_sink, replace=False)) if n_sink else None
    kbar = G.gpu_block_means(k, M, B)
    scores, kept = G.gpu_block_scores(q, focus, counts, k, kbar, M, B, n_keep)
    out, lse = G.gpu_sparse_attn(q, active, counts, k, v, M, B, kept, sinks)
    o2 = q[:, :n_act] if over else torch.empty_like(out)
    s2, k2, l2 = torch.empty_like(scores), torch.empty_like(kept), torch.empty_like(lse)
    s = fb.make_shape(q, k, v, M, B, o2)
    fb.sparse_layer(q, focus, active, counts, k, v, kbar, s, n_keep, sinks, n_sink, s2, k2, o2, l2,
                    G.ws(fb.workspace_bytes(fb.FN_SPARSE_LAYER, s, n_act, n_keep, n_sink)))
    torch.cuda.synchronize()
    assert torch.equal(s2, scores) and torch.equal(k2, kept)
    if over:  # the merge of the splits rounds in other places
        G.assert_attention_close(o2, out.double().cpu().numpy())
        assert torch.allclose(l2, lse, atol=2e-3)
    else:
        assert torch.equal(o2, out) and torch.equal(l2, lse)


@pytest.mark.parametrize("d,H,n_keep,n_sink", [
    (128, 120, 6, 2), (128, 4, 6, 2),      # eight sub-tiles; with four heads the relevances come from the attention kernel
    (64, 100, 6, 2), (64, 60, 13, 40),     # eight, sixteen
    (64, 4, 11, 5),                        # thirteen, relevances in the attention kernel
])
@pytest.mark.parametrize("over", ["queries", "queries_reversed", "reversed", "keys", "values", "means", "focus"])
def test_outputs_that_share_memory_with_an_input(G, d, H, n_keep, n_sink, over):
    """Short key lists whose output (a compact tensor, so that the rows of one head lie on those of other heads), log-sum-exps, scores or
    block list lie over an input: read before they are written, as with key splits.  ("reversed": only the heads in descending order.)"""
    M, B, N, n_gen, cap = 512, 16, 20, 40, 16
    rng = np.random.default_rng(H + d)
    src = [_rand_bf16(201 + i, H, r, d).to(G.DEV) for i, r in enumerate((n_gen, M + N, M + N))]
    active, counts = G.i32(np.sort(rng.choice(n_gen, cap, replace=False))), G.i32([9, cap])
    rows, sinks = G.i32(np.sort(rng.choice(n_gen, max(9, n_keep), replace=False))), G.i32(rng.choice(M, n_sink, replace=False))
    means, n_b = G.gpu_block_means(src[1], M, B), M // B

    for call in ("attention", "layer", "scan"):
        if over in ("means", "focus") and call != "layer":
            continue
        got = []
        for shared in (False, True):
            q, k, v = (t.clone() for t in src)
            kbar, focus = means.clone(), rows.clone()
            out = torch.empty((H, cap, d), dtype=torch.bfloat16, device=G.DEV)
            lse = torch.empty((H, cap), device=G.DEV)
            scores, kept = torch.empty(n_b, device=G.DEV), G.i32(np.zeros(n_keep))
            if shared:
                if over in ("queries", "queries_reversed", "keys", "values"):
                    out = {"keys": k, "values": v}.get(over, q).view(-1)[:H * cap * d].view(H, cap, d)
                elif over == "means":   # the log-sum-exps at its start, the scores at its end
                    lse, scores = kbar.view(-1)[:H * cap].view(H, cap), kbar.view(-1)[-n_b:]
                elif over == "focus":
                    kept = focus[:n_keep]
            s = fb.make_shape(q, k, v, M, B, out)
            reverse, first = over.endswith("reversed") and shared, out
            if reverse:   # heads in descending order: the first one last
                s.o_stride_h, first = -s.o_stride_h, out[H - 1]
            if call == "attention":
                blocks = G.i32(np.arange(1, 2 * n_keep, 2))
                fb.sparse_attn(q, active, counts, k, v, s, blocks, n_keep, sinks, n_sink, first, lse,
                               G.ws(fb.workspace_bytes(fb.FN_SPARSE_ATTN, s, cap, n_keep, n_sink)))
            else:
                fb.sparse_layer(q, focus, active, counts, k, v, kbar if call == "layer" else None, s, n_keep, sinks, n_sink, scores, kept, first, lse,
                                G.ws(fb.workspace_bytes(fb.FN_SPARSE_LAYER, s, cap, n_keep, n_sink)))
            torch.cuda.synchronize()
            got.append((out.flip(0) if reverse else out.clone(), lse.clone(), scores.clone(), kept.clone()))
        (o0, l0, s0, k0), (o1, l1, s1, k1) = got
        G.assert_attention_close(o1, o0.double().cpu().numpy())   # the merge of the splits rounds in other places
        assert torch.allclose(l0, l1, atol=2e-3)
        if call != "attention":
            assert torch.equal(s0, s1) and torch.equal(k0, k1)


@pytest.mark.parametrize("H,d,n_keep,n_act", [
    (32, 128, 5, 16), (32, 128, 16, 9), (28, 128, 18, 16),   # three key splits, eight, nine
    (64, 64, 9, 16), (64, 64, 32, 13), (60, 64, 34, 16),     # five, sixteen, seventeen
    (40, 128, 12, 40),                                       # more rows than one query tile
])
def test_combine_of_few_splits(G, H, d, n_keep, n_act):
    """A wavefront or a workgroup merges the splits of a row: an empty split (ids outside the prompt), lse, rows past the count left alone."""
    M, B, N, cap = 4096, 64, 0, n_act + 2
    q, k, v = (_rand_bf16(171 + i, H, r, d).to(G.DEV) for i, r in enumerate((cap, M + N, M + N)))
    listed = np.arange(0, 64, 64 // n_keep)[:n_keep]
    listed[:2] = [-1, 64]                                    # the four sub-tiles of the first split
    out = torch.full((H, cap, d), 7.0, dtype=torch.bfloat16, device=G.DEV)
    lse = torch.full((H, cap), 9.0, device=G.DEV)
    s = fb.make_shape(q, k, v, M, B, out)
    buf = torch.full((fb.workspace_bytes(fb.FN_SPARSE_ATTN, s, cap, n_keep, 0),), 0xFF, dtype=torch.uint8, device=G.DEV)
    fb.sparse_attn(q, G.i32(np.arange(cap)), G.i32([1, n_act]), k, v, s, G.i32(listed), n_keep, None, 0, out, lse, buf)
    some, act = [0, H // 2, H - 1], np.arange(n_act)
    ref, ref_lse = fo.sparse_attention(G.to_np(q[some]), act, G.to_np(k[some]), G.to_np(v[some]), fo.attention_index_set([], listed[2:], M, B), M)
    G.assert_attention_close(out[some, :n_act], ref)
    assert np.allclose(lse[some, :n_act].cpu().numpy(), ref_lse, atol=2e-3)
    assert bool((out[:, n_act:] == 7).all()) and bool((lse[:, n_act:] == 9).all())


def test_sparse_attn_dense_reduction(G):
    # keep every block, every row a query: plain bidirectional attention over all M+N keys
    H, M, N, d, B, n_gen = 4, 3000, 72, 128, 128, 64
    n_b = -(-M // B)
    out, lse, ref, _ = _attn_case(G, H, M, N, d, B, n_gen, np.arange(n_gen), np.arange(n_b), [])
    G.assert_attention_close(out, ref)
    q, k, v = (_rand_bf16(11 + i, H, r, d).double() for i, r in enumerate((n_gen, M + N, M + N)))
    sdpa = torch.nn.functional.scaled_dot_product_attention(q, k, v).numpy()
    G.assert_attention_close(out, sdpa)


def test_sparse_attn_union_is_a_set(G):
    H, M, N, d, B, n_gen = 2, 1024, 32, 128, 64, 16
    active = np.arange(16)
    base = _attn_case(G, H, M, N, d, B, n_gen, active, [3, 9], [700, 5])[0]
    # sinks inside kept blocks, repeated sinks, out-of-range entries and -1 padding change nothing
    # (the split of the key axis differs with the list lengths, so equality holds up to the rounding of the merge)
    same, _, ref, _ = _attn_case(G, H, M, N, d, B, n_gen, active, [3, -1, 9, 16], [700, 5, 200, 600, 700, 5, -1, 5000])
    G.assert_attention_close(same, ref)
    assert (base.float() - same.float()).abs().max() <= 4e-3
    # order of the lists is irrelevant
    perm = _attn_case(G, H, M, N, d, B, n_gen, active, [9, 3], [5, 700])[0]
    assert (base.float() - perm.float()).abs().max() <= 4e-3


def test_sparse_attn_counts_and_untouched_rows(G):
    H, M, N, d, B, n_gen = 2, 512, 32, 64, 64, 32
    active = [1, 4, 6, 30, 31]
    canary = torch.full((H, 8, d), 123.0, dtype=torch.bfloat16, device=G.DEV)
    q, k, v = (_rand_bf16(21 + i, H, r, d).to(G.DEV) for i, r in enumerate((n_gen, M + N, M + N)))
    a_dev = G.i32(active + [7, 7, 7])                      # slots past counts[1] must be ignored
    out, lse = G.gpu_sparse_attn(q, a_dev, G.i32([0, 5]), k, v, M, B, G.i32([0, 5]), G.i32([100]), out=canary)
    I_p = fo.attention_index_set([100], [0, 5], M, B)
    ref, _ = fo.sparse_attention(G.to_np(q), active, G.to_np(k), G.to_np(v), I_p, M)
    G.assert_attention_close(out[:, :5], ref)
    assert (out[:, 5:] == 123.0).all()


def test_sparse_attn_empty_key_set(G):
    H, M, d = 2, 256, 64
    q, k, v = (_rand_bf16(31 + i, H, r, d).to(G.DEV) for i, r in enumerate((8, M, M)))
    out, lse = G.gpu_sparse_attn(q, G.i32([0, 1, 2]), None, k, v, M, 64, None, G.i32([-1, 9999]))
    assert (out == 0).all() and torch.isinf(lse).all() and (lse < 0).all()


def test_sparse_attn_single_key_returns_that_value_row(G):
    H, M, d = 2, 256, 128
    q, k, v = (_rand_bf16(41 + i, H, r, d).to(G.DEV) for i, r in enumerate((8, M, M)))
    out, _ = G.gpu_sparse_attn(q, G.i32([3, 5]), None, k, v, M, 64, None, G.i32([77]))
    assert torch.equal(out[:, 0], v[:, 77]) and torch.equal(out[:, 1], v[:, 77])


def test_sparse_attn_is_deterministic_and_linear_in_v(G):
    H, M, N, d, B, n_gen = 4, 2048, 64, 128, 128, 64
    q, k, v = (_rand_bf16(51 + i, H, r, d).to(G.DEV) for i, r in enumerate((n_gen, M + N, M + N)))
    args = (G.i32(np.arange(0, 64, 4)), None, k)
    o1, _ = G.gpu_sparse_attn(q, *args, v, M, B, G.i32([1, 7, 8]), G.i32([900, 1500]))
    o2, _ = G.gpu_sparse_attn(q, *args, v, M, B, G.i32([1, 7, 8]), G.i32([900, 1500]))
    assert torch.equal(o1, o2)
    o3, _ = G.gpu_sparse_attn(q, *args, (v.float() * 2).to(torch.bfloat16), M, B, G.i32([1, 7, 8]), G.i32([900, 1500]))
    assert torch.equal(o3.float(), o1.float() * 2)         # scaling by two is exact in bf16


@pytest.mark.parametrize("n_act", [16, 30, 50])
@pytest.mark.parametrize("ascending", [True, False])
def test_sparse_attn_many_sinks_inside_and_outside_kept_blocks(G, n_act, ascending):
    """Eq. 8 as a set with hundreds of sinks: about a third of them fall inside kept blocks and a few are listed twice;
    an ascending list (what focus_find_sinks writes) and a shuffled one must both be attended exactly once."""
    H, M, N, d, B, n_gen = 2, 8192, 48, 128, 64, 64
    rng = np.random.default_rng(1000 + n_act)
    n_b = M // B
    kept = np.sort(rng.choice(n_b, 40, replace=False))
    sinks = rng.choice(M, 200, replace=False)
    sinks = np.concatenate([sinks, sinks[:7]])                  # seven positions named twice
    sinks = np.sort(sinks) if ascending else rng.permutation(sinks)
    inside = np.isin(sinks // B, kept).sum()
    assert 30 < inside < 120
    active = np.sort(rng.choice(n_gen, n_act, replace=False))
    out, lse, ref, ref_lse = _attn_case(G, H, M, N, d, B, n_gen, active, kept, sinks, seed=70)
    G.assert_attention_close(out, ref)
    assert np.allclose(lse.cpu().numpy(), ref_lse, atol=2e-3)


@pytest.mark.parametrize("n_act", [16, 30])
@pytest.mark.parametrize("n_sink,n_keep", [(1, 0), (2, 3), (31, 70), (32, 70), (33, 70)])
@pytest.mark.parametrize("ascending", [True, False])
def test_sparse_attn_sink_lists_of_one_sub_tile(G, n_act, n_sink, n_keep, ascending):
    """Up to 32 sinks are one sub-tile, held in registers: inside and outside kept blocks, listed twice, out of range."""
    H, M, N, d, B, n_gen = 2, 8192, 48, 64, 64, 64
    rng = np.random.default_rng(n_sink)
    kept = np.sort(rng.choice(M // B, n_keep, replace=False))
    sinks = rng.choice(M, n_sink, replace=False)
    if n_sink > 4:
        sinks[:3] = sinks[4], M + 3, -1
        sinks[5] = kept[-1] * B + 7
    sinks = np.sort(sinks) if ascending else rng.permutation(sinks)
    out, lse, ref, ref_lse = _attn_case(G, H, M, N, d, B, n_gen, np.arange(n_act) * 2, kept, sinks, seed=90)
    G.assert_attention_close(out, ref)
    assert np.allclose(lse.cpu().numpy(), ref_lse, atol=2e-3)


@pytest.mark.parametrize("n_act", [9, 40])
def test_sparse_attn_unattended_rows_may_hold_inf_or_nan(G, n_act):
    """Rows outside I_p must not influence the result (Eq. 8, Eq. 9), whatever they hold: sink slots that hold no key
    (dropped, repeated or out-of-range entries, padding) and the clamped slots of ragged tiles read some row of K / V,
    and that row has to be one of the attended ones.  Every unattended row of K and V is filled with inf / NaN here."""
    H, M, N, d, B, n_gen = 2, 1000, 21, 128, 48, 48
    rng = np.random.default_rng(77 + n_act)
    kept = [2, 7, 20]                                            # block 20 is the ragged last block (rows 960..999)
    sinks = [5, 130, 131, 5, 2000, -1, 333, 98, 340]             # 130, 131, 98 and 340 lie in kept blocks; 5 twice; two invalid
    active = np.sort(rng.choice(n_gen, n_act, replace=False))
    q, k, v = (_rand_bf16(300 + i, H, r, d) for i, r in enumerate((n_gen, M + N, M + N)))
    I_p = fo.attention_index_set(sinks, kept, M, B)
    attended = np.zeros(M + N, bool)
    attended[I_p] = True
    attended[M:] = True
    ref, ref_lse = fo.sparse_attention(G.to_np(q), active, G.to_np(k), G.to_np(v), I_p, M)
    bad = torch.tensor(~attended)
    k[:, bad] = float("inf")
    v[:, bad] = float("nan")
    v[:, 0] = float("inf")                                       # row 0 is not attended
    assert not attended[0]
    out, lse = G.gpu_sparse_attn(q.to(G.DEV), G.i32(active), None, k.to(G.DEV), v.to(G.DEV), M, B, G.i32(kept), G.i32(sinks))
    G.assert_attention_close(out, ref)
    assert np.allclose(lse.cpu().numpy(), ref_lse, atol=2e-3)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("H,n_act,loop", [
    (2, 20, False), (2, 100, False),                             # one 32-query tile, several query groups: a sub-tile per slot
    (64, 16, True), (64, 20, True), (64, 40, True), (32, 100, True),   # one, one, two tiles and query groups: slots walk several sub-tiles
])
def test_sparse_attn_unattended_rows_may_hold_inf_or_nan_in_every_kernel(G, H, n_act, loop, d):
    """As above, for every tiling of the queries, with and without a key loop; a sink list of more than one sub-tile, unsorted, with
    entries in kept blocks, repeated, negative and past the prompt."""
    M, N, B, n_gen = 2500, 21, 48, 112
    n_b = -(-M // B)                                             # 53 blocks, the last one ragged (rows 2496 .. 2499)
    rng = np.random.default_rng(78 + n_act)
    kept = np.sort(rng.choice(n_b - 1, 29, replace=False)).tolist() + [n_b - 1]
    sinks = rng.permutation(np.concatenate([rng.choice(M, 36, replace=False), [kept[0] * B, -1, M, 7, 7, 2 * M]])).tolist()
    n_sub, per_head = 30 * 2 + 1 + 2, max(1, 512 // (H * (-(-n_act // 32) if n_act > 64 else 1)))
    assert (per_head * 4 < n_sub) == loop                        # the split plan: 512 workgroups, four sub-tiles each at a time
    active = np.sort(rng.choice(n_gen, n_act, replace=False))
    q, k, v = (_rand_bf16(320 + i, H, r, d) for i, r in enumerate((n_gen, M + N, M + N)))
    I_p = fo.attention_index_set(sinks, kept, M, B)
    attended = np.zeros(M + N, bool)
    attended[I_p] = True
    attended[M:] = True
    ref, ref_lse = fo.sparse_attention(G.to_np(q), active, G.to_np(k), G.to_np(v), I_p, M)
    bad = torch.tensor(~attended)
    k[:, bad] = float("inf")
    v[:, bad] = float("nan")
    out, lse = G.gpu_sparse_attn(q.to(G.DEV), G.i32(active), None, k.to(G.DEV), v.to(G.DEV), M, B, G.i32(kept), G.i32(sinks))
    G.assert_attention_close(out, ref)
    assert np.allclose(lse.cpu().numpy(), ref_lse, atol=2e-3)


@pytest.mark.parametrize("probe,H", [(False, 1 << 13), (True, 1 << 14)])
def test_more_query_groups_than_one_grid_axis_holds(G, probe, H):
    """2^24 workgroups of 256 threads (heads x query groups) do not fit the 2^32 threads of one grid axis.  All heads share Q, K, V and
    the output, where they write the same values; the log-sum-exps, and the column mass in the probe layer, tell whether all have run."""
    n_q, d, L = 1 << 16, 64, 1
    q, k, v = (_rand_bf16(310 + i, 1, r, d).to(G.DEV).expand(H, r, d) for i, r in enumerate((n_q, L, L)))
    store = torch.full((1, n_q, d), float("nan"), dtype=torch.bfloat16, device=G.DEV)
    out, lse = store.expand(H, n_q, d), torch.full((H, n_q), float("nan"), device=G.DEV)
    s = fb.make_shape(q, k, v, L, 64, out)
    active, one, col = torch.arange(n_q, dtype=torch.int32, device=G.DEV), G.i32([0]), torch.full((L,), float("nan"), device=G.DEV)
    w = G.ws(fb.workspace_bytes(fb.FN_PROBE_LAYER if probe else fb.FN_SPARSE_ATTN, s, n_q, 1, 0))
    if probe:
        sinks = G.i32(None, 1)
        fb.probe_layer(q, active, None, k, v, s, 1, out, lse, col, sinks, w)
        assert col.item() == 1.0 and sinks.item() == 0                  # sums of powers of two
    else:
        fb.sparse_attn(q, active, None, k, v, s, one, 1, None, 0, out, lse, w)
    torch.cuda.synchronize()
    assert torch.equal(store[0], v[0].expand(n_q, d))                   # one key
    ref = torch.matmul(q[0].double(), k[0, 0].double()) / math.sqrt(d)
    assert torch.allclose(lse[0].double(), ref, atol=1e-5)
    for h in range(0, H, 1 << 10):
        assert torch.equal(lse[h:h + (1 << 10)], lse[:1].expand(1 << 10, n_q))


# ------------------------------------------------------------------------------------------------ probe layer
@pytest.mark.parametrize("H,M,N,d,B,n_gen,n_act,n_sink", [
    (4, 1024, 32, 64, 64, 32, 8, 2),          # the tiny shape: a single key split
    (3, 2050, 33, 128, 128, 80, 16, 4),       # 16 queries: logits kept from the attention pass
    (2, 8192, 64, 128, 128, 64, 16, 20),      # several splits, radix Top-N
    (2, 4100, 30, 128, 64, 64, 28, 7),        # two query tiles: column sums from a second pass over K
    (2, 3000, 0, 64, 64, 96, 72, 41),         # five query tiles (two groups), d = 64, no response rows
    (3, 96, 33, 128, 32, 32, 16, 4),          # five sub-tiles, the fewest that one workgroup of eight wavefronts takes
    (2, 256, 0, 128, 64, 64, 5, 3),           # eight, the most at d = 128
    (2, 224, 33, 128, 32, 40, 16, 2),         # nine
    (40, 128, 1, 64, 32, 64, 14, 1),          # d = 64: five
    (3, 320, 30, 64, 64, 64, 9, 3),           # eleven, for twelve wavefronts
    (2, 480, 20, 64, 32, 40, 14, 2),          # sixteen, the most
    (2, 512, 20, 64, 32, 40, 14, 2),          # seventeen
])
def test_probe_layer(G, H, M, N, d, B, n_gen, n_act, n_sink):
    """Dense attention of the active queries over every key plus the sinks it implies, in one call: the attention equals
    focus_sparse_attn with every block kept (bit for bit when the tiles coincide), the column masses and sinks match
    the oracle (and focus_find_sinks to rounding)."""
    q, k, v = (_rand_bf16(81 + i, H, r, d).to(G.DEV) for i, r in enumerate((n_gen, M + N, M + N)))
    act = np.sort(np.random.default_rng(84).choice(n_gen, n_act, replace=False))
    cap = n_act + 2
    active, counts = G.i32(list(act) + [-1] * (cap - n_act)), G.i32([0, n_act])
    out, lse, col, sinks = G.gpu_probe_layer(q, active, counts, k, v, M, B, n_sink)
    n_b = -(-M // B)
    out_d, lse_d = G.gpu_sparse_attn(q, active, counts, k, v, M, B, G.i32(np.arange(n_b)), None)
    if M % B == 0 and B % 32 == 0:     # the 32-row tiles of both paths coincide: same arithmetic in the same order
        assert torch.equal(out[:, :n_act], out_d[:, :n_act]) and torch.equal(lse[:, :n_act], lse_d[:, :n_act])
    else:                              # the dense path tiles the key axis without regard to block boundaries
        assert np.allclose(G.to_np(out[:, :n_act]), G.to_np(out_d[:, :n_act]), atol=2e-3)
        assert np.allclose(lse[:, :n_act].cpu().numpy(), lse_d[:, :n_act].cpu().numpy(), atol=1e-5)
    Q, K, V = G.to_np(q), G.to_np(k), G.to_np(v)
    ref, ref_lse = fo.sparse_attention(Q, act, K, V, np.arange(M), M)
    G.assert_attention_close(out[:, :n_act], ref)
    assert np.allclose(lse[:, :n_act].cpu().numpy(), ref_lse, atol=2e-3)
    Sref = fo.sink_scores(Q, act, K)
    S = col.cpu().numpy().astype(np.float64)
    assert np.allclose(S, Sref, rtol=2e-4, atol=1e-9) and S.sum() == pytest.approx(1.0, abs=1e-4)
    assert fo.decision_margin(Sref, n_sink, np.arange(M + N) < M) > 1e-5, "test inputs produce a near-tie; pick another seed"
    assert sinks.cpu().tolist() == fo.select_sinks(Sref, M, n_sink).tolist()
    assert sinks.cpu().tolist() == fo.select_sinks(S, M, n_sink).tolist()
    col2, sinks2 = G.gpu_find_sinks(q, active, counts, k, M, B, n_sink)
    assert np.allclose(col2.cpu().numpy(), S, rtol=1e-5, atol=1e-12) and torch.equal(sinks, sinks2)


# ------------------------------------------------------------------------------------------------ fused layer call
@pytest.mark.parametrize("H,M,N,d,B,n_gen,n_f,n_act,n_keep,n_sink", [
    (4, 1024, 32, 64, 64, 32, 8, 8, 4, 2),
    (8, 4096, 64, 128, 128, 64, 16, 16, 5, 4),        # 32 blocks, several splits per head
    (3, 3000, 40, 128, 48, 48, 5, 40, 9, 7),          # ragged, three query tiles
    (2, 16384, 64, 128, 64, 64, 16, 16, 25, 4),       # exactly 256 blocks: the most with one key per thread of the ranking
    (2, 8192, 64, 128, 16, 64, 16, 16, 40, 4),        # 512 blocks
    (2, 16385, 64, 64, 64, 64, 16, 16, 30, 4),        # one block more than a workgroup has threads
    (2, 8208, 0, 64, 16, 64, 4, 50, 257, 40),         # 513 blocks, two query tiles per slot
    (1, 16384, 64, 128, 16, 64, 4, 20, 1024, 5),      # the most blocks with four keys per thread of the ranking, all kept
    (5, 16384, 7, 64, 16, 64, 9, 30, 500, 90),
    (2, 16400, 64, 64, 16, 64, 9, 30, 11, 3),         # ... and one more
    (2, 2048, 0, 64, 128, 16, 3, 16, 16, 0),          # every block kept, no response rows, no sinks
    (4, 4096, 64, 128, 64, 64, 8, 28, 20, 6),         # two query tiles per workgroup, Top-C inside the kernel
    (4, 2048, 32, 64, 32, 80, 8, 72, 30, 40),         # five query tiles (two groups of four), d = 64, unsorted sinks
    (3, 1500, 10, 64, 50, 40, 4, 20, 12, 33),         # two query tiles, d = 64, ragged blocks
    (2, 16384, 64, 128, 64, 64, 4, 36, 128, 163),     # the paper's proportions at 16K: half the blocks, 1 % sinks
    (32, 4096, 64, 64, 16, 64, 16, 16, 64, 4),        # d = 64, 256 blocks: 17 splits of four sub-tiles
    (16, 4096, 30, 64, 16, 64, 8, 16, 250, 4),        # 63 splits
    (32, 16384, 64, 64, 16, 64, 4, 16, 125, 4),       # 1024 blocks: 32 splits; the list lies over the histograms, as in the next three
    (32, 4112, 64, 64, 16, 64, 16, 9, 94, 40),        # 257 blocks, 25 splits, two sub-tiles of sinks
    (32, 32768, 33, 64, 16, 64, 8, 11, 124, 3),       # 2048 blocks: 32 splits
    (3, 32768, 5, 64, 16, 64, 5, 16, 2048, 35),       # all of them kept: the whole place is in use, key loop
    (37, 1000, 8, 128, 64, 100, 90, 10, 5, 3),        # more than eight groups of heads, more than 64 focus rows
    (33, 2000, 8, 64, 64, 100, 33, 40, 5, 3),
])
def test_sparse_layer_equals_block_scores_then_sparse_attn(G, H, M, N, d, B, n_gen, n_f, n_act, n_keep, n_sink):
    rng = np.random.default_rng(M + n_keep)
    q, k, v = (_rand_bf16(61 + i, H, r, d).to(G.DEV) for i, r in enumerate((n_gen, M + N, M + N)))
    focus = G.i32(np.sort(rng.choice(n_gen, n_f, replace=False)))
    active = G.i32(np.sort(rng.choice(n_gen, n_act, replace=False)))
    sinks = G.i32(rng.choice(M, n_sink, replace=False)) if n_sink else None
    counts = G.i32([n_f, n_act])
    scores, kept = G.gpu_block_scores(q, focus, counts, k, None, M, B, n_keep)
    out, lse = G.gpu_sparse_attn(q, active, counts, k, v, M, B, kept, sinks)
    for kbar in (None, G.gpu_block_means(k, M, B)):
        for _ in range(2):                                  # twice: arrival counters must be reusable
            s2, k2, o2, l2 = G.gpu_sparse_layer(q, focus, active, counts, k, v, kbar, M, B, n_keep, sinks)
            assert torch.equal(s2, scores) and torch.equal(k2, kept)
            assert torch.equal(o2, out) and torch.equal(l2, lse)
    # and against the oracle
    lay = fo.focus_layer(G.to_np(q), G.to_np(k), G.to_np(v), focus.cpu().numpy(), active.cpu().numpy(),
                         [] if sinks is None else sinks.cpu().numpy(), M, B, n_keep)
    assert kept.cpu().tolist() == lay["blocks"].tolist()
    G.assert_attention_close(out, lay["out"])


@pytest.mark.parametrize("H,M,N,d,B,n_act,n_keep,n_sink", [
    (2, 1025, 64, 128, 1, 16, 30, 4),       # one block more than four keys per thread
    (9, 32768, 33, 64, 16, 16, 7, 3),       # 2048 blocks, the most; two groups of heads, one with one head
    (2, 2048, 5, 64, 1, 40, 2048, 0),       # ... all kept, two query tiles of 32
    (3, 24001, 40, 128, 16, 24, 900, 240),  # 1501 blocks, one tile of 32, a key loop
    (40, 1700, 16, 128, 1, 16, 1600, 17),   # ten groups of heads: more parts than are requested first
    (2, 1100, 16, 64, 1, 70, 300, 33),      # several query groups
    (2, 2049, 64, 128, 1, 16, 30, 4),       # one more than the most: a launch ranks them
])
def test_sparse_layer_of_many_blocks(G, H, M, N, d, B, n_act, n_keep, n_sink):
    """Ranked inside the attention kernel or, with the least workspace, by a launch of its own: the same as the separate calls."""
    rng, n_gen = np.random.default_rng(M), 80
    q, k, v = (_rand_bf16(91 + i, H, r, d).to(G.DEV) for i, r in enumerate((n_gen, M + N, M + N)))
    k[:, 3 * B:4 * B] = k[:, 7 * B:8 * B]                   # equal relevances: ties go to the lower block
    focus, active = (G.i32(np.sort(rng.choice(n_gen, n, replace=False))) for n in (9, n_act))
    sinks = G.i32(rng.choice(M, n_sink, replace=False)) if n_sink else None
    counts = G.i32([9, n_act])
    scores, kept = G.gpu_block_scores(q, focus, counts, k, None, M, B, n_keep)
    out, lse = G.gpu_sparse_attn(q, active, counts, k, v, M, B, kept, sinks)
    kbar = G.gpu_block_means(k, M, B)
    o2 = torch.empty_like(out)
    s = fb.make_shape(q, k, v, M, B, o2)
    least = max(fb.workspace_bytes(fb.FN_BLOCK_SCORES, s), fb.workspace_bytes(fb.FN_SPARSE_ATTN, s, n_act, n_keep, n_sink))
    full = fb.workspace_bytes(fb.FN_SPARSE_LAYER, s, n_act, n_keep, n_sink)
    assert full >= least
    for nbytes in (full, least, full):
        s2, k2, l2 = torch.full_like(scores, -1.0), torch.full_like(kept, -9), torch.empty_like(lse)
        o2.fill_(7.0)
        fb.sparse_layer(q, focus, active, counts, k, v, kbar, s, n_keep, sinks, n_sink, s2, k2, o2, l2, G.ws(nbytes))
        torch.cuda.synchronize()
        assert torch.equal(s2, scores) and torch.equal(k2, kept)
        assert torch.equal(o2, out) and torch.equal(l2, lse)
    for nbytes in (full, least, full):                      # the relevances from a scan of K: per head, added up by groups of four in between
        s2, k2, l2 = torch.full_like(scores, -1.0), torch.full_like(kept, -9), torch.empty_like(lse)
        o2.fill_(7.0)
        fb.sparse_layer(q, focus, active, counts, k, v, None, s, n_keep, sinks, n_sink, s2, k2, o2, l2, G.ws(nbytes))
        torch.cuda.synchronize()
        assert torch.equal(s2, scores) and torch.equal(k2, kept)
        assert torch.equal(o2, out) and torch.equal(l2, lse)


@pytest.mark.parametrize("H,M,N,B,n_keep,splits", [
    (32, 4096, 0, 32, 128, 8),    # 32 splits with the full workspace; with the least a key loop in 8
    (32, 4096, 64, 64, 32, 8),    # 17, and a key loop in 8
    (16, 8192, 1, 32, 256, 16),   # a key loop in 32 and in 16
    (300, 256, 0, 32, 8, 1),      # 2, and a key loop in one: no workspace at all
])
def test_least_workspace_of_64_columns(G, H, M, N, B, n_keep, splits):
    """d = 64, up to 16 queries: the workspace of fewer key splits is taken, too, one byte less is not, and nothing is written past it."""
    d, n_act = 64, 11
    q, k, v = (_rand_bf16(121 + i, H, r, d).to(G.DEV) for i, r in enumerate((16, M + N, M + N)))
    focus, active, counts = G.i32(np.arange(4)), G.i32(np.arange(16)), G.i32([4, n_act])
    up = lambda x: (x + 255) // 256 * 256
    least = up(H * 16 * splits * d * 4) + up(H * 16 * splits * 8) if splits > 1 else 0
    kbar = G.gpu_block_means(k, M, B)
    scores, kept = G.gpu_block_scores(q, focus, counts, k, kbar, M, B, n_keep)
    out = torch.empty((H, 16, d), dtype=torch.bfloat16, device=G.DEV)
    s = fb.make_shape(q, k, v, M, B, out)
    assert fb.workspace_bytes(fb.FN_SPARSE_ATTN, s, 16, n_keep, 0) > max(least, 256)
    rows = np.concatenate([np.arange(b * B, min((b + 1) * B, M)) for b in kept.tolist()])
    ref, ref_lse = fo.sparse_attention(G.to_np(q), np.arange(n_act), G.to_np(k), G.to_np(v), rows, M)
    extra = fb.workspace_bytes(fb.FN_BLOCK_SCORES, s)
    for layer, nbytes in ((False, least), (True, extra + max(least, 256))):
        buf = torch.full((nbytes + 4096,), 0x5B, dtype=torch.uint8, device=G.DEV)
        lse, s2, k2 = torch.full((H, 16), 9.0, device=G.DEV), torch.empty_like(scores), torch.empty_like(kept)

        def call(w):
            if layer:
                fb.sparse_layer(q, focus, active, counts, k, v, kbar, s, n_keep, None, 0, s2, k2, out, lse, w)
            else:
                fb.sparse_attn(q, active, counts, k, v, s, kept, n_keep, None, 0, out, lse, w if nbytes else None)
        out.fill_(7.0)
        call(buf[:nbytes])
        torch.cuda.synchronize()
        assert bool((buf[nbytes:] == 0x5B).all())
        assert not layer or (torch.equal(s2, scores) and torch.equal(k2, kept))
        G.assert_attention_close(out[:, :n_act], ref)
        assert np.allclose(lse[:, :n_act].cpu().numpy(), ref_lse, atol=2e-3)
        if nbytes:
            with pytest.raises(fb.FocusError):
                call(buf[:nbytes - 1])


# ------------------------------------------------------------------------------------------------ whole layer on the workloads
@pytest.mark.parametrize("name", ["tiny", "ctx8k", "ctx16k", "ctx32k", "paper32k", "paper32k_gen256", "ctx128k"])
def test_workload_layer_end_to_end(G, name):
    w = fi.WORKLOADS[name]
    # one realised tensor feeds both sides: generated on the host and uploaded, except for the 128K context, whose
    # 1.6 G elements are generated on the device and downloaded for the oracle
    q, k, v = (t.to(G.DEV) for t in fi.layer_qkv(w, 0, device=G.DEV if name == "ctx128k" else "cpu"))
    conf = fi.confidence(w)
    Q, K, V = G.to_np(q), G.to_np(k), G.to_np(v)
    # oracle
    focus_ref = fo.select_focus(conf.numpy(), None, w.k_focus)
    active_ref = fo.expand_window(focus_ref, w.window, 0, w.n_gen)
    S_ref = fo.sink_scores(Q, active_ref, K)
    sinks_ref = fo.select_sinks(S_ref, w.n_ctx, w.n_sink)
    lay = fo.focus_layer(Q, K, V, focus_ref, active_ref, sinks_ref, w.n_ctx, w.block, w.n_keep)
    # index parity is only well posed away from near-ties; fp32 reordering noise is below 1e-6 of the score spread
    min_margin = 1e-5 if name.startswith("paper32k") else 1e-4      # selecting hundreds of items leaves smaller gaps
    assert fo.decision_margin(S_ref, w.n_sink, np.arange(w.n_kv) < w.n_ctx) > min_margin
    assert fo.decision_margin(lay["R"], w.n_keep) > min_margin
    # device, chained without host round trips of the index sets
    focus, active, counts = G.gpu_select(conf.numpy(), fi.masked_all(w).numpy(), w.k_focus, w.window, 0, w.n_gen)
    col, sinks = G.gpu_find_sinks(q, active, counts, k, w.n_ctx, w.block, w.n_sink)
    scores, kept = G.gpu_block_scores(q, focus, counts, k, None, w.n_ctx, w.block, w.n_keep)
    out, lse = G.gpu_sparse_attn(q, active, counts, k, v, w.n_ctx, w.block, kept, sinks)
    n_q = len(active_ref)
    assert counts.cpu().tolist() == [len(focus_ref), n_q]
    assert focus.cpu().tolist() == focus_ref.tolist()
    assert active.cpu().tolist() == active_ref.tolist() + [-1] * (active.numel() - n_q)
    assert sinks.cpu().tolist() == sinks_ref.tolist()
    assert kept.cpu().tolist() == lay["blocks"].tolist()
    assert np.allclose(col.cpu().numpy(), S_ref, rtol=2e-4, atol=1e-10)
    assert np.allclose(scores.cpu().numpy(), lay["R"], atol=2e-6)
    G.assert_attention_close(out[:, :n_q], lay["out"])
    assert np.allclose(lse.cpu().numpy()[:, :n_q], lay["lse"], atol=2e-3)
    # the fused per-layer call gives the same bits as the two separate calls
    s2, k2, o2, _ = G.gpu_sparse_layer(q, focus, active, counts, k, v, None, w.n_ctx, w.block, w.n_keep, sinks)
    assert torch.equal(s2, scores) and torch.equal(k2, kept) and torch.equal(o2[:, :n_q], out[:, :n_q])
    # dense comparison baseline through the same entry point: every block kept
    n_b = w.n_blocks
    dense, _ = G.gpu_sparse_attn(q, active, counts, k, v, w.n_ctx, w.block, G.i32(np.arange(n_b)), None)
    I_all = fo.attention_index_set([], np.arange(n_b), w.n_ctx, w.block)
    G.assert_attention_close(dense[:, :n_q], fo.sparse_attention(Q, active_ref, K, V, I_all, w.n_ctx)[0])


def test_stack_reuses_probe_layer_sinks(G):
    # a short stack shaped like the tiny workload: sinks found at layer 1 are handed, as the same device buffer, to layers 2..4
    w = fi.strong_sinks(fi.TINY).with_(n_layers=5, probe_layer=1, first_sparse_layer=2)
    conf = fi.confidence(w)
    tensors = {l: tuple(t.to(G.DEV) for t in fi.layer_qkv(w, l)) for l in range(w.n_layers)}
    step = fo.focus_step(conf.numpy(), None, w.k_focus, w.window, 0, w.n_gen,
                         lambda l: tuple(G.to_np(t) for t in tensors[l]), w.probe_layer, range(2, 5), w.n_ctx, w.block,
                         w.n_keep, w.n_sink)
    assert step["sinks"].tolist() == list(w.sink_positions)          # the planted keys are the sinks
    focus, active, counts = G.gpu_select(conf.numpy(), None, w.k_focus, w.window, 0, w.n_gen)
    qp, kp, _ = tensors[w.probe_layer]
    _, sinks = G.gpu_find_sinks(qp, active, counts, kp, w.n_ctx, w.block, w.n_sink)
    frozen = sinks.clone()
    assert sinks.cpu().tolist() == step["sinks"].tolist()
    for l in range(2, 5):
        q, k, v = tensors[l]
        _, kept = G.gpu_block_scores(q, focus, counts, k, None, w.n_ctx, w.block, w.n_keep)
        out, _ = G.gpu_sparse_attn(q, active, counts, k, v, w.n_ctx, w.block, kept, sinks)
        assert torch.equal(sinks, frozen)                              # reused unchanged
        assert kept.cpu().tolist() == step["layers"][l]["blocks"].tolist()
        G.assert_attention_close(out, step["layers"][l]["out"])


def test_stack32k_full_size_step_against_the_oracle(G):
    """The 32-layer, 32K-context workload at full size, as bench.py times it: block means from the block-entry cache
    refresh, query selection, sinks at layer 16, then layers 17..31 through focus_sparse_layer with those cached means.
    Every layer's kept blocks bit-exact and output within tolerance of oracle.focus_step; the sink buffer is the same
    after every layer; one HIP-graph replay of the whole step reproduces the eager bits."""
    from paper_2602_02159_amd.step import FocusStep
    w = fi.STACK32K
    sparse_ids = list(range(w.first_sparse_layer, w.n_layers))
    conf, masked = fi.confidence(w, G.DEV), fi.masked_all(w, G.DEV)
    probe = fi.layer_qkv(w, w.probe_layer, G.DEV, which="qkv")
    layers, kbars = [], []
    for l in sparse_ids:                                         # block entry of layer l: cache and block means in one pass
        q, k_new, v_new = fi.layer_qkv(w, l, G.DEV)
        k_cache, v_cache = torch.empty_like(k_new), torch.empty_like(v_new)
        kbar = torch.empty(w.n_heads, w.n_blocks, w.head_dim, dtype=torch.float32, device=G.DEV)
        fb.cache_refresh(k_cache, v_cache, fb.make_shape(q, k_cache, v_cache, w.n_ctx, w.block), k_new, v_new, kbar)
        torch.cuda.synchronize()
        assert torch.equal(k_cache, k_new) and torch.equal(v_cache, v_new)
        del k_new, v_new
        layers.append((q, k_cache, v_cache))
        kbars.append(kbar)
    st = FocusStep(conf, masked, probe, layers, w.n_ctx, w.block, w.k_focus, w.window, w.n_keep, w.n_sink, cached_means=True,
                   kbars=kbars)
    # eager, one call at a time
    st.issue("select")
    st.issue("find_sinks")
    torch.cuda.synchronize()
    frozen = st.sink_idx.clone()
    for i in range(len(layers)):
        st.issue("sparse_layer_cached", i)
        torch.cuda.synchronize()
        assert torch.equal(st.sink_idx, frozen)                  # handed on unchanged (cross-layer reuse)
    # oracle, one layer's tensors on the host at a time
    tensors = {w.probe_layer: probe}
    tensors.update({l: t for l, t in zip(sparse_ids, layers)})
    ref = fo.focus_step(conf.cpu().numpy(), None, w.k_focus, w.window, 0, w.n_gen, lambda l: tuple(G.to_np(t) for t in tensors[l]),
                        w.probe_layer, sparse_ids, w.n_ctx, w.block, w.n_keep, w.n_sink)
    n_q = len(ref["active"])
    assert st.counts.cpu().tolist() == [len(ref["focus"]), n_q]
    assert st.focus_idx.cpu().tolist() == ref["focus"].tolist() and st.active_idx.cpu().tolist()[:n_q] == ref["active"].tolist()
    assert fo.decision_margin(ref["S"], w.n_sink, np.arange(w.n_kv) < w.n_ctx) > 1e-4
    assert frozen.cpu().tolist() == ref["sinks"].tolist()
    for i, l in enumerate(sparse_ids):
        lay = ref["layers"][l]
        assert fo.decision_margin(lay["R"], w.n_keep) > 1e-4
        assert st.bufs[i]["kept"].cpu().tolist() == lay["blocks"].tolist(), f"layer {l}"
        assert np.allclose(st.bufs[i]["scores"].cpu().numpy(), lay["R"], atol=2e-6)
        G.assert_attention_close(st.bufs[i]["out"][:, :n_q], lay["out"])
    # the whole step as one graph, outputs wiped first
    eager = [(b["out"].clone(), b["kept"].clone()) for b in st.bufs]
    st.capture()
    for b in st.bufs:
        b["out"].zero_()
        b["kept"].fill_(-3)
    st.sink_idx.fill_(-3)
    torch.cuda.synchronize()
    st.run()
    torch.cuda.synchronize()
    assert torch.equal(st.sink_idx, frozen)
    assert all(torch.equal(o, b["out"]) and torch.equal(kp, b["kept"]) for (o, kp), b in zip(eager, st.bufs))


def test_step_driver_graph_with_confidence_probe_layer_and_dense_tail(G):
    """The whole step as the driver sequences it and a HIP graph replays it: confidence from logits, query selection,
    the probe layer's dense attention with the sinks as a by-product, sparse layers, and a dense last layer."""
    from paper_2602_02159_amd.step import FocusStep
    w = fi.strong_sinks(fi.TINY).with_(n_layers=5, probe_layer=1, first_sparse_layer=2, window=2)
    tensors = {l: tuple(t.to(G.DEV) for t in fi.layer_qkv(w, l)) for l in range(w.n_layers)}
    vocab = 5003
    g = torch.Generator().manual_seed(123)
    logits = (torch.randn(w.n_gen, vocab + 5, generator=g) * 2.5).to(torch.bfloat16).to(G.DEV)[:, :vocab]
    masked = (torch.arange(w.n_gen) % 5 != 0).to(torch.uint8)
    conf = torch.zeros(w.n_gen, dtype=torch.float32, device=G.DEV)
    st = FocusStep(conf, masked.to(G.DEV), tensors[w.probe_layer], [tensors[l] for l in (2, 3, 4)], w.n_ctx, w.block,
                   w.k_focus, w.window, w.n_keep, w.n_sink, logits=logits, dense_tail=1)
    st.use_probe_layer = True
    # oracle
    tok_ref, conf_ref = fo.token_confidence(G.to_np(logits), masked.numpy())
    focus_ref = fo.select_focus(conf_ref.astype(np.float32), masked.numpy(), w.k_focus)
    active_ref = fo.expand_window(focus_ref, w.window, 0, w.n_gen)
    np_l = {l: tuple(G.to_np(t) for t in tensors[l]) for l in tensors}
    Qp, Kp, Vp = np_l[w.probe_layer]
    sinks_ref = fo.select_sinks(fo.sink_scores(Qp, active_ref, Kp), w.n_ctx, w.n_sink)
    probe_ref, _ = fo.sparse_attention(Qp, active_ref, Kp, Vp, np.arange(w.n_ctx), w.n_ctx)
    lay_ref = [fo.focus_layer(*np_l[l], focus_ref, active_ref, sinks_ref, w.n_ctx, w.block, w.n_keep) for l in (2, 3)]
    dense_ref, _ = fo.sparse_attention(*np_l[4][:1], active_ref, *np_l[4][1:], np.arange(w.n_ctx), w.n_ctx)

    def check():
        n_a = len(active_ref)
        assert st.tokens.cpu().tolist() == tok_ref.tolist()
        assert np.allclose(st.conf.cpu().numpy(), conf_ref, rtol=2e-5)
        assert st.counts.cpu().tolist() == [len(focus_ref), n_a]
        assert st.focus_idx.cpu().tolist()[:len(focus_ref)] == focus_ref.tolist()
        assert st.active_idx.cpu().tolist()[:n_a] == active_ref.tolist()
        assert st.sink_idx.cpu().tolist() == sinks_ref.tolist() == list(w.sink_positions)
        G.assert_attention_close(st.probe_out[:, :n_a], probe_ref)
        for i in range(2):
            assert st.bufs[i]["kept"].cpu().tolist() == lay_ref[i]["blocks"].tolist()
            G.assert_attention_close(st.bufs[i]["out"][:, :n_a], lay_ref[i]["out"])
        G.assert_attention_close(st.bufs[2]["out"][:, :n_a], dense_ref)

    st.run()
    torch.cuda.synchronize()
    check()
    eager = [b["out"].clone() for b in st.bufs]
    st.capture()
    for _ in range(3):                                   # replays, with the buffers wiped in between
        for b in st.bufs:
            b["out"].zero_()
        st.conf.zero_()
        st.sink_idx.fill_(-3)
        torch.cuda.synchronize()
        st.run()
        torch.cuda.synchronize()
        check()
        assert all(torch.equal(a, b["out"]) for a, b in zip(eager, st.bufs))


@pytest.mark.parametrize("n_act,n_sink,n_keep", [(16, 4, 7), (28, 60, 40), (64, 327, 128), (112, 20, 16)])
def test_results_are_bit_identical_from_run_to_run(G, n_act, n_sink, n_keep):
    """Nothing in the path depends on the order in which workgroups or atomics happen to land: twelve runs of the probe
    layer and the fused sparse layer (one, two and four query tiles per workgroup, several query groups) give the same
    bits every time."""
    H, M, N, d, B, n_gen = 8, 16384, 64, 128, 64, 128
    q, k, v = (_rand_bf16(211 + i, H, r, d).to(G.DEV) for i, r in enumerate((n_gen, M + N, M + N)))
    rng = np.random.default_rng(n_act)
    active = np.sort(rng.choice(n_gen, n_act, replace=False))
    focus = active[:: max(1, n_act // 8)]
    a_dev, f_dev, counts = G.i32(list(active)), G.i32(list(focus)), G.i32([len(focus), n_act])
    first = None
    for _ in range(12):
        out_p, lse_p, col, sinks = G.gpu_probe_layer(q, a_dev, counts, k, v, M, B, n_sink)
        scores, kept, out, lse = G.gpu_sparse_layer(q, f_dev, a_dev, counts, k, v, None, M, B, n_keep, sinks)
        got = [t.clone() for t in (out_p[:, :n_act], lse_p[:, :n_act], col, sinks, scores, kept, out[:, :n_act], lse[:, :n_act])]
        if first is None:
            first = got
        else:
            assert all(torch.equal(a, b) for a, b in zip(first, got))


# ------------------------------------------------------------------------------------------------ randomized shapes
def _random_configs(n, seed):
    rng = np.random.default_rng(seed)
    out = []
    for _ in range(n):
        d = int(rng.choice([64, 128]))
        H = int(rng.choice([1, 2, 3, 5]))
        M = int(rng.integers(33, 3000))
        N = int(rng.integers(0, 100))
        B = int(rng.choice([16, 32, 48, 64, 100, 128]))
        n_gen = int(rng.integers(1, 131))
        n_act = int(rng.integers(1, min(n_gen, 80) + 1))
        n_b = -(-M // B)
        n_keep = int(rng.integers(0, n_b + 1)) if rng.random() < 0.3 else int(rng.integers(0, min(n_b, 12) + 1))
        n_sink = int(rng.integers(0, min(M, 40) + 1))
        out.append((H, M, N, d, B, n_gen, n_act, n_keep, n_sink))
    return out


@pytest.mark.parametrize("cfg", _random_configs(64, 20260301), ids=lambda c: "-".join(map(str, c)))
def test_randomized_shapes_against_the_oracle(G, cfg):
    """Seeded random shapes (ragged everything, every query-tile count, zero kept blocks or sinks now and then): block
    scores, sink scores and the attention over a random kept set, each against the oracle."""
    H, M, N, d, B, n_gen, n_act, n_keep, n_sink = cfg
    rng = np.random.default_rng(sum(cfg))
    n_b = -(-M // B)
    q, k, v = (_rand_bf16(161 + i, H, r, d).to(G.DEV) for i, r in enumerate((n_gen, M + N, M + N)))
    Q, K, V = G.to_np(q), G.to_np(k), G.to_np(v)
    active = np.sort(rng.choice(n_gen, n_act, replace=False))
    focus = np.sort(rng.choice(active, max(1, n_act // 2), replace=False))
    pad = min(2, n_gen - n_act)    # the capacity of the active list may not exceed n_gen
    a_dev, f_dev = G.i32(list(active) + [-1] * pad), G.i32(list(focus) + [-1])
    counts = G.i32([len(focus), n_act])
    # block scores (values always; the Top-C only where no decision is a near-tie)
    R_ref = fo.block_relevance(Q, focus, fo.block_means(K, M, B))
    scores, kept_dev = G.gpu_block_scores(q, f_dev, counts, k, None, M, B, n_keep)
    assert np.allclose(scores.cpu().numpy(), R_ref, atol=2e-6 * max(1.0, np.abs(R_ref).max()))
    if 0 < n_keep < n_b and fo.decision_margin(R_ref, n_keep) > 1e-4:
        assert kept_dev.cpu().tolist() == fo.top_indices(R_ref, n_keep).tolist()
    # sink scores
    S_ref = fo.sink_scores(Q, active, K)
    col, sinks_dev = G.gpu_find_sinks(q, a_dev, counts, k, M, B, n_sink)
    assert np.allclose(col.cpu().numpy(), S_ref, rtol=2e-4, atol=1e-9)
    if 0 < n_sink < M and fo.decision_margin(S_ref, n_sink, np.arange(M + N) < M) > 1e-4:
        assert sinks_dev.cpu().tolist() == fo.select_sinks(S_ref, M, n_sink).tolist()
    # attention over a random kept set and random sinks (unsorted, with a repeat)
    kept = rng.choice(n_b, n_keep, replace=False) if n_keep else np.zeros(0, dtype=np.int64)
    sinks = rng.choice(M, n_sink, replace=False) if n_sink else np.zeros(0, dtype=np.int64)
    if n_sink > 1:
        sinks = np.concatenate([sinks, sinks[:1]])
    out, lse = G.gpu_sparse_attn(q, a_dev, counts, k, v, M, B, G.i32(kept) if len(kept) else None, G.i32(sinks) if len(sinks) else None)
    I_p = fo.attention_index_set(sinks, kept, M, B)
    if len(I_p) + N == 0:
        return   # nothing to attend to: covered by the dedicated empty-set test
    ref, ref_lse = fo.sparse_attention(Q, active, K, V, I_p, M)
    G.assert_attention_close(out[:, :n_act], ref)
    assert np.allclose(lse.cpu().numpy()[:, :n_act], ref_lse, atol=2e-3)


@pytest.mark.parametrize("cfg", _random_configs(32, 20260302), ids=lambda c: "-".join(map(str, c)))
def test_randomized_shapes_fused_layer_probe_layer_and_block_entry(G, cfg):
    """The same kind of seeded shapes through the fused calls: focus_sparse_layer against the oracle's layer (and bit
    for bit against the separate calls), focus_probe_layer against the oracle's dense attention and sinks, and the two
    block-entry calls against the oracle."""
    H, M, N, d, B, n_gen, n_act, n_keep, n_sink = cfg
    rng = np.random.default_rng(sum(cfg) + 1)
    n_b, L = -(-M // B), M + N
    n_keep = max(n_keep, 1)
    q, k, v = (_rand_bf16(171 + i, H, r, d).to(G.DEV) for i, r in enumerate((n_gen, L, L)))
    Q, K, V = G.to_np(q), G.to_np(k), G.to_np(v)
    active = np.sort(rng.choice(n_gen, n_act, replace=False))
    focus = np.sort(rng.choice(active, max(1, n_act // 3), replace=False))
    a_dev, f_dev, counts = G.i32(list(active)), G.i32(list(focus)), G.i32([len(focus), n_act])
    # probe layer
    out_p, lse_p, col, sinks_dev = G.gpu_probe_layer(q, a_dev, counts, k, v, M, B, n_sink)
    S_ref = fo.sink_scores(Q, active, K)
    assert np.allclose(col.cpu().numpy(), S_ref, rtol=2e-4, atol=1e-9)
    ref_p, ref_lse_p = fo.sparse_attention(Q, active, K, V, np.arange(M), M)
    G.assert_attention_close(out_p[:, :n_act], ref_p)
    assert np.allclose(lse_p.cpu().numpy()[:, :n_act], ref_lse_p, atol=2e-3)
    sinks_ref = fo.select_sinks(S_ref, M, n_sink)
    sure_sinks = not (0 < n_sink < M) or fo.decision_margin(S_ref, n_sink, np.arange(L) < M) > 1e-4
    if sure_sinks:
        assert sinks_dev.cpu().tolist() == sinks_ref.tolist()
    # fused sparse layer with the device's sinks
    scores, kept, out, lse = G.gpu_sparse_layer(q, f_dev, a_dev, counts, k, v, None, M, B, n_keep, sinks_dev if n_sink else None)
    s2, k2 = G.gpu_block_scores(q, f_dev, counts, k, None, M, B, n_keep)
    o2, l2 = G.gpu_sparse_attn(q, a_dev, counts, k, v, M, B, k2, sinks_dev if n_sink else None)
    assert torch.equal(scores, s2) and torch.equal(kept, k2) and torch.equal(out[:, :n_act], o2[:, :n_act])
    lay = fo.focus_layer(Q, K, V, focus, active, np.array(sinks_dev.cpu().tolist(), dtype=np.int64), M, B, n_keep)
    if n_keep == n_b or fo.decision_margin(lay["R"], n_keep) > 1e-4:
        assert kept.cpu().tolist() == lay["blocks"].tolist()
        G.assert_attention_close(out[:, :n_act], lay["out"])
    # block entry: cache rewrite + block means, then every position attends to every key
    k_cache, v_cache = torch.zeros_like(k), torch.zeros_like(v)
    kbar = torch.empty(H, n_b, d, dtype=torch.float32, device=G.DEV)
    fb.cache_refresh(k_cache, v_cache, fb.make_shape(q, k_cache, v_cache, M, B), k, v, kbar)
    q_all = _rand_bf16(175, H, L, d).to(G.DEV)
    out_all = torch.empty_like(q_all)
    lse_all = torch.empty(H, L, dtype=torch.float32, device=G.DEV)
    fb.refresh_attn(q_all, k_cache, v_cache, fb.make_shape(q_all, k_cache, v_cache, M, B, out_all), out_all, lse_all)
    torch.cuda.synchronize()
    assert torch.equal(k_cache, k) and torch.equal(v_cache, v)
    assert np.allclose(kbar.cpu().numpy(), fo.block_means(K, M, B), rtol=1e-5, atol=1e-5)
    rows = np.unique(rng.integers(0, L, 24))
    ref_all, ref_lse_all = fo.sparse_attention(G.to_np(q_all), rows, K, V, np.arange(M), M)
    G.assert_attention_close(out_all[:, rows], ref_all)
    assert np.allclose(lse_all.cpu().numpy()[:, rows], ref_lse_all, atol=2e-3)


# ------------------------------------------------------------------------------------------------ grouped-query attention
@pytest.mark.parametrize("H_kv,group,M,N,d,B,n_gen,k,window,n_keep,n_sink", [
    (2, 4, 2048, 32, 128, 64, 32, 6, 0, 5, 3),       # 24 query rows per K/V head: two query tiles
    (4, 7, 4096, 64, 128, 128, 64, 4, 8, 8, 20),     # 28 heads on 4 K/V heads, window-expanded queries: several query groups
    (3, 2, 1000, 37, 64, 48, 40, 16, 0, 4, 2),       # ragged sizes, d = 64
])
def test_grouped_query_attention_through_the_row_view(G, H_kv, group, M, N, d, B, n_gen, k, window, n_keep, n_sink):
    """Several query heads per K/V head: the device runs H_kv heads over the [H_kv, group * n_gen, d] view of Q with the
    expanded index lists and reads every K/V head once; the oracle runs all H_q heads separately against K/V repeated
    per query head.  Sinks, kept blocks and attention must agree."""
    H_q, L = H_kv * group, M + N
    q = _rand_bf16(141, H_q, n_gen, d).to(G.DEV)                      # head-major: [H_q, n_gen, d]
    k_, v_ = _rand_bf16(142, H_kv, L, d).to(G.DEV), _rand_bf16(143, H_kv, L, d).to(G.DEV)
    conf = np.random.default_rng(144).random(n_gen).astype(np.float32)
    # oracle: plain multi-head attention over repeated K/V
    Q, K, V = G.to_np(q), np.repeat(G.to_np(k_), group, axis=0), np.repeat(G.to_np(v_), group, axis=0)
    focus_ref = fo.select_focus(conf, None, k)
    active_ref = fo.expand_window(focus_ref, window, 0, n_gen)
    S_ref = fo.sink_scores(Q, active_ref, K)
    sinks_ref = fo.select_sinks(S_ref, M, n_sink)
    lay = fo.focus_layer(Q, K, V, focus_ref, active_ref, sinks_ref, M, B, n_keep)
    assert fo.decision_margin(S_ref, n_sink, np.arange(L) < M) > 1e-5 and fo.decision_margin(lay["R"], n_keep) > 1e-5
    # device
    focus, active, counts = G.gpu_select(conf, None, k, window, 0, n_gen)
    f2 = torch.full((group * focus.numel(),), -7, dtype=torch.int32, device=G.DEV)
    a2 = torch.full((group * active.numel(),), -7, dtype=torch.int32, device=G.DEV)
    c2 = torch.zeros(2, dtype=torch.int32, device=G.DEV)
    fb.expand_groups(focus, active, counts, n_gen, group, f2, a2, c2)
    torch.cuda.synchronize()
    n_f, n_a = len(focus_ref), len(active_ref)
    assert c2.cpu().tolist() == [group * n_f, group * n_a]
    want_a = [g * n_gen + i for g in range(group) for i in active_ref.tolist()]
    assert a2.cpu().tolist() == want_a + [-1] * (a2.numel() - len(want_a))
    want_f = [g * n_gen + i for g in range(group) for i in focus_ref.tolist()]
    assert f2.cpu().tolist() == want_f + [-1] * (f2.numel() - len(want_f))
    qv = q.view(H_kv, group * n_gen, d)                               # the same memory, one row list per K/V head
    col, sinks = G.gpu_find_sinks(qv, a2, c2, k_, M, B, n_sink)
    scores, kept = G.gpu_block_scores(qv, f2, c2, k_, None, M, B, n_keep)
    out, lse = G.gpu_sparse_attn(qv, a2, c2, k_, v_, M, B, kept, sinks)
    assert np.allclose(col.cpu().numpy(), S_ref, rtol=2e-4, atol=1e-10)
    assert sinks.cpu().tolist() == sinks_ref.tolist()
    assert np.allclose(scores.cpu().numpy(), lay["R"], atol=2e-6)
    assert kept.cpu().tolist() == lay["blocks"].tolist()
    # output slot g * n_a + a of K/V head kv is active query a of query head kv * group + g
    got = out[:, :group * n_a].reshape(H_kv, group, n_a, d).reshape(H_q, n_a, d)
    G.assert_attention_close(got, lay["out"])


# ------------------------------------------------------------------------------------------------ block-entry refresh
@pytest.mark.parametrize("H,M,N,d", [(4, 1024, 32, 64), (2, 2050, 33, 128), (3, 100, 7, 128), (1, 5, 0, 64), (2, 4096, 64, 128),
                                     (2, 40, 9, 128), (2, 64, 32, 64), (33, 300, 20, 128)])   # two and three key sub-tiles; a head count that is no multiple of 8
def test_refresh_attn_equals_full_bidirectional_attention(G, H, M, N, d):
    """Every position attends to every position: against the oracle's dense reduction, an independent fp64
    scaled_dot_product_attention, and focus_sparse_attn with everything kept."""
    L = M + N
    q, k, v = (_rand_bf16(101 + i, H, L, d).to(G.DEV) for i in range(3))
    out = torch.full((H, L, d), float("nan"), dtype=torch.bfloat16, device=G.DEV)
    lse = torch.full((H, L), float("nan"), dtype=torch.float32, device=G.DEV)
    s = fb.make_shape(q, k, v, M, 64, out)
    fb.refresh_attn(q, k, v, s, out, lse)
    torch.cuda.synchronize()
    Q, K, V = G.to_np(q), G.to_np(k), G.to_np(v)
    ref, ref_lse = fo.sparse_attention(Q, np.arange(L), K, V, np.arange(M), M)
    G.assert_attention_close(out, ref)
    assert np.allclose(lse.cpu().numpy(), ref_lse, atol=2e-3)
    sdpa = torch.nn.functional.scaled_dot_product_attention(torch.from_numpy(Q), torch.from_numpy(K), torch.from_numpy(V))
    G.assert_attention_close(out, sdpa.numpy())
    n_b = -(-M // 64)
    out2, lse2 = G.gpu_sparse_attn(q, G.i32(np.arange(L)), None, k, v, M, 64, G.i32(np.arange(n_b)), None)
    # the two kernels round differently (this one sums the bf16-rounded probabilities): close, not identical
    G.assert_attention_close(out, G.to_np(out2))
    assert np.allclose(lse.cpu().numpy(), lse2.cpu().numpy(), atol=1e-3)


@pytest.mark.parametrize("H,n_q,L,d", [
    (256, 256, 20, 128),   # 256-query blocks only: one key sub-tile,
    (256, 250, 130, 64),   # ... fewer than the ring holds,
    (256, 256, 259, 128),  # ... once around it and a ragged one,
    (40, 1100, 1100, 128), # ... and a ragged query block
    (64, 1032, 1032, 64),  # a full round of blocks, the last tile of every head on its own
    (72, 1000, 300, 128),  # a round of blocks, the others as single tiles
    (3, 2100, 70, 64),     # single tiles only, fewer key sub-tiles than wavefronts
    (1, 1, 33, 128),
])
def test_refresh_attn_cut_into_blocks_and_tiles(G, H, n_q, L, d):
    q, k, v = (_rand_bf16(161 + i, H, r, d).to(G.DEV) for i, r in enumerate((n_q, L, L)))
    out = torch.full((H, n_q, d), float("nan"), dtype=torch.bfloat16, device=G.DEV)
    lse = torch.full((H, n_q), float("nan"), dtype=torch.float32, device=G.DEV)
    fb.refresh_attn(q, k, v, fb.make_shape(q, k, v, L, 64, out), out, lse)
    Q, K, V = (t.float().cpu() for t in (q, k, v))
    s = torch.matmul(Q, K.transpose(1, 2).contiguous()) / math.sqrt(d)
    G.assert_attention_close(out, torch.matmul(torch.softmax(s, -1), V).numpy())
    assert np.allclose(lse.cpu().numpy(), torch.logsumexp(s, -1).numpy(), atol=2e-3)


@pytest.mark.parametrize("offset", [0.0, 40.0])      # 40: the maximum of a row moves with nearly every sub-tile
@pytest.mark.parametrize("H,n_q,L,d", [
    (70, 256, 577, 128),   # 140 half blocks: an odd number of key sub-tiles, the last of one row
    (70, 256, 640, 128),   # ... an even number of whole ones
    (64, 470, 1000, 128),  # half blocks of every head's last seven tiles as well, the last tile ragged and one missing
    (130, 263, 748, 128),  # a round of half blocks, the others as single tiles
    (130, 404, 811, 128),  # half blocks of whole ones and of every head's last tiles, the others as single tiles
    (24, 3567, 1300, 128), # a round of blocks, then 160 half blocks; an odd number of sub-tiles
    (96, 678, 836, 128),   # whole blocks, then half blocks of every head's last tiles
    (130, 771, 1639, 128), # a round of blocks, a round of half blocks, single tiles
    (64, 512, 1100, 64),   # half blocks of 64 columns, a ragged last sub-tile of one half
    (64, 500, 1121, 64),   # ... and of the other
    (70, 452, 2004, 64),   # half blocks of whole ones and of the last tiles, then single tiles
    (130, 787, 2028, 64),  # a round of blocks, a round of half blocks, single tiles
    (8, 1500, 1490, 128),  # quarters, the last tile of a head missing: one part has a sub-tile less than the others,
    (8, 1500, 1537, 128),  # ... three have, and the fourth's last one has a single row;
    (9, 1000, 330, 128),   # ... a few sub-tiles each, the last tile ragged
    (24, 3298, 645, 128),  # a round of blocks, then quarters
    (70, 912, 475, 128),   # whole blocks, then quarters of every head's last tiles
    (130, 546, 461, 128),  # a round of blocks, quarters of the other four and of the last tiles
])
def test_refresh_attn_half_blocks(G, H, n_q, L, d, offset):
    q, k, v = (_rand_bf16(171 + i, H, r, d).to(G.DEV) for i, r in enumerate((n_q, L, L)))
    k += (offset / L * torch.arange(L, device=G.DEV)[None, :, None] * torch.sign(q[:, :1].float())).to(torch.bfloat16)
    out = torch.full((H, n_q, d), float("nan"), dtype=torch.bfloat16, device=G.DEV)
    lse = torch.full((H, n_q), float("nan"), dtype=torch.float32, device=G.DEV)
    fb.refresh_attn(q, k, v, fb.make_shape(q, k, v, L, 64, out), out, lse)
    # float64 on the device, a head at a time: float32 would leave the large logits 2e-5 of themselves
    for h in range(H):
        s = torch.matmul(q[h].double(), k[h].double().t()) / math.sqrt(d)
        G.assert_attention_close(out[h], torch.matmul(torch.softmax(s, -1), v[h].double()).cpu().numpy())
        # sums of rounded probabilities (whole blocks) are off by up to 2^-9 of themselves; the size of a logit scales its fp32 rounding
        assert torch.allclose(lse[h].double(), torch.logsumexp(s, -1), atol=2.0 ** -8, rtol=1e-5)
    out2 = torch.zeros_like(out)
    fb.refresh_attn(q, k, v, fb.make_shape(q, k, v, L, 64, out2), out2, None)
    assert torch.equal(out, out2)


@pytest.mark.parametrize("H,n_q,L,d", [
    (70, 256, 577, 128), (64, 470, 1000, 128), (64, 500, 1121, 64),   # half blocks
    (8, 1500, 1490, 128), (9, 1000, 330, 128),                        # quarters
    (256, 250, 300, 128), (256, 250, 300, 64),                        # whole blocks
    (3, 100, 300, 128), (3, 100, 300, 64),                            # single tiles
])
def test_refresh_attn_logits_of_minus_infinity(G, H, n_q, L, d):
    """Some queries of every tile have logits of -inf (a product of 2^65 and -2^65) for some keys: all that one part of a block, or one
    wavefront, sees at first or at all.  They count for nothing; a query with no other key gets a row of zeros."""
    q, k, v = (_rand_bf16(175 + i, H, r, d) for i, r in enumerate((n_q, L, L)))
    key, sub = torch.arange(L), torch.arange(L) // 32
    sets = [sub % 2 == 0, sub % 2 == 1, sub % 4 != 3, sub % 8 != 5, sub < 3, key < L - 1, key >= 0]   # query i: set i mod 8, or none
    row = torch.arange(n_q) % 8
    dead = torch.zeros(n_q, L, dtype=torch.bool)
    for c, keys in enumerate(sets):
        q[:, :, c] = torch.where(row == c, 2.0 ** 65, 0.0).to(torch.bfloat16)
        k[:, :, c] = torch.where(keys, -2.0 ** 65, 0.0).to(torch.bfloat16)
        dead |= (row == c)[:, None] & keys
    q, k, v, dead = (t.to(G.DEV) for t in (q, k, v, dead))
    out = torch.full((H, n_q, d), float("nan"), dtype=torch.bfloat16, device=G.DEV)
    lse = torch.full((H, n_q), float("nan"), dtype=torch.float32, device=G.DEV)
    fb.refresh_attn(q, k, v, fb.make_shape(q, k, v, L, 64, out), out, lse)
    n = len(sets)
    for h in range(H):
        s = torch.matmul(q[h, :, n:].double(), k[h, :, n:].double().t()).div(math.sqrt(d)).masked_fill(dead, -math.inf)
        G.assert_attention_close(out[h], torch.matmul(torch.softmax(s, -1).nan_to_num(0.0), v[h].double()).cpu().numpy())
        assert torch.allclose(lse[h].double(), torch.logsumexp(s, -1), atol=2.0 ** -8, rtol=1e-5)   # (bound of rounded sums)
    out2 = torch.zeros_like(out)
    fb.refresh_attn(q, k, v, fb.make_shape(q, k, v, L, 64, out2), out2, None)
    assert torch.equal(out, out2)


@pytest.mark.parametrize("offset", [0.0, 40.0])      # 40: the maximum of a row moves with nearly every sub-tile
@pytest.mark.parametrize("H,n_q,L", [
    (8, 1024, 255),      # 256 tiles of 64 columns: one per compute unit; a sub-tile per wavefront, the last ragged
    (9, 1000, 257),      # 288: two of them share some; a second sub-tile for one wavefront
    (8, 2080, 2080),     # 520: more than are resident at once
    (32, 1032, 1032),    # whole blocks and a ragged one of 32 heads, all as tiles
])
def test_refresh_attn_tiles_of_64_columns(G, H, n_q, L, offset):
    d = 64
    q, k, v = (_rand_bf16(191 + i, H, r, d).to(G.DEV) for i, r in enumerate((n_q, L, L)))
    k += (offset / L * torch.arange(L, device=G.DEV)[None, :, None] * torch.sign(q[:, :1].float())).to(torch.bfloat16)
    out = torch.full((H, n_q, d), float("nan"), dtype=torch.bfloat16, device=G.DEV)
    lse = torch.full((H, n_q), float("nan"), dtype=torch.float32, device=G.DEV)
    fb.refresh_attn(q, k, v, fb.make_shape(q, k, v, L, 64, out), out, lse)
    Q, K, V = (t.float().cpu() for t in (q, k, v))
    s = torch.matmul(Q, K.transpose(1, 2).contiguous()) / math.sqrt(d)
    G.assert_attention_close(out, torch.matmul(torch.softmax(s, -1), V).numpy())
    # the log-sum-exps of the tiles are those of unrounded sums; their size scales the fp32 rounding of the logits
    assert np.allclose(lse.cpu().numpy(), torch.logsumexp(s, -1).numpy(), atol=2e-3, rtol=1e-5)
    out2 = torch.zeros_like(out)
    fb.refresh_attn(q, k, v, fb.make_shape(q, k, v, L, 64, out2), out2, None)
    assert torch.equal(out, out2)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("H,n_q,L", [(256, 256, 24), (256, 256, 300), (3, 40, 24), (3, 100, 300)])   # 256-query blocks; single tiles
def test_refresh_attn_divides_by_the_probabilities_it_adds_up(G, H, n_q, L, d):
    """Every row is normalised by the sum of the bf16 probabilities that enter the PV product, in both kernels: the output is then a
    weighted mean of V.  With |v - c_col| <= eps it is off by at most 2^-9 max|v - o| <= 2^-8 eps (a probability is off by 2^-9 of
    itself) before it is stored, whatever c_col; dividing by the unrounded sum would add up to 2^-9 |c_col|.  For c_col in (2, 4) the store
    adds half a unit, 2^-7; 2e-5 is left for fp32."""
    g = torch.Generator().manual_seed(197 + L + d)
    q, k = ((_rand_bf16(194 + i, H, r, d).float() * 1.5).to(torch.bfloat16) for i, r in enumerate((n_q, L)))
    eps = 2.0 ** -6                                                     # the spacing of bf16 between 2 and 4
    col = 2.0 + eps * torch.randint(2, 126, (1, 1, d), generator=g)
    v = (col + eps * torch.randint(-1, 2, (H, L, d), generator=g)).to(torch.bfloat16)
    out = torch.empty(H, n_q, d, dtype=torch.bfloat16, device=G.DEV)
    lse = torch.empty(H, n_q, device=G.DEV)
    qd, kd, vd = (t.to(G.DEV) for t in (q, k, v))
    fb.refresh_attn(qd, kd, vd, fb.make_shape(qd, kd, vd, L, 64, out), out, lse)
    s = torch.matmul(q.double(), k.double().transpose(1, 2).contiguous()) / math.sqrt(d)
    err = (out.cpu().double() - torch.matmul(torch.softmax(s, -1), v.double())).abs().max().item()
    assert err <= 2.0 ** -7 + 2.0 ** -8 * eps + 2e-5
    out2 = torch.empty_like(out)
    fb.refresh_attn(qd, kd, vd, fb.make_shape(qd, kd, vd, L, 64, out2), out2, None)
    assert torch.equal(out, out2)                                       # whether the log-sum-exp is wanted or not
    assert np.allclose(lse.cpu().numpy(), torch.logsumexp(s, -1).numpy(), atol=2.0 ** -8)   # rounded sums are off by up to 2^-9 of themselves


@pytest.mark.parametrize("d", [64, 128])
def test_refresh_attn_running_maximum_keeps_moving(G, d):
    """Keys grow along the key axis and the queries are large, so the row maxima rise in almost every sub-tile and the
    softmax is close to one-hot: the rescale branch of the kernel runs all the way through, not only at the start."""
    H, M, N = 3, 3000, 77
    L = M + N
    grow = (1.0 + 4.0 * torch.arange(L) / L).view(1, L, 1)
    q = (_rand_bf16(191, H, L, d).float() * 2.0).to(torch.bfloat16).to(G.DEV)
    k = (_rand_bf16(192, H, L, d).float() * grow).to(torch.bfloat16).to(G.DEV)
    v = _rand_bf16(193, H, L, d).to(G.DEV)
    out = torch.empty(H, L, d, dtype=torch.bfloat16, device=G.DEV)
    lse = torch.empty(H, L, dtype=torch.float32, device=G.DEV)
    fb.refresh_attn(q, k, v, fb.make_shape(q, k, v, M, 64, out), out, lse)
    torch.cuda.synchronize()
    ref, ref_lse = fo.sparse_attention(G.to_np(q), np.arange(L), G.to_np(k), G.to_np(v), np.arange(M), M)
    G.assert_attention_close(out, ref)
    assert np.allclose(lse.cpu().numpy(), ref_lse, rtol=1e-5, atol=2e-3)
    # the same inputs through the step's attention kernel with every block kept
    out2, _ = G.gpu_sparse_attn(q, G.i32(np.arange(L)), None, k, v, M, 64, G.i32(np.arange(-(-M // 64))), None)
    G.assert_attention_close(out2, ref)


def test_refresh_attn_full_size_sampled_rows(G):
    """The launch bench.py --full-refresh times (32 heads, 32768 + 64 keys, d = 128, every position a query), checked on
    sampled (head, row) pairs the oracle computes one by one."""
    H, M, N, d = 32, 32768, 64, 128
    L = M + N
    q, k, v = (_rand_bf16(131 + i, H, L, d).to(G.DEV) for i in range(3))
    out = torch.full((H, L, d), float("nan"), dtype=torch.bfloat16, device=G.DEV)
    lse = torch.full((H, L), float("nan"), dtype=torch.float32, device=G.DEV)
    fb.refresh_attn(q, k, v, fb.make_shape(q, k, v, M, 128, out), out, lse)
    torch.cuda.synchronize()
    assert not torch.isnan(out.float()).any() and not torch.isnan(lse).any()
    rows = np.array([0, 1, 31, 32, 127, 128, 16383, 16384, 32767, 32768, 32800, 32831])
    for h in (0, 13, 31):
        ref, ref_lse = fo.sparse_attention(G.to_np(q[h:h + 1]), rows, G.to_np(k[h:h + 1]), G.to_np(v[h:h + 1]), np.arange(M), M)
        G.assert_attention_close(out[h:h + 1, rows], ref)
        assert np.allclose(lse[h:h + 1, rows].cpu().numpy(), ref_lse, atol=2e-3)


def test_refresh_attn_strided_output_and_fewer_queries_than_keys(G):
    H, M, N, d, n_q = 2, 700, 20, 128, 333
    q = _rand_bf16(111, n_q, H, d).to(G.DEV).permute(1, 0, 2)            # [L, H, d] storage
    k, v = _rand_bf16(112, H, M + N, d).to(G.DEV), _rand_bf16(113, H, M + N, d).to(G.DEV)
    buf = torch.full((H, n_q, 2 * d), 7.0, dtype=torch.bfloat16, device=G.DEV)
    out = buf[:, :, :d]                                                    # row stride 2 d: the other half must stay untouched
    s = fb.make_shape(q, k, v, M, 64, out)
    fb.refresh_attn(q, k, v, s, out, None)
    torch.cuda.synchronize()
    ref, _ = fo.sparse_attention(G.to_np(q), np.arange(n_q), G.to_np(k), G.to_np(v), np.arange(M), M)
    G.assert_attention_close(out, ref)
    assert (buf[:, :, d:] == 7.0).all()


@pytest.mark.parametrize("H,M,N,B,d", [(4, 1024, 64, 64, 128), (3, 1000, 37, 128, 64), (2, 70, 0, 32, 128), (2, 4100, 300, 128, 128)])
def test_cache_refresh_copies_every_row_and_emits_block_means(G, H, M, N, B, d):
    """Block entry: the caches equal the new states bit for bit (strided cache, padding untouched), K_bar equals the
    oracle's block means and, bit for bit, focus_block_means of the new K."""
    L = M + N
    k_new, v_new = _rand_bf16(121, H, L, d).to(G.DEV), _rand_bf16(122, H, L, d).to(G.DEV)
    kbuf = torch.full((H, L + 3, d + 8), 5.0, dtype=torch.bfloat16, device=G.DEV)
    vbuf = torch.full((H, L + 3, d + 8), 6.0, dtype=torch.bfloat16, device=G.DEV)
    k_cache, v_cache = kbuf[:, :L, :d], vbuf[:, :L, :d]
    n_b = -(-M // B)
    kbar = torch.full((H, n_b, d), float("nan"), dtype=torch.float32, device=G.DEV)
    s = fb.make_shape(k_new[:, :1], k_cache, v_cache, M, B)
    fb.cache_refresh(k_cache, v_cache, s, k_new, v_new, kbar)
    torch.cuda.synchronize()
    K_ref, V_ref = fo.cache_update(np.zeros((H, L, d)), np.zeros((H, L, d)), G.to_np(k_new), G.to_np(v_new), np.arange(L), 0)
    assert np.array_equal(G.to_np(k_cache), K_ref) and np.array_equal(G.to_np(v_cache), V_ref)
    assert (kbuf[:, L:] == 5.0).all() and (kbuf[:, :, d:] == 5.0).all() and (vbuf[:, L:] == 6.0).all() and (vbuf[:, :, d:] == 6.0).all()
    ref = fo.block_means(G.to_np(k_new), M, B)
    assert np.allclose(kbar.cpu().numpy(), ref, rtol=1e-5, atol=1e-5)
    kbar2 = torch.empty_like(kbar)
    fb.block_means(k_new, fb.make_shape(k_new[:, :1], k_new, v_new, M, B), kbar2)
    torch.cuda.synchronize()
    assert torch.equal(kbar, kbar2)
    # copy only
    kbuf.fill_(1.0)
    fb.cache_refresh(k_cache, v_cache, s, k_new, v_new, None)
    torch.cuda.synchronize()
    assert torch.equal(k_cache, k_new)


def test_block_entry_then_step_uses_the_refreshed_cache_and_means(G):
    """A block entry followed by a sparse step (Alg. 1): the caches are rewritten and K_bar formed in one pass, every
    position attends densely over the new cache, and the next step's block scoring from those cached means picks the
    same blocks, with the same scores bit for bit, as scoring from the raw keys."""
    H, M, N, d, B, n_gen = 4, 4096, 64, 128, 64, 64
    L = M + N
    k_new, v_new = _rand_bf16(151, H, L, d).to(G.DEV), _rand_bf16(152, H, L, d).to(G.DEV)
    k_cache, v_cache = torch.zeros_like(k_new), torch.zeros_like(v_new)
    n_b = M // B
    kbar = torch.empty(H, n_b, d, dtype=torch.float32, device=G.DEV)
    q_all = _rand_bf16(153, H, L, d).to(G.DEV)
    out_all = torch.empty_like(q_all)
    fb.cache_refresh(k_cache, v_cache, fb.make_shape(q_all, k_cache, v_cache, M, B), k_new, v_new, kbar)
    fb.refresh_attn(q_all, k_cache, v_cache, fb.make_shape(q_all, k_cache, v_cache, M, B, out_all), out_all, None)
    torch.cuda.synchronize()
    rows = np.array([0, 77, M - 1, M, L - 1])
    ref, _ = fo.sparse_attention(G.to_np(q_all), rows, G.to_np(k_new), G.to_np(v_new), np.arange(M), M)
    G.assert_attention_close(out_all[:, rows], ref)
    # the following step: queries of the generation block, scoring from the cached means against scoring from raw K
    q = q_all[:, M:M + n_gen].contiguous()
    conf = np.random.default_rng(154).random(n_gen).astype(np.float32)
    focus, active, counts = G.gpu_select(conf, None, 16, 0, 0, n_gen)
    s_raw, kept_raw = G.gpu_block_scores(q, focus, counts, k_cache, None, M, B, 6)
    s_mean, kept_mean = G.gpu_block_scores(q, focus, counts, None, kbar, M, B, 6)
    assert torch.equal(s_raw, s_mean) and torch.equal(kept_raw, kept_mean)
    R = fo.block_relevance(G.to_np(q), fo.select_focus(conf, None, 16), fo.block_means(G.to_np(k_new), M, B))
    assert np.allclose(s_mean.cpu().numpy(), R, atol=2e-6)
    assert kept_mean.cpu().tolist() == fo.top_indices(R, 6).tolist()


@pytest.mark.parametrize("H,M,N,B,d", [
    (4, 1024, 32, 64, 64),      # single tiles only
    (3, 1000, 37, 128, 128),    # an odd number of chunks, ragged blocks
    (40, 1060, 40, 64, 128),    # blocks, the last of each head padded
    (129, 240, 17, 64, 128),    # whole blocks, then tiles with the copy behind them
    (17, 1950, 41, 64, 64),     # ... half blocks, then tiles
    (129, 1760, 33, 64, 128),   # ... blocks, half blocks, then tiles
    (97, 700, 37, 64, 128),     # blocks, then quarters with the copy behind them
    (256, 256, 0, 128, 64),     # whole blocks only, the copy's chunks behind them
    (32, 1000, 24, 64, 128),    # half blocks only,
    (32, 1000, 24, 130, 64),    # ... of 64 columns, chunks of more rows than are requested at once,
    (8, 1470, 31, 150, 128),    # ... quarters
    (128, 500, 44, 50, 64),     # whole blocks and 128 tiles of 64 columns, which get a compute unit each beside the chunks of the copy
    (129, 500, 44, 50, 64),     # 145 tiles, which share theirs
    (1, 30, 0, 32, 64),
    (1, 30, 0, 32, 128),
])
def test_block_entry_equals_the_two_calls(G, H, M, N, B, d):
    L, n_b = M + N, -(-M // B)
    store = [_rand_bf16(171 + i, L, H, d).to(G.DEV) for i in range(2)]
    k_new, v_new = (t.transpose(0, 1) for t in store)  # strides of their own
    q = _rand_bf16(173, H, L, d).to(G.DEV)
    res = []
    for fused in (False, True):
        kc, vc, out = (torch.full((H, L, d), float("nan"), dtype=torch.bfloat16, device=G.DEV) for _ in range(3))
        kbar, lse = torch.full((H, n_b, d), float("nan"), device=G.DEV), torch.full((H, L), float("nan"), device=G.DEV)
        s = fb.make_shape(q, kc, vc, M, B, out)
        if fused:
            fb.block_entry(kc, vc, s, q, k_new, v_new, kbar, out, lse)
        else:
            fb.cache_refresh(kc, vc, s, k_new, v_new, kbar)
            fb.refresh_attn(q, kc, vc, s, out, lse)
        torch.cuda.synchronize()
        res.append((kc, vc, kbar, out, lse))
    assert all(torch.equal(a, b) for a, b in zip(*res))


def test_block_entry_with_more_chunks_than_one_launch_holds(G):
    """2^24 chunks of the cache refresh do not fit behind the query tiles in one launch (fewer than 2^32 threads, 512 per two
    chunks); with blocks of one row K_bar is K itself, and the heads share the new states so that the inputs stay small."""
    H, M, d, n_q = 32, (1 << 19) + 3, 64, 33
    k_new, v_new = (_rand_bf16(181 + i, 1, M, d).to(G.DEV).expand(H, M, d) for i in range(2))
    q = _rand_bf16(183, H, n_q, d).to(G.DEV)
    kc, vc = (torch.full((H, M, d), float("nan"), dtype=torch.bfloat16, device=G.DEV) for _ in range(2))
    kbar = torch.full((H, M, d), float("nan"), device=G.DEV)
    out, out2 = (torch.full((H, n_q, d), float("nan"), dtype=torch.bfloat16, device=G.DEV) for _ in range(2))
    fb.block_entry(kc, vc, fb.make_shape(q, kc, vc, M, 1, out), q, k_new, v_new, kbar, out, None)
    fb.refresh_attn(q, kc, vc, fb.make_shape(q, kc, vc, M, 1, out2), out2, None)
    torch.cuda.synchronize()
    assert torch.equal(out, out2) and not torch.isnan(out.float()).any()
    for h in range(H):
        assert torch.equal(kc[h], k_new[0]) and torch.equal(vc[h], v_new[0]) and torch.equal(kbar[h], k_new[0].float())


def test_refresh_attn_with_more_tiles_than_one_launch_holds(G):
    """Seven tiles of every head would be 2^23 tiles and more, 512 threads each, past what a launch holds; all heads share Q, K, V and
    the output (they write the same values), and the log-sum-exp tells whether every head has run."""
    H, n_q, d, L = (1 << 23) // 7 + 1, 224, 64, 1
    q, k, v = (_rand_bf16(184 + i, 1, r, d).to(G.DEV).expand(H, r, d) for i, r in enumerate((n_q, L, L)))
    store = torch.full((1, n_q, d), float("nan"), dtype=torch.bfloat16, device=G.DEV)
    out = store.expand(H, n_q, d)
    lse = torch.full((H, n_q), float("nan"), device=G.DEV)
    fb.refresh_attn(q, k, v, fb.make_shape(q, k, v, L, 64, out), out, lse)
    torch.cuda.synchronize()
    assert torch.equal(store[0], v[0].expand(n_q, d))                   # one key
    ref = torch.matmul(q[0].double(), k[0, 0].double()) / math.sqrt(d)
    assert torch.allclose(lse[0].double(), ref, atol=1e-5) and torch.equal(lse, lse[:1].expand_as(lse))


def test_block_entry_calls_replay_in_a_hip_graph(G):
    """The block-entry calls and the group expansion enqueue kernels only, so they can be captured: three replays, the
    outputs wiped in between, each equal to the eager result bit for bit."""
    H, M, N, d, B, n_gen, group = 2, 1500, 36, 128, 64, 32, 3
    L = M + N
    k_new, v_new, q_all = (_rand_bf16(201 + i, H, L, d).to(G.DEV) for i in range(3))
    k_cache, v_cache, out = torch.zeros_like(k_new), torch.zeros_like(v_new), torch.zeros_like(q_all)
    kbar = torch.zeros(H, -(-M // B), d, dtype=torch.float32, device=G.DEV)
    lse = torch.zeros(H, L, dtype=torch.float32, device=G.DEV)
    focus, active, counts = G.gpu_select(np.random.default_rng(204).random(n_gen).astype(np.float32), None, 5, 2, 0, n_gen)
    f2, a2, c2 = G.i32(None, group * focus.numel()), G.i32(None, group * active.numel()), G.i32(None, 2)
    s_c = fb.make_shape(q_all, k_cache, v_cache, M, B)
    s_a = fb.make_shape(q_all, k_cache, v_cache, M, B, out)

    def enqueue():
        fb.expand_groups(focus, active, counts, n_gen, group, f2, a2, c2)
        fb.cache_refresh(k_cache, v_cache, s_c, k_new, v_new, kbar)
        fb.refresh_attn(q_all, k_cache, v_cache, s_a, out, lse)

    outputs = (f2, a2, c2, k_cache, v_cache, kbar, out, lse)
    enqueue()
    torch.cuda.synchronize()
    eager = [t.clone() for t in outputs]
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        enqueue()
    for _ in range(3):
        for t in outputs:
            t.zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(eager, outputs))


@pytest.mark.parametrize("use_graph", [False, True])
@pytest.mark.parametrize("H,M,N,d,B,n_gen,k,window,n_keep,n_sink,n_layers,l_dense,dense_tail", [
    (4, 1024, 32, 64, 64, 32, 8, 2, 4, 2, 5, 1, 1),          # the tiny shape; dense, probe, sparse, sparse, dense tail
    (2, 1000, 40, 128, 48, 40, 5, 4, 6, 3, 4, 0, 0),         # ragged prompt and blocks; the first layer is the probe
    (3, 2048, 64, 128, 128, 64, 16, 0, 3, 4, 6, 2, 2),       # 16 queries, block 128
])
def test_decoder_block_entry_then_sparse_steps_against_the_oracle(G, use_graph, H, M, N, d, B, n_gen, k, window, n_keep, n_sink,
                                                                  n_layers, l_dense, dense_tail):
    """Alg. 1 across a block entry: FocusDecoder (block-entry cache refresh with K_bar, dense attention of every position;
    then steps of query selection, per-layer cache update, dense prefix, probe layer with the sinks, sparse layers from
    the cached K_bar, dense tail) against oracle.decode_block over two steps — index sets and caches bit-exact, outputs
    within tolerance — eagerly and as two HIP graphs."""
    from paper_2602_02159_amd.step import FocusDecoder
    L = M + N
    rng = np.random.default_rng(H * 100 + n_layers)
    dec = FocusDecoder(n_layers, l_dense, dense_tail, H, d, M, N, n_gen, M, B, k, window, n_keep, n_sink, G.DEV)
    cap = dec.max_active
    if use_graph:
        dec.capture()
    # the "model": random states; two keys per head carry a shared direction so that the sinks are well separated
    u = rng.standard_normal(d)
    u /= np.linalg.norm(u)
    gain = math.sqrt(6.0 * math.sqrt(d))
    planted = sorted(rng.choice(M, n_sink, replace=False).tolist())
    bf = lambda x: torch.from_numpy(x).to(torch.bfloat16)
    ent = {}
    for l in range(n_layers):
        q_all, k_all, v_all = (rng.standard_normal((H, L, d)) for _ in range(3))
        k_all[:, planted] += gain * u
        ent[l] = (bf(q_all), bf(k_all), bf(v_all))
    steps = []
    masked = np.ones(n_gen, dtype=np.uint8)
    for t in range(2):
        per_layer = {}
        for l in range(n_layers):
            q = rng.standard_normal((H, n_gen, d)) + gain * u
            per_layer[l] = (bf(q), bf(rng.standard_normal((H, cap, d))), bf(rng.standard_normal((H, cap, d))))
        steps.append({"conf": rng.random(n_gen).astype(np.float32), "masked": masked.copy(), "k": k, "tensors": per_layer})
        masked[rng.choice(n_gen, 3, replace=False)] = 0          # three positions are unmasked between the steps
    np_of = lambda ts: tuple(G.to_np(x) for x in ts)
    kw = dict(n_layers=n_layers, l_dense=l_dense, dense_tail=dense_tail, n_ctx=M, row_base=M, block=B, window=window, lo=0, hi=n_gen,
              n_keep=n_keep, n_sink=n_sink)
    o_steps = [{"conf": s["conf"], "masked": s["masked"], "k": k, "layer": (lambda pl: (lambda l: np_of(pl[l])))(s["tensors"])}
               for s in steps]
    refs = [fo.decode_block(lambda l: np_of(ent[l]), o_steps[:t], **kw) for t in (0, 1, 2)]   # after the entry, after step 1, after step 2

    # ---- block entry
    for l in range(n_layers):
        for dst, src in zip((dec.q_all[l], dec.k_all[l], dec.v_all[l]), ent[l]):
            dst.copy_(src)
    dec.run_entry()
    torch.cuda.synchronize()
    for l in range(n_layers):
        assert torch.equal(dec.k_cache[l].cpu(), ent[l][1]) and torch.equal(dec.v_cache[l].cpu(), ent[l][2])
        G.assert_attention_close(dec.out_all[l], refs[0]["entry"][l])
        if dec.is_sparse(l):
            assert np.allclose(dec.kbar[l].cpu().numpy(), fo.block_means(G.to_np(ent[l][1]), M, B), atol=2e-6 * math.sqrt(B))
    kbar_entry = [None if kb is None else kb.clone() for kb in dec.kbar]

    # ---- two steps
    for t, s in enumerate(steps):
        ref = refs[t + 1]["steps"][t]
        n_a = len(ref["active"])
        assert fo.decision_margin(ref["S"], n_sink, np.arange(L) < M) > 1e-4
        dec.conf.copy_(torch.from_numpy(s["conf"]))
        dec.masked.copy_(torch.from_numpy(s["masked"]))
        for l in range(n_layers):
            for dst, src in zip((dec.q[l], dec.k_new[l], dec.v_new[l]), s["tensors"][l]):
                dst.copy_(src)
            dec.out[l].zero_()
        dec.sink_idx.fill_(-3)
        dec.run_step()
        torch.cuda.synchronize()
        assert dec.counts.cpu().tolist() == [len(ref["focus"]), n_a]
        assert dec.focus_idx.cpu().tolist()[:len(ref["focus"])] == ref["focus"].tolist()
        assert dec.active_idx.cpu().tolist()[:n_a] == ref["active"].tolist()
        assert dec.sink_idx.cpu().tolist() == ref["sinks"].tolist() == planted
        for l in range(n_layers):
            lay = ref["layers"][l]
            assert (lay["kind"] == "sparse") == dec.is_sparse(l)
            if dec.is_sparse(l):
                assert fo.decision_margin(lay["R"], n_keep) > 1e-4
                assert dec.kept[l].cpu().tolist() == lay["blocks"].tolist(), f"step {t} layer {l}"
                assert torch.equal(dec.kbar[l], kbar_entry[l])                       # frozen since the block entry
            G.assert_attention_close(dec.out[l][:, :n_a], lay["out"])
            # Eq. 3: exactly the active rows took their new states, in every layer; the copies are exact
            assert np.array_equal(G.to_np(dec.k_cache[l]).astype(np.float64), refs[t + 1]["K_cache"][l]), f"step {t} layer {l}"
            assert np.array_equal(G.to_np(dec.v_cache[l]).astype(np.float64), refs[t + 1]["V_cache"][l])
    assert refs[2]["steps"][0]["active"].tolist() != refs[2]["steps"][1]["active"].tolist()   # the two steps refresh different rows


# ------------------------------------------------------------------------------------------------ around the step
@pytest.mark.parametrize("n_rows,vocab,pad", [(5, 1000, 0), (3, 8, 0), (4, 13, 3), (64, 126464, 0), (7, 131077, 11), (2, 40000, 8)])
def test_token_confidence(G, n_rows, vocab, pad):
    """Eq. 2 on bf16 logits: the arg max is exact (bf16 rows hold many exactly equal maxima: the lower id wins), the
    confidence agrees with the float64 oracle to fp32 summation accuracy."""
    stride = -(-(vocab + pad) // 8) * 8
    g = torch.Generator().manual_seed(90 + vocab)
    buf = (torch.randn(n_rows, stride, generator=g) * 3.0).to(torch.bfloat16)
    buf[0, : vocab // 2] = buf[0, : vocab // 2].clamp(max=2.0)             # a plateau: thousands of tokens share the maximum
    if n_rows > 2:
        buf[2, ::3] = float("-inf")                                         # excluded tokens
    logits = buf.to(G.DEV)[:, :vocab]
    masked = (torch.arange(n_rows) % 4 != 1).to(torch.uint8)
    for m in (None, masked):
        tok = G.i32(None, n_rows)
        conf = torch.full((n_rows,), float("nan"), dtype=torch.float32, device=G.DEV)
        w = G.ws(fb.token_confidence_workspace(n_rows, vocab))
        w.fill_(0xEE)
        fb.token_confidence(logits, None if m is None else m.to(G.DEV), tok, conf, w)
        torch.cuda.synchronize()
        ref_tok, ref_conf = fo.token_confidence(G.to_np(logits), None if m is None else m.numpy())
        assert tok.cpu().tolist() == ref_tok.tolist()
        assert np.allclose(conf.cpu().numpy(), ref_conf, rtol=2e-5, atol=0)
    # the result is the input of Eq. 4 as it stands
    focus, _, _ = G.gpu_select(conf.cpu().numpy(), masked.numpy(), min(2, n_rows), 0, 0, n_rows)
    assert focus.cpu().tolist()[: len(fo.select_focus(ref_conf, masked.numpy(), min(2, n_rows)))] == \
        fo.select_focus(ref_conf.astype(np.float32), masked.numpy(), min(2, n_rows)).tolist()


def test_token_confidence_uniform_row(G):
    logits = torch.zeros(2, 4096, dtype=torch.bfloat16, device=G.DEV)
    tok, conf = G.i32(None, 2), torch.zeros(2, dtype=torch.float32, device=G.DEV)
    fb.token_confidence(logits, None, tok, conf, G.ws(fb.token_confidence_workspace(2, 4096)))
    torch.cuda.synchronize()
    assert tok.cpu().tolist() == [0, 0] and np.allclose(conf.cpu().numpy(), 1.0 / 4096, rtol=1e-6)


@pytest.mark.parametrize("H,M,N,d,cap,n_act,base", [(4, 100, 32, 64, 8, 5, 100), (32, 2048, 64, 128, 36, 28, 2048 + 16), (2, 64, 16, 128, 16, 16, 64)])
def test_cache_update(G, H, M, N, d, cap, n_act, base):
    """Eq. 3: exactly the rows of the refreshed positions change, bit for bit; strided cache layout, spare slots,
    negative and out-of-range entries are skipped."""
    rng = np.random.default_rng(H + M)
    L = M + N
    kc = _rand_bf16(95, L, H, d).to(G.DEV).permute(1, 0, 2)                  # cache stored [L, H, d]
    vc = _rand_bf16(96, H, L, d).to(G.DEV)
    kn, vn = _rand_bf16(97, H, cap, d).to(G.DEV), _rand_bf16(98, H, cap, d).to(G.DEV)
    span = L - base
    act = np.sort(rng.choice(span, min(n_act, span), replace=False)).tolist()
    lst = act + [-1] * (cap - len(act))
    if len(act) < cap:
        lst[len(act)] = 3                                                    # a stale entry past the count must be ignored
    k_before, v_before = kc.clone(), vc.clone()
    s = fb.make_shape(kn, kc, vc, M, 64)
    fb.cache_update(kc, vc, s, kn, vn, G.i32(lst), G.i32([0, len(act)]), base)
    torch.cuda.synchronize()
    K_ref, V_ref = fo.cache_update(G.to_np(k_before), G.to_np(v_before), G.to_np(kn), G.to_np(vn), act, base)
    assert np.array_equal(G.to_np(kc), K_ref) and np.array_equal(G.to_np(vc), V_ref)
    # entries that map outside the cache or are negative: nothing happens
    k2, v2 = kc.clone(), vc.clone()
    fb.cache_update(kc, vc, s, kn, vn, G.i32([-5, span, span + 7] + [-1] * (cap - 3)), None, base)
    torch.cuda.synchronize()
    assert torch.equal(kc, k2) and torch.equal(vc, v2)


@pytest.mark.parametrize("H,M,N,d,B,n_gen,n_act,n_keep,means", [
    (32, 2048, 64, 128, 64, 64, 36, 9, "cached"),    # the update beside the relevances: five workgroups per head,
    (6, 1000, 40, 64, 16, 33, 17, 20, "cached"),     # ... more of them than the relevances have, a ragged last one
    (1, 70000, 16, 64, 32, 16, 16, 40, "cached"),    # ... one head, many slices of relevances, ranked by a launch of their own
    (4, 256, 8, 128, 16, 8, 5, 3, "cached"),         # one launch for the layer: the update has its own
    (5, 700, 30, 128, 64, 30, 9, 4, "scan"),         # block means from K, which the update may touch
])
def test_update_and_sparse_layer_in_one_call(G, H, M, N, d, B, n_gen, n_act, n_keep, means):
    """The caches and outputs of the two calls one after the other, bit for bit; entries that are negative or map outside the cache are skipped."""
    L, n_sink, base = M + N, 3, M - 2                                       # (the first positions lie in the prompt)
    q, kn, vn = (_rand_bf16(301 + i, H, r, d).to(G.DEV) for i, r in enumerate((n_gen, n_gen, n_gen)))
    rng = np.random.default_rng(M)
    act = np.sort(rng.choice(min(n_gen, N + 2), n_act, replace=False)).tolist()
    lst = act + [N + 5] + [-1] * n_gen
    active, counts = G.i32(lst[:n_gen]), G.i32([2, n_act])
    focus, sinks = G.i32(act[:2]), G.i32([0, 7, M // 2])
    kbar = _rand_bf16(307, H, -(-M // B), d).float().to(G.DEV) if means == "cached" else None
    res = []
    for together in (False, True):
        kc = _rand_bf16(305, L, H, d).to(G.DEV).permute(1, 0, 2)             # cache stored [L, H, d]
        vc = _rand_bf16(306, H, L, d).to(G.DEV)
        out = torch.zeros((H, n_gen, d), dtype=torch.bfloat16, device=G.DEV)
        lse, scores, kept = torch.zeros((H, n_gen), device=G.DEV), torch.zeros(-(-M // B), device=G.DEV), G.i32(None, n_keep)
        s = fb.make_shape(q, kc, vc, M, B, out)
        ws = G.ws(fb.workspace_bytes(fb.FN_SPARSE_LAYER, s, n_gen, n_keep, n_sink))
        if together:
            fb.update_sparse_layer(kc, vc, kn, vn, base, q, focus, active, counts, kbar, s, n_keep, sinks, n_sink, scores, kept, out, lse, ws)
        else:
            fb.cache_update(kc, vc, s, kn, vn, active, counts, base)
            fb.sparse_layer(q, focus, active, counts, kc, vc, kbar, s, n_keep, sinks, n_sink, scores, kept, out, lse, ws)
        res.append((kc, vc, scores, kept, out[:, :n_act], lse[:, :n_act]))
    torch.cuda.synchronize()
    assert torch.equal(res[0][0][:, base + act[0]], kn[:, 0])
    for a, b in zip(*res):
        assert torch.equal(a, b)
