"""Running top-k ranking on the GPU against the oracle, bit-exact (App. B.3, App. C,
Sec. 3.1 eq. teacher_label). Priorities are compared in float32 on both sides (the
ranking is an integer decided by them); ranks, cutoffs, labels and boundary tokens
must match exactly."""
import ctypes
import heapq
import math

import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
import paper_2607_05061_amd as kv  # noqa: E402

pytestmark = pytest.mark.gpu


def _expected(scores, log_gamma, s, w, k, queries=None):
    B, H, T = scores.shape
    exp = {n: np.empty((B, H, T), dtype=np.int64) for n in ("rank", "cutoff", "label", "boundary", "evict")}
    for b in range(B):
        for h in range(H):
            lg = 0.0 if log_gamma is None else log_gamma[h]
            prio = oracle.static_priority_f32(scores[b, h], lg)
            rank = oracle.ranks_from_priority(prio)
            tau = oracle.running_cutoff_fenwick(rank, s, w, k)
            y, tb = oracle.teacher_labels(rank, tau, s, w, queries)
            exp["rank"][b, h], exp["cutoff"][b, h] = rank, tau
            exp["label"][b, h], exp["boundary"][b, h] = y, tb
            exp["evict"][b, h] = oracle.eviction_times(rank, tau, s, w)
    return exp


def _run(scores, log_gamma, s, w, k, labels=True, evict=True):
    sc = torch.from_numpy(scores).to("cuda")
    lg = torch.from_numpy(np.asarray(log_gamma, dtype=np.float32)).to("cuda") if log_gamma is not None else None
    out = kv.kvpop_running_topk(sc, s, w, k, log_gamma=lg, labels=labels, evict=evict)
    torch.cuda.synchronize()
    return {n: v.cpu().numpy().astype(np.int64) for n, v in out.items()}


def test_hand_case():
    scores = np.array([[[5.0, 2.0, 4.0, 1.0, 3.0]]], dtype=np.float32)  # ranks (0, 3, 1, 4, 2)
    got = _run(scores, None, 1, 1, 2)
    np.testing.assert_array_equal(got["rank"][0, 0], [0, 3, 1, 4, 2])
    np.testing.assert_array_equal(got["cutoff"][0, 0], [5, 5, 5, 3, 3])
    np.testing.assert_array_equal(got["label"][0, 0], [0, 0, 1, 1, -1])
    np.testing.assert_array_equal(got["boundary"][0, 0], [-1, -1, 1, 1, 1])
    np.testing.assert_array_equal(got["evict"][0, 0], [5, 5, 5, 4, 5])


CASES = [
    # B, H, T, s, w, k
    (1, 1, 1, 0, 0, 1),
    (1, 2, 2, 0, 1, 1),
    (2, 3, 17, 1, 2, 3),
    (1, 2, 300, 4, 16, 20),
    (2, 2, 1000, 4, 64, 128),
    (1, 1, 4097, 4, 256, 1000),
    (1, 2, 513, 0, 0, 1),
    (1, 1, 600, 10, 5, 700),   # never saturated
    (1, 1, 50, 60, 3, 2),      # sinks beyond T: nothing eligible
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "B%dH%dT%d_s%dw%dk%d" % c)
@pytest.mark.parametrize("decay", [False, True])
def test_matches_oracle(case, decay):
    B, H, T, s, w, k = case
    rng = np.random.default_rng(T * 7 + k)
    scores = rng.standard_normal((B, H, T)).astype(np.float32) * 3
    log_gamma = np.log(rng.uniform(0.99, 0.9999, size=H)).astype(np.float32) if decay else None
    got = _run(scores, log_gamma, s, w, k)
    exp = _expected(scores, log_gamma, s, w, k)
    for n in ("rank", "cutoff", "label", "boundary", "evict"):
        np.testing.assert_array_equal(got[n], exp[n], err_msg=n)


def test_ties_break_to_earlier_position():
    rng = np.random.default_rng(3)
    scores = (np.round(rng.standard_normal((2, 2, 700)) * 2) / 2).astype(np.float32)  # many exact ties
    got = _run(scores, None, 2, 8, 40)
    exp = _expected(scores, None, 2, 8, 40)
    for n in ("rank", "cutoff", "label", "boundary", "evict"):
        np.testing.assert_array_equal(got[n], exp[n], err_msg=n)


def test_ties_across_sorted_chunks():
    """Exact ties spanning the 4096-position chunks that the ranking sorts one
    workgroup each (three whole chunks and a ragged one): every tie still breaks to the
    earlier position, an all-equal sequence ranks by position, and -0.0 ties +0.0."""
    rng = np.random.default_rng(8)
    T = 3 * 4096 + 123
    scores = (np.round(rng.standard_normal((1, 3, T)) * 2) / 2).astype(np.float32)
    scores[0, 1] = 1.5
    scores[0, 2, ::2] = -0.0
    scores[0, 2, 1::2] = 0.0
    scores[0, 2, 5000:5010] = 2.0
    got = _run(scores, None, 4, 256, 2016)
    exp = _expected(scores, None, 4, 256, 2016)
    for n in ("rank", "cutoff", "label", "boundary", "evict"):
        np.testing.assert_array_equal(got[n], exp[n], err_msg=n)
    np.testing.assert_array_equal(got["rank"][0, 1], np.arange(T))


def test_labels_optional():
    scores = np.random.default_rng(4).standard_normal((1, 2, 200)).astype(np.float32)
    got = _run(scores, None, 1, 4, 10, labels=False, evict=False)
    assert set(got) == {"rank", "cutoff"}
    exp = _expected(scores, None, 1, 4, 10)
    np.testing.assert_array_equal(got["cutoff"], exp["cutoff"])


def test_paper_budget_at_benchmark_size():
    """The paper's budget (s=4, w=256, k=2016) on the Qwen3-8B-shaped T=32768 layout
    (B=4, 8 KV heads) with learned-decay-range log gammas: ranks and cutoffs of every
    sequence exactly, labels and boundaries on sampled queries."""
    B, H, T, s, w, k = 4, 8, 32768, 4, 256, 2016
    rng = np.random.default_rng(5)
    scores = rng.standard_normal((B, H, T)).astype(np.float32)
    log_gamma = (math.log(0.999) + rng.random(H) * (math.log(0.999999) - math.log(0.999))).astype(np.float32)
    got = _run(scores, log_gamma, s, w, k)
    qs = sorted(set(rng.integers(0, T, 64).tolist()) | {0, s + w - 1, s + w, s + w + k - 2, s + w + k - 1, T - 1})
    for b, h in [(0, 0), (1, 5), (3, 7)]:
        e = _expected(scores[b:b + 1, h:h + 1], log_gamma[h:h + 1], s, w, k, queries=qs)
        np.testing.assert_array_equal(got["rank"][b, h], e["rank"][0, 0])
        np.testing.assert_array_equal(got["cutoff"][b, h], e["cutoff"][0, 0])
        np.testing.assert_array_equal(got["evict"][b, h], e["evict"][0, 0])
        np.testing.assert_array_equal(got["label"][b, h, qs], e["label"][0, 0, qs])
        np.testing.assert_array_equal(got["boundary"][b, h, qs], e["boundary"][0, 0, qs])
    # every sequence: ranks are a permutation, cutoffs monotone once saturated
    for b in range(B):
        for h in range(H):
            assert np.array_equal(np.sort(got["rank"][b, h]), np.arange(T))
            c = got["cutoff"][b, h]
            assert np.all(np.diff(c[s + w + k - 1:]) <= 0) and np.all(c[:s + w + k - 1] == T)


def test_long_context_t131072():
    """T = 131072 (the long-context workload's length), paper budget, decay on: ranks,
    cutoffs and eviction queries of two heads in full, labels and boundaries sampled."""
    H, T, s, w, k = 4, 131072, 4, 256, 2016
    rng = np.random.default_rng(21)
    scores = rng.standard_normal((1, H, T)).astype(np.float32)
    log_gamma = np.log(np.linspace(0.999, 0.999999, H)).astype(np.float32)
    got = _run(scores, log_gamma, s, w, k)
    qs = sorted(set(rng.integers(0, T, 48).tolist()) | {0, s + w + k - 1, T - 1})
    for h in (0, 3):
        e = _expected(scores[:, h:h + 1], log_gamma[h:h + 1], s, w, k, queries=qs)
        for n in ("rank", "cutoff", "evict"):
            np.testing.assert_array_equal(got[n][0, h], e[n][0, 0], err_msg=n)
        np.testing.assert_array_equal(got["label"][0, h, qs], e["label"][0, 0, qs])
        np.testing.assert_array_equal(got["boundary"][0, h, qs], e["boundary"][0, 0, qs])


@pytest.mark.parametrize("T", [32771, 32772, 40000, 136072])
def test_ragged_chunks_and_runs(T):
    """Several sorted chunks of 4096 positions, the last one of 3, 4 or 3136 (T = 32771,
    32772, 40000), and two runs of chunks, the second of 5000 positions (T = 136072).
    Ranks, cutoffs and eviction queries of every position exactly, labels and boundaries
    on sampled queries."""
    s, w, k = 4, 256, 2016
    rng = np.random.default_rng(T)
    scores = rng.standard_normal((1, 2, T)).astype(np.float32)
    log_gamma = np.log(np.array([0.9999, 0.99999])).astype(np.float32)
    got = _run(scores, log_gamma, s, w, k)
    qs = sorted(set(rng.integers(0, T, 40).tolist()) | {0, s + w + k - 1, T - 1})
    for h in range(2):
        e = _expected(scores[:, h:h + 1], log_gamma[h:h + 1], s, w, k, queries=qs)
        for n in ("rank", "cutoff", "evict"):
            np.testing.assert_array_equal(got[n][0, h], e[n][0, 0], err_msg=n)
        np.testing.assert_array_equal(got["label"][0, h, qs], e["label"][0, 0, qs])
        np.testing.assert_array_equal(got["boundary"][0, h, qs], e["boundary"][0, 0, qs])


def test_many_sequences_of_ragged_length():
    """64 sequences of T = 12411 (a ragged last block of queries, and more workgroups of
    queries than the chip holds at once). Ranks, cutoffs and eviction queries of three
    sequences exactly, labels and boundaries on sampled queries."""
    B, H, T, s, w, k = 8, 8, 12411, 4, 256, 2016
    rng = np.random.default_rng(77)
    scores = rng.standard_normal((B, H, T)).astype(np.float32)
    log_gamma = np.log(np.linspace(0.999, 0.99999, H)).astype(np.float32)
    got = _run(scores, log_gamma, s, w, k)
    qs = sorted(set(rng.integers(0, T, 48).tolist()) | {0, s + w + k - 2, s + w + k - 1, T - 1})
    for b, h in [(0, 0), (3, 5), (7, 7)]:
        e = _expected(scores[b:b + 1, h:h + 1], log_gamma[h:h + 1], s, w, k, queries=qs)
        for n in ("rank", "cutoff", "evict"):
            np.testing.assert_array_equal(got[n][b, h], e[n][0, 0], err_msg=n)
        np.testing.assert_array_equal(got["label"][b, h, qs], e["label"][0, 0, qs])
        np.testing.assert_array_equal(got["boundary"][b, h, qs], e["boundary"][0, 0, qs])


def _cutoffs_by_heap(rank, s, w, k):
    """The running cutoff from its definition with a heap of the k smallest ranks so far,
    for lengths at which the oracle's Fenwick scan takes too long."""
    T = rank.shape[0]
    cut, kept, ranks = np.full(T, T, dtype=np.int64), [], rank.tolist()
    for q in range(s + w, T):
        heapq.heappush(kept, -ranks[q - w])
        if len(kept) > k:
            heapq.heappop(kept)
        if len(kept) == k:
            cut[q] = -kept[0]
    return cut


EDGES = [
    # T, s, w, k: one token to each side of a query block, a sorted chunk, a run and the
    # widest census
    (1023, 0, 0, 100), (1025, 4, 0, 1024), (2049, 4, 1, 700), (4096, 4, 256, 2016), (4097, 0, 64, 1),
    (8193, 3, 256, 4000), (131072, 4, 256, 2016), (131073, 4, 256, 2016), ((1 << 20) + 100003, 4, 256, 2016),
]


@pytest.mark.parametrize("kind", ["rising", "falling", "waves"])
@pytest.mark.parametrize("case", EDGES, ids=lambda c: "T%d_s%dw%dk%d" % c)
def test_edges_of_blocks_chunks_and_runs(case, kind):
    """Scores that keep every arriving token (rising), none (falling) or stretches of them
    (waves, with ties), at the sizes where the ranking's pieces end."""
    T, s, w, k = case
    rng = np.random.default_rng(T + len(kind))
    t = np.arange(T, dtype=np.float32)
    scores = {"rising": t * 0.01 + rng.standard_normal(T) * 0.1, "falling": rng.standard_normal(T) * 0.1 - t * 0.01,
              "waves": np.round(np.sin(t / 311.0) * 40 + rng.standard_normal(T)) / 4}[kind].astype(np.float32)
    got = _run(scores[None, None], None, s, w, k)
    rank = oracle.ranks_from_priority(oracle.static_priority_f32(scores, 0.0))
    np.testing.assert_array_equal(got["rank"][0, 0], rank)
    cut = _cutoffs_by_heap(rank, s, w, k) if T > 5000 else oracle.running_cutoff_fenwick(rank, s, w, k)
    np.testing.assert_array_equal(got["cutoff"][0, 0], cut)
    np.testing.assert_array_equal(got["evict"][0, 0], oracle.eviction_times(rank, cut, s, w))
    qs = sorted(set(rng.integers(0, T, 24).tolist()) | {0, min(T - 1, s + w + k - 1), T - 1})
    y, tb = oracle.teacher_labels(rank, cut, s, w, qs)
    np.testing.assert_array_equal(got["label"][0, 0, qs], y[qs])
    np.testing.assert_array_equal(got["boundary"][0, 0, qs], tb[qs])


@pytest.mark.parametrize("k", [1, 128, 1023, 1024, 1025])
@pytest.mark.parametrize("kind", ["rising", "low_start", "waves"])
def test_budgets_around_a_block_of_queries(k, kind):
    """Budgets up to, at and above the 1024 queries of a block, with scores of which every
    arrival is kept (rising), every arrival but the first few tokens' places (low_start: the
    first 200 tokens outrank all later ones) or stretches (waves): the block's candidates
    then end among its own tokens, among old ones, or span all later tokens' ranks."""
    T, s, w = 20003, 4, 64
    rng = np.random.default_rng(k + len(kind))
    t = np.arange(T, dtype=np.float32)
    scores = {"rising": t * 0.01, "low_start": t * 0.01 + 1e4 * (t < 200),
              "waves": np.sin(t / 911.0) * 40 + rng.standard_normal(T)}[kind].astype(np.float32)
    got = _run(scores[None, None], None, s, w, k)
    rank = oracle.ranks_from_priority(oracle.static_priority_f32(scores, 0.0))
    cut = _cutoffs_by_heap(rank, s, w, k)
    np.testing.assert_array_equal(got["rank"][0, 0], rank)
    np.testing.assert_array_equal(got["cutoff"][0, 0], cut)
    np.testing.assert_array_equal(got["evict"][0, 0], oracle.eviction_times(rank, cut, s, w))
    qs = sorted(set(rng.integers(0, T, 24).tolist()) | {s + w + k - 1, T - 1})
    y, tb = oracle.teacher_labels(rank, cut, s, w, qs)
    np.testing.assert_array_equal(got["label"][0, 0, qs], y[qs])
    np.testing.assert_array_equal(got["boundary"][0, 0, qs], tb[qs])


def _ms(f, n=3):
    f()
    best = math.inf
    for _ in range(n):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        f()
        b.record()
        b.synchronize()
        best = min(best, a.elapsed_time(b))
    return best


@pytest.mark.parametrize("kind", ["rising", "low_start"])
def test_small_budget_costs_no_more_than_a_large_one(kind):
    """The work per query block does not grow with T where a block brings more kept tokens
    than the budget holds: 4 million rising scores with k = 128 take about the time of
    k = 2016 (0.33 ms; a scan past the block's last cutoff would read the whole ranking in
    each of the 4096 blocks: 10 ms)."""
    T = 1 << 22
    t = torch.arange(T, device="cuda", dtype=torch.float32)
    scores = (t * 0.01 + (1e6 * (t < 200) if kind == "low_start" else 0.0))[None, None].contiguous()
    ws = torch.empty(kv.kvpop_running_topk_workspace_size(1, 1, T), dtype=torch.uint8, device="cuda")
    small = _ms(lambda: kv.kvpop_running_topk(scores, 4, 64, 128, workspace=ws))
    large = _ms(lambda: kv.kvpop_running_topk(scores, 4, 64, 2016, workspace=ws))
    assert small <= 4 * large, "k = 128: %.3f ms, k = 2016: %.3f ms" % (small, large)


@pytest.mark.parametrize("case", [(5003, 0, 0, 5003), (12411, 4, 64, 9000), (12411, 4, 64, 1 << 30),
                                  (140003, 7, 256, 140000), ((1 << 20) + 100003, 4, 64, 1 << 20)],
                         ids=lambda c: "T%d_s%dw%dk%d" % c)
def test_boundary_tokens_before_a_late_saturation(case):
    """Budgets so large that most or all queries keep every eligible token: the boundary
    token is the kept one with the largest rank, on each side of the query block from which
    it comes from the census instead of a scan of the earlier ranks."""
    T, s, w, k = case
    rng = np.random.default_rng(T)
    scores = rng.standard_normal(T).astype(np.float32)
    got = _run(scores[None, None], None, s, w, k)
    rank = oracle.ranks_from_priority(oracle.static_priority_f32(scores, 0.0))
    cut = _cutoffs_by_heap(rank, s, w, k)
    np.testing.assert_array_equal(got["cutoff"][0, 0], cut)
    largest = np.maximum.accumulate(rank[s:T - w])  # over the eligible tokens, at query s + w + i
    last = min(T - w - s, k - 1)                    # queries before saturation
    at = np.empty(T, dtype=np.int64)
    at[rank] = np.arange(T)
    np.testing.assert_array_equal(got["boundary"][0, 0, :s + w], -1)
    np.testing.assert_array_equal(got["boundary"][0, 0, s + w:s + w + last], at[largest[:last]])
    np.testing.assert_array_equal(got["boundary"][0, 0, s + w + last:], at[cut[s + w + last:]])


def test_a_budget_of_every_token_costs_no_more_than_a_large_one():
    """The boundary tokens before saturation cost the same work per block at any T: 8
    sequences of 4 million with k = T in about the time of k = 2016 (6.4 ms; 39 ms if each
    block scanned all earlier ranks)."""
    T = 1 << 22
    scores = torch.randn(1, 8, T, device="cuda")
    ws = torch.empty(kv.kvpop_running_topk_workspace_size(1, 8, T), dtype=torch.uint8, device="cuda")
    full = _ms(lambda: kv.kvpop_running_topk(scores, 4, 64, T, workspace=ws))
    large = _ms(lambda: kv.kvpop_running_topk(scores, 4, 64, 2016, workspace=ws))
    assert full <= 4 * large, "k = T: %.3f ms, k = 2016: %.3f ms" % (full, large)


def test_more_than_2_pow_32_query_threads():
    """2^21 + 64 sequences of 1025 positions, two blocks of 1024 queries each: over 2^32
    work-items of queries. With s = w = 0 the last cutoff of every sequence is k - 1, and the
    queries before saturation keep everything; three sequences exactly. 88 GB of memory."""
    if torch.cuda.mem_get_info()[0] < 110e9:
        pytest.skip("needs 110 GB of free memory")
    n, T, k = (1 << 21) + 64, 1025, 100
    scores = torch.randn(n, 1, T, device="cuda", generator=torch.Generator("cuda").manual_seed(9))
    ws = torch.empty(kv.kvpop_running_topk_workspace_size(n, 1, T), dtype=torch.uint8, device="cuda")
    rank, cut = (torch.full((n, 1, T), -7, dtype=torch.int32, device="cuda") for _ in range(2))
    d = kv.KvpopTopkDims(n, 1, T)
    st = kv.lib().kvpop_running_topk(ctypes.byref(d), scores.data_ptr(), None, 0, 0, k, rank.data_ptr(),
                                     cut.data_ptr(), None, None, None, ws.data_ptr(), ws.numel(),
                                     torch.cuda.current_stream().cuda_stream)
    assert st == kv.KVPOP_OK
    assert bool((cut[..., :k - 1] == T).all()) and bool((cut[..., T - 1] == k - 1).all())
    for i in (0, (1 << 20) + 3, n - 1):
        e = _expected(scores[i:i + 1].cpu().numpy(), None, 0, 0, k)
        np.testing.assert_array_equal(rank[i].cpu().numpy(), e["rank"][0])
        np.testing.assert_array_equal(cut[i].cpu().numpy(), e["cutoff"][0])
    del scores, ws, rank, cut
    torch.cuda.empty_cache()
