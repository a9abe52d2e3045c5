"""Parity of the fused target epilogue (App. D.4 step 5) with the oracle.

scores[b, h, t] = log(agg_g m_bar + eps) - log N_t is compared in absolute terms:
a 2e-3 relative error on the masses is at most ~2e-3 on their logarithm, so the bar
is |gpu - oracle| <= 2e-3 (+ 1e-5 for the fp32 logarithm itself).
"""
import ctypes
import math

import numpy as np
import pytest

import oracle
import workload

torch = pytest.importorskip("torch")
import paper_2607_05061_amd as kv  # noqa: E402

pytestmark = pytest.mark.gpu
ABS = 2e-3 + 1e-5


def _dev(bits):
    return torch.from_numpy(np.ascontiguousarray(bits).view(np.int16)).view(torch.bfloat16).to("cuda")


def _cfg(B, Hq, Hkv, T, D, seed, kind="rope", sink=False):
    return dict(seed=seed, B=B, Hq=Hq, Hkv=Hkv, T=T, D=D, scale=1.0 / math.sqrt(D), kind=kind, sink=sink,
                bands=[(0, -1)])


def _scores(w, window, horizon, agg, eps, normalize, bias=None, write_mass=False):
    q, k = _dev(w.q_bits), _dev(w.k_bits)
    bias = w.bias if bias is None else bias
    b = torch.from_numpy(np.ascontiguousarray(bias, dtype=np.float32)).to("cuda") if bias is not None else None
    lse = kv.kvpop_row_lse(q, k, w.scale, key_bias=b)
    sc, out = kv.kvpop_future_attn_scores(q, k, lse, w.scale, window, horizon, agg=agg, eps=eps,
                                          normalize=normalize, key_bias=b, write_mass=write_mass)
    mass = kv.kvpop_future_attn_from_lse(q, k, lse, w.scale, window, horizon, key_bias=b)
    torch.cuda.synchronize()
    return (sc.cpu().numpy().astype(np.float64), None if out is None else out.cpu().numpy(),
            mass.cpu().numpy())


def _check(got, ref, what):
    fin = np.isfinite(ref)
    assert np.array_equal(np.isfinite(got), fin), what + ": infinite entries differ"
    assert np.all(got[~fin] == ref[~fin]), what
    err = np.abs(got[fin] - ref[fin])
    assert err.max() <= ABS, "%s: max abs err %.3e" % (what, err.max())


CASES = [
    # B, Hq, Hkv, T, D, window, horizon
    (1, 4, 1, 300, 128, 0, -1),
    (2, 8, 2, 257, 128, 1, 64),
    (1, 6, 2, 200, 64, 3, -1),
    (1, 5, 1, 130, 128, 0, 10),
    (1, 16, 2, 96, 128, 1, -1),
    (1, 1, 1, 70, 64, 0, 0),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "B%dHq%dHkv%dT%dD%d_w%d_h%d" % c)
@pytest.mark.parametrize("agg", ["max", "mean"])
def test_scores_match_oracle(case, agg):
    B, Hq, Hkv, T, D, win, hor = case
    w = workload.make(_cfg(B, Hq, Hkv, T, D, seed=T + Hq))
    m_ref = oracle.future_mass(w.q_bits, w.k_bits, w.scale, None, win, hor)
    for eps, normalize in [(1e-8, True), (1e-3, False), (0.0, True)]:
        got, out, mass = _scores(w, win, hor, agg, eps, normalize, write_mass=True)
        ref = oracle.target_scores(m_ref, Hkv, win, hor, agg=agg, eps=eps, normalize=normalize)
        _check(got, ref, "case %s agg %s eps %g norm %s" % (case, agg, eps, normalize))
        # the per-head masses written by the fused kernel are the plain pass-2 masses,
        # bit for bit (a launch this small spreads plain pass 2's query heads over
        # more workgroups; each still sums its keys' terms in the same order)
        np.testing.assert_array_equal(out, mass)


def test_scores_with_sink_and_masked_keys():
    T = 400
    w = workload.make(_cfg(1, 8, 2, T, 128, seed=41, sink=True))
    bias = w.bias.copy()
    bias[5::9] = -np.inf
    m_ref = oracle.future_mass(w.q_bits, w.k_bits, w.scale, bias, 1, 50)
    for agg in ("max", "mean"):
        got, _, _ = _scores(w, 1, 50, agg, 1e-8, True, bias=bias)
        _check(got, oracle.target_scores(m_ref, 2, 1, 50, agg=agg, eps=1e-8), "sink/masked " + agg)


def test_scores_full_size_sampled():
    """T=32768 benchmark workload: the last 48 keys of two KV heads (all 4 query
    heads each) against the oracle's columns."""
    w = workload.make("qwen3_8b_t32k")
    got, out, mass = _scores(w, 0, -1, "max", 1e-8, True, write_mass=True)
    # the fused and plain launches sum every key's terms in one order
    np.testing.assert_array_equal(out, mass)
    cols = list(range(w.T - 48, w.T))
    for b, h in [(0, 2), (3, 7)]:
        m = np.stack([oracle.future_mass_columns(w.q_bits[b, h * 4 + g], w.k_bits[b, h], w.scale, cols)
                      for g in range(4)])
        r = np.log(m.max(axis=0) + 1e-8) - np.log(np.maximum(1, w.T - np.array(cols)))
        assert np.max(np.abs(got[b, h, cols] - r)) <= ABS


def test_scores_one_batch_row_full_length():
    """B = 1, T = 32768: plain pass 2 and the scores' call with an array for the masses
    spread each key block's query heads over two workgroups, in one form (masses bit for
    bit), and keys of the last key blocks match the oracle's columns."""
    w = workload.make("qwen3_8b_t32k", B=1)
    _, out, mass = _scores(w, 0, -1, "mean", 1e-8, True, write_mass=True)
    np.testing.assert_array_equal(out, mass)
    cols = [32000, 32300, 32511, 32512] + list(range(w.T - 8, w.T))
    for qh in (5, 26):
        m = oracle.future_mass_columns(w.q_bits[0, qh], w.k_bits[0, qh // 4], w.scale, cols)
        rel = np.abs(mass[0, qh, cols] - m) / m
        assert rel.max() <= 2e-3, "qh %d: mass max rel err %.3e" % (qh, rel.max())


FORMS = [
    # B, Hq, Hkv, T, D, (window, horizon): on each side of the lines between pass 2's launch
    # forms (key subtiles per wave, query heads per workgroup; 0: whole sweeps); n = ceil(T / 256)
    # B Hkv blocks, n G pairs
    (1, 4, 2, 511, 128, (0, -1)),      # one extra head of 511 rows: fused epilogue, 2 / 0
    (1, 4, 2, 512, 128, (0, -1)),      # 512: heads spread, epilogue after them, 2 / 1
    (2, 6, 2, 300, 64, (1, 150)),      # odd group, lookahead of exactly T / 2: 2 / 1
    (2, 6, 2, 300, 64, (1, 149)),      # a short band: 2 / 0
    (4, 32, 8, 2287, 128, (0, -1)),    # under 4096 positions, n = 288, 576 workgroups: 2 / 2
    (4, 32, 8, 1900, 64, (0, -1)),     # n = 256, 480 workgroups: 2 / 1
    (8, 32, 8, 2100, 64, (0, -1)),     # n = 576: 4 / 2
    (8, 16, 8, 2100, 128, (0, -1)),    # n = 576, two heads are all: 4 / 0
    (1, 48, 8, 4096, 64, (0, -1)),     # 4096 positions, 768 pairs: 2 / 1
    (2, 32, 8, 4096, 128, (0, -1)),    # n = 256, 1024 pairs: 2 / 2
    (2, 32, 8, 4600, 128, (0, -1)),    # 1152 pairs: 4 / 1
    (2, 32, 8, 4600, 64, (0, -1)),     # D = 64: 2 / 2
    (4, 24, 4, 4300, 64, (0, -1)),     # G = 6: 2 / 2
    (1, 16, 8, 8191, 128, (0, -1)),    # n = 256, 512 pairs: 2 / 1
    (1, 24, 8, 8192, 128, (0, -1)),    # 768 pairs: 4 / 1
    (1, 32, 8, 7900, 64, (0, -1)),     # 992 pairs below 8192 positions: 2 / 2
    (1, 32, 8, 8192, 64, (0, -1)),     # 1024 pairs: 4 / 1
    (4, 32, 8, 4096, 64, (0, -1)),     # n = 512: 4 / 1
    (8, 32, 8, 4096, 128, (0, -1)),    # n = 1024, 4096 pairs: 4 / 2
    (8, 64, 8, 3900, 128, (0, -1)),    # n = 1024, 8192 pairs: 4 / 0
    (8, 16, 8, 4096, 64, (0, -1)),     # n = 1024, G = 2, D = 64: 4 / 1
]


def _scores_without_masses(q, k, lse, scale, win, hor, agg, bias):
    """kvpop_future_attn_scores with out = NULL: always the fused epilogue."""
    B, Hq, T, D = q.shape
    d = kv.KvpopDims(B, Hq, k.shape[1], T, D, float(scale))
    sc = torch.full((B, k.shape[1], T), float("nan"), device="cuda")
    st = kv.lib().kvpop_future_attn_scores(
        ctypes.byref(d), q.data_ptr(), k.data_ptr(), bias.data_ptr() if bias is not None else None, lse.data_ptr(), win,
        hor, kv.KVPOP_AGG_MAX if agg == "max" else kv.KVPOP_AGG_MEAN, 1e-8, 1, None, sc.data_ptr(),
        torch.cuda.current_stream().cuda_stream)
    assert st == kv.KVPOP_OK
    return sc


@pytest.mark.parametrize("agg", ["max", "mean"])
@pytest.mark.parametrize("biased", [False, True], ids=["plain", "biased"])
@pytest.mark.parametrize("case", FORMS, ids=lambda c: "B%dHq%dHkv%dT%dD%d_%d_%d" % (c[:5] + c[5]))
def test_spread_and_fused_epilogues_agree(case, biased, agg):
    """The epilogue fused into pass 2 (the C entry without an array for the masses), and the
    binding's call with and without masses: masses equal to plain pass 2's bit for bit, and
    scores that are the epilogue of those masses to the rounding of two float32 logarithms
    (1e-5) and, fused, of sums of up to T terms in another order (T 2^-24 at most, their
    square root in practice: 1e-5 too). Biased: keys at -inf, mass 0, and one at -40, whose
    block takes the exact sweep."""
    B, Hq, Hkv, T, D, (win, hor) = case
    w = workload.make(dict(seed=T + Hq, B=1, Hq=Hq, Hkv=Hkv, T=T, D=D, scale=1.0 / math.sqrt(D), kind="rope",
                           sink=False, bands=[(0, -1)]))
    q, k = (_dev(x).expand(B, -1, -1, -1).contiguous() for x in (w.q_bits, w.k_bits))
    bias = None
    if biased:
        bias = torch.zeros(T, device="cuda")
        bias[5::97] = -math.inf
        bias[T // 3] = -40.0
    lse = kv.kvpop_row_lse(q, k, w.scale, key_bias=bias)
    a, none = kv.kvpop_future_attn_scores(q, k, lse, w.scale, win, hor, agg=agg, key_bias=bias)
    b, mass = kv.kvpop_future_attn_scores(q, k, lse, w.scale, win, hor, agg=agg, key_bias=bias, write_mass=True)
    fused = _scores_without_masses(q, k, lse, w.scale, win, hor, agg, bias)
    plain = kv.kvpop_future_attn_from_lse(q, k, lse, w.scale, win, hor, key_bias=bias)
    assert none is None
    assert torch.equal(mass, plain)
    if biased:
        assert bool((plain[..., 5::97] == 0).all())
    m = plain.double().view(B, Hkv, Hq // Hkv, T)
    t = torch.arange(T, device="cuda")
    count = ((t + (hor if hor >= 0 else T)).clamp(max=T - 1) - (t + win) + 1).clamp(min=1)
    ref = ((m.amax(2) if agg == "max" else m.mean(2)) + 1e-8).log() - count.double().log()
    for what, got in (("binding", a), ("with masses", b), ("fused", fused)):
        err = (got.double() - ref).abs().max().item()
        assert err <= 2e-5, "%s: %.2e" % (what, err)


@pytest.mark.parametrize("case", [
    # B, H, T, D: n = ceil(T / 256) B H key blocks, on each side of 512, 704 and 768
    (4, 8, 3800, 128), (4, 8, 4096, 128), (4, 8, 5300, 64), (4, 8, 5376, 128), (4, 8, 5500, 128), (4, 8, 5900, 64),
    (4, 8, 6000, 64), (4, 8, 6300, 128),
], ids=lambda c: "B%dH%dT%dD%d" % c)
def test_masses_of_one_query_head_per_kv_head(case):
    """G = 1: no heads to spread, so the epilogue is always fused. Its masses equal plain
    pass 2's bit for bit, at every number of key blocks."""
    B, H, T, D = case
    w = workload.make(dict(seed=T, B=B, Hq=H, Hkv=H, T=T, D=D, scale=1.0 / math.sqrt(D), kind="rope", sink=False,
                           bands=[(0, -1)]))
    q, k = _dev(w.q_bits), _dev(w.k_bits)
    lse = kv.kvpop_row_lse(q, k, w.scale)
    _, mass = kv.kvpop_future_attn_scores(q, k, lse, w.scale, 0, -1, write_mass=True)
    plain = kv.kvpop_future_attn_from_lse(q, k, lse, w.scale, 0, -1)
    assert torch.equal(mass, plain)
