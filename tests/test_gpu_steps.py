"""Series whose level jumps (a noisy periodic signal, switched on and off): a
chunk of the screening holds both levels, so its FP16 values resolve the signal
poorly and the error bound decides little.  A dense round then hands over more
pairs than its list holds; it gives up, the sweeps decide, and no later length
of the call tries again.  Heatmaps never take a dense round: every row and
count equals theirs, and the first length's distances are checked in FP64."""

import math
import sys

import numpy as np
import pytest

from parity_helpers import close_ed

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

KEYS = ("idx", "len", "nn_dist", "nn_idx", "count")


def _dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


def _say(*a):
    print("[case]", *a, file=sys.stderr, flush=True)


def stepped(n, m, jump, seed):
    """A sine of twice the noise's power; levels 0 and `jump` deviations of the
    noise in turn, 150 to 600 points each."""
    rng = np.random.default_rng([seed, n])
    T = 2.0 * np.sin(2.0 * np.pi * np.arange(n) / (0.8 * m)) + rng.standard_normal(n)
    p, on = 0, False
    while p < n:
        q = p + int(rng.integers(150, 600))
        T[p:q] += jump if on else 0.0
        p, on = q, not on
    return T


def _profile(T, m):
    """Largest correlation of every window with a non-self match, in FP64."""
    w = T.unfold(0, m, 1)
    w = w - w.mean(1, keepdim=True)
    w = w / w.norm(dim=1, keepdim=True)
    N = w.shape[0]
    col = torch.arange(N, device=T.device)
    out = []
    for a in range(0, N, 2048):
        r = w[a:a + 2048] @ w.t().contiguous()
        r[(col[None, :] - col[a:a + 2048, None]).abs() < m] = -2.0
        out.append(r.max(1).values)
    return torch.cat(out).clamp(-1.0, 1.0)


@pytest.mark.parametrize("jump", [500.0, 1000.0, 3000.0])
@pytest.mark.parametrize("n", [9000, 20011])
@pytest.mark.parametrize("dist_bits", [32, 64])
def test_a_dense_round_that_cannot_decide_gives_up(dist_bits, n, jump):
    from paper_2304_01660_amd import api
    dev = _dev()
    minL, maxL, k = 64, 68, 2
    _say("steps", dist_bits, n, jump)
    T = torch.from_numpy(stepped(n, minL, jump, 11)).to(dev)
    # every first pass covers all columns, so what the selection evaluates beside
    # it are the bounds of dense rounds
    opts = dict(dist_bits=dist_bits, near_cols=1 << 30, return_stats=True)
    plain = api.discords(T, minL, maxL, k, **opts)
    swept = api.discord_heatmap(T, minL, maxL, k, **opts)
    for key in KEYS:
        assert torch.equal(plain[key], swept[key]), key
    rho = _profile(T, minL)
    d = torch.sqrt(2.0 * minL * (1.0 - rho)).cpu().numpy()
    r = float(swept["range"][0])
    assert np.all(close_ed(plain["nn_dist"][:k].cpu().numpy(), np.sort(d)[::-1][:k], minL))
    if not close_ed(d, np.full_like(d, r), minL).any():
        assert int(plain["count"][0]) == int((d >= r).sum())
    # one range search more than the sweeps need: the round that gave up (FP32
    # sweeps repeat a range search of their own where their guard band is wide)
    if dist_bits == 64:
        assert plain["stats"]["range_searches"] <= swept["stats"]["range_searches"] + 1
    # and it gave up early: its rows (about all of them at r = sqrt(m) / 2)
    # against a part of the columns
    N = n - minL + 1
    left = int((d >= r).sum())
    assert math.isclose(r, math.sqrt(minL) / 2) and left > 1024
    if n > 16384:
        st = plain["stats"]
        assert st["kernel_evals"][1] == 0
        assert 0 < st["evals_select"] - st["kernel_evals"][0] < 0.5 * left * N


def test_a_batch_of_stepped_series_equals_single_searches():
    from paper_2304_01660_amd import api
    dev = _dev()
    vals = [torch.from_numpy(stepped(n, 64, j, 12)).to(dev)
            for n, j in ((9000, 1000.0), (1200, 500.0), (12000, 0.0), (8300, 3000.0))]
    _say("steps batch")
    res = api.discords_batched(vals, [64] * 4, [67] * 4, 2)
    for b in range(4):
        one = api.discords(vals[b], 64, 67, 2)
        for key in KEYS:
            assert torch.equal(res[b][key], one[key]), (b, key)


@pytest.mark.parametrize("jump", [90.0, 110.0, 130.0, 150.0])
def test_candidates_of_a_dense_round_beyond_one_exact_pass(jump):
    """Jumps of about a hundred deviations: the bounds still tell range discords
    from the rest, but leave one to several thousand rows that may be among the
    k best, up to and past what the exact pass takes in parts."""
    from paper_2304_01660_amd import api
    dev = _dev()
    T = torch.from_numpy(stepped(20011, 64, jump, 3)).to(dev)
    for k in (2, 64):  # a part carries the k best so far
        _say("parts", jump, k)
        plain = api.discords(T, 64, 66, k)
        swept = api.discord_heatmap(T, 64, 66, k)
        for key in KEYS:
            assert torch.equal(plain[key], swept[key]), (k, key)
    vals = [torch.from_numpy(stepped(n, 64, j, 3)).to(dev)
            for n, j in ((20011, jump), (9000, 0.0), (16011, 1000.0), (14000, jump))]
    res = api.discords_batched(vals, [64] * 4, [66] * 4, 2)
    for b in range(4):
        one = api.discord_heatmap(vals[b], 64, 66, 2)
        for key in KEYS:
            assert torch.equal(res[b][key], one[key]), (b, key)


def test_a_long_series_throws_no_dense_round_away():
    """Beats between quiet baselines, half a million points: between one and
    three thousand candidates at several lengths."""
    from paper_2304_01660_amd import api, synth
    dev = _dev()
    n, minL, maxL, k = 487755, 38, 42, 5
    T, _ = synth.ecg_like(np.random.default_rng([3, n, 43]), n, 5, maxL=43)
    T = torch.from_numpy(synth.fp32_canonical(T)).to(dev)
    _say("parts", n)
    plain = api.discords(T, minL, maxL, k, dist_bits=64, return_stats=True)
    swept = api.discord_heatmap(T, minL, maxL, k, dist_bits=64, return_stats=True)
    for key in KEYS:
        assert torch.equal(plain[key], swept[key]), key
    assert plain["stats"]["range_searches"] == swept["stats"]["range_searches"]


@pytest.mark.parametrize("n, minL, maxL, call", [(14098, 36, 46, "heatmap"), (9000, 300, 306, "heatmap"),
                                                 (20011, 64, 72, "search")])
def test_lengths_that_sweep_ask_for_it_at_once(monkeypatch, n, minL, maxL, call):
    """A heatmap whose lengths keep more range discords than the exact pass
    takes, windows past 256 points, and a search whose dense rounds gave up: a
    round is issued per range search and for the first change of kind, not one
    more per length that finds out that it needs sweeps."""
    from paper_2304_01660_amd import _lib, api, synth
    dev = _dev()
    if call == "search":
        T = stepped(n, minL, 1000.0, 11)
    else:
        T, _ = synth.ecg_like(np.random.default_rng([3, n, maxL]), n, 5, maxL=maxL)
    T = torch.from_numpy(T).to(dev)
    plain = _lib.make_options

    def timed(*a, **kw):  # with timing a launch of rounds is one round
        o = plain(*a, **kw)
        o.flags |= _lib.FLAG_TIME_KERNELS
        return o

    monkeypatch.setattr(_lib, "make_options", timed)
    f = api.discord_heatmap if call == "heatmap" else api.discords
    _say("sweeping lengths", call, n, minL)
    out = f(T, minL, maxL, 5, return_stats=True)
    st = out["stats"]
    issued = st["kernel_launches"][4]
    _say(st["range_searches"], "range searches", issued, "rounds", out["count"].tolist())
    assert issued <= st["range_searches"] + 3


@pytest.mark.parametrize("n, band", [(30000, 1), (66000, 0)])
def test_sweeps_without_witnesses_find_the_range_discords(n, band):
    """White noise with windows past 256 points: thousands of range discords at
    every length, so that from the third on the sweeps keep no witnesses (in
    tiles of 512 rows where the series is long): every length's range discords
    and distances in FP64, and the same rows without a heatmap."""
    from paper_2304_01660_amd import api
    dev = _dev()
    minL, maxL, k = 300, 304, 3
    T = torch.from_numpy(np.random.default_rng([66, n]).standard_normal(n)).to(dev)
    _say("no witnesses", n, band)
    heat = api.discord_heatmap(T, minL, maxL, k, band_pass=band)
    plain = api.discords(T, minL, maxL, k, band_pass=band)
    for key in KEYS:
        assert torch.equal(heat[key], plain[key]), key
    assert int(heat["count"][1:].min()) > 1024
    for m in range(minL, maxL + 1):
        P = torch.sqrt(2.0 * m * (1.0 - _profile(T, m))).cpu().numpy()
        row = heat["heat"][m - minL, :n - m + 1].cpu().numpy()
        r = float(heat["range"][m - minL])
        far = ~close_ed(P, np.full_like(P, r), m)
        np.testing.assert_array_equal((row > 0.0)[far], (P >= r)[far])
        member = row > 0.0
        assert np.all(close_ed(np.sqrt(2.0 * m * row[member]), P[member], m))
        assert int(member.sum()) == int(heat["count"][m - minL])


@pytest.mark.parametrize("chunk", [64, 128, 1024])
def test_the_first_pass_of_a_dense_round_may_be_cut(chunk):
    """Tiles of 128 rows and chunks of 64 columns: a dense round's first pass of
    16,384 columns would take 200,000 workgroups, past the cap; the bounds cover
    what it leaves out."""
    from paper_2304_01660_amd import api, synth
    dev = _dev()
    rng = np.random.default_rng([100, 100000])
    T, _ = synth.inject_bursts(rng, synth.random_walk(rng, 100000), 5, maxL=66)
    T = torch.from_numpy(synth.fp32_canonical(T)).to(dev)
    _say("first pass", chunk)
    plain = api.discords(T, 64, 66, 3, rows_near=128, chunk_cols=chunk)
    swept = api.discord_heatmap(T, 64, 66, 3)
    for key in KEYS:
        assert torch.equal(plain[key], swept[key]), key


def test_a_length_whose_witnesses_all_fail_does_not_end_dense_rounds():
    """Short windows of a noisy beat train: most rows are range discords of the
    first length, so that the second length's witnesses fail and it sweeps; the
    lengths after it take dense rounds again, which refine nothing."""
    from paper_2304_01660_amd import api, synth
    dev = _dev()
    n, minL, maxL, k = 260000, 26, 36, 8
    T, _ = synth.ecg_like(np.random.default_rng([3, n, maxL]), n, 5, maxL=maxL)
    T = torch.from_numpy(synth.fp32_canonical(T)).to(dev)
    _say("failed witnesses", n)
    plain = api.discords(T, minL, maxL, k, return_stats=True)
    swept = api.discord_heatmap(T, minL, maxL, k, return_stats=True)
    for key in KEYS:
        assert torch.equal(plain[key], swept[key]), key
    two = api.discords(T, minL, minL + 1, k, return_stats=True)
    _say([x["stats"]["evals_refine"] for x in (two, plain, swept)], plain["count"].tolist())
    # no more refinement than the first two lengths' beside one length's sweep
    assert plain["stats"]["evals_refine"] <= 2 * two["stats"]["evals_refine"] + n * n // 4
