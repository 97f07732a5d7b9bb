"""Rounds without sweeps: the witness test, the second chances and the
screened exact pass, at the sizes where they can go wrong -- series around the
screening's smallest size and around multiples of its 512-column chunks and
128-column blocks, windows around the 256-offset staging chunk, flat
stretches, a series with a huge spike (which widens the screening's error
bound) -- against profiles in FP64 by plain matrix products
of the reference's z-normalised windows: the top-k rows, and through the
heatmap every length's range discords with their exact distances.  Tolerance
as in the other parity tests (ED^2 = 2m (1 - rho), rho to 1e-12)."""

import sys

import numpy as np
import pytest

from oracle import bruteforce as bf
from paper_2304_01660_amd import synth
from parity_helpers import close_ed

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SCREEN_MIN = 8192  # subsequences; longer series are screened


def _dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


def _say(*a):
    print("[case]", *a, file=sys.stderr, flush=True)


def _series(kind, n, seed):
    rng = np.random.default_rng([seed, n])
    if kind in ("rw", "ecg", "noise"):
        return synth.small_random(seed, n, kind)
    if kind == "flat":  # plateaus of up to 150 points between walks
        T = np.cumsum(rng.standard_normal(n))
        for _ in range(max(2, n // 1500)):
            p = int(rng.integers(0, n - 200))
            T[p:p + int(rng.integers(60, 150))] = T[p]
        return T
    if kind == "spike":
        T = synth.small_random(seed, n, "ecg")
        T[n // 3] += 1.0e6
        return T
    raise ValueError(kind)


def _profile(T, m, dev):
    """Distance of every subsequence to its nearest non-self match."""
    Z, _, _, flat = bf.znorm_windows(T, m)
    Z = torch.from_numpy(np.ascontiguousarray(Z)).to(dev)
    f = torch.from_numpy(flat).to(dev)
    N = Z.shape[0]
    Zt = Z.t().contiguous()
    i = torch.arange(N, device=dev)
    best = []
    for a in range(0, N, 2048):
        rows = i[a:a + 2048]
        rho = Z[a:a + 2048] @ Zt / m
        rho[f[a:a + 2048][:, None] & f[None, :]] = 1.0
        rho[(i[None, :] - rows[:, None]).abs() < m] = -2.0
        best.append(rho.max(1).values)
    rho = torch.cat(best).clamp(-1.0, 1.0)
    return torch.sqrt(2.0 * m * (1.0 - rho)).cpu().numpy()


CASES = [
    # kind, N at minL, minL, maxL, k
    ("rw", SCREEN_MIN, 20, 23, 3),
    ("ecg", SCREEN_MIN + 1, 31, 35, 2),
    ("noise", SCREEN_MIN + 1, 17, 20, 1),
    ("rw", 8704, 64, 67, 1),            # 17 chunks of 512
    ("ecg", 8705 + 2, 64, 67, 3),       # N crosses 8705 -> 8704 on the way
    ("ecg", 8833, 255, 258, 2),         # windows around 256 offsets
    ("rw", 9000, 511, 513, 2),
    ("flat", 8400, 40, 44, 2),
    ("flat", 1500, 12, 16, 3),
    ("spike", 8300, 50, 54, 2),
    ("rw", 400, 3, 6, 64),              # k at its largest
]


@pytest.mark.parametrize("dist_bits", [32, 64])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_search_and_heatmap_match_bruteforce(case, dist_bits):
    from paper_2304_01660_amd import api
    dev = _dev()
    kind, N, minL, maxL, k = CASES[case]
    n = N + minL - 1
    T = _series(kind, n, 700 + case)
    _say("witness", dist_bits, case, CASES[case], n)
    Td = torch.from_numpy(T).to(dev)
    out = api.discord_heatmap(Td, minL, maxL, k, dist_bits=dist_bits, return_stats=True)
    plain = api.discords(Td, minL, maxL, k, dist_bits=dist_bits)
    for key in ("idx", "len", "nn_dist", "nn_idx", "count"):
        assert torch.equal(out[key], plain[key]), key
    heat = out["heat"].cpu().numpy()
    rng = out["range"].cpu().numpy()
    cnt = out["count"].cpu().numpy()
    nn = out["nn_dist"].cpu().numpy()
    idx = out["idx"].cpu().numpy()
    nbr = out["nn_idx"].cpu().numpy()
    for m in range(minL, maxL + 1):
        li = m - minL
        Nm = n - m + 1
        P = _profile(T, m, dev)
        r = rng[li]
        row = heat[li, :Nm]
        assert np.all(heat[li, Nm:] == 0.0)
        top = np.sort(P)[::-1][:k]
        rows = slice(li * k, (li + 1) * k)
        assert np.all(close_ed(nn[rows], top, m))
        assert np.all(close_ed(nn[rows], P[idx[rows]], m))
        assert np.all(np.abs(nbr[rows] - idx[rows]) >= m)
        for i, j, d in zip(idx[rows], nbr[rows], nn[rows]):
            x, y = T[i:i + m], T[j:j + m]
            if x.std() > 0.0 and y.std() > 0.0:
                rho = np.mean((x - x.mean()) * (y - y.mean())) / (x.std() * y.std())
                assert close_ed(d, np.sqrt(max(0.0, 2.0 * m * (1.0 - rho))), m)
        if r <= 0:
            continue
        member = row > 0.0
        far = ~close_ed(P, np.full_like(P, r), m)
        np.testing.assert_array_equal(member[far], (P >= r)[far])
        assert int(member.sum()) == int(cnt[li])
        assert np.all(close_ed(np.sqrt(2.0 * m * row[member]), P[member], m))


def test_batch_of_screened_and_small_series_equals_single_searches():
    """Candidate groups numbered across series of uneven size."""
    from paper_2304_01660_amd import api
    dev = _dev()
    spec = [("rw", 300, 10, 14), ("ecg", 9500, 60, 66), ("noise", 2000, 12, 14),
            ("rw", 12000, 33, 37), ("flat", 5000, 20, 24), ("ecg", 700, 40, 41)]
    vals = [torch.from_numpy(_series(kind, n, 800 + q)).to(dev)
            for q, (kind, n, _, _) in enumerate(spec)]
    lo = [x[2] for x in spec]
    hi = [x[3] for x in spec]
    for band in (0, 1):
        _say("witness batch", band)
        res = api.discords_batched(vals, lo, hi, 2, band_pass=band)
        for b in range(len(spec)):
            one = api.discords(vals[b], lo[b], hi[b], 2)
            for key in ("idx", "len", "nn_dist", "nn_idx", "count"):
                assert torch.equal(res[b][key], one[key]), (b, key)


@pytest.mark.parametrize("one_past", [0, 1])
def test_refinement_items_of_one_column(one_past):
    """The last item on the left of the series' last tile holds only column 0,
    the only neighbour of one row; so the row is no range discord."""
    from paper_2304_01660_amd import api
    dev = _dev()
    N, m = 1088 + one_past, 255
    T = np.random.default_rng([1088, m]).standard_normal(N + m - 1)
    T[671:671 + m + 3] = T[671]  # a wide guard: the refinement decides
    T[5:5 + m] = T[1047:1047 + m]
    _say("one column", N)
    out = api.discord_heatmap(torch.from_numpy(T).to(dev), m, m, 2)
    r = float(out["range"][0])
    P = _profile(T, m, dev)
    far = ~close_ed(P, np.full_like(P, r), m)
    member = out["heat"].cpu().numpy()[0, :N] > 0.0
    np.testing.assert_array_equal(member[far], (P >= r)[far])


@pytest.mark.parametrize("minL", [31, 64, 96, 127, 255])
@pytest.mark.parametrize("N", [1025, 1088, 1537, 8193])
def test_many_range_discords_match_the_heatmaps_sweeps(N, minL):
    """White noise: at the second range most or all subsequences are range
    discords, which a plain search bounds on the matrix cores and a heatmap
    sweeps for.  Lists one past a tile of 64 rows, columns one past a chunk of
    512, windows around the operand steps of 32 and around 128 and 256."""
    from paper_2304_01660_amd import api
    dev = _dev()
    k, n = 2, N + minL - 1
    T = np.random.default_rng([N, minL]).standard_normal(n)
    T[n // 2:n // 2 + minL + 3] = T[n // 2]       # flat rows, each other's neighbours
    T[5:5 + minL] = T[n - 40 - minL:n - 40]       # a pair without distance
    _say("dense", N, minL)
    Td = torch.from_numpy(T).to(dev)
    plain = api.discords(Td, minL, minL + 2, k)
    swept = api.discord_heatmap(Td, minL, minL + 2, k)
    for key in ("idx", "len", "nn_dist", "nn_idx", "count"):
        assert torch.equal(plain[key], swept[key]), key
    r = float(swept["range"][0])
    P = _profile(T, minL, dev)
    far = ~close_ed(P, np.full_like(P, r), minL)
    if r > 0 and bool(far.all()):
        assert int(plain["count"][0]) == int((P >= r).sum())
    res = api.discords_batched([Td, Td[:n - 1].contiguous()], [minL] * 2, [minL + 2] * 2, k)
    for key in ("idx", "len", "nn_dist", "nn_idx", "count"):
        assert torch.equal(res[0][key], plain[key]), key


@pytest.mark.parametrize("seed", [4, 35, 52])
def test_a_window_flat_at_one_length_starts_its_witness_anew(seed):
    """White noise with one stretch of 200 values around 1e-12: its window is
    flat at m = 200, where its correlation with window 0 counts as 0, and just
    above the flat threshold at m = 201, where half of either window's variance
    is its last value and the rest correlates -1, so that the two do not
    correlate.  The window is one of the 64 discords there."""
    from paper_2304_01660_amd import api
    dev = _dev()
    m, k = 200, 64
    rng = np.random.default_rng([seed, m])
    T = rng.standard_normal(1200 + m)
    p = 700
    w, s = T[:m] - T[:m].mean(), T[:m].std()
    last = np.sqrt(m * (m + 1) / m)  # f d^2 = m s^2, f = m / (m + 1)
    T[m] = T[:m].mean() + last * s
    T[p:p + m] = -w / s * 0.9e-12
    T[p + m] = last * 0.9e-12
    _, _, _, flat = bf.znorm_windows(T, m)
    assert flat.sum() == 1 and flat[p] and not bf.znorm_windows(T, m + 1)[3].any()
    _say("flat then not", seed)
    out = api.discord_heatmap(torch.from_numpy(T).to(dev), m, m + 1, k)
    P = _profile(T, m + 1, dev)
    r = float(out["range"][1])
    assert P[p] > np.sort(P)[-k]
    far = ~close_ed(P, np.full_like(P, r), m + 1)
    member = out["heat"].cpu().numpy()[1, :P.shape[0]] > 0.0
    np.testing.assert_array_equal(member[far], (P >= r)[far])
    assert p in out["idx"].cpu().numpy()[k:]


@pytest.mark.parametrize("sizes", [(9000, 8500), (12000, 300, 30000, 9001, 700), (300000, 9500, 260000)])
def test_batches_small_and_large_equal_single_searches(sizes):
    """The screening takes candidate groups one at a time or four, and the exact
    pass 512 or 1024 workgroups, by the batch's chunks: up to 1024 of 512 columns
    and beyond."""
    from paper_2304_01660_amd import api
    dev = _dev()
    vals = [torch.from_numpy(_series("ecg" if q % 2 else "rw", n, 810 + q)).to(dev)
            for q, n in enumerate(sizes)]
    lo = [30 + 20 * q for q in range(len(sizes))]
    hi = [a + 6 for a in lo]
    _say("batch chunks", sizes)
    res = api.discords_batched(vals, lo, hi, 3)
    for b, T in enumerate(vals):
        one = api.discords(T, lo[b], hi[b], 3)
        for key in ("idx", "len", "nn_dist", "nn_idx", "count"):
            assert torch.equal(res[b][key], one[key]), (b, key)
