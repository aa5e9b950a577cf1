"""Parity of atts_calibrate_online / atts_classify_ordinal with the oracle: ranks, classes and
thresholds bit-exact, p-values equal to the oracle's binary64 p rounded once to fp32."""
import numpy as np
import pytest
import torch

from oracle import atts_oracle as O
from synth import WORKLOADS, lognormal_scores
from util import announce, dev

pytestmark = pytest.mark.gpu


def _classify(A, calib, test, alphas, want_p=True, want_q=True):
    M = len(test)
    t = dev(np.asarray(test, dtype=np.float32))
    ranks = torch.full((M,), -7, dtype=torch.int32, device="cuda")
    cls = torch.full((M,), 99, dtype=torch.uint8, device="cuda")
    p = torch.empty(M, dtype=torch.float32, device="cuda") if want_p else None
    q = torch.empty(len(alphas), dtype=torch.float32, device="cuda") if want_q else None
    A.atts_classify_ordinal(calib, t, alphas, ranks, p, cls, q)
    torch.cuda.synchronize()
    return (ranks.cpu().numpy(), cls.cpu().numpy(), None if p is None else p.cpu().numpy(),
            None if q is None else q.cpu().numpy())


def _check_against_oracle(A, calib, cal_np, test, alphas, brute=True):
    ranks, cls, p, q = _classify(A, calib, test, alphas)
    n = len(cal_np)
    c = (O.rank_counts if brute else O.rank_counts_sorted)(cal_np, test)
    r = O.reject_ranks(alphas, n)
    assert np.array_equal(ranks.astype(np.int64), c)
    assert np.array_equal(cls, O.classify(c, r))
    assert np.array_equal(p, O.p_values(c, n).astype(np.float32))
    assert np.array_equal(q, O.quantile_thresholds(cal_np, r).astype(np.float32), equal_nan=True)
    # decisions only (ranks = NULL): the threshold form of the same rule must give the same classes and thresholds
    M = len(test)
    cls2 = torch.full((M,), 77, dtype=torch.uint8, device="cuda")
    q2 = torch.empty(len(alphas), dtype=torch.float32, device="cuda")
    A.atts_classify_ordinal(calib, dev(np.asarray(test, dtype=np.float32)), alphas, None, None, cls2, q2)
    torch.cuda.synchronize()
    assert np.array_equal(cls2.cpu().numpy(), cls)
    assert np.array_equal(q2.cpu().numpy(), q, equal_nan=True)
    if M > 1:                                                  # pointers that are not 16- / 4-byte aligned
        t_all = dev(np.asarray(test, dtype=np.float32))
        cls3 = torch.full((M,), 77, dtype=torch.uint8, device="cuda")
        A.atts_classify_ordinal(calib, t_all[1:], alphas, None, None, cls3[1:], None)
        torch.cuda.synchronize()
        assert np.array_equal(cls3.cpu().numpy()[1:], cls[1:])
    return ranks, cls


def test_small_with_ties_and_special_values():
    import paper_2509_15148_amd as A
    announce("calib small/special")
    cal = np.array([0.5, 1.0, 1.0, 2.0, 2.0, 2.0, 3.5, 4.0, 4.0, -0.0, 0.0, np.inf, -np.inf, np.nan, 1e-45, -1e-45],
                   dtype=np.float32)
    test = np.array([2.0, 0.25, 5.0, 1.0, 3.75, 0.0, -0.0, np.nan, np.inf, -np.inf, 1e-45, -3.0], dtype=np.float32)
    c = A.Calib(64)
    A.atts_calibrate_online(c, dev(cal))
    assert A.atts_calib_size(c) == len(cal)
    for alphas in ([0.3], [0.3, 0.75], [0.01, 0.5, 0.5, 0.99]):
        _check_against_oracle(A, c, cal.astype(np.float64), test, alphas)
    out = torch.empty(len(cal), dtype=torch.float32, device="cuda")
    A.atts_calib_export(c, out)
    got = out.cpu().numpy()
    assert np.isnan(got[0]) and np.array_equal(got[1:], np.sort(cal[~np.isnan(cal)]))
    # empty test batch: only the thresholds are produced
    ranks, cls, p, q = _classify(A, c, np.zeros(0, np.float32), [0.3])
    assert len(ranks) == 0 and q[0] == O.quantile_thresholds(cal.astype(np.float64), O.reject_ranks([0.3], len(cal)))[0]


@pytest.mark.parametrize("sizes", [(1,), (7, 1, 300), (2047, 2048, 2049, 5), (8191, 8193, 5), (65536, 65537, 16, 65535),
                                   (20000, 3, 70001), (200000, 131072 + 17),
                                   # set sizes at and around whole index nodes (32, 1024, 32768 keys)
                                   (31, 1, 1, 991, 1, 31743, 1, 1)])
def test_online_appends_span_sort_chunks_and_merge_paths(sizes):
    """Batches of one sorted run (up to 8192 keys) and of several, one below, at and above those limits; after every append the
    state must equal the sorted union."""
    import paper_2509_15148_amd as A
    announce("calib appends", sizes)
    total = sum(sizes)
    allv = np.round(lognormal_scores(total, seed=sum(sizes)), 3)       # rounding plants many ties
    c = A.Calib(total)
    test = np.concatenate([lognormal_scores(500, seed=77), allv[:50]])
    lo = 0
    for s in sizes:
        A.atts_calibrate_online(c, dev(allv[lo:lo + s]))
        lo += s
        assert A.atts_calib_size(c) == lo
        out = torch.empty(lo, dtype=torch.float32, device="cuda")
        A.atts_calib_export(c, out)
        assert np.array_equal(out.cpu().numpy(), np.sort(allv[:lo]))
        _check_against_oracle(A, c, allv[:lo].astype(np.float64), test, [0.05, 0.2], brute=lo <= 30000)


@pytest.mark.parametrize("base,sizes", [(0, (48,)), (0, (49,)), (700, (47, 48, 49, 50)), (0, (512,)), (3, (510, 511, 512, 513)),
                                        ((1 << 21) - 1000, (512, 48, 440, 1, 30))])
def test_appends_sorted_inside_the_merge(base, sizes):
    """One below, at and above the sizes of the batches that the merge workgroups rank or sort themselves, and of the set that lets
    them; ties, NaN and both infinities in the batch.  The state equals the sorted union after every append."""
    import paper_2509_15148_amd as A
    announce("calib inline sort", base, sizes)
    allv = np.round(lognormal_scores(base + sum(sizes), seed=base % 1000 + 3), 2)
    allv[base:base + 3] = [np.nan, np.inf, -np.inf]
    c = A.Calib(base + sum(sizes))
    if base:
        A.atts_calibrate_online(c, dev(allv[:base]))
    lo = base
    for n in sizes:
        A.atts_calibrate_online(c, dev(allv[lo:lo + n]))
        lo += n
        out = torch.empty(lo, dtype=torch.float32, device="cuda")
        A.atts_calib_export(c, out)
        held, finite = out.cpu().numpy(), allv[:lo][~np.isnan(allv[:lo])]
        nan = lo - len(finite)
        assert np.isnan(held[:nan]).all() and np.array_equal(held[nan:], np.sort(finite))


@pytest.mark.parametrize("base,sizes", [(0, (1, 3, 4, 5)), (1000, (16, 63, 64, 65)), (5000, (255, 256, 257)), (37, (511, 512, 513, 1024, 1025)),
                                        (2047, (1, 2049, 4096, 4097)), ((1 << 19) - 300, (100, 200, 1, 17))])
def test_small_appends_at_the_edges_of_their_kernels(base, sizes):
    """Batches sorted inside the merge (up to 256 scores into up to 2^19 keys) and by one workgroup of 64 ... 1024
    threads (512 ... 8192 keys), one below, at and above each limit; ties with the set and inside the batch, NaN, zeros
    of both signs and infinities in the batch.  Integer work: every comparison exact."""
    import paper_2509_15148_amd as A
    announce("calib small appends", base, sizes)
    allv = np.round(lognormal_scores(base + sum(sizes), seed=base + 9), 2)
    lo = base
    for i, n in enumerate(sizes):                              # special values at the batch's ends and inside
        special = np.array([np.nan, np.inf, -np.inf, -0.0, 0.0, 1e-45, np.nan], dtype=np.float32)
        if n > 16:
            allv[lo + 1:lo + 4] = special[:3]
            allv[lo + n - 4:lo + n] = special[3:]
        lo += n
    c = A.Calib(base + sum(sizes))
    if base:
        A.atts_calibrate_online(c, dev(allv[:base]))
    test = np.concatenate([lognormal_scores(100, seed=78), allv[:50], allv[-50:]])
    lo = base
    for n in sizes:
        A.atts_calibrate_online(c, dev(allv[lo:lo + n]))
        lo += n
        out = torch.empty(lo, dtype=torch.float32, device="cuda")
        A.atts_calib_export(c, out)
        held, finite = out.cpu().numpy(), allv[:lo][~np.isnan(allv[:lo])]
        nan = lo - len(finite)
        assert np.isnan(held[:nan]).all() and np.array_equal(held[nan:], np.sort(finite))
        _check_against_oracle(A, c, allv[:lo].astype(np.float64), test, [0.05, 0.2], brute=lo <= 30000)


@pytest.mark.parametrize("n", [8193, 10016, 65535, 131072, 131073, 262145, 524288, 524289])
@pytest.mark.parametrize("kind", ["spread", "one value", "few values", "descending", "clustered"])
def test_batches_of_several_runs(n, kind):
    """Batches sorted as runs of 2048 / 4096 / 8192 keys that are cut at sampled keys, at the limits of each run length and of the
    radix sort above them.  Equal splitters (ties), descending and clustered scores fill the buckets unevenly; zeros of both
    signs, infinities and NaN among them.  Integer work: the state equals the sorted batch."""
    import paper_2509_15148_amd as A
    announce("calib batch", n, kind)
    x = lognormal_scores(n, seed=n)
    if kind == "one value":
        x[:] = 2.5
    elif kind == "few values":
        x = np.round(x)
    elif kind == "descending":
        x = -np.sort(-x)
    elif kind == "clustered":
        x[: n - n // 9] = np.float32(1.0) + np.float32(2.0) ** -23 * (np.arange(n - n // 9) % 700)
    special = np.array([np.nan, np.inf, -np.inf, -0.0, 0.0, 1e-45, np.nan], dtype=np.float32)
    x[[0, 1, 2, n // 2, n // 3, n - 2, n - 1]] = special
    c = A.Calib(n)
    A.atts_calibrate_online(c, dev(x))
    out = torch.empty(n, dtype=torch.float32, device="cuda")
    A.atts_calib_export(c, out)
    held, finite = out.cpu().numpy(), x[~np.isnan(x)]
    assert np.isnan(held[:n - len(finite)]).all() and np.array_equal(held[n - len(finite):], np.sort(finite))


@pytest.mark.parametrize("n", [1, 40, 9000, 300000])
@pytest.mark.parametrize("m", [(1 << 19) - 1, 1 << 19, (1 << 20) - 1, 1 << 20, (1 << 20) + 513])
def test_classification_workgroup_sizes(n, m):
    """Fewer and more test scores than the lines between the two workgroup sizes and one score a thread or several, ragged ends, sets of no, one and two index levels
    below the staged one; scores outside the set's range, ties and NaN among them.  Integer work: every rank exact."""
    import paper_2509_15148_amd as A
    announce("classify", n, m)
    cal = np.round(lognormal_scores(n, seed=n), 4)
    test = lognormal_scores(m, seed=m)
    test[: m // 2] = np.round(test[: m // 2], 4)
    test[[0, 1, m - 3, m - 2, m - 1]] = np.array([-1.0, np.inf, np.nan, cal[0], -np.inf], dtype=np.float32)
    c = A.Calib(n)
    A.atts_calibrate_online(c, dev(cal))
    ranks, cls, p, q = _classify(A, c, test, [0.05, 0.2])
    want = O.rank_counts_sorted(cal.astype(np.float64), test)
    assert np.array_equal(ranks.astype(np.int64), want)
    assert np.array_equal(cls, O.classify(want, O.reject_ranks([0.05, 0.2], n)))


@pytest.mark.parametrize("n", [9000, 300000, 9000000])
@pytest.mark.parametrize("m", [1, 2, 3, 4, 5, 6, 65, 257, 258])
def test_classification_of_a_few_scores(n, m):
    """Quads of lanes with work for one, two or more of them, in every wavefront and in the last one only; one to three index
    levels below the staged one.  The first scores are in turn a NaN and below all of the set: lanes without work ahead of others."""
    import paper_2509_15148_amd as A
    announce("classify few", n, m)
    cal = np.round(lognormal_scores(n, seed=n % 1000), 4)
    c = A.Calib(n)
    A.atts_calibrate_online(c, dev(cal))
    for first in ([], [np.nan], [-1.0, np.nan]):
        test = np.round(lognormal_scores(m, seed=m), 4)
        test[:len(first)] = first[:m]
        ranks, cls, _, _ = _classify(A, c, test, [0.05, 0.2])
        want = O.rank_counts_sorted(cal.astype(np.float64), test)
        assert np.array_equal(ranks.astype(np.int64), want)
        assert np.array_equal(cls, O.classify(want, O.reject_ranks([0.05, 0.2], n)))


@pytest.mark.parametrize("n", [20000, 32768, 32769, 65536, 65537])
def test_bucket_sizes_and_limits(n):
    """Batches around the line between buckets of 8 and of 16 samples.  Whole blocks of 64 equal keys, one key above a block, runs that
    end inside a block of 64 and inside a 16-byte piece: the limits of a bucket fall on and beside block edges in every run."""
    import paper_2509_15148_amd as A
    announce("bucket limits", n)
    rng = np.random.default_rng(n)
    for m in (n, n - 1, n - 61):
        v = np.concatenate([np.repeat(rng.lognormal(size=m // 128 + 1), 64), rng.lognormal(size=m // 3), np.repeat(rng.lognormal(size=m // 300 + 1), 65),
                            [np.nan, np.inf, -np.inf, 0.0, -0.0], rng.lognormal(size=m)]).astype(np.float32)[:m]
        v = rng.permutation(v) if m % 2 else np.sort(v)
        c = A.Calib(m)
        A.atts_calibrate_online(c, dev(v))
        out = torch.empty(m, dtype=torch.float32, device="cuda")
        A.atts_calib_export(c, out)
        torch.cuda.synchronize()
        got, ref = out.cpu().numpy(), np.sort(v)                       # NaN last there, first here
        k = int(np.isnan(v).sum())
        assert np.isnan(got[:k]).all() and np.array_equal(got[k:], ref[:m - k] if k else ref), m
        c.close()


@pytest.mark.parametrize("base,sizes", [(0, (1023, 1, 1, 1022, 1, 1)), (900, (60, 64, 65)), ((1 << 18) - 513, (512, 1, 1, 600)),
                                        ((1 << 18) - 5000, (4096, 4097)), (300000, (700, 65536, 262145)), (5, (20000,)), (40000, (9,))])
@pytest.mark.parametrize("where", ["spread", "one place", "below", "above", "ties"])
def test_merge_segments_and_splits(base, sizes, where):
    """Totals around whole segments of 1024 and 2048 keys and around the line between them, batches one below, at and above 64, 64^2
    and 64^3 keys (rounds of the split search), larger and smaller than the set; the batch spread over the set, in one place of it, outside
    it on either side, or all ties with it."""
    import paper_2509_15148_amd as A
    announce("merge segments", base, sizes, where)
    rng = np.random.default_rng(base + len(sizes))
    total = base + sum(sizes)
    c = A.Calib(total)
    have = np.round(rng.lognormal(size=base), 3).astype(np.float32)
    if base:
        A.atts_calibrate_online(c, dev(have))
    for n in sizes:
        v = {"spread": lambda: np.round(rng.lognormal(size=n), 3), "one place": lambda: 1.0 + 1e-6 * rng.random(n), "below": lambda: -rng.random(n),
             "above": lambda: 1e6 + rng.random(n), "ties": lambda: np.full(n, have[base // 2] if base else 1.0)}[where]().astype(np.float32)
        A.atts_calibrate_online(c, dev(v))
        have = np.concatenate([have, v])
        out = torch.empty(len(have), dtype=torch.float32, device="cuda")
        A.atts_calib_export(c, out)
        torch.cuda.synchronize()
        assert np.array_equal(out.cpu().numpy(), np.sort(have)), n
        probe = np.concatenate([rng.choice(have, 300), [0.0, 2e6, -2.0]]).astype(np.float32)         # the index levels written with it
        ranks = _classify(A, c, probe, [0.1])[0]
        assert np.array_equal(ranks.astype(np.int64), O.rank_counts_sorted(have, probe))
    c.close()


@pytest.mark.parametrize("n", [(1 << 19) + 1, 4096 * 256, 4096 * 256 + 1, 4096 * 257 - 1, 4096 * 512, 4096 * 513 + 77, 5000003])
@pytest.mark.parametrize("kind", ["spread", "one value", "high digits", "bits"])
def test_radix_sort_groups_of_tiles(n, kind):
    """Tiles around one, two and more a group, partly filled last tiles and groups; one digit only, few high digits, all bit patterns
    (NaN, infinities and zeros of both signs among them)."""
    import paper_2509_15148_amd as A
    announce("radix groups", n, kind)
    rng = np.random.default_rng(n)
    v = {"spread": lambda: rng.lognormal(size=n), "one value": lambda: np.full(n, 0.75), "high digits": lambda: 1.0 + 1e-3 * rng.random(n),
         "bits": lambda: rng.integers(0, 1 << 32, n, dtype=np.uint64).astype(np.uint32).view(np.float32)}[kind]().astype(np.float32)
    c = A.Calib(n)
    A.atts_calibrate_online(c, dev(v))
    out = torch.empty(n, dtype=torch.float32, device="cuda")
    A.atts_calib_export(c, out)
    torch.cuda.synchronize()
    got, k = out.cpu().numpy(), int(np.isnan(v).sum())
    assert np.isnan(got[:k]).all() and np.array_equal(got[k:], np.sort(v)[:n - k])
    c.close()


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 63, 255, 1021, 1024, 4099, 8191, 8192, 8193, 262144, 262145])
@pytest.mark.parametrize("m", [1, 255, 256, 700])
def test_staged_levels_of_every_length(n, m):
    """The staged level read in 16-byte pieces and searched by three probes a step: lengths around whole pieces, whole batches of
    them and the most that is staged; scores below, in and above the set, NaN and ties; thresholds inside and outside the set."""
    import paper_2509_15148_amd as A
    announce("staged level", n, m)
    rng = np.random.default_rng(n * 7 + m)
    cal = np.round(rng.lognormal(size=n), 4).astype(np.float32)
    test = np.concatenate([rng.choice(cal, m), [np.nan, -1.0, np.inf, cal.max(), cal.min()], np.round(rng.lognormal(size=m), 4)]).astype(np.float32)[-m:]
    c = A.Calib(n)
    A.atts_calibrate_online(c, dev(cal))
    _check_against_oracle(A, c, cal, test, [0.001, 0.05, 0.2, 0.999], brute=n < 5000)
    c.close()


def test_capacity_and_argument_errors():
    import paper_2509_15148_amd as A
    announce("calib errors")
    c = A.Calib(10)
    x = dev(np.arange(8, dtype=np.float32))
    with pytest.raises(A.AttsError) as e:                      # classify on an empty set
        _classify(A, c, np.zeros(3, np.float32), [0.1])
    assert e.value.code == A.ERR_INVALID_ARG
    A.atts_calibrate_online(c, x)
    with pytest.raises(A.AttsError) as e:
        A.atts_calibrate_online(c, x)
    assert e.value.code == A.ERR_CAPACITY and A.atts_calib_size(c) == 8
    A.atts_calibrate_online(c, x[:0])                          # empty append is a no-op
    for bad in ([], [0.0], [1.0], [0.3, 0.2], [0.1] * 9, [float("nan")]):
        with pytest.raises(A.AttsError) as e:
            _classify(A, c, np.zeros(3, np.float32), bad)
        assert e.value.code == A.ERR_INVALID_ARG
    with pytest.raises(A.AttsError) as e:                      # p-values need the ranks
        A.atts_classify_ordinal(c, x[:3], [0.5], None, torch.empty(3, device="cuda"), torch.empty(3, dtype=torch.uint8, device="cuda"), None)
    assert e.value.code == A.ERR_INVALID_ARG
    A.atts_calib_reset(c)
    assert A.atts_calib_size(c) == 0
    A.atts_calibrate_online(c, x[:3])
    _check_against_oracle(A, c, np.arange(3, dtype=np.float64), np.array([-1, 0, 1.5, 2, 9], np.float32), [0.5])


def test_calibration_only_workload_full_size():
    """The calibration-only workload at its published size: 2^20 lognormal scores, 16 online steps
    of 65,536 appended + 65,536 classified at alpha = (0.05, 0.2).  Every rank and class is checked
    against the oracle's sort-based count; 128 sampled test scores per step against the double sum."""
    import paper_2509_15148_amd as A
    wl = WORKLOADS["calib"]
    announce("calib full workload", wl.n_cal, wl.n_new, wl.n_steps)
    cal = lognormal_scores(wl.n_cal, wl.seed)
    c = A.Calib(wl.n_cal + wl.n_steps * wl.n_new)
    A.atts_calibrate_online(c, dev(cal))
    rng = np.random.default_rng(1)
    counts = np.zeros(3, dtype=np.int64)
    for step in range(wl.n_steps):
        new = lognormal_scores(wl.n_new, wl.seed + 1000 + step)
        test = lognormal_scores(wl.n_test, wl.seed + 2000 + step)
        A.atts_calibrate_online(c, dev(new))
        cal = np.concatenate([cal, new])
        ranks, cls, p, q = _classify(A, c, test, list(wl.alphas))
        cal64 = cal.astype(np.float64)
        cs = O.rank_counts_sorted(cal64, test)
        r = O.reject_ranks(wl.alphas, len(cal))
        assert np.array_equal(ranks.astype(np.int64), cs), step
        assert np.array_equal(cls, O.classify(cs, r)), step
        assert np.array_equal(q, O.quantile_thresholds(cal64, r).astype(np.float32))
        cls2 = torch.empty(wl.n_test, dtype=torch.uint8, device="cuda")
        A.atts_classify_ordinal(c, dev(test), list(wl.alphas), None, None, cls2, None)
        assert np.array_equal(cls2.cpu().numpy(), cls), step
        idx = rng.choice(wl.n_test, 128, replace=False)
        assert np.array_equal(ranks[idx].astype(np.int64), O.rank_counts(cal64, test[idx]))
        counts += np.bincount(cls, minlength=3)
    frac = counts / counts.sum()
    assert abs(frac[2] - 0.05) < 0.005 and abs(frac[1] + frac[2] - 0.2) < 0.01     # take-over rate ~ alpha


def test_streaming_merge_sizes():
    """Batches and totals above 2^22 keys take the streaming merge (4096-key segments, splits found by a
    separate kernel) in both its pairwise and its final form; smaller appends into the large set, ragged
    lengths and ties included.  The state must equal the sorted union after every append."""
    import paper_2509_15148_amd as A
    sizes = ((1 << 22) + 12345, 5_000_000, 70_001, 17, 8192)
    announce("calib streaming merge", sizes)
    total = sum(sizes)
    allv = np.round(lognormal_scores(total, seed=4242), 4)
    c = A.Calib(total)
    test = np.concatenate([lognormal_scores(4000, seed=78), allv[:96], np.array([0.0, np.inf, -1.0, np.nan], np.float32)])
    lo = 0
    for s in sizes:
        A.atts_calibrate_online(c, dev(allv[lo:lo + s]))
        lo += s
        out = torch.empty(lo, dtype=torch.float32, device="cuda")
        A.atts_calib_export(c, out)
        assert np.array_equal(out.cpu().numpy(), np.sort(allv[:lo])), s
        _check_against_oracle(A, c, allv[:lo].astype(np.float64), test, [0.05, 0.2], brute=False)
    idx = np.arange(0, len(test), 64)
    ranks = _classify(A, c, test[idx], [0.05, 0.2])[0]
    assert np.array_equal(ranks.astype(np.int64), O.rank_counts(allv.astype(np.float64), test[idx]))


@pytest.mark.parametrize("kind", ["lognormal", "clustered"])
def test_large_set_rank_search_with_guessed_window(kind):
    """Sets of 2^24 scores and more: the rank search first tries a two-line window picked by linear interpolation
    inside a 256-key block and falls back to the two index levels when the window does not bracket the score.
    Smooth data takes the window almost always; clustered data (long runs of equal scores, gaps of several orders of
    magnitude, sub-normals) defeats the guess.  Every rank and class against the oracle's sort-based count, sampled
    ones against the double sum."""
    import paper_2509_15148_amd as A
    n, m = (1 << 24) + 4321, 1 << 18
    announce("calib guessed window", kind, n, m)
    rng = np.random.default_rng(11)
    if kind == "lognormal":
        cal = lognormal_scores(n, seed=606)
        test = lognormal_scores(m, seed=607)
    else:
        parts = [np.full(n // 3, 1.0, np.float32), lognormal_scores(n // 3, seed=608) * np.float32(1e-30),
                 (rng.integers(0, 50, n - 2 * (n // 3)) * 1000.0).astype(np.float32)]
        cal = np.concatenate(parts)
        rng.shuffle(cal)
        test = np.concatenate([cal[: m // 2], lognormal_scores(m // 4, seed=609) * np.float32(1e-30),
                               (rng.random(m - m // 2 - m // 4) * 60000.0 - 5000.0).astype(np.float32)])
    c = A.Calib(n)
    A.atts_calibrate_online(c, dev(cal))
    ranks, cls, p, q = _classify(A, c, test, [0.05, 0.2])
    cal64 = cal.astype(np.float64)
    want = O.rank_counts_sorted(cal64, test)
    assert np.array_equal(ranks.astype(np.int64), want)
    r = O.reject_ranks([0.05, 0.2], n)
    assert np.array_equal(cls, O.classify(want, r))
    assert np.array_equal(q, O.quantile_thresholds(cal64, r).astype(np.float32))
    idx = rng.choice(m, 24, replace=False)
    assert np.array_equal(ranks[idx].astype(np.int64), O.rank_counts(cal64, test[idx]))


def test_out_of_cache_size_sampled():
    """2^28 resident scores + one append of 2^24 (the out-of-cache variant that bench.py times): the coarsest
    index level no longer fits LDS whole, so the strided top level + window search is exercised.  Ranks of
    sampled test scores against the oracle's double sum; the exported state must be ascending and keep every
    score (sum of ranks of the extreme probes)."""
    import paper_2509_15148_amd as A
    n0, n1 = 1 << 28, 1 << 24
    announce("calib out-of-cache", n0, n1)
    g = torch.Generator(device="cuda").manual_seed(99)
    cal0 = torch.randn(n0, device="cuda", generator=g).exp_()
    cal1 = torch.randn(n1, device="cuda", generator=g).exp_()
    c = A.Calib(n0 + n1)
    A.atts_calibrate_online(c, cal0)
    A.atts_calibrate_online(c, cal1)
    assert A.atts_calib_size(c) == n0 + n1
    out = torch.empty(n0 + n1, dtype=torch.float32, device="cuda")
    A.atts_calib_export(c, out)
    assert bool((out[1:] >= out[:-1]).all())
    del out
    host = np.concatenate([cal0.cpu().numpy(), cal1.cpu().numpy()])
    del cal0, cal1
    test = np.concatenate([lognormal_scores(60, seed=5), host[:3], np.array([0.0, 1e30], np.float32)]).astype(np.float32)
    ranks, cls, p, q = _classify(A, c, test, [0.05, 0.2])
    n = len(host)
    want = O.rank_counts(host.astype(np.float64), test)
    assert np.array_equal(ranks.astype(np.int64), want)
    r = O.reject_ranks([0.05, 0.2], n)
    assert np.array_equal(cls, O.classify(want, r))
    assert np.array_equal(p, O.p_values(want, n).astype(np.float32))
    assert ranks[-2] == n and ranks[-1] == 0
    # thresholds: the (n + 1 - r)-th smallest, by partition instead of a full sort
    for l in range(2):
        kth = n + 1 - int(r[l])
        assert q[l] == np.partition(host, kth - 1)[kth - 1]


def test_export_import_round_trip():
    """Checkpoint / resume of the online calibration state: a handle restored from an export gives the same ranks,
    classes and thresholds bit for bit, before and after further appends to both."""
    import paper_2509_15148_amd as A
    announce("calib export/import")
    for n0, n1 in ((16, 5), (1000, 37), (70000, 9000), (300000, 70001)):
        cal = lognormal_scores(n0, 901).astype(np.float32)
        cal[:: max(n0 // 7, 1)] = cal[0]
        if n0 > 100:
            cal[3], cal[5], cal[9], cal[11] = np.nan, -0.0, 0.0, np.inf
        more = lognormal_scores(n1, 902).astype(np.float32)
        test = np.concatenate([lognormal_scores(3000, 903).astype(np.float32), cal[:50],
                               np.array([np.nan, 0.0, -0.0, np.inf, -np.inf], dtype=np.float32)])
        alphas = [0.05, 0.2]
        a = A.Calib(n0 + n1)
        A.atts_calibrate_online(a, dev(cal[: n0 // 2]))
        A.atts_calibrate_online(a, dev(cal[n0 // 2:]))
        saved = torch.empty(n0, dtype=torch.float32, device="cuda")
        A.atts_calib_export(a, saved)
        b = A.Calib(n0 + n1)
        A.atts_calibrate_online(b, dev(more))                     # old contents are replaced by the import
        A.atts_calib_import(b, saved)
        assert A.atts_calib_size(b) == n0
        ra = _classify(A, a, test, alphas)
        rb = _classify(A, b, test, alphas)
        for x, y in zip(ra, rb):
            assert np.array_equal(x, y, equal_nan=True)
        _check_against_oracle(A, b, cal.astype(np.float64), test, alphas, brute=n0 <= 1000)
        A.atts_calibrate_online(a, dev(more))
        A.atts_calibrate_online(b, dev(more))
        ra = _classify(A, a, test, alphas)
        rb = _classify(A, b, test, alphas)
        for x, y in zip(ra, rb):
            assert np.array_equal(x, y, equal_nan=True)
        with pytest.raises(A.AttsError) as e:
            A.atts_calib_import(b, torch.zeros(n0 + n1 + 1, dtype=torch.float32, device="cuda"))
        assert e.value.code == A.ERR_CAPACITY
        A.atts_calib_import(b, torch.zeros(0, dtype=torch.float32, device="cuda"))
        assert A.atts_calib_size(b) == 0
        a.close()
        b.close()


@pytest.mark.parametrize("n", [1, 1000, 20001])
@pytest.mark.parametrize("m", [(1 << 17) - 1, 1 << 17, (1 << 19) - 1, 1 << 19, (1 << 20) - 1, 1 << 20])
def test_rank_search_on_both_sides_of_its_sizes(n, m):
    """The three forms of the rank search, on each side of the numbers of scores where one follows the other: ranks,
    classes, thresholds and p-values exactly the oracle's.  Half of the scores tie with the set's."""
    import paper_2509_15148_amd as A
    announce("calib rank search sizes", n, m)
    cal = lognormal_scores(n, seed=31)
    test = lognormal_scores(m, seed=32)
    test[::2] = cal[np.arange(len(test[::2])) % n]
    calib = A.Calib(n)
    A.atts_calibrate_online(calib, dev(cal))
    _check_against_oracle(A, calib, cal, test, [0.05, 0.2, 0.5], brute=False)
