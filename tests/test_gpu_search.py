"""GPU parity of the boxcar filter, the exact sigma-cut and peak finding
(section 2.3) against the oracle, through the C ABI."""
import numpy as np
import pytest

import oracle
from oracle.peaks import series_events
import synth
from gpu_common import events_equal, log, small_case, small_search, survey_case, to_dev, torch_dev

pytestmark = pytest.mark.gpu


def _series_dev(out_np, u16):
    torch = torch_dev()
    if u16:
        return to_dev(out_np.astype(np.uint16).view(np.int16))
    return to_dev(out_np.astype(np.int32))


def test_boxcar_filter_small_config():
    from paper_1112_0065_amd import _lib as L
    torch = torch_dev()
    fb, dly, x, out = small_case()
    bw, _ = small_search()
    for u16 in (False, True):
        s = _series_dev(out, u16)
        for first, count in [(0, 100), (37, 5), (99, 1)]:
            dst = torch.empty((len(fb.widths), count, bw.shape[2]), dtype=torch.int32, device="cuda")
            L.boxcar_filter(s, 100, out.shape[1], fb.widths, first, count, dst)
            torch.cuda.synchronize()
            assert (dst.cpu().numpy() == bw[:, first:first + count]).all(), (u16, first)


def test_boxcar_uint32_wrap():
    """Running sums far beyond 2^32 wrap; the windows stay exact."""
    from paper_1112_0065_amd import _lib as L
    torch = torch_dev()
    s = np.full((2, 300000), 60000, dtype=np.int64)
    s[1, ::7] = 0
    ref = oracle.boxcar(s, [1, 16, 300])
    dst = torch.empty((3, 2, ref.shape[2]), dtype=torch.int32, device="cuda")
    L.boxcar_filter(_series_dev(s, False), 2, s.shape[1], [1, 16, 300], 0, 2, dst)
    torch.cuda.synchronize()
    assert (dst.cpu().numpy() == ref).all()


def _find(series_np, widths, k, u16, capacity=1 << 16):
    from paper_1112_0065_amd import _lib as L
    torch = torch_dev()
    ndm, nout = series_np.shape
    s = _series_dev(series_np, u16)
    ws = torch.empty(max(256, L.find_peaks_workspace_bytes(ndm, nout, widths)), dtype=torch.uint8,
                     device="cuda")
    ev = torch.empty(max(capacity, 1) * 40, dtype=torch.uint8, device="cuda")
    n = L.find_peaks(s, ndm, nout, widths, k, ev, capacity, ws)
    stats = L.find_peaks_read_stats(ws, ndm, nout, widths)
    return L.events_from_buffer(ev, n), stats


def _ref_stats(bw, k):
    nw, ndm = bw.shape[:2]
    s1 = np.empty((nw, ndm), np.int64)
    s2 = np.empty((nw, ndm), object)
    thr = np.empty((nw, ndm), np.int64)
    for w in range(nw):
        for d in range(ndm):
            n, a, b = oracle.series_stats(bw[w, d])
            s1[w, d], s2[w, d] = a, b
            t = oracle.threshold_level(n, a, b, k)
            thr[w, d] = -1 if t is None else t
    return s1, s2, thr


def test_find_peaks_small_config():
    fb, dly, x, out = small_case()
    bw, ref_ev = small_search()
    s1, s2, thr = _ref_stats(bw, fb.snr_thresh)
    assert len(ref_ev) > 0
    for u16 in (False, True):
        log("find_peaks small config u16", u16, "ref events", len(ref_ev))
        ev, (g1, g2, gt) = _find(out, fb.widths, fb.snr_thresh, u16)
        assert (g1 == s1).all() and (g2 == s2).all() and (gt == thr).all()
        events_equal(ev, ref_ev)


@pytest.mark.parametrize("k", [0.5, 1.0, 2.0, 2.75, 3.0, 4.5])
def test_find_peaks_thresholds_and_ties(k):
    """Random series with many events; k values with exact ties possible."""
    rng = np.random.default_rng(int(k * 100))
    series = rng.integers(0, 12, size=(9, 4000)).astype(np.int64)
    series[3, 100:140] = 40        # a long run
    series[5, :] = 7               # constant series: D = 0 for every width
    series[6, 3990:] = 30          # run touching the end
    series[7, :20] = 30            # run at the start
    series[8, :] = np.tile([0, 11], 2000)   # ~2000 one-sample runs in one segment
    widths = [1, 2, 3, 8]
    bw = oracle.boxcar(series, widths)
    ref = oracle.find_events(bw, k)
    s1, s2, thr = _ref_stats(bw, k)
    for u16 in (False, True):
        ev, (g1, g2, gt) = _find(series, widths, k, u16)
        assert (g1 == s1).all() and (g2 == s2).all() and (gt == thr).all()
        events_equal(ev, ref)


@pytest.mark.parametrize("k", [1.0, 2.0])
def test_find_peaks_runs_leave_the_segment_window(k):
    """Runs that start in one 8192-position segment and go on past its
    running-sum window (so their walk continues on the series in global
    memory, over several 64-position steps): a long run across a segment
    boundary, a run whose peak lies beyond the window, a plateau (the peak is
    its first position), and a run that reaches the end of the data."""
    rng = np.random.default_rng(5)
    series = rng.integers(0, 12, size=(5, 40000)).astype(np.int64)
    series[0, 8000:9600] = 60
    series[1, 16000:16500] = 50
    series[1, 16400:16450] = 80
    series[2, 30000:] = 40
    series[3, 8100:8192 + 64 * 3] = 45
    series[4, 24500:24576 + 200] = 30
    series[4, 24576 + 100:24576 + 130] = 90
    widths = [1, 4, 64]
    bw = oracle.boxcar(series, widths)
    ref = oracle.find_events(bw, k)
    seg = 8192
    crossing = [e for e in ref if e[3] >= (e[2] // seg + 1) * seg + widths[-1] - widths[e[0]]]
    assert len(crossing) >= 12
    s1, s2, thr = _ref_stats(bw, k)
    for u16 in (False, True):
        log("find_peaks window-crossing runs k", k, "u16", u16, "ref events", len(ref))
        ev, (g1, g2, gt) = _find(series, widths, k, u16)
        assert (g1 == s1).all() and (g2 == s2).all() and (gt == thr).all()
        events_equal(ev, ref)


def test_find_peaks_capacity_overflow():
    from paper_1112_0065_amd import _lib as L
    rng = np.random.default_rng(3)
    series = rng.integers(0, 12, size=(4, 3000)).astype(np.int64)
    widths = [1, 2]
    ref = oracle.find_events(oracle.boxcar(series, widths), 1.0)
    assert len(ref) > 20
    with pytest.raises(L.DedispError) as e:
        _find(series, widths, 1.0, False, capacity=10)
    assert e.value.status == L.ERR_CAPACITY
    ev, _ = _find(series, widths, 1.0, False, capacity=len(ref))
    events_equal(ev, ref)


def test_find_peaks_bad_args():
    from paper_1112_0065_amd import _lib as L
    series = np.zeros((2, 100), np.int64)
    for widths, k, st in [([4, 2], 3.0, L.ERR_INVALID_ARG), ([1, 200], 3.0, L.ERR_TOO_FEW_SAMPLES),
                          ([1], 0.0, L.ERR_INVALID_ARG), ([1], float("nan"), L.ERR_INVALID_ARG)]:
        with pytest.raises(L.DedispError) as e:
            _find(series, widths, k, False)
        assert e.value.status == st


def test_survey_search_sampled_series():
    """Full-size survey beam: dedisperse + find_peaks on the GPU; the events
    and statistics of sampled DM rows equal the oracle's for those rows."""
    from paper_1112_0065_amd import _lib as L
    torch = torch_dev()
    fb = survey_case()
    p = L.dedisp_plan_create(fb.nchans, fb.f_top, fb.df, fb.tsamp, fb.dm_list)
    dly = oracle.delay_table(fb.nchans, fb.f_top, fb.df, fb.tsamp, fb.dm_list)
    nout = fb.nsamps - p.max_delay
    inp = to_dev(fb.packed)
    ws = torch.empty(L.dedisp_workspace_bytes(p, fb.nsamps), dtype=torch.uint8, device="cuda")
    out = torch.empty((1200, nout), dtype=torch.int16, device="cuda")
    L.dedisp_execute(p, inp, fb.nsamps, out, ws)
    pws = torch.empty(L.find_peaks_workspace_bytes(1200, nout, fb.widths), dtype=torch.uint8,
                      device="cuda")
    evb = torch.empty((1 << 20) * 40, dtype=torch.uint8, device="cuda")
    n = L.find_peaks(out, 1200, nout, fb.widths, fb.snr_thresh, evb, 1 << 20, pws)
    ev = L.events_from_buffer(evb, n)
    g1, g2, gt = L.find_peaks_read_stats(pws, 1200, nout, fb.widths)
    log("survey events", n)
    keys = [(int(e["width_idx"]), int(e["dm_idx"]), int(e["t_start"])) for e in ev]
    assert keys == sorted(keys)
    rng = np.random.default_rng(11)
    rows = sorted({0, 1199} | {int(np.argmin(np.abs(fb.dm_list - pu.dm))) for pu in fb.pulses[:4]}
                  | set(rng.integers(0, 1200, 2).tolist()))
    x = oracle.unpack_2bit(fb.packed, fb.nsamps, fb.nchans)
    ref_rows = oracle.dedisperse(x, dly[rows], nout=nout)
    for k, d in enumerate(rows):
        bw = oracle.boxcar(ref_rows[k:k + 1], fb.widths)
        for wi in range(len(fb.widths)):
            nn, a, b = oracle.series_stats(bw[wi, 0])
            assert g1[wi, d] == a and g2[wi, d] == b
            t = oracle.threshold_level(nn, a, b, fb.snr_thresh)
            assert gt[wi, d] == (-1 if t is None else t)
            ref_ev = series_events(bw[wi, 0], fb.snr_thresh, wi, d)
            got = [e for e in ev if int(e["width_idx"]) == wi and int(e["dm_idx"]) == d]
            events_equal(got, ref_ev)
    # every injected pulse whose S/N, after 2-bit quantisation (efficiency
    # ~0.94) and the smearing by the distance to the nearest trial DM, stays
    # >= 10 is detected near its DM and time
    for pu in fb.pulses:
        d = int(np.argmin(np.abs(fb.dm_list - pu.dm)))
        smear = abs(pu.dm - fb.dm_list[d]) * 20476.0 / 1000.0
        if 0.94 * pu.snr * np.sqrt(pu.width / (pu.width + smear)) < 10:
            continue
        hit = [e for e in ev if abs(int(e["dm_idx"]) - d) <= 3 and
               abs(int(e["t_peak"]) - pu.t0) <= pu.width + 64]
        assert hit, (pu.dm, pu.t0, pu.width, pu.snr)


def test_find_peaks_large_values_exact():
    """Windows whose boxcars exceed 2^26 take the 128-bit square-sum path."""
    rng = np.random.default_rng(21)
    series = rng.integers(0, 1 << 20, size=(3, 20000)).astype(np.int64)
    series[1, 5000:5040] = (1 << 21)
    widths = [1, 16, 128]
    bw = oracle.boxcar(series, widths)
    assert bw.max() >= (1 << 26)
    ref = oracle.find_events(bw, 3.0)
    s1, s2, thr = _ref_stats(bw, 3.0)
    ev, (g1, g2, gt) = _find(series, widths, 3.0, False)
    assert (g1 == s1).all() and (g2 == s2).all() and (gt == thr).all()
    events_equal(ev, ref)


def test_find_peaks_square_sum_near_2_64():
    """Full 8192-position segments whose boxcars lie just below 2^26: each
    segment's sum of squares exceeds 2^64 (8192 x (5e7)^2 = 2.0e19), so the
    64-bit fast path must not take them; the sums stay exact."""
    rng = np.random.default_rng(95)
    series = rng.integers(95000, 100000, size=(2, 20000)).astype(np.int64)
    widths = [1, 512]
    bw = oracle.boxcar(series, widths)
    assert int(bw.max()) < (1 << 26)
    seg_s2 = int((bw[1, 0, :8192].astype(object) ** 2).sum())
    assert seg_s2 >= (1 << 64)
    ref = oracle.find_events(bw, 3.0)
    s1, s2, thr = _ref_stats(bw, 3.0)
    ev, (g1, g2, gt) = _find(series, widths, 3.0, False)
    assert (g1 == s1).all() and (g2 == s2).all() and (gt == thr).all()
    events_equal(ev, ref)


@pytest.mark.parametrize("k", [6.0, 1.0e6])
def test_find_peaks_wide_integer_paths(k):
    """Series of 2^18 values uniform below 2^27 with widths up to 16: at
    k = 1e6, k^2 D exceeds 2^104 (the digit-by-digit square root) and
    S1 + isqrt(k^2 D) + 1 exceeds 2^64 (the bit-serial division); at k = 6
    both stay on their fast paths.  Thresholds equal the oracle's."""
    rng = np.random.default_rng(26)
    series = rng.integers(0, 1 << 27, size=(2, 1 << 18)).astype(np.int64)
    widths = [1, 16]
    bw = oracle.boxcar(series, widths)
    assert int(bw.max()) < (1 << 31)
    s1, s2, thr = _ref_stats(bw, k)
    if k > 1000:
        n = bw.shape[2]
        d = n * int(s2[1, 0]) - int(s1[1, 0]) ** 2
        assert int(k * k) * d >= (1 << 104)
        assert int(s1[1, 0]) + int(k * np.sqrt(float(d))) >= (1 << 64)
    ref = oracle.find_events(bw, k)
    ev, (g1, g2, gt) = _find(series, widths, k, False)
    assert (g1 == s1).all() and (g2 == s2).all() and (gt == thr).all()
    events_equal(ev, ref)


@pytest.mark.parametrize("nout", [3 * 8192 + 512, 3 * 8192 + 514, 8192 + 1024])
def test_find_peaks_uint16_window_loads(nout):
    """uint16 series whose rows are a multiple of 4 samples take the
    statistics pass's 8-byte window loads (from sample 0 in a row's first
    segment, whole 8192-position segments and a ragged last one); the other
    row lengths take the per-sample loads.  Survey-level values, pulses that
    cross segment edges, and one row of values near 2^16 (width-512 boxcars
    just below 2^25, the largest the register fast path takes) -- all equal
    the oracle."""
    rng = np.random.default_rng(nout)
    series = rng.integers(1400, 1700, size=(5, nout)).astype(np.int64)
    series[1, 8150:8260] += 400            # across the first segment edge
    series[2, :40] += 600                  # at the start of the row
    series[3, nout - 30:] += 500           # at the end of the row
    series[4, :] = rng.integers(60000, 65536, size=nout)
    widths = [1 << i for i in range(10)]
    bw = oracle.boxcar(series, widths)
    ref = oracle.find_events(bw, 6.0)
    s1, s2, thr = _ref_stats(bw, 6.0)
    log("uint16 window loads nout", nout, "ref events", len(ref))
    ev, (g1, g2, gt) = _find(series, widths, 6.0, True)
    assert (g1 == s1).all() and (g2 == s2).all() and (gt == thr).all()
    events_equal(ev, ref)


@pytest.mark.parametrize("ndm,nout,nw", [
    (5, 700, 4),         # one segment per series: its count is the series' total
    (1300, 9001, 4),     # two segments; two steps of the one-block series scan
    (2100, 90, 32),      # 67 200 series: more than one block scans
])
def test_event_slots_over_series_and_segments(ndm, nout, nw):
    """Every event lands in its slot whatever scans the series' counts and
    however many segments come before its own in the series."""
    rng = np.random.default_rng(ndm)
    series = rng.integers(0, 40, size=(ndm, nout)).astype(np.int64)
    series[rng.integers(ndm, size=ndm // 2), rng.integers(nout, size=ndm // 2)] += 200
    widths = list(range(1, nw + 1))
    ref = oracle.find_events(oracle.boxcar(series, widths), 4.0)
    for u16 in (False, True):
        ev, _ = _find(series, widths, 4.0, u16, capacity=1 << 19)
        events_equal(ev, ref)


@pytest.mark.parametrize("widths,nout", [
    ([1, 2, 4, 8], 8192 + 7),                        # the last window ends the row; one whole segment
    ([1, 2, 4, 8, 16], 8192 + 15),                   # one position more than a segment less one
    ([3, 4, 10, 64], 16384 + 64),                    # odd first width; one position in the third segment
    ([2, 6, 100, 512, 1020], 16384 + 1019 + 511),    # even widths, the widest that fits; ragged tail
    ([1, 2, 4, 8, 16, 32, 64, 128, 256, 512, 514, 600], 12001),
    ([1, 2, 4, 1022], 20002),                        # too wide: the 32-bit form
    ([1, 2, 4, 7, 8], 9000),                         # an odd width further on: the 32-bit form
])
def test_statistics_forms_and_their_limits(widths, nout):
    """The 16-bit statistics pass (rows at every alignment, whole and ragged
    segments), its 32-bit halves for windows of a wide span, the general sums
    for large values, and the lists it does not take: sums, cuts and events
    equal the oracle's."""
    rng = np.random.default_rng(nout)
    ndm = 7
    series = rng.normal(1500.0, 30.0, size=(ndm, nout)).round().astype(np.int64)
    series[1, 3000:3600] += 60                   # spans more than 2^14
    series[2] += (400 * np.sin(np.arange(nout) / 2000.0)).astype(np.int64)   # a drifting baseline
    series[3] = 60000 + series[3] % 64           # near the largest 16-bit value
    series[4, nout - 40:] += 80                  # into the last window
    series[5] = 1500                             # constant
    for big in (False, True):
        if big:
            series[0] += 1 << 21                 # int32 only: beyond the fast forms
            series[6, ::2] = 0
        ref_ev = oracle.find_events(oracle.boxcar(series, widths), 5.0)
        s1, s2, thr = _ref_stats(oracle.boxcar(series, widths), 5.0)
        for u16 in (False,) if big else (True, False):
            ev, (g1, g2, gt) = _find(series, widths, 5.0, u16, capacity=1 << 18)
            assert (g1 == s1).all() and (g2 == s2).all() and (gt == thr).all(), (big, u16)
            events_equal(ev, ref_ev)


def test_statistics_square_sums_use_all_32_bits():
    """Windows that span just under 2^14: a thread's 16 squares sum to nearly
    2^32."""
    nout = 8192 + 511
    series = np.zeros((2, nout), np.int64)
    series[0, ::512] = 2 * 16000                 # +-16000 around a mean of 62.5
    series[1, 100:8200:1024] = 16000
    for widths in ([1, 2, 4, 256, 512], [2, 4, 8, 512]):
        s1, s2, thr = _ref_stats(oracle.boxcar(series, widths), 3.0)
        for u16 in (True, False):
            _, (g1, g2, gt) = _find(series, widths, 3.0, u16, capacity=1 << 18)
            assert (g1 == s1).all() and (g2 == s2).all() and (gt == thr).all(), u16


def _window_extremes(nout):
    """Series at the limits of the statistics pass's forms: the largest 16-bit
    value, blocks of the smallest and largest value (the widest span of centred
    running sums), a strong drift, pulses, and a whole row near one value."""
    t = np.arange(nout)
    return np.stack([
        np.where(t // 2304 % 2 == 0, 65535, 0),
        np.where(t < nout // 2, 65535, 0),
        np.full(nout, 65535),
        (15000 + 9000 * np.sin(t / 3000.0)).astype(np.int64),
        1500 + 2000 * (t % 2500 < 300),
        np.where(t % 4096 == 4095, 65535, 0),
        (t * 65535) // nout,
    ]).astype(np.int64)


@pytest.mark.parametrize("widths", [[1, 2, 4, 8], [1, 64, 256, 512], [2, 16, 514, 1020], [2, 4, 6, 1020]])
@pytest.mark.parametrize("nout", [700 + 1020, 4096 + 1019, 4097 + 1019, 8192 + 1019, 8192 + 3 * 4096 + 1019 + 5])
def test_statistics_of_wide_spans(widths, nout):
    """Windows whose centred running sums span more than 16 bits, whole and
    ragged, around half a segment: sums, cuts and events equal the oracle's."""
    series = _window_extremes(nout)
    bw = oracle.boxcar(series, widths)
    s1, s2, thr = _ref_stats(bw, 5.0)
    ref = oracle.find_events(bw, 5.0)
    for u16 in (True, False):
        ev, (g1, g2, gt) = _find(series, widths, 5.0, u16, capacity=1 << 18)
        assert (g1 == s1).all() and (g2 == s2).all() and (gt == thr).all(), u16
        events_equal(ev, ref)


@pytest.mark.parametrize("top", [(1 << 17) - 1, 1 << 17, (1 << 18) + 1, (1 << 19) - 1, 1 << 19, 1 << 21])
@pytest.mark.parametrize("widths", [[1, 2, 4, 8], [1, 2, 62, 64], [1, 2, 4, 66], [1, 2, 128, 130], [2, 4, 256, 512]])
def test_statistics_of_large_int32_values(top, widths):
    """int32 samples around 2^17, 2^19 (where centred running sums give way to
    plain ones) and, times the widest boxcar, around 2^25 and 2^26 (64- and
    128-bit square sums): sums, cuts and events equal the oracle's."""
    nout = 8192 + 4500
    rng = np.random.default_rng(top % 97 + widths[-1])
    t = np.arange(nout)
    series = np.stack([np.full(nout, top), np.where(t // 2304 % 2 == 0, top, 0),
                       np.where(t < 4608, top, 0), rng.integers(0, top + 1, size=nout),
                       top - rng.integers(0, 64, size=nout)]).astype(np.int64)
    bw = oracle.boxcar(series, widths)
    s1, s2, thr = _ref_stats(bw, 3.0)
    ref = oracle.find_events(bw, 3.0)
    ev, (g1, g2, gt) = _find(series, widths, 3.0, False, capacity=1 << 18)
    assert (g1 == s1).all() and (g2 == s2).all() and (gt == thr).all()
    events_equal(ev, ref)


def test_statistics_time_of_wide_spans():
    """A window that the 16-bit sums do not take costs a few passes over LDS,
    not another kind of arithmetic: per position and width a 32-bit read and a
    64-bit multiply-add in place of half a packed word's, so a search of only
    such windows takes at most twice one of none.  (Strong drift, and int32
    values above 2^17; nothing is above the cut, so the rest is the same.)"""
    import time
    from paper_1112_0065_amd import _lib as L
    torch = torch_dev()
    ndm, nout, widths = 600, 200003, [1 << i for i in range(10)]
    g = torch.Generator(device="cuda").manual_seed(1)
    quiet = 12000 + torch.randint(0, 100, (ndm, nout), generator=g, device="cuda", dtype=torch.int32)
    t = torch.arange(nout, device="cuda").float()
    drift = quiet + (5000 * torch.sin(t / 3000.0)).to(torch.int32)
    large = quiet + 60000 + torch.randint(0, 1 << 17, (ndm, nout), generator=g, device="cuda", dtype=torch.int32) // 64 * 64
    ws = torch.empty(L.find_peaks_workspace_bytes(ndm, nout, widths), dtype=torch.uint8, device="cuda")
    ev = torch.empty(40 << 10, dtype=torch.uint8, device="cuda")

    def us(series, w):
        def run():
            assert L.find_peaks(series, ndm, nout, w, 1000.0, ev, 1 << 10, ws) == 0
        for _ in range(3):
            run()
        times = []
        for _ in range(7):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            for _ in range(5):
                run()
            times.append(time.perf_counter() - t0)
        return 2e5 * sorted(times)[3]

    for name, a, b, w in (("u16 drift", quiet.to(torch.int16), drift.to(torch.int16), widths),
                          ("i32 drift", quiet, drift, widths), ("i32 large", quiet, large, widths[:8])):
        q, x = us(a, w), us(b, w)
        log(name, "quiet us", q, "wide us", x)
        assert x <= 2.0 * q, name


def test_statistics_packed_square_sums_use_all_32_bits():
    """The packed form's accumulators near their limit: centred running sums
    that alternate between 0 and 16000 (a span the form takes) give boxcars of
    +-16000 at width 512, so a thread's 16 squares sum to 0.95 x 2^32."""
    nout = 9216
    series = np.full((3, nout), 30000, np.int64)
    for row, off in enumerate((256, 257, 300)):
        at = np.arange(off, nout, 512)
        series[row, at[0::2]] += 16000
        series[row, at[1::2]] -= 16000
    for widths in ([2, 4, 8, 512], [1, 2, 4, 256, 512]):
        # the form's own conditions: the span of the centred running sums of the
        # window, and a thread's squares (positions 2 t and 2 t + 1 mod 512 of half a segment)
        for row in range(3):
            c = int(series[row].astype(np.float64).mean() + 0.5)
            p = np.concatenate([[0], np.cumsum(series[row] - c)])[:8192 + 512]
            assert c == 30000 and p.max() - min(p.min(), 0) <= (1 << 14) - 1
            b = p[512:512 + 8192] - p[:8192]
            sq = (b[:4096].reshape(8, 256, 2).astype(np.int64) ** 2).sum(axis=(0, 2))
            assert (1 << 31) < sq.max() < (1 << 32)
        s1, s2, thr = _ref_stats(oracle.boxcar(series, widths), 3.0)
        for u16 in (True, False):
            _, (g1, g2, gt) = _find(series, widths, 3.0, u16, capacity=1 << 18)
            assert (g1 == s1).all() and (g2 == s2).all() and (gt == thr).all(), u16


def _us(run, calls=3, rounds=5):
    """Median time of one call, us (find_peaks waits for the GPU by itself)."""
    import time
    torch = torch_dev()
    run()
    times = []
    for _ in range(rounds):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(calls):
            run()
        times.append((time.perf_counter() - t0) / calls)
    return 1e6 * sorted(times)[rounds // 2]


@pytest.mark.parametrize("nseg", [2048, 2049])
def test_event_slots_of_long_series(nseg):
    """The event slots of a series of at most 2048 segments and of a longer one:
    events in every segment's place, equal to the oracle's."""
    rng = np.random.default_rng(nseg)
    widths = [1, 3]
    nout = (nseg - 1) * 8192 + 77 + widths[-1] - 1
    series = rng.integers(0, 40, size=(2, nout)).astype(np.int64)
    for row, step in enumerate((3001, 90001)):
        series[row, 5::step] += 400
    ref = oracle.find_events(oracle.boxcar(series, widths), 12.0)
    assert len(ref) > nseg
    for u16 in (True, False):
        ev, _ = _find(series, widths, 12.0, u16, capacity=1 << 16)
        events_equal(ev, ref)


def test_time_of_a_long_series_is_linear():
    """What the events of a series cost (every segment has one) grows with its
    segments, not with their square: per segment 32768 of them take no more than
    4096, half as much again allowed."""
    from paper_1112_0065_amd import _lib as L
    torch = torch_dev()
    widths = [1 << i for i in range(10)]
    g = torch.Generator(device="cuda").manual_seed(2)
    cost = {}
    for lg in (25, 28):
        nout = (1 << lg) + 511
        quiet = torch.randint(1000, 1100, (1, nout), generator=g, device="cuda", dtype=torch.int16)
        pulses = quiet.clone()
        pulses[:, 4000::8192] += 3000
        ws = torch.empty(L.find_peaks_workspace_bytes(1, nout, widths), dtype=torch.uint8, device="cuda")
        ev = torch.empty(40 << 20, dtype=torch.uint8, device="cuda")
        nseg, t = 1 << (lg - 13), []
        for series in (quiet, pulses):
            n = L.find_peaks(series, 1, nout, widths, 20.0, ev, 1 << 20, ws)
            assert n == 0 if series is quiet else n >= nseg
            t.append(_us(lambda: L.find_peaks(series, 1, nout, widths, 20.0, ev, 1 << 20, ws)))
        cost[lg] = (t[1] - t[0]) / nseg
        log("segments", nseg, "quiet us", t[0], "events us", t[1], "per segment", cost[lg])
    assert cost[28] <= 1.5 * cost[25]


@pytest.mark.parametrize("ndm,nout,k", [
    (60, 8192 + 303, 1.2), (4096, 90, 5.0),                           # the largest blocks
    (4097, 90, 5.0), (1290, 8192 + 303, 1.2), (32768, 40, 1.2),       # the middle ones: by number or by cut
    (32769, 40, 1.2),                                                 # the smallest
])
def test_list_passes_with_every_block_size(ndm, nout, k):
    """The count and write passes on both sides of the lines between their block
    sizes (4096 and 32768 segments in all, a cut that noise passes): every series
    listed, one with more runs in a segment than the passes list at once, equal to the
    oracle's."""
    rng = np.random.default_rng(ndm)
    widths = [1, 2]
    series = rng.integers(0, 4, size=(ndm, nout)).astype(np.int64)
    at = rng.integers(0, nout, size=ndm)
    series[np.arange(ndm), at] += 60
    if nout > 8192:
        series[:, 100:] = 0           # (few runs elsewhere)
        series[3, ::3] += 60          # 2832 runs, 2731 of them in the first segment
    ref = oracle.find_events(oracle.boxcar(series, widths), k)
    assert len(ref) > ndm
    for u16 in (True, False):
        ev, _ = _find(series, widths, k, u16, capacity=1 << 20)
        events_equal(ev, ref)


def test_time_of_listed_segments_on_both_sides_of_the_line():
    """With every segment listed, a segment's share of a search of 30500 segments
    (the larger blocks) is that of 36600 (the smaller ones), 15% allowed."""
    from paper_1112_0065_amd import _lib as L
    torch = torch_dev()
    widths, nout = [1 << i for i in range(10)], 500000
    g = torch.Generator(device="cuda").manual_seed(4)
    per = []
    for ndm in (500, 600):
        x = torch.randn((ndm, nout), generator=g, device="cuda").mul_(30).add_(1500).round_().to(torch.int16)
        ws = torch.empty(L.find_peaks_workspace_bytes(ndm, nout, widths), dtype=torch.uint8, device="cuda")
        ev = torch.empty(40 << 20, dtype=torch.uint8, device="cuda")
        n = L.find_peaks(x, ndm, nout, widths, 4.0, ev, 1 << 20, ws)
        segments = ndm * -(-(nout - 511) // 8192)
        per.append(_us(lambda: L.find_peaks(x, ndm, nout, widths, 4.0, ev, 1 << 20, ws)) / segments)
        log("segments", segments, "events", n, "us per segment", per[-1])
        assert n > segments
    assert per[0] <= 1.15 * per[1]
