"""GPU parity of baseline (red-noise) removal (section 2.3) against the
oracle through the C ABI, and what it buys the search: a slow baseline
wiggle inflates every series' sigma so that the sigma-cut misses the
injected pulses; with the running mean removed they are all found."""
import numpy as np
import pytest

import oracle
from gpu_common import events_equal, log, to_dev, torch_dev

pytestmark = pytest.mark.gpu


def _dev(a, u16):
    return to_dev(a.astype(np.uint16).view(np.int16) if u16 else a.astype(np.int32))


def _run(series, radius, offset, in_u16, out_u16):
    from paper_1112_0065_amd import _lib as L
    torch = torch_dev()
    ndm, nout = series.shape
    out = torch.empty((ndm, nout - 2 * radius), dtype=torch.int16 if out_u16 else torch.int32,
                      device="cuda")
    L.baseline_remove(_dev(series, in_u16), ndm, nout, radius, offset, out)
    torch.cuda.synchronize()
    o = out.cpu().numpy()
    return o.view(np.uint16).astype(np.int64) if out_u16 else o.astype(np.int64)


@pytest.mark.parametrize("radius", [0, 1, 7, 2048, 8192])
def test_matches_oracle(radius):
    rng = np.random.default_rng(radius)
    nout = 30001 + 2 * radius
    s = rng.integers(0, 3073, size=(5, nout))
    ref = oracle.baseline_remove(s, radius, 3072)
    for in_u16, out_u16 in [(True, True), (True, False), (False, True), (False, False)]:
        got = _run(s, radius, 3072, in_u16, out_u16)
        assert (got == ref).all(), (radius, in_u16, out_u16)


@pytest.mark.parametrize("nres", [1, 255, 1025, 4095, 4096, 4097, 16383, 16385, 16447, 16384 + 4096 + 2049])
def test_lengths_around_a_step(nres):
    # steps of 4096 (16-bit) or 2048 (32-bit) outputs, then of 1024, then rows of
    # 64 to the end of a segment of 16384; odd lengths put the rows at odd samples
    # and the first segment's end up to 63 outputs later
    rng = np.random.default_rng(nres)
    for radius in (0, 3, 600):
        s = rng.integers(0, 3073, size=(3, nres + 2 * radius))
        s[1] = 3072
        ref = oracle.baseline_remove(s, radius, 3072)
        for in_u16, out_u16 in [(True, True), (True, False), (False, True), (False, False)]:
            got = _run(s, radius, 3072, in_u16, out_u16)
            assert (got == ref).all(), (radius, in_u16, out_u16)


def test_red_noise_removed_pulses_kept():
    from paper_1112_0065_amd import _lib as L
    torch = torch_dev()
    rng = np.random.default_rng(3)
    ndm, nout = 8, 200_000
    t = np.arange(nout)
    noise = np.rint(30 * rng.standard_normal((ndm, nout))).astype(np.int64)
    wiggle = np.rint(40 * np.sin(2 * np.pi * t / 20000.0)).astype(np.int64)
    s = 1536 + noise + wiggle
    pulses = [(20000, 16), (77000, 64), (150000, 4)]
    for t0, w in pulses:
        s[:, t0:t0 + w] += int(round(12 * 30 / np.sqrt(w)))      # S/N ~12 at width w
    widths = [1, 4, 16, 64, 256]

    def search(series):
        n = series.shape[1]
        ws = torch.empty(L.find_peaks_workspace_bytes(ndm, n, widths), dtype=torch.uint8,
                         device="cuda")
        evb = torch.empty((1 << 18) * 40, dtype=torch.uint8, device="cuda")
        k = L.find_peaks(_dev(series, True), ndm, n, widths, 6.0, evb, 1 << 18, ws)
        return L.events_from_buffer(evb, k)

    R = 1024
    flat = _run(s, R, 3072, True, True)
    assert (flat == oracle.baseline_remove(s, R, 3072)).all()
    before, after = search(s), search(flat)

    def near(ev, shift):
        return np.array([any(abs(int(e["t_peak"]) + shift - t0) <= w + 300 for t0, w in pulses)
                         for e in ev], bool)

    nb, na = near(before, 0), near(after, R)

    def found(ev, shift):
        return sum(any(abs(int(e["t_peak"]) + shift - t0) <= w + 300 for e in ev)
                   for t0, w in pulses)

    log("events before", len(before), "false", int((~nb).sum()), "pulses found", found(before, 0),
        "| after", len(after), "false", int((~na).sum()), "pulses found", found(after, R))
    # the wiggle inflates every series' sigma and hides the pulses; with the
    # running mean removed every pulse is found, with no false events
    assert found(before, 0) < len(pulses) and found(after, R) == len(pulses)
    assert (~na).sum() <= 2 and na.sum() > 10 * max(1, nb.sum())
    # the events of the flattened series are those of the oracle chain
    events_equal(after, oracle.find_events(oracle.boxcar(oracle.baseline_remove(s, R, 3072),
                                                         widths), 6.0))


def test_bad_arguments():
    from paper_1112_0065_amd import _lib as L
    torch = torch_dev()
    s = _dev(np.zeros((2, 100), np.int64), True)
    out = torch.empty((2, 100), dtype=torch.int16, device="cuda")
    for r, st in [(-1, L.ERR_INVALID_ARG), (8193, L.ERR_INVALID_ARG), (50, L.ERR_TOO_FEW_SAMPLES)]:
        with pytest.raises(L.DedispError) as e:
            L.baseline_remove(s, 2, 100, r, 0, out)
        assert e.value.status == st


@pytest.mark.parametrize("nres", [63, 64, 65, 1023, 1024, 1087, 1599, 1600, 2047, 2048])
def test_lengths_of_short_rows(nres):
    """Rows around a step of the short form and the lengths where it ends, windows
    wider and narrower than the row, every output alignment."""
    rng = np.random.default_rng(nres)
    for radius in (0, 5, 900):
        s = rng.integers(0, 4000, size=(5, nres + 2 * radius)).astype(np.int64)
        ref = oracle.baseline_remove(s, radius, 3000)
        for u16 in (True, False):
            for o16 in (True, False):
                got = _run(s, radius, 3000, u16, o16)
                assert (got == ref).all(), (radius, u16, o16)


def test_time_of_short_rows():
    """65535 rows of 300 outputs are the samples of 1200 rows of 16384: a wave per row
    starts 55 times as often, with one window to sum and one step each, in at most two
    and a half times the time."""
    import time
    from paper_1112_0065_amd import _lib as L
    torch = torch_dev()
    us = []
    for ndm, nres in ((1200, 16384), (65535, 300)):
        s = torch.randint(100, 2000, (ndm, nres + 14), device="cuda", dtype=torch.int32).to(torch.int16)
        out = torch.empty((ndm, nres), dtype=torch.int16, device="cuda")
        times = []
        for _ in range(9):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            for _ in range(30):
                L.baseline_remove(s, ndm, nres + 14, 7, 3072, out)
            torch.cuda.synchronize()
            times.append((time.perf_counter() - t0) / 30)
        us.append(1e6 * sorted(times)[4])
    log("us", us)
    assert us[1] <= 2.5 * us[0]
