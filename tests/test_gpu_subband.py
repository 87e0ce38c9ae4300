"""GPU parity of subband (two-stage) dedispersion against the oracle,
through the C ABI: exact integers for every (subbands, group) shape tried,
both output types, ragged groups, the shortest input, the survey beam on
sampled trials, and the exact reduction to direct dedispersion."""
import numpy as np
import pytest

import oracle
from oracle.subband import effective_delays, subband_dedisperse
import synth
from gpu_common import log, small_case, survey_case, to_dev, torch_dev

pytestmark = pytest.mark.gpu


def _run(fb, plan, nsub, group, u16=True, packed=None, nsamps=None):
    from paper_1112_0065_amd import _lib as L
    torch = torch_dev()
    nsamps = fb.nsamps if nsamps is None else nsamps
    packed = fb.packed if packed is None else packed
    sb = L.dedisp_subband_create(plan, nsub, group)
    nout = nsamps - sb.max_delay
    ws = torch.empty(L.dedisp_subband_workspace_bytes(sb, nsamps), dtype=torch.uint8, device="cuda")
    out = torch.empty((len(fb.dm_list), nout), dtype=torch.int16 if u16 else torch.int32,
                      device="cuda")
    L.dedisp_subband_execute(sb, to_dev(packed), nsamps, out, ws)
    torch.cuda.synchronize()
    o = out.cpu().numpy()
    return sb, (o.view(np.uint16).astype(np.int64) if u16 else o.astype(np.int64))


@pytest.mark.parametrize("nsub,group", [(1, 1), (4, 3), (16, 4), (64, 1), (32, 16), (8, 7), (2, 9)])
def test_small_config_matches_oracle(nsub, group):
    from paper_1112_0065_amd import _lib as L
    fb, dly, x, direct = small_case()
    plan = L.dedisp_plan_create(fb.nchans, fb.f_top, fb.df, fb.tsamp, fb.dm_list)
    ref = subband_dedisperse(x, fb.f_top, fb.df, fb.tsamp, fb.dm_list, nsub, group)
    for u16 in (True, False):
        sb, got = _run(fb, plan, nsub, group, u16)
        assert sb.ncoarse == (100 + group - 1) // group
        assert got.shape == ref.shape and (got == ref).all(), (nsub, group, u16)
    if (nsub, group) == (1, 1):
        assert (got == direct).all()       # one subband, one trial per group: the direct sum
    log(f"nsub {nsub} group {group}: {ref.shape}, span {sb.span}")


def test_shortest_input_and_bad_arguments():
    from paper_1112_0065_amd import _lib as L
    fb, dly, x, direct = small_case()
    plan = L.dedisp_plan_create(fb.nchans, fb.f_top, fb.df, fb.tsamp, fb.dm_list)
    sb = L.dedisp_subband_create(plan, 16, 4)
    nsamps = sb.max_delay + 1                       # one output sample
    bpt = fb.nchans // 4
    packed = fb.packed[:nsamps * bpt]
    _, got = _run(fb, plan, 16, 4, packed=packed, nsamps=nsamps)
    ref = subband_dedisperse(x[:, :nsamps], fb.f_top, fb.df, fb.tsamp, fb.dm_list, 16, 4)
    assert got.shape == (100, 1) and (got == ref).all()
    assert L.dedisp_subband_workspace_bytes(sb, sb.max_delay) == 0
    for nsub, group in ((3, 1), (128, 1), (16, 0), (16, 17)):    # 128: subbands of 2 channels
        with pytest.raises(L.DedispError) as ei:
            L.dedisp_subband_create(plan, nsub, group)
        assert ei.value.status == L.ERR_INVALID_ARG
    torch = torch_dev()
    ws = torch.empty(1 << 20, dtype=torch.uint8, device="cuda")
    out = torch.empty((100, 1), dtype=torch.int16, device="cuda")
    with pytest.raises(L.DedispError) as ei:
        L.dedisp_subband_execute(sb, to_dev(packed), sb.max_delay, out, ws)
    assert ei.value.status == L.ERR_TOO_FEW_SAMPLES


def test_survey_beam_sampled_trials():
    """1024 channels, 2^19 samples, 1200 trials; 32 subbands, groups of 8:
    sampled trials equal the oracle's effective-delay sum."""
    from paper_1112_0065_amd import _lib as L
    fb = survey_case()
    plan = L.dedisp_plan_create(fb.nchans, fb.f_top, fb.df, fb.tsamp, fb.dm_list)
    sb, got = _run(fb, plan, 32, 8)
    eff = effective_delays(fb.nchans, fb.f_top, fb.df, fb.tsamp, fb.dm_list, 32, 8)
    assert sb.max_delay == int(eff.max()) or sb.max_delay >= int(eff.max())
    nout = fb.nsamps - sb.max_delay
    assert got.shape == (1200, nout)
    x = oracle.unpack_2bit(fb.packed, fb.nsamps, fb.nchans)
    rows = [0, 3, 4, 599, 1195, 1199]
    ref = oracle.dedisperse(x, eff[rows], nout=nout)
    for k, d in enumerate(rows):
        assert (got[d] == ref[k]).all(), d
    log(f"survey subband: span {sb.span}, max delay {sb.max_delay}, ncoarse {sb.ncoarse}")


@pytest.mark.parametrize("extra", [1, 2, 2047, 2049])
def test_output_lengths_around_a_tile(extra):
    """Outputs that end at, before and after a stage-2 tile, rows of odd
    length (pairs of samples off word alignment), trials at odd and even
    offsets; both output types."""
    from paper_1112_0065_amd import _lib as L
    fb, dly, x, direct = small_case()
    plan = L.dedisp_plan_create(fb.nchans, fb.f_top, fb.df, fb.tsamp, fb.dm_list)
    nsamps = L.dedisp_subband_create(plan, 8, 3).max_delay + extra
    ref = subband_dedisperse(x[:, :nsamps], fb.f_top, fb.df, fb.tsamp, fb.dm_list, 8, 3)
    for u16 in (True, False):
        _, got = _run(fb, plan, 8, 3, u16, packed=fb.packed[:nsamps * fb.nchans // 4], nsamps=nsamps)
        assert got.shape == ref.shape == (len(fb.dm_list), extra) and (got == ref).all(), u16


def test_time_of_large_groups():
    """A group of 16 trials sums half the coarse series that groups of 8 do, and the
    same fine ones: it takes no longer (a tenth allowed for the wider staged rows)."""
    import time
    from paper_1112_0065_amd import _lib as L
    torch = torch_dev()
    nchans, ndm, nsamps = 1024, 400, 1 << 18
    plan = L.dedisp_plan_create(nchans, 1581.8, -400.0 / nchans, 64e-6, np.linspace(0.0, 300.0, ndm))
    x = torch.randint(0, 256, (nsamps * nchans // 4,), dtype=torch.uint8, device="cuda")
    us = {}
    for group in (8, 16):
        sb = L.dedisp_subband_create(plan, 16, group)
        ws = torch.empty(L.dedisp_subband_workspace_bytes(sb, nsamps), dtype=torch.uint8, device="cuda")
        out = torch.empty((ndm, nsamps - sb.max_delay), dtype=torch.int16, device="cuda")
        times = []
        for _ in range(6):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            for _ in range(5):
                L.dedisp_subband_execute(sb, x, nsamps, out, ws)
            torch.cuda.synchronize()
            times.append((time.perf_counter() - t0) / 5)
        us[group] = 1e6 * sorted(times)[2]
    log("us by group", us)
    assert us[16] <= 1.1 * us[8]


def test_widest_spread_of_a_group():
    """A group whose subband delays spread over just what a staged row holds, and
    one past it, which is refused."""
    from paper_1112_0065_amd import _lib as L
    nchans, ndm, nsub, group = 16, 8, 4, 8

    def plan_of(dm):
        return L.dedisp_plan_create(nchans, 400.0, -10.0, 1e-3, np.linspace(0.0, dm, ndm))

    def span_of(dm):
        d = oracle.delay_table(nchans, 400.0, -10.0, 1e-3, np.linspace(0.0, dm, ndm))[:, ::nchans // nsub]
        return int((d.max(axis=0) - d.min(axis=0)).max())

    lo, hi = 0.0, 1e5
    for _ in range(60):
        mid = 0.5 * (lo + hi)
        lo, hi = (mid, hi) if span_of(mid) <= 7152 else (lo, mid)
    assert 7140 < span_of(lo) <= 7152 < span_of(hi)
    sb = L.dedisp_subband_create(plan_of(lo), nsub, group)
    assert sb.span == span_of(lo)
    nsamps = sb.max_delay + 4099
    packed = np.random.default_rng(5).integers(0, 256, nsamps * nchans // 4).astype(np.uint8)

    class Beam:
        dm_list = np.linspace(0.0, lo, ndm)

    Beam.nsamps, Beam.packed = nsamps, packed
    x = oracle.unpack_2bit(packed, nsamps, nchans)
    ref = subband_dedisperse(x, 400.0, -10.0, 1e-3, Beam.dm_list, nsub, group)
    for u16 in (True, False):
        _, got = _run(Beam, plan_of(lo), nsub, group, u16)
        assert got.shape == ref.shape and (got == ref).all(), u16
    with pytest.raises(L.DedispError) as ei:
        L.dedisp_subband_create(plan_of(hi), nsub, group)
    assert ei.value.status == L.ERR_UNSUPPORTED


def test_first_stage_that_fits_no_lds_tile_is_refused():
    """Coarse trials so far apart that not even blocks of 4 of them fit a block's LDS:
    the two-stage plan is made, its execution refused, and the library works on."""
    from paper_1112_0065_amd import _lib as L
    torch = torch_dev()
    nchans, ndm = 16, 8
    plan = L.dedisp_plan_create(nchans, 400.0, -10.0, 1e-3, np.linspace(0.0, 7000.0, ndm))
    sb = L.dedisp_subband_create(plan, 2, 1)
    nsamps = sb.max_delay + 100
    x = torch.zeros(nsamps * nchans // 4, dtype=torch.uint8, device="cuda")
    ws = torch.empty(L.dedisp_subband_workspace_bytes(sb, nsamps), dtype=torch.uint8, device="cuda")
    out = torch.empty((ndm, 100), dtype=torch.int16, device="cuda")
    with pytest.raises(L.DedispError) as ei:
        L.dedisp_subband_execute(sb, x, nsamps, out, ws)
    assert ei.value.status == L.ERR_UNSUPPORTED
    fb, _, _, direct = small_case()
    _, got = _run(fb, L.dedisp_plan_create(fb.nchans, fb.f_top, fb.df, fb.tsamp, fb.dm_list), 1, 1)
    assert (got == direct).all()
