"""GPU parity of the multibeam coincidence RFI mask (section 2.1) against the
oracle, through the C ABI: zero-DM series and cut levels bit-exact, mask
bit-exact, over the 1024-channel fast path, the any-width path, thresholds
with ties, vote counts at the edges, constant beams and bad arguments."""
import numpy as np
import pytest

import oracle
import synth
from gpu_common import log, to_dev, torch_dev

pytestmark = pytest.mark.gpu


def _run(packed, nchans, nsamps, k, min_beams):
    from paper_1112_0065_amd import _lib as L
    torch = torch_dev()
    ins = [to_dev(p) for p in packed]
    ws = torch.empty(L.dedisp_rfi_mask_workspace_bytes(len(ins), nsamps), dtype=torch.uint8,
                     device="cuda")
    mask = torch.empty(nsamps, dtype=torch.uint8, device="cuda")
    n = L.dedisp_rfi_mask(ins, nchans, nsamps, k, min_beams, mask, ws)
    z, thr = L.dedisp_rfi_mask_read_stats(ws, len(ins), nsamps)
    return n, mask.cpu().numpy().astype(bool), z, thr


def _check(packed, nchans, nsamps, k, min_beams):
    zs = [oracle.zero_dm_series(p, nsamps, nchans) for p in packed]
    ref_mask, votes, ref_thr = oracle.rfi_mask(zs, k, min_beams)
    n, mask, z, thr = _run(packed, nchans, nsamps, k, min_beams)
    assert (z == np.array(zs)).all()
    assert thr.tolist() == [-1 if t is None else t for t in ref_thr]
    assert (mask == ref_mask).all() and n == int(ref_mask.sum())
    return n


@pytest.mark.parametrize("nchans", [64, 1024, 20])
def test_mask_matches_oracle(nchans):
    nsamps = 1 << 14
    packed, imps, amps, _ = synth.make_coincidence_beams(5, nbeams=13, nsamps=nsamps, nchans=nchans)
    for k, m in [(3.0, 4), (1.0, 4), (2.5, 1), (3.0, 13), (3.0, 14)]:
        n = _check(packed, nchans, nsamps, k, m)
        log("coincidence", nchans, k, m, "masked", n)


def test_constant_and_ragged_beams():
    nsamps = 5003                                  # not a multiple of any block
    rng = np.random.default_rng(2)
    q = [rng.integers(0, 4, size=(nsamps, 64), dtype=np.uint8) for _ in range(5)]
    q[1][:] = 2                                    # constant beam: D = 0
    q[0][100:103] = 3
    q[2][100:103] = 3
    q[3][100:103] = 3
    packed = [synth.pack_2bit(x) for x in q]
    n = _check(packed, 64, nsamps, 3.0, 3)
    assert n >= 3


@pytest.mark.parametrize("nchans", [4, 60, 64, 68, 128, 132, 256, 260, 512, 1000, 1024, 1028, 2048, 2052,
                                    4096, 4100, 21844])
def test_sample_sizes_and_alignments(nchans):
    """Groups of 1 to 64 lanes per sample, a shared last piece of 16 bytes,
    several pieces per lane, samples at any byte; 1 to 9001 samples (one to
    several blocks of 8192, fewer than four for the vote)."""
    from paper_1112_0065_amd import _lib as L
    torch = torch_dev()
    rng = np.random.default_rng(nchans)
    for nsamps in (1, 3, 5, 2049, 9001):
        packed = [rng.integers(0, 256, size=nsamps * nchans // 4, dtype=np.uint8) for _ in range(3)]
        zs = [oracle.zero_dm_series(p, nsamps, nchans) for p in packed]
        ref_mask, _, ref_thr = oracle.rfi_mask(zs, 1.0, 2)
        for at in (0, 1, 6):
            ins = [to_dev(np.concatenate([np.zeros(at, np.uint8), p]))[at:] for p in packed]
            ws = torch.empty(L.dedisp_rfi_mask_workspace_bytes(3, nsamps), dtype=torch.uint8, device="cuda")
            mask = torch.full((nsamps + 3,), 7, dtype=torch.uint8, device="cuda")
            n = L.dedisp_rfi_mask(ins, nchans, nsamps, 1.0, 2, mask[:nsamps], ws)
            z, thr = L.dedisp_rfi_mask_read_stats(ws, 3, nsamps)
            got = mask.cpu().numpy()
            assert (z == np.array(zs)).all(), (nsamps, at)
            assert thr.tolist() == [-1 if t is None else t for t in ref_thr]
            assert (got[:nsamps] == ref_mask).all() and n == int(ref_mask.sum())
            assert (got[nsamps:] == 7).all()


def test_full_chunk_1024_channels():
    """13 beams x 2^17 samples x 1024 channels (one streaming chunk of the
    survey backend)."""
    nsamps = 1 << 17
    packed, imps, amps, _ = synth.make_coincidence_beams(11, nbeams=13, nsamps=nsamps)
    n = _check(packed, 1024, nsamps, 3.0, 4)
    inside = np.zeros(nsamps, bool)
    for im in imps:
        inside[im.t:im.t + im.width] = True
    log("full chunk: impulses", len(imps), "masked", n, "impulse samples", int(inside.sum()))
    assert 0 < n <= inside.sum()


def test_bad_arguments():
    from paper_1112_0065_amd import _lib as L
    torch = torch_dev()
    p = to_dev(np.zeros(64 * 16, np.uint8))
    ws = torch.empty(1 << 16, dtype=torch.uint8, device="cuda")
    mask = torch.empty(64, dtype=torch.uint8, device="cuda")
    for args, st in [((64, 64, 0.0, 4), L.ERR_INVALID_ARG), ((64, 64, 3.0, 0), L.ERR_INVALID_ARG),
                     ((62, 64, 3.0, 4), L.ERR_INVALID_ARG), ((64, 0, 3.0, 4), L.ERR_INVALID_ARG)]:
        with pytest.raises(L.DedispError) as e:
            L.dedisp_rfi_mask([p], *args, mask, ws)
        assert e.value.status == st
    assert L.dedisp_rfi_mask_workspace_bytes(65, 100) == 0


@pytest.mark.parametrize("nchans,aligned", [(1024, True), (64, True), (20, True), (1024, False)])
def test_apply_matches_oracle(nchans, aligned):
    """The mask computed on the GPU, applied on the GPU in place, equals the
    oracle's replacement of the flagged samples, byte for byte, on 16-byte
    rows, short rows and misaligned buffers."""
    from paper_1112_0065_amd import _lib as L
    torch = torch_dev()
    nsamps = 1 << 14
    packed, imps, amps, _ = synth.make_coincidence_beams(8, nbeams=13, nsamps=nsamps, nchans=nchans,
                                                         impulse_rate=20.0)
    zs = [oracle.zero_dm_series(p, nsamps, nchans) for p in packed]
    ref_mask, _, _ = oracle.rfi_mask(zs, 3.0, 4)
    assert ref_mask.sum() > 0
    bufs = []
    for p in packed:
        if aligned:
            bufs.append(to_dev(p))
        else:                                  # a view one byte into a larger buffer
            big = to_dev(np.concatenate([np.zeros(1, np.uint8), p]))
            bufs.append(big[1:])
    ws = torch.empty(L.dedisp_rfi_mask_workspace_bytes(13, nsamps), dtype=torch.uint8, device="cuda")
    mask = torch.empty(nsamps, dtype=torch.uint8, device="cuda")
    L.dedisp_rfi_mask(bufs, nchans, nsamps, 3.0, 4, mask, ws)
    L.dedisp_rfi_apply(bufs, nchans, nsamps, mask)
    torch.cuda.synchronize()
    for b, p in enumerate(packed):
        want = oracle.replace_masked(oracle.unpack_2bit(p, nsamps, nchans), ref_mask)
        got = oracle.unpack_2bit(bufs[b].cpu().numpy(), nsamps, nchans)
        assert (got == want).all(), b
    # applied data no longer flags the same samples
    n2 = L.dedisp_rfi_mask(bufs, nchans, nsamps, 3.0, 4, mask, ws)
    assert not (mask.cpu().numpy().astype(bool) & ref_mask).any()
    log(f"nchans {nchans}: {int(ref_mask.sum())} samples replaced, {n2} flagged after")
