"""The strip dedispersion kernel against the oracle, bit for bit, where its tiles, channel
groups, staging passes and edge path end: output lengths about multiples of its tile, channel
counts about multiples of its groups and steps, narrow and wide blocks of trials, delays that
put staged rows before the first and past the last sample, several pitches."""

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

TILE = 864

CASES = [
    # nchan, n_out, f_top, foff, dms
    *[(nchan, TILE + 1, 1500.0, 1.0, list(np.arange(33) * 2.0)) for nchan in (1, 2, 7, 8, 9, 15, 16, 17, 31, 33)],
    *[(24, n_out, 1500.0, 2.0, list(np.arange(32) * 1.0))
      for n_out in (1, 3, 127, 128, TILE - 1, TILE, TILE + 127, 2 * TILE - 4, 2 * TILE, 2 * TILE + 5, 5 * TILE + 333)],
    (40, 3 * TILE + 1, 1500.0, 2.0, [0.0]),                          # one trial
    (40, 3 * TILE - 1, 1500.0, 2.0, [700.0]),                        # one far trial
    (40, 2 * TILE + 9, 1200.0, 4.0, list(np.arange(65) * 9.0)),      # wide steps: few trials a block, long delays
    (200, 4 * TILE, 1500.0, 0.5, list(np.arange(40) * 0.05)),        # hardly any drift: long runs
    (130, 2500, 1300.0, 2.0, list(np.arange(96) * 4.0)),
    (64, 6000, 400.0, 1.0, list(np.arange(20) * 1.5)),               # steep: short runs
    (513, 1800, 1500.0, 0.25, list(np.arange(31) * 3.0)),
]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_strip_kernel_matches_oracle(case):
    import torch
    from paper_2101_00941_amd import Plan
    nchan, n_out, f_top, foff, dms = CASES[case]
    probe = Plan(nchan, 1 << 24, f_top, foff, 64e-6, dms, [1], 6.0, host_only=True)
    nsamp = n_out + probe.info["maxshift"]
    plan = Plan(nchan, nsamp, f_top, foff, 64e-6, dms, [1], 6.0)
    strip = [v for v, i in enumerate(Plan.variants()) if i["layout"] == 8]
    assert strip and plan.variant in strip
    rng = np.random.default_rng(case)
    x = rng.integers(0, 256, (nchan, nsamp), dtype=np.uint8)
    x[:, rng.integers(0, nsamp, 4)] = 255
    x[:, rng.integers(0, nsamp, 4)] = 0
    want = oracle.dedisperse(x, plan.shifts().astype(np.int64), nsamp)
    # the tightest pitch and wider ones (multiples of 16, as the call asks); bytes past a row's
    # samples hold 255
    tight = (nsamp + 15) // 16 * 16
    for pitch, first in ((tight, 0), (tight + 16 * (1 + case % 3), 16), ((nsamp + 255) // 256 * 256, 0)):
        buf = torch.full((first + nchan * pitch,), 255, dtype=torch.uint8, device="cuda")
        xd = buf[first:].view(nchan, pitch)
        xd[:, :nsamp] = torch.from_numpy(x).cuda()
        guard = -7
        out = torch.full((len(dms), (n_out + 5 + case % 2) // 4 * 4 + 4), guard, dtype=torch.int32, device="cuda")
        plan.dedisperse(xd, n_in=nsamp, out=out)
        got = out.cpu().numpy()
        assert np.array_equal(got[:, :n_out], want), (case, pitch, first)
        assert (got[:, n_out:] == guard).all(), (case, pitch, first)


@pytest.mark.parametrize("pitch", [(1 << 26) - 16, 1 << 26, (1 << 26) + 16])
def test_strip_kernel_wide_pitch(pitch):
    """Row distances about the largest that the kernel reaches with 31-bit offsets."""
    import torch
    from paper_2101_00941_amd import Plan
    nchan, dms = 37, list(np.arange(33) * 2.0)
    probe = Plan(nchan, 1 << 24, 1500.0, 1.0, 64e-6, dms, [1], 6.0, host_only=True)
    nsamp = TILE + 200 + probe.info["maxshift"]
    plan = Plan(nchan, nsamp, 1500.0, 1.0, 64e-6, dms, [1], 6.0)
    x = np.random.default_rng(pitch).integers(0, 256, (nchan, nsamp), dtype=np.uint8)
    want = oracle.dedisperse(x, plan.shifts().astype(np.int64), nsamp)
    xd = torch.empty((nchan, pitch), dtype=torch.uint8, device="cuda")
    xd[:, :nsamp] = torch.from_numpy(x).cuda()
    got = plan.dedisperse(xd, n_in=nsamp)
    assert np.array_equal(got[:, :want.shape[1]].cpu().numpy(), want)
