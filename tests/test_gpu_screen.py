"""The integer-screened single-pulse detection against the oracle where its runs, tiles and
width rules end: planes drawn directly, so that any pitch, alignment, number of trials and
starts, width list and share of passing cells can be had. Candidate positions and widths are
equal; S/N is one float32 rounding of the oracle's float64 value."""

import numpy as np
import pytest

import oracle
from tests.gpu_util import assert_candidates_equal, say

pytestmark = pytest.mark.gpu

POW2 = [1, 2, 4, 8, 16, 32, 64, 128, 256]


def _search(D, widths, thr, block, full_width, shift, pad, t_begin=0, t_end=None, t_total=None, want_best=False):
    """Search a plane whose rows start `shift` dwords past a 16-byte boundary and are `pad`
    columns longer than it is wide; the columns around it hold a large value."""
    import torch
    from paper_2101_00941_amd import Plan, candidates_as_tuples, candidates_to_numpy
    ndm, n = D.shape
    # a plan for its trials, widths and threshold: at (almost) one DM there are no delays
    plan = Plan(16, n, 1500.0, 1.0, 64e-6, np.arange(ndm) * 1e-9, widths, thr, block, boxcar_full_width=full_width)
    pitch = n + pad
    buf = torch.full((shift + ndm * pitch,), 4080, dtype=torch.int32, device="cuda")
    dd = torch.as_strided(buf, (ndm, pitch), (pitch, 1), shift)
    dd[:, :n] = torch.from_numpy(D.astype(np.int32)).cuda()
    cand, count, _ = plan.single_pulse(dd, dd_n=n, t_begin=t_begin, t_end=t_end, t_total=t_total, cap=1 << 18,
                                       want_best=want_best)
    torch.cuda.synchronize()
    return candidates_as_tuples(candidates_to_numpy(cand, count)), int(count.item())


def _plane(ndm, n, seed):
    rng = np.random.default_rng(seed)
    D = np.clip(np.rint(rng.normal(2000, 60, (ndm, n))), 0, 4080).astype(np.int64)
    for _ in range(1 + n // 400):   # bright samples, also at both ends of rows and tiles
        d, t, w = int(rng.integers(ndm)), int(rng.integers(n)), int(rng.integers(1, 20))
        D[max(0, d - 1):d + 2, t:t + w] += int(rng.integers(150, 900))
    D[0, 0] = D[-1, n - 1] = 4080
    for t in range(256, n, 1024):
        D[int(rng.integers(ndm)), t - int(rng.integers(0, 2))] = 4000
    return np.minimum(D, 4080)


CASES = [
    # ndm, starts, widths, threshold, stat block, full width, dword shift, pad
    (1, 1, [1], 0.0, 256, 0, 0, 0),
    (1, 255, [1], 2.0, 256, 0, 1, 1),
    (2, 256, [1, 2], 3.0, 256, 0, 3, 2),
    (3, 257, [1, 2, 4], 3.0, 512, 0, 2, 3),
    (5, 2047, POW2[:6], 4.0, 256, 0, 0, 1),
    (4, 2048, POW2, 4.0, 512, 0, 1, 0),
    (7, 2049, POW2, 5.0, 32768, 0, 2, 5),
    (33, 20481, POW2, 4.5, 4096, 0, 0, 3),
    (9, 5000, POW2, 1.0, 1024, 0, 0, 0),      # most rows have many passing cells
    (6, 4097, POW2, 3.0, 2048, 1, 0, 1),      # hierarchy: strides 2 .. 256
    (6, 4097, POW2[:8], 3.0, 2048, 16, 1, 2),
    (5, 3001, [1, 2, 4, 8, 12], 3.0, 1024, 0, 0, 0),
    (5, 3001, [3, 5, 6, 7, 9, 255], 3.0, 1024, 0, 3, 1),
    (4, 2500, [1, 3, 10, 50, 249], 2.0, 512, 10, 0, 0),
    (4, 3000, [2, 4, 8, 256], 3.0, 1024, 0, 0, 2),
    (3, 3000, [1, 2, 4, 257], 3.0, 1024, 0, 1, 0),      # past one group of 256 columns
    (3, 3000, [1, 64, 511, 512, 1024], 3.0, 1024, 64, 0, 1),
    (4, 2600, [1 << k for k in range(11)], 3.0, 256, 0, 2, 0),
    (2, 300000, POW2, 5.0, 32768, 0, 0, 0),
    (401, 6000, POW2[:6], 4.0, 2048, 0, 0, 0),          # several tiles a run
]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_screened_detection_matches_oracle(case):
    ndm, starts, widths, thr, block, full_width, shift, pad = CASES[case]
    n = starts + widths[-1] - 1
    D = _plane(ndm, n, 100 + case)
    kw = dict(boxcar_full_width=full_width) if full_width else {}
    want, _ = oracle.single_pulse(D, 0, 0, starts, starts, widths, thr, block, **kw)
    got, count = _search(D, widths, thr, block, full_width, shift, pad)
    say(f"case {case}: {len(want)} candidates")
    assert count == len(want)
    assert_candidates_equal(got, want)


@pytest.mark.parametrize("a,b,open_end", [(0, 700, True), (512, 1400, True), (1024, 3801, False)])
@pytest.mark.parametrize("widths", [POW2[:5], [1, 3, 300]])
def test_screened_detection_of_a_range(a, b, open_end, widths):
    starts, block = 3801, 512
    D = _plane(6, starts + widths[-1] - 1, 7)
    total = -1 if open_end else starts
    want, _ = oracle.single_pulse(D, 0, a, b, total, widths, 3.0, block)
    got, _ = _search(D, widths, 3.0, block, 0, 0, 1, t_begin=a, t_end=b, t_total=total)
    assert len(want) > 0
    assert_candidates_equal(got, want)
