"""The two kernels that a new plan's launches choose from, against the oracle bit for bit: the strip
kernel set as the plan's variant, so that it also takes the small shapes that a new plan leaves to
the step kernel, and the step kernel in the batched and the decimated-range calls."""

import numpy as np
import pytest

import oracle
from tests.gpu_util import assert_candidates_equal
from tests.test_gpu_strip import CASES

pytestmark = pytest.mark.gpu

STEP = 25


@pytest.mark.parametrize("case", range(len(CASES)))
def test_chosen_strip_kernel_matches_oracle(case):
    import torch
    from paper_2101_00941_amd import Plan
    nchan, n_out, f_top, foff, dms = CASES[case]
    probe = Plan(nchan, 1 << 24, f_top, foff, 64e-6, dms, [1], 6.0, host_only=True)
    nsamp = n_out + probe.info["maxshift"]
    plan = Plan(nchan, nsamp, f_top, foff, 64e-6, dms, [1], 6.0)
    x = np.random.default_rng(50 + case).integers(0, 256, (nchan, nsamp), dtype=np.uint8)
    want = oracle.dedisperse(x, plan.shifts().astype(np.int64), nsamp)
    pitch = (nsamp + 15) // 16 * 16
    xd = torch.full((nchan, pitch), 255, dtype=torch.uint8, device="cuda")
    xd[:, :nsamp] = torch.from_numpy(x).cuda()
    for v in [plan.variant, STEP]:
        plan.set_variant(v)
        out = torch.full((len(dms), (n_out + 3) // 4 * 4 + 4), -7, dtype=torch.int32, device="cuda")
        got = plan.dedisperse(xd, n_in=nsamp, out=out).cpu().numpy()
        assert np.array_equal(got[:, :n_out], want), v
        assert (got[:, n_out:] == -7).all(), v


def _beams():
    from paper_2101_00941_amd import Plan
    out = []
    for i, (nchan, nsamp, ndm) in enumerate([(16, 9000, 20), (100, 12001, 70), (64, 5000, 33)]):
        dms = np.arange(ndm) * 1.0
        rng = np.random.default_rng(i)
        x = np.clip(rng.normal(128, 16, (nchan, nsamp)), 0, 255).astype(np.uint8)
        x[:, nsamp // 3:nsamp // 3 + 6] = np.minimum(x[:, nsamp // 3:nsamp // 3 + 6].astype(int) + 40, 255)
        args = (nsamp, 1500.0, 100.0 / nchan, 64e-6, dms, [1, 2, 4, 8], 6.0)
        out.append((Plan(nchan, *args, 4096), x, nsamp, oracle.run(x, *args, stat_block=4096)["candidates"]))
    return out


def test_batch_of_step_kernel_matches_oracle():
    import torch
    from paper_2101_00941_amd import batch_run, candidates_as_tuples
    beams = _beams()
    dev = []
    for _, x, nsamp, _ in beams:
        d = torch.full((x.shape[0], (nsamp + 255) // 256 * 256), 255, dtype=torch.uint8, device="cuda")
        d[:, :nsamp] = torch.from_numpy(x).cuda()
        dev.append(d)
    cands, counts, info = batch_run([(b[0], d, b[2]) for b, d in zip(beams, dev)], variant=STEP, work_bytes=64 << 20,
                                    cap=4096)
    assert info["variant"] == STEP
    for (_, _, _, want), c, n in zip(beams, cands, counts):
        assert len(want) > 0 and n == len(want)
        assert_candidates_equal(candidates_as_tuples(c), want)


def test_ranges_of_step_kernel_match_oracle():
    import torch
    from paper_2101_00941_amd import RangePlan, candidates_as_tuples, candidates_to_numpy
    nchan, nsamp, dms, widths = 64, 40000, np.arange(90) * 1.0, [1, 2, 4, 8]
    rng = np.random.default_rng(9)
    x = np.clip(rng.normal(128, 16, (nchan, nsamp)), 0, 255).astype(np.uint8)
    x[:, 20000:20008] = np.minimum(x[:, 20000:20008].astype(int) + 40, 255)
    first, factor = [0, 40], [1, 2]
    args = (nsamp, 1450.0, 300.0 / nchan, 64e-6, dms, widths, 6.0)
    want = oracle.run_ranges(x, *args, 8192, first, factor)["candidates"]
    rp = RangePlan(nchan, *args, first, factor, 8192)
    xd = torch.full((nchan, (nsamp + 255) // 256 * 256), 255, dtype=torch.uint8, device="cuda")
    xd[:, :nsamp] = torch.from_numpy(x).cuda()
    for v in (None, STEP):
        if v is not None:
            rp.set_variant(v)
        cand, count = rp.run(xd, n_in=nsamp, cap=1 << 14)
        torch.cuda.synchronize()
        assert int(count.item()) == len(want) and len(want) > 0
        assert_candidates_equal(candidates_as_tuples(candidates_to_numpy(cand, count)), want)
