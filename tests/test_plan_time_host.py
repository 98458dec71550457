"""The time a plan takes to make (CPU only): steep trial steps, whose blocks of trials are short,
must not cost many times what the same number of trials and channels costs with a small step. The
search for the longest block has to turn lengths down without going through the whole band."""

import time

import numpy as np
import pytest


@pytest.mark.parametrize("nchan,f_top,foff,step", [(1024, 1450.0, 300.0 / 1024, 20.0), (512, 150.0, 0.05, 1.0)])
def test_steep_plans_are_made_as_fast_as_gentle_ones(nchan, f_top, foff, step):
    from paper_2101_00941_amd import Plan

    def make(s):
        t = time.perf_counter()
        Plan(nchan, 1 << 24, f_top, foff, 64e-6, np.arange(500) * s, [1], 6.0, host_only=True)
        return time.perf_counter() - t
    pairs = [(make(step), make(step / 400)) for _ in range(7)]
    steep, gentle = (min(p[i] for p in pairs) for i in range(2))
    print(f"{nchan} channels: steep {1e3 * steep:.1f} ms, gentle {1e3 * gentle:.1f} ms")
    # a steep plan has up to 32 times as many blocks, whose tables are written in one pass (2 to 6
    # times the time); going through the band for every length that a block is tried at took 50 times
    assert steep < 16 * gentle
