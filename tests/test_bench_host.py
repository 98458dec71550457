"""What bench.py's line says of the kernel that it timed (CPU only)."""

import bench


def test_roofline_names_the_kernel_of_the_layout():
    adds, ms, nbytes = 10 ** 13, 100.0, 8 * 10 ** 11
    strip, step = (bench.mfma_roofline(layout, adds, ms, nbytes) for layout in (8, 4))
    assert strip["kernel"].startswith("dedisp_strip_kernel") and step["kernel"].startswith("dedisp_kernel")
    for r in (strip, step):
        assert r["bound"] == "mfma" and r["achieved"] == 100.0 and r["frac"] == 100.0 / r["peak"]
        assert r["hbm_frac"] == 1.0
        assert not any(k.startswith("alu") for k in r)      # no fraction of a unit that the kernel does not use
