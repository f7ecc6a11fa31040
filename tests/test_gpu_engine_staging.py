"""The engine keeps the field copies' pinned staging buffers between its jobs."""
import gc

import pytest

pytestmark = pytest.mark.gpu

SLAB = 4 << 20  # bytes of a staging buffer


def _pinned():
    """device-file mappings of a staging buffer's size"""
    n = 0
    with open("/proc/self/maps") as fh:
        for line in fh:
            a, b = (int(x, 16) for x in line.split()[0].split("-"))
            n += b - a == SLAB and "/dev/dri/" in line
    return n


def test_staging_outlives_the_last_job():
    import paper_1812_03191_amd as dfm

    cfg = dict(nx=16, ny=16, nz=16, nlevels=1, dx0=0.05, GM=0.01, eps=0.1, L=0.0, mach=0.5, chi=0.1)
    gc.collect()  # runs of earlier tests
    eng = dfm.Engine(dfm.engine_job_bytes(cfg) + (1 << 20))
    held = []
    for _ in range(2):
        s = eng.admit(cfg, 2)
        while eng.active()[0]:
            eng.step(1)
        before = _pinned()
        eng.field(s, 0, "rho", (16, 16, 16))
        read = _pinned()
        eng.release(s)
        held.append((read - before, _pinned() - read))
    # the first read pins a pair (unless another run of this process holds one);
    # no release gives it back while the engine lives
    assert held in ([(2, 0), (0, 0)], [(0, 0), (0, 0)]), held
    if held[0][0]:
        last = _pinned()
        del eng
        assert _pinned() <= last - 2
