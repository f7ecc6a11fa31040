"""Every launch of a nested step is timed under its kind: the launches of each kind
per coarse step."""
import pytest

pytestmark = pytest.mark.gpu


def _counts(dfm, n, levels, prec=0, steps=2, quadrant=False, criterion=False, **switches):
    r = dfm.Run(*n, nlevels=levels, dx0=0.02 * 2 ** (levels - 1), precision=prec, seed=17, noise_amp=1e-3,
                quadrant=quadrant)
    r.set_boundaries(int(quadrant))
    r.set_perturber(0.01, 0.04, 1e-3, 0.6, 0.1)
    r.set_subcycling(int(criterion))
    for name, on in switches.items():
        getattr(r, f"set_{name}_fusion")(on)
    dfm.timing_enable(r.handle, 4096)
    r.step(steps)
    return {k: c for k, (_, c) in dfm.timing_read(r.handle).items() if c}


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("levels", [2, 3, 4])
def test_frontier_sums(levels, prec):
    import paper_1812_03191_amd as dfm

    # one before each step of a level that has a finer one
    got = _counts(dfm, (32, 24, 28), levels, prec, steps=2)
    assert got["front"] == 2 * (2 ** (levels - 1) - 1), got


def test_steps_under_the_criterion():
    import paper_1812_03191_amd as dfm

    got = _counts(dfm, (32, 24, 28), 2, steps=3, criterion=True)
    assert got["dt"] == 3 and got["force"] == 3 and got["front"] == 3, got
