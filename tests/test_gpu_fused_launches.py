"""Which launches a step takes: the fused ones wherever they apply, and the separate
ones where a switch asks for them or the ghost shell is too narrow.  (The tests
that compare the two forms' values are about two forms only if this holds.)"""
import pytest

pytestmark = pytest.mark.gpu


def _counts(dfm, n, levels, prec, chunk=0, quadrant=False, walls=False, transport=True, finish=True, kick=True):
    r = dfm.Run(*n, nlevels=levels, dx0=0.02 * 2 ** (levels - 1), precision=prec, seed=17, noise_amp=1e-3,
                tile_chunk=chunk, quadrant=quadrant)
    r.set_boundaries(int(quadrant or walls))
    r.set_perturber(0.01, 0.04, 1e-3, 0.6, 0.1)
    r.set_transport_fusion(transport)
    r.set_finish_fusion(finish)
    r.set_kick_fusion(kick)
    dfm.timing_enable(r.handle, 4096)
    r.step(2)
    c = {k: v / 2 for k, (_, v) in dfm.timing_read(r.handle).items()}
    return tuple(c[k] for k in ("kick_compress", "kick", "compress", "pass_xy", "pass_x", "pass_y", "pass_z_finish",
                                "pass_z", "rebuild_kick"))


ROWS = [2, 30, 34, 62, 64, 66, 96, 126, 128, 130, 156, 190, 254, 256]


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("chunk", [0, 2])
@pytest.mark.parametrize("nx", ROWS)
def test_single_level(nx, chunk, prec):
    import paper_1812_03191_amd as dfm

    n = (nx, 22, 14)
    assert _counts(dfm, n, 1, prec, chunk) == (1, 0, 0, 1, 0, 0, 1, 0, 0)
    assert _counts(dfm, n, 1, prec, chunk, finish=False) == (1, 0, 0, 1, 0, 0, 0, 1, 1)
    assert _counts(dfm, n, 1, prec, chunk, transport=False) == (1, 0, 0, 0, 1, 1, 1, 0, 0)
    # the finish needs the fused kick's own set of face velocities
    assert _counts(dfm, n, 1, prec, chunk, kick=False) == (0, 1, 1, 1, 0, 0, 0, 1, 1)
    assert _counts(dfm, n, 1, prec, chunk, walls=True) == (1, 0, 0, 1, 0, 0, 0, 1, 1)


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("quadrant", [False, True])
@pytest.mark.parametrize("n,levels", [((16, 16, 16), 2), ((16, 16, 16), 3), ((32, 24, 28), 3), ((32, 28, 40), 3),
                                      ((32, 28, 28), 4), ((104, 32, 36), 3), ((200, 28, 28), 2)])
def test_nested(n, levels, quadrant, prec):
    import paper_1812_03191_amd as dfm

    steps = [2 ** l for l in range(levels)]
    # a middle level's first sub-step needs its cells to five beyond what the next
    # level's ghosts read of them, 8 - n/4 cells outside (two along a mirror plane's
    # normal, one at least), and the finish six entries of the shell of ten
    beyond = max(max(1, 8 - m // 4) for m in n)
    if quadrant:
        # the covered cells lie at the planes: the far side has half the cells between
        beyond = max(max(1, 8 - n[0] // 4), 2)
    wide = beyond + 5 <= 6
    fin = sum(s if wide or l == levels - 1 else s // 2 for l, s in enumerate(steps) if l)
    lev = sum(steps)
    # the second sub-steps of the finest level start kicked
    pairs = steps[-1] // 2
    kc = lev - pairs if prec else 1 + fin - pairs
    apart = lev - pairs - kc
    assert _counts(dfm, n, levels, prec, quadrant=quadrant) == \
        (kc, apart, apart + pairs, lev, 0, 0, fin, lev - fin, lev - fin)
    # each pass apart: no finish, in FP64 no fused kick on the finer levels
    kc = lev if prec else 1
    assert _counts(dfm, n, levels, prec, quadrant=quadrant, finish=False) == \
        (kc, lev - kc, lev - kc, lev, 0, 0, 0, lev, lev)
    assert _counts(dfm, n, levels, prec, quadrant=quadrant, transport=False) == \
        (kc, lev - kc, lev - kc, 0, lev, lev, 0, lev, lev)
