"""Kernels at the edges of their tiles and splits, against the fp64 oracle.

Bounds: sums run in fp64, so an fp32 output differs from the oracle by its own
rounding (2^-24 relative, 6e-8) plus fp64 terms below it; 2e-7 leaves a factor
of three.
"""

import numpy as np
import pytest
import torch

from gpu_common import rel_l2, require_gpu, say
from oracle import static as ostatic
from oracle.dynamic import WindowOracle
from synth import GradientStream, get_workload

pytestmark = pytest.mark.gpu

F32_TOL = 2e-7


@pytest.fixture(scope="module")
def dev():
    return require_gpu()


def _stream(d, m, lam, seed, **kw):
    wl = get_workload("dyn_d1m_m256").scaled(d=d, m=m, lam=lam, scale_d=d, **kw)
    return GradientStream(wl, seed=seed)


# one tile with one, a few and many splits of the slab range; a second tile of
# a single row; three tiles
@pytest.mark.parametrize("d,m", [(2048, 1), (2049, 127), (150_001, 128), (150_001, 129), (70_000, 256)])
def test_window_gram_reduction(dev, d, m):
    from paper_2107_03356_amd import Window
    say("window Gram d =", d, "m =", m)
    gs = _stream(d, m, 1e-4, seed=m)
    G0 = gs.window()
    win = Window(d, m, 1e-4, G0=G0.to(dev), device=dev)
    x = gs.queries(0, 1)
    y = win.ihvp(x.to(dev)).cpu().numpy()[0]
    assert win.status() == 0
    yo = WindowOracle(d, m, 1e-4, G0=G0.numpy()).ihvp(x.numpy())[0]
    assert rel_l2(y, yo) < F32_TOL


# one wide block: a single tile (m <= 128) split many times, three tiles; the
# fp64 sums bound the diagonal at 1e-11
@pytest.mark.parametrize("d,m", [(40_000, 64), (65_540, 128), (30_000, 200)])
def test_wide_block_gram_reduction(dev, d, m):
    from paper_2107_03356_amd import StaticBlocks
    say("wide block d =", d, "m =", m)
    gs = _stream(d, m, 1e-4, seed=d)
    G = gs.window()
    sb = StaticBlocks(G.to(dev).contiguous(), d, 1e-4)
    diag = sb.inv_diag(fp64=True).cpu().numpy()
    assert sb.status() == 0
    assert np.max(np.abs(diag / ostatic.inv_diag(G.numpy(), 1e-4, d) - 1.0)) < 1e-11
