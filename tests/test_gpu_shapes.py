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
# a single row; three tiles; 28 and 36 tiles (one thread an element from 32 on)
@pytest.mark.parametrize("d,m", [(2048, 1), (2049, 127), (150_001, 128), (150_001, 129), (70_000, 256), (6000, 896),
                                 (6000, 897), (30_000, 897)])
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


# the same for several blocks in 2 to 4 splits each, on both sides of 32 tiles
@pytest.mark.parametrize("m,B,nb", [(100, 4100, 31), (100, 8192, 33), (300, 6148, 5), (300, 4096, 6)])
def test_split_blocks_gram_reduction(dev, m, B, nb):
    from paper_2107_03356_amd import StaticBlocks
    say("split blocks m =", m, "B =", B, "nb =", nb)
    G = _stream(B * nb, m, 1e-4, seed=m + B).window()
    sb = StaticBlocks(G.to(dev).contiguous(), B, 1e-4)
    diag = sb.inv_diag(fp64=True).cpu().numpy()
    assert sb.status() == 0
    assert np.max(np.abs(diag / ostatic.inv_diag(G.numpy(), 1e-4, B) - 1.0)) < 1e-11


# fast mode: m and B on both sides of the 32-row pieces, the 64-row padding, the
# 128- and 256-row tiles, 16-column chunks in odd number, a split block (B > 2048)
FAST_SHAPES = [(1, 4, 3), (31, 20, 5), (33, 36, 4), (64, 128, 3), (65, 132, 3), (128, 256, 2), (129, 260, 2),
               (255, 300, 2), (256, 256, 2), (257, 512, 2), (320, 1040, 2), (513, 2048, 1), (200, 2052, 1),
               (130, 4100, 2)]
# batches whose factor runs its large products in 256-tiles: whole tiles, one
# ragged tile in either direction, two levels of them (512 and 256 of m = 1024)
FAST_SHAPES += [(512, 16, 130), (520, 16, 70), (700, 32, 40), (1024, 64, 40), (1100, 32, 36), (1024, 16, 130)]


# split blocks on both sides of the line between eight threads and one an element
# (8 tiles of 256, 32 of 128), with padding rows, in 2 to 4 splits
FAST_SHAPES += [(200, 4100, 7), (200, 4100, 8), (330, 6148, 3), (100, 4096, 31), (100, 4096, 32)]


@pytest.mark.parametrize("m,B,nb", FAST_SHAPES)
def test_fast_gram_and_w(dev, m, B, nb):
    """The inverse diagonal (Gram, factor, W) and the IHVP of a second block.

    S_j = 1 - lam * diag_j is a sum of m squares of W, each with the rounding of
    fp32 sums over k <= max(m, 2048) terms: (sqrt(k) + 2) 2^-24 = 2.8e-6
    relative at most for well-conditioned blocks; the sums run over groups of 16
    and the rounding of a group's terms stays below the accumulator's, so that
    1e-6 (measured: 1e-8 to 2e-7) holds for all of them.
    """
    from paper_2107_03356_amd import StaticBlocks
    say("fast shapes", m, B, nb)
    base = get_workload("static_d4.19m_b2048_m1024")
    wl = base.scaled(d=B * nb, m=m, block=B, lam=1e-4, scale_d=base.d)
    gs = GradientStream(wl, seed=m + B)
    G = gs.rows(0, m)
    Gd = G.to(dev).contiguous()
    sb = StaticBlocks(Gd, B, wl.lam, fp32=True)
    S = 1.0 - wl.lam * sb.inv_diag(fp64=True).cpu().numpy()
    X = gs.queries(0, 1)
    Y = sb.ihvp(X.to(dev)).cpu().numpy()[0]
    assert sb.status() == 0
    assert np.array_equal(Gd.cpu().numpy(), G.numpy())
    Sref = 1.0 - wl.lam * ostatic.inv_diag(G.numpy(), wl.lam, B)
    # 1 - lam diag itself carries fp64 rounding of 1
    assert np.max(np.abs(S - Sref) / (np.abs(Sref) + 1e-9)) < 4e-6
    assert rel_l2(S, Sref) < 1e-6
    assert rel_l2(Y, ostatic.ihvp(G.numpy(), wl.lam, B, X.numpy())[0]) < 1e-6


@pytest.mark.parametrize("m,B,nb", [(1024, 64, 140), (1024, 2048, 6), (700, 4096, 2), (366, 500, 8)])
def test_fast_diagonal_is_unbiased(dev, m, B, nb):
    """The mean signed relative error of S = 1 - lam * diag over all coordinates.

    A, L^-1 and W are each rounded to fp32 once, to either side: 3 x 2^-25 = 9e-8
    even if every one of them fell to the same side, and the panels of a
    128-column node, still updated in fp32 16 columns at a time, lose at most an
    eighth of the squares sum_k L_ik^2 (2.2e-7 of S at m = 1024, B = 64, less
    elsewhere). Sums that lose the small terms added to a large one are far
    outside: -1.8e-6, -1.9e-7, -1.1e-7 and -1.0e-7 with C in the accumulators of
    the factor's updates.
    """
    from paper_2107_03356_amd import StaticBlocks
    say("fast bias", m, B, nb)
    base = get_workload("static_d4.19m_b2048_m1024")
    wl = base.scaled(d=B * nb, m=m, block=B, lam=1e-4, scale_d=base.d)
    G = GradientStream(wl, seed=m + B).rows(0, m)
    sb = StaticBlocks(G.to(dev).contiguous(), B, wl.lam, fp32=True)
    S = 1.0 - wl.lam * sb.inv_diag(fp64=True).cpu().numpy()
    assert sb.status() == 0
    Sref = 1.0 - wl.lam * ostatic.inv_diag(G.numpy(), wl.lam, B)
    mean = float(np.mean((S - Sref) / (Sref + 1e-9)))
    say("mean signed relative error of S", f"{mean:+.1e}")
    assert abs(mean) < (3.1e-7 if B == 64 else 9e-8)


# one row: S_j = g_j^2 / (|g|^2 + lam), so a Gram entry's own error; the 256-tile
# kernel at |g_i|^2 = m lam
@pytest.mark.parametrize("m,gain", [(1, 900.0), (200, 1.0)])
def test_fast_gram_sums_keep_low_bits(dev, m, gain):
    """The mean signed relative error of S, from sums of 2048 squares.

    The sum is rounded after every 16 columns to either side, A, L^-1 and W once:
    the mean over 64 blocks (m = 1: 64 Gram entries) stays below one rounding,
    2^-24 = 6e-8. Accumulating in the bf16 MFMA, which cuts what lies below a
    larger accumulator's last bits, leaves the sums low by several times that.
    """
    from paper_2107_03356_amd import StaticBlocks
    say("fast Gram sums", m)
    B, nb, lam = 2048, 64, 1e-3
    g = torch.Generator().manual_seed(m)
    G = torch.randn((m, B * nb), generator=g) * float(np.sqrt(gain * m * lam / B))
    sb = StaticBlocks(G.to(dev).contiguous(), B, lam, fp32=True)
    S = 1.0 - lam * sb.inv_diag(fp64=True).cpu().numpy()
    assert sb.status() == 0
    Sref = 1.0 - lam * ostatic.inv_diag(G.numpy(), lam, B)
    mean = float(np.mean((S - Sref) / (Sref + 1e-9)))
    say("mean signed relative error of S", f"{mean:+.1e}")
    assert abs(mean) < 6e-8


@pytest.mark.parametrize("bad", [float("nan"), float("inf"), -float("inf"), 3.4e38])
@pytest.mark.parametrize("m,B", [(20, 36), (300, 256)])
def test_fast_bad_block_is_reported_and_alone(dev, m, B, bad):
    """A value that is not finite, or whose square is not (3.4e38 also rounds to
    infinity as bf16), is reported; the other blocks' results are what they are
    without it. Columns of zeros and of values whose low parts are subnormal as
    bf16 next to it change nothing: their S is 0 to fp64."""
    from paper_2107_03356_amd import MFAC_ENONFINITE, StaticBlocks
    say("fast bad block", m, B, bad)
    nb, lam = 5, 1e-3
    g = torch.Generator().manual_seed(m)
    G = torch.randn((m, B * nb), generator=g) * 0.01
    G[:, 3 * B] = 0.0
    G[:, 3 * B + 1] = 1e-38
    G[:, 3 * B + 2] = -3e-41
    X = torch.randn((1, B * nb), generator=g)
    good = StaticBlocks(G.to(dev).contiguous(), B, lam, fp32=True)
    dg, Yg = good.inv_diag(fp64=True).cpu().numpy(), good.ihvp(X.to(dev)).cpu().numpy()[0]
    assert good.status() == 0
    dref = ostatic.inv_diag(G.numpy(), lam, B)
    assert np.max(np.abs(dg / dref - 1.0)) < 1e-6
    np.testing.assert_allclose(dg[3 * B:3 * B + 3], 1.0 / lam, rtol=1e-15)
    assert rel_l2(Yg, ostatic.ihvp(G.numpy(), lam, B, X.numpy())[0]) < 1e-6
    G[m // 2, 2 * B + 5] = bad
    sb = StaticBlocks(G.to(dev).contiguous(), B, lam, fp32=True)
    d, Y = sb.inv_diag(fp64=True).cpu().numpy(), sb.ihvp(X.to(dev)).cpu().numpy()[0]
    assert sb.status() == MFAC_ENONFINITE
    others = np.r_[0:2 * B, 3 * B:5 * B]
    np.testing.assert_array_equal(d[others], dg[others])
    np.testing.assert_array_equal(Y[others], Yg[others])


# m below and above the tiles, up to the fast mode's largest; few blocks and many
@pytest.mark.parametrize("m,B,nb", [(3, 8, 5), (256, 64, 600), (300, 2048, 2), (511, 1024, 3), (1000, 500, 4),
                                    (1025, 128, 2), (2049, 256, 2), (4096, 64, 2)])
def test_fast_obs_update_without_and_with_w(dev, m, B, nb):
    """The OBS correction before and after another query. Against the oracle both
    carry the fp32 factor's rounding
    (bound 4e-6: S's of test_fast_gram_and_w, and theta / diag in fp32)."""
    from paper_2107_03356_amd import StaticBlocks
    say("fast obs_update", m, B, nb)
    base = get_workload("static_d4.19m_b2048_m1024")
    wl = base.scaled(d=B * nb, m=m, block=B, lam=1e-4, scale_d=base.d)
    gs = GradientStream(wl, seed=m + B)
    G, theta = gs.rows(0, m), gs.theta()
    Gd = G.to(dev).contiguous()
    sb = StaticBlocks(Gd, B, wl.lam, fp32=True)
    mask = (torch.arange(wl.d) % 3 != 0).to(torch.uint8)
    d1 = sb.obs_update(theta.to(dev), mask.to(dev)).cpu().numpy()
    sb.ihvp(gs.queries(0, 1).to(dev))
    d2 = sb.obs_update(theta.to(dev), mask.to(dev)).cpu().numpy()
    assert sb.status() == 0
    assert np.array_equal(Gd.cpu().numpy(), G.numpy())
    ref = ostatic.obs_update(G.numpy(), wl.lam, B, theta.numpy(), mask.numpy())
    assert rel_l2(d1, ref) < 4e-6
    assert rel_l2(d2, ref) < 4e-6


@pytest.mark.parametrize("m,B,nb", [(3, 8, 5), (130, 300, 6), (256, 64, 600)])
def test_fast_queries_do_not_read_g(dev, m, B, nb):
    """G may be reused once the precompute (and any keep-mask) is done: the
    queries answer from the W in the workspace, whatever was called before, and
    the same call gives the same bits before and after the others."""
    from paper_2107_03356_amd import StaticBlocks
    say("fast queries without G", m, B, nb)
    base = get_workload("static_d4.19m_b2048_m1024")
    wl = base.scaled(d=B * nb, m=m, block=B, lam=1e-4, scale_d=base.d)
    gs = GradientStream(wl, seed=m + B)
    G, theta, X = gs.rows(0, m), gs.theta(), gs.queries(0, 1)
    Gd = G.to(dev).contiguous()
    sb = StaticBlocks(Gd, B, wl.lam, fp32=True)
    mask = (torch.arange(wl.d) % 3 != 0).to(torch.uint8)
    d1 = sb.obs_update(theta.to(dev), mask.to(dev)).cpu().numpy()
    Gd.fill_(7.0)
    d2 = sb.obs_update(theta.to(dev), mask.to(dev)).cpu().numpy()
    Y = sb.ihvp(X.to(dev)).cpu().numpy()[0]
    d3 = sb.obs_update(theta.to(dev), mask.to(dev)).cpu().numpy()
    assert sb.status() == 0
    np.testing.assert_array_equal(d1, d2)
    np.testing.assert_array_equal(d1, d3)
    assert rel_l2(Y, ostatic.ihvp(G.numpy(), wl.lam, B, X.numpy())[0]) < 1e-6
    assert rel_l2(d1, ostatic.obs_update(G.numpy(), wl.lam, B, theta.numpy(), mask.numpy())) < 4e-6


# units of 2048, 1024, 512 and 256 columns in the one-vector passes: fewer units
# than work-groups, just over a multiple of them, a ragged last unit; m below and
# at the rows in flight, and rows that no round of the pass divides; one to many
# row groups in pass 1
@pytest.mark.parametrize("d,m", [(1, 1), (255, 3), (2049, 33), (66_001, 31), (131_073, 65), (269_722, 40),
                                 (525_000, 17), (530_000, 5), (1_050_000, 9), (200_000, 33), (200_003, 65),
                                 (733_330, 40), (600_001, 100)])
def test_single_vector_units(dev, d, m):
    from paper_2107_03356_amd import Window
    say("single-vector units d =", d, "m =", m)
    gs = _stream(d, m, 1e-3, seed=d)
    G0 = gs.window()
    win = Window(d, m, 1e-3, G0=G0.to(dev), device=dev)
    orc = WindowOracle(d, m, 1e-3, G0=G0.numpy())
    x = gs.queries(0, 1)
    assert rel_l2(win.ihvp(x.to(dev)).cpu().numpy()[0], orc.ihvp(x.numpy())[0]) < F32_TOL
    for t in range(2):
        g = gs.step_row(t)
        y = win.replace(g.to(dev)).cpu().numpy()
        assert rel_l2(y, orc.slide(g.numpy())) < F32_TOL
    # a known sequence, in both directions of the fused pass
    Gn = torch.stack([gs.step_row(2 + t) for t in range(3)])
    Yn = win.replace_seq(Gn.to(dev)).cpu().numpy()
    for t in range(3):
        assert rel_l2(Yn[t], orc.slide(Gn[t].numpy())) < F32_TOL
    assert win.status() == 0


# keys over every digit of the selection: one value for all, two values, 36
# decades, neighbouring doubles; fewer keys than a wave up to several rounds of
# the grid; ranks at both ends and inside ties
@pytest.mark.parametrize("fast", [False, True])
@pytest.mark.parametrize("d,kind", [(4, "wide"), (1020, "ties"), (4100, "zeros"), (70_000, "wide"),
                                    (70_000, "equal"), (300_004, "near"), (4_300_000, "ties")])
def test_keep_mask_selection(dev, d, kind, fast):
    """The mask against the oracle's ranking of the scores the call returns: exact."""
    from oracle import mask as omask
    from paper_2107_03356_amd import StaticBlocks
    say("keep-mask selection", d, kind, fast)
    g = torch.Generator().manual_seed(d)
    u = torch.rand(d, generator=g)
    theta = {"wide": 10.0 ** (36 * u - 18), "equal": torch.full((d,), 0.05), "zeros": torch.where(u < 0.6, 0.0, u),
             "ties": torch.floor(u * 7), "near": 1.0 + u * 1e-3}[kind].float()
    # one equal gradient row: every diagonal entry is the same
    sb = StaticBlocks(torch.full((1, d), 0.01, device=dev), 4, 1e-2, fp32=fast)
    for keep in sorted({1, d // 3, d // 2, d - 1} - {0}):
        mask, scores = sb.obs_mask(theta.to(dev), keep)
        assert sb.status() == 0
        np.testing.assert_array_equal(mask.cpu().numpy(), omask.keep_mask(scores.cpu().numpy(), keep))


# the one-launch step of small windows: rows in 8 column ranges, rows that 16
# waves do not divide, the largest windows it takes (32 rows times slabs) and the
# first it does not, vectors off 16-byte alignment
@pytest.mark.parametrize("d,m,off", [(32_768, 2, 0), (40_000, 1, 0), (5, 32, 1), (5, 64, 1), (2049, 15, 0), (2048, 32, 3), (4095, 16, 1),
                                     (4096, 17, 0), (2048, 33, 0), (2048, 31, 0), (10_000, 6, 2), (10_241, 6, 0)])
def test_small_window_step(dev, d, m, off):
    from paper_2107_03356_amd import Window
    say("small window d =", d, "m =", m, "offset", off)
    gs = _stream(d, m, 1e-3, seed=d + m)
    win, orc = Window(d, m, 1e-3, max_queries=1, device=dev), WindowOracle(d, m, 1e-3)
    win.set_refactor_period(7)
    gbuf, ybuf = torch.empty(d + 4, device=dev), torch.full((d + 4,), 7.0, device=dev)
    for t in range(2 * m + 9):
        g = gs.row(t)
        gbuf[off:off + d] = g.to(dev)
        if t % 5 == 4:   # the separate kernels between two one-launch steps
            x = gs.queries(t, 1)
            y, Y = win.replace(gbuf[off:off + d].clone(), X=x.to(dev))
            yo = orc.slide(g.numpy())
            assert rel_l2(Y.cpu().numpy()[0], orc.ihvp(x.numpy())[0]) < F32_TOL
        elif t % 5 == 3:   # the slot given
            head, steps = win.info()
            y = win.replace(gbuf[off:off + d], slot=head, y_out=ybuf[off:off + d])
            assert win.info() == (head, steps + 1)
            win.set_head((head + 1) % m, steps + 1)
            yo = orc.slide(g.numpy())
        else:
            y = win.replace(gbuf[off:off + d], y_out=ybuf[off:off + d])
            yo = orc.slide(g.numpy())
        assert rel_l2(y.cpu().numpy(), yo) < F32_TOL, t
        assert win.status() == 0
        assert float(ybuf[off + d]) == 7.0 and (off == 0 or float(ybuf[off - 1]) == 7.0)
    np.testing.assert_array_equal(win.get_rows(0, 1).cpu().numpy()[0], orc.G[0].astype(np.float32))


@pytest.mark.parametrize("bad", [float("nan"), float("inf"), -float("inf"), 1e30])
@pytest.mark.parametrize("d,m", [(4096, 16), (300, 3)])
def test_small_window_step_reports_bad_gradients(dev, d, m, bad):
    """A gradient that is not finite is reported by the one-launch step; a window
    whose bad row is overwritten and rebuilt works on. 1e30 is finite (its square
    is summed in fp64) and reported by neither path."""
    from paper_2107_03356_amd import MFAC_ENONFINITE, Window
    say("small window, bad gradient", d, m, bad)
    gs = _stream(d, m, 1e-3, seed=d)
    win, orc = Window(d, m, 1e-3, device=dev), WindowOracle(d, m, 1e-3)
    for t in range(m):
        g = gs.row(t)
        assert rel_l2(win.replace(g.to(dev)).cpu().numpy(), orc.slide(g.numpy())) < F32_TOL
    g = gs.row(m).to(dev)
    g[d // 3] = bad
    win.replace(g)
    assert win.status() == (0 if bad == 1e30 else MFAC_ENONFINITE)
    win.set_rows(0, gs.row(m + 1)[None].to(dev))   # the bad row was slot 0
    win.rebuild()
    assert win.status() == 0
    rows = np.stack([gs.row(m + 1).numpy()] + [gs.row(t).numpy() for t in range(1, m)])
    orc = WindowOracle(d, m, 1e-3, G0=rows)
    x = gs.queries(0, 1)
    assert rel_l2(win.ihvp(x.to(dev)).cpu().numpy()[0], orc.ihvp(x.numpy())[0]) < F32_TOL
