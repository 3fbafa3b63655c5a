"""GPU parity: every HIP kernel against the FP64 oracle on the same seeded inputs.

Tolerances (relative L2, ||gpu - oracle|| / ||oracle||): 1e-5 for the projector,
backprojector, ramp filter and normalisation; 1e-4 for full FBP and TV iterates.
"""
import math

import numpy as np
import pytest
import torch

import oracle
import synth
import paper_1306_1392_amd as ph

pytestmark = pytest.mark.gpu

TOL_OP = 1e-5
TOL_PIPE = 1e-4


def rel(a, b):
    a = a.detach().double().cpu().numpy() if torch.is_tensor(a) else np.asarray(a, dtype=np.float64)
    b = np.asarray(b, dtype=np.float64)
    return float(np.linalg.norm(a.ravel() - b.ravel()) / np.linalg.norm(b.ravel()))


def pair(nx, ny, nb, K, axis, shifts=None, s=1.0, scan=ph.SCAN_180, span=None, overlap=0.0, jitter=0.0, seed=0):
    span = span if span is not None else (math.pi if scan == ph.SCAN_180 else 2 * math.pi)
    ang = synth.uniform_angles(K, span)
    if jitter:
        ang = ang + np.random.default_rng(seed).uniform(-jitter, jitter, K) * span / K
    sh = None if shifts is None else np.random.default_rng(seed + 1).normal(0, shifts, K)
    return (ph.Geometry(nx, ny, nb, ang, axis, sh, scan, s, overlap),
            oracle.Geom(nx, ny, nb, ang, axis, sh, scan, s, overlap))


CASES = {
    "cfg1_256": dict(nx=256, ny=256, nb=256, K=180, axis=127.5),
    "odd_shift": dict(nx=77, ny=53, nb=101, K=61, axis=49.3, shifts=0.5, jitter=0.3),
    "wide_det": dict(nx=96, ny=96, nb=160, K=45, axis=81.25, shifts=0.5),
    "pix_0p7": dict(nx=70, ny=70, nb=64, K=50, axis=30.8, s=0.7),
    "pix_1p6": dict(nx=40, ny=50, nb=100, K=33, axis=50.0, s=1.6),
    "pix_0p4": dict(nx=60, ny=48, nb=50, K=37, axis=24.6, s=0.4, shifts=0.3),   # > 6 candidates per line
    # wider than the 224-position staged segment of six candidates: interior blocks take 16-byte reads
    "pix_0p7_wide": dict(nx=288, ny=264, nb=210, K=40, axis=104.5, s=0.7, shifts=0.3),
    "tiny": dict(nx=5, ny=3, nb=7, K=4, axis=3.0),
    "scan360": dict(nx=64, ny=64, nb=72, K=100, axis=36.4, scan=ph.SCAN_360),
}


@pytest.fixture(scope="module")
def gen():
    return np.random.default_rng(1234)


@pytest.mark.parametrize("case", list(CASES))
@pytest.mark.parametrize("tile,persistent", [(-1, False), (0, False), (3, True), (1, False), (2, True), (5, False),
                                             (5, True), (4, False)])
def test_backproject_parity(dev, gen, case, tile, persistent):
    g, og = pair(**CASES[case])
    plan = ph.Plan(g, n_slices=2)
    plan.set_tiles(tile, persistent)
    y = gen.standard_normal((2, g.n_angles, g.n_det)).astype(np.float32)
    out = ph.backproject(plan, torch.from_numpy(y).to(dev))
    ref = oracle.backproject(y, og)
    assert rel(out, ref) <= TOL_OP, (case, tile, persistent, rel(out, ref))


@pytest.mark.parametrize("case", ["odd_shift", "pix_0p7", "pix_1p6", "tiny", "scan360"])
@pytest.mark.parametrize("tile", [0, 1, 2, 3, 4])
def test_bp_two_slices_equal_one_slice_kernel(dev, gen, case, tile):
    """Two slices per backprojector workgroup (the automatic choice on uniform plans) against one
    slice per workgroup with the same tile: equal bit for bit, with an odd slice count (the last
    slice runs as a pair with itself) and an accumulating beta."""
    g, og = pair(**CASES[case])
    plan = ph.Plan(g, n_slices=3)
    y = torch.from_numpy(gen.standard_normal((3, g.n_angles, g.n_det)).astype(np.float32)).to(dev)
    base = torch.from_numpy(gen.standard_normal((3, g.n_y, g.n_x)).astype(np.float32)).to(dev)
    outs = []
    for per in (1, 2):
        plan.set_tiles(tile, False)
        plan.set_bp_slices(per)
        o = base.clone()
        ph.backproject(plan, y, out=o, alpha=0.75, beta=0.5)
        outs.append(o)
    torch.cuda.synchronize()
    assert torch.equal(outs[0], outs[1]), (case, tile, float((outs[0] - outs[1]).abs().max()))
    ref = 0.75 * oracle.backproject(y.cpu().numpy(), og) + 0.5 * base.double().cpu().numpy()
    assert rel(outs[1], ref) <= TOL_OP, (case, tile, rel(outs[1], ref))


@pytest.mark.parametrize("S,case", [(520, dict(nx=101, ny=97, nb=104, K=9, axis=51.3, shifts=0.4)),
                                    (59, dict(nx=430, ny=417, nb=431, K=34, axis=214.0)),
                                    (29, dict(nx=540, ny=556, nb=310, K=6, axis=280.0, scan=2)),
                                    (16, dict(nx=736, ny=736, nb=530, K=5, axis=264.2, s=0.7)),
                                    (24, dict(nx=613, ny=620, nb=600, K=3, axis=299.5)),
                                    (48, dict(nx=1024, ny=1017, nb=800, K=3, axis=399.5))])
def test_bp_matrix_core_kernel(dev, gen, S, case):
    """Plans of many slices sum on the matrix cores (32 slices per workgroup and a rest of 16): every slice equals the
    one-slice kernel within twice the operator tolerance, and sampled slices the oracle, with an accumulating beta;
    rows that grow by factors of 1e3 along the projections (the slices' scales follow), a zero slice; odd image sizes,
    half acquisition, rows that end inside and outside the image."""
    g, og = pair(**case)
    plan = ph.Plan(g, n_slices=S)
    y = gen.standard_normal((S, g.n_angles, g.n_det)).astype(np.float32)
    y *= (10.0 ** gen.uniform(-6, 6, S)).astype(np.float32)[:, None, None]
    y[5] *= (1e3 ** np.arange(g.n_angles) % 1e15 + 1).astype(np.float32)[:, None]
    y[2] = 0.0
    yt = torch.from_numpy(y).to(dev)
    base = torch.from_numpy(gen.standard_normal((S, g.n_y, g.n_x)).astype(np.float32)).to(dev)
    outs = []
    for per in (0, 1):
        plan.set_bp_slices(per)
        o = base.clone()
        ph.backproject(plan, yt, out=o, alpha=0.75, beta=0.5)
        outs.append((o, ph.backproject(plan, yt)))
    torch.cuda.synchronize()
    for s in range(S):
        if s != 2:
            assert rel(outs[0][1][s], outs[1][1][s].cpu().numpy()) <= 2 * TOL_OP, s
            assert rel(outs[0][0][s], outs[1][0][s].cpu().numpy()) <= 2 * TOL_OP, s
    assert not outs[0][1][2].any() and torch.equal(outs[0][0][2], 0.5 * base[2])
    assert not torch.equal(outs[0][1], outs[1][1])      # the matrix-core kernel ran
    for s in (0, 5, S - 1):
        assert rel(outs[0][1][s], oracle.backproject(y[s], og)) <= TOL_OP, s


def test_bp_matrix_core_kernel_non_finite(dev, gen):
    """Infinite and NaN bins reach the pixels that they reach in the one-slice kernel, and no others."""
    N, K, S = 101, 8, 520
    g, og = pair(nx=N, ny=N, nb=N, K=K, axis=50.0)
    y = torch.from_numpy(gen.standard_normal((S, K, N)).astype(np.float32)).to(dev)
    y[3, 5, 20], y[7, 2, 30], y[40, 0, 55], y[40, 1, 55] = float("inf"), float("nan"), float("inf"), -float("inf")
    y[519, 7, N - 1] = float("nan")
    plan = ph.Plan(g, n_slices=S)
    a = ph.backproject(plan, y)
    plan.set_bp_slices(1)
    b = ph.backproject(plan, y)
    assert torch.equal(torch.isnan(a), torch.isnan(b)) and torch.equal(torch.isinf(a), torch.isinf(b))
    fin = torch.isfinite(b)
    assert rel(torch.where(fin, a, 0.0), torch.where(fin, b, 0.0).cpu().numpy()) <= 2 * TOL_OP


def positions(g, axis):
    """t of every pixel at every projection, FP64 [K][n_y][n_x]."""
    x, y = np.arange(g.n_x) - 0.5 * (g.n_x - 1), np.arange(g.n_y) - 0.5 * (g.n_y - 1)
    a = np.asarray(g.angles)[:, None, None]
    return axis + np.cos(a) * x + np.sin(a) * y[:, None]


@pytest.mark.parametrize("value", [1e5, 1e6, 1e8, 1e12, 1e30, 3.4028235e38])
def test_bp_matrix_core_kernel_beside_a_large_bin(dev, gen, value):
    """One bin far above all others (a dead detector element), in the first, a middle and the last projections: a pixel that
    it does not touch keeps its own sum.  Bins of 0.2 to 1: every term of the general kernels, and so of the sum, is good
    to their coordinates (4e-6 bins), and a split term to 2^-21; 1e-5 of the pixel for both."""
    N, K, S = 125, 61, 1024
    g, og = pair(nx=N, ny=121, nb=N, K=K, axis=61.7)
    y = gen.uniform(0.2, 1.0, (S, K, N)).astype(np.float32)
    hot = [(1, 0, 60), (40, 2, 33), (300, 30, 50), (301, 31, 97), (1022, K - 1, 20), (1023, K - 3, 5)]
    for s, k, j in hot:
        y[s, k, j] = value
    plan = ph.Plan(g, n_slices=S)
    yt = torch.from_numpy(y).to(dev)
    a = ph.backproject(plan, yt).double().cpu().numpy()
    plan.set_bp_slices(1)
    b = ph.backproject(plan, yt).double().cpu().numpy()
    assert bool((a != b).any())                         # the matrix-core kernel ran
    t = positions(g, 61.7)
    for s, k, j in hot:
        off = np.abs(t[k] - j) > 1.0 + 1e-4
        ref = oracle.backproject(y[s], og)
        for out in (a[s], b[s]):
            assert np.abs(out - ref)[off].max() <= 1e-5 * ref[off].max(), (s, value)
            assert (np.abs(out - ref)[off] <= 1e-5 * ref[off]).all(), (s, value)
            assert np.abs(out - ref)[~off].max() <= 1e-5 * value, (s, value)


def test_bp_matrix_core_kernel_wide_range(dev, gen):
    """Rows that fall by a factor at one bin, pixels on either side of it; slices that begin with zeros or with far smaller
    values than end them, and the other way round; whole slices near either end of float32; every row or column of another
    magnitude.  Every pixel is good to 1e-5 of the sum of its own terms' magnitudes, and to what 1e-6 bin (half of it the
    coordinates' fixed point) changes in them."""
    N, K, S = 125, 48, 1024
    g, og = pair(nx=N, ny=121, nb=N, K=K, axis=62.2)
    y = gen.standard_normal((S, K, N)).astype(np.float32)
    falls = {3: 1e-4, 4: 1e-7, 5: 1e-9, 6: 1e-12, 7: 1e-20, 8: 1e-30}
    for s, f in falls.items():
        y[s, :, 45:] *= np.float32(f)
    y[20, :10] = 0.0
    y[21, :10] *= np.float32(1e-25)
    y[22, 10:] *= np.float32(1e-25)
    y[23, :5], y[23, 5:] = y[23, :5] * np.float32(1e-33), 0.0
    y[23, 40, 50] = 3e38
    y[24] *= np.float32(1e-33)
    y[25] *= np.float32(1e35)
    y[26] *= (10.0 ** gen.uniform(-30, 0, (K, 1))).astype(np.float32)
    y[27] *= (10.0 ** gen.uniform(-30, 0, (1, N))).astype(np.float32)
    plan = ph.Plan(g, n_slices=S)
    out = ph.backproject(plan, torch.from_numpy(y).to(dev)).double().cpu().numpy()
    t = positions(g, 62.2)

    def difference(rows, t):    # of the two bins of every pixel, summed
        q = np.pad(rows.astype(np.float64), ((0, 0), (1, 2)))
        j = np.clip(np.floor(t).astype(int) + 1, 0, N + 1).reshape(K, -1)
        d = np.abs(np.take_along_axis(q, j + 1, 1) - np.take_along_axis(q, j, 1)).reshape(t.shape)
        return np.where((t >= -1.0) & (t < N), d, 0.0)

    for s in [0, *falls, *range(20, 28)]:
        change = np.maximum(difference(y[s], t - 1e-6), difference(y[s], t + 1e-6)).sum(0)
        bound = 1e-5 * oracle.backproject(np.abs(y[s]), og) + 1e-6 * change
        assert (np.abs(out[s] - oracle.backproject(y[s], og)) <= bound).all(), s


def test_bp_matrix_core_kernel_all_large_and_nan_columns(dev, gen):
    """A column of the detector that is dead in every projection and slice, and one that is NaN in some: most pixels are
    summed apart from the matrix product, with an accumulating beta."""
    N, K, S = 125, 24, 1024
    g, og = pair(nx=N, ny=121, nb=N, K=K, axis=62.3)   # (no pixel lies on a bin at any angle)
    y = gen.uniform(0.2, 1.0, (S, K, N)).astype(np.float32)
    y[:, :, 30] = 1e15
    y[100:200, :, 80] = float("nan")
    yt = torch.from_numpy(y).to(dev)
    base = torch.from_numpy(gen.uniform(0.0, 1.0, (S, 121, N)).astype(np.float32)).to(dev)
    plan = ph.Plan(g, n_slices=S)
    a = ph.backproject(plan, yt, out=base.clone(), alpha=0.75, beta=0.5)
    plan.set_bp_slices(1)
    b = ph.backproject(plan, yt, out=base.clone(), alpha=0.75, beta=0.5)
    assert bool((torch.isnan(a) == torch.isnan(b)).all())
    clear = torch.from_numpy((np.abs(positions(g, 62.3) - 30) > 1.0001).all(0)).to(dev) & torch.isfinite(b)
    assert int(clear.sum()) > 1000 * S
    assert bool(((a - b).abs()[clear] <= 2e-5 * b.abs()[clear]).all())


@pytest.mark.parametrize("ny,nx,S", [(121, 125, 1024), (128, 97, 1024), (65, 1001, 256), (1001, 65, 256), (500, 511, 62)])
def test_cp_primal_step_on_matrix_cores_sizes(dev, gen, ny, nx, S):
    """The primal step's quads of pixels at the image's edges, last columns that are not a whole quad, more slices than a
    multiple of 32: against the one-slice kernel and the oracle."""
    g, og = pair(nx=nx, ny=ny, nb=90, K=5, axis=44.3, s=0.9)
    y = gen.standard_normal((S, 5, 90)).astype(np.float32)
    yt, res = torch.from_numpy(y).to(dev), []
    for per in (0, 1):
        plan = ph.Plan(g, n_slices=S)
        plan.set_bp_slices(per)
        res.append(ph.reconstruct_slices(plan, sino=yt, method=ph.TV_CP, lam=0.05, n_iter=3, op_norm=60.0))
    assert bool((res[0] != res[1]).any())               # the matrix-core kernel ran
    for s in (0, S // 2, S - 1):
        ref = oracle.cp_tv(y[s].astype(np.float64), og, 0.05, 3, 60.0)
        assert rel(res[0][s], ref) <= TOL_PIPE and rel(res[1][s], ref) <= TOL_PIPE, s
    assert rel(res[0], res[1].cpu().numpy()) <= TOL_PIPE


@pytest.mark.parametrize("S,case", [(1000, dict(nx=101, ny=97, nb=104, K=41, axis=51.3, shifts=0.4)),
                                    (60, dict(nx=430, ny=417, nb=431, K=62, axis=214.0)),
                                    (62, dict(nx=540, ny=556, nb=310, K=110, axis=280.0, scan=2)),
                                    (16, dict(nx=800, ny=800, nb=577, K=90, axis=287.2, s=0.7)),
                                    (48, dict(nx=1024, ny=1017, nb=800, K=49, axis=399.5))])
def test_bp_matrix_core_kernel_where_it_is_chosen(dev, gen, S, case):
    """Plans that run on the matrix cores (get_tiles says so): every slice against the one-slice kernel, and sampled ones
    against the oracle, both to the operator tolerances; half acquisition, small pixels, odd sizes, a rest of 16 slices."""
    g, og = pair(**case)
    plan = ph.Plan(g, n_slices=S)
    assert plan.get_tiles()[0] == -1
    y = gen.standard_normal((S, g.n_angles, g.n_det)).astype(np.float32)
    y *= (10.0 ** gen.uniform(-6, 6, S)).astype(np.float32)[:, None, None]
    yt = torch.from_numpy(y).to(dev)
    a = ph.backproject(plan, yt)
    plan.set_bp_slices(1)
    b = ph.backproject(plan, yt)
    d = ((a - b).double().flatten(1).norm(dim=1) / b.double().flatten(1).norm(dim=1)).max()
    assert 0.0 < float(d) <= 2 * TOL_OP
    for s in (0, S // 2, S - 1):
        assert rel(a[s], oracle.backproject(y[s], og)) <= TOL_OP, s


@pytest.mark.parametrize("S,n,K,matrix", [
    (60, 512, 120, True), (28, 600, 200, True), (32, 512, 90, True), (64, 2048, 1800, True), (1024, 256, 180, True),
    (24, 640, 300, False), (48, 430, 300, False), (64, 1100, 14, False), (520, 101, 61, False), (33, 2048, 100, False)])
def test_bp_matrix_core_rule(dev, S, n, K, matrix):
    """Which of the two kernels a plan's backprojections run on, well on either side of where they take the same time."""
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the rule counts compute units")
    g, _ = pair(nx=n, ny=n, nb=n, K=K, axis=0.5 * (n - 1))
    assert (ph.Plan(g, n_slices=S).get_tiles()[0] == -1) == matrix


@pytest.mark.parametrize("S,K", [(1024, 5), (1003, 33), (1007, 70)])
def test_bp_matrix_core_kernel_sums_apart(dev, gen, S, K):
    """Pixels summed apart from the matrix product: more and fewer slices than go side by side, marked ones among others,
    sums over less than, just more than and some chunks of projections; and in the primal step (one Chambolle-Pock
    iteration from zero is a multiple of the backprojection)."""
    g, og = pair(nx=125, ny=121, nb=100, K=K, axis=49.3)
    y = gen.uniform(0.2, 1.0, (S, K, 100)).astype(np.float32)
    hot = sorted(set(gen.integers(0, S, 60)) | {0, 1, 2, S - 1})
    y[hot, :, 40] = 1e13
    yt = torch.from_numpy(y).to(dev)
    far = (np.abs(positions(g, 49.3) - 40) > 1.0001).all(0)
    assert far.sum() > 200
    out = ph.backproject(ph.Plan(g, n_slices=S), yt).cpu().numpy()
    step = ph.reconstruct_slices(ph.Plan(g, n_slices=S), sino=yt, method=ph.TV_CP, lam=0.05, n_iter=1, op_norm=60.0)
    step = step.cpu().numpy()
    for s in hot + [3, S // 2]:
        ref = oracle.backproject(y[s], og)[far]
        assert np.abs(out[s][far] / ref - 1.0).max() <= 1e-5, s
        r = step[s][far] / ref
        assert np.abs(r / np.median(step[3][far] / oracle.backproject(y[3], og)[far]) - 1.0).max() <= 2e-5, s


def test_bp_tiles_read_and_set_keep_the_kernel(dev, gen):
    """set_tiles(*get_tiles()) changes nothing: a plan on the matrix cores reports -1, as created and after an autotune; one
    with a set tile, one that is too small and one of other slices per workgroup report a tile."""
    g, og = pair(nx=125, ny=121, nb=125, K=90, axis=62.3)
    S = 1024
    y = torch.from_numpy(gen.standard_normal((S, 90, 125)).astype(np.float32)).to(dev)
    plan = ph.Plan(g, n_slices=S)
    first = ph.backproject(plan, y)
    assert plan.get_tiles() == (-1, 0)
    for tune in (False, True):
        if tune:
            plan.autotune(y, torch.empty_like(first), reps=3)
            first = ph.backproject(plan, y)
        plan.set_tiles(*plan.get_tiles())
        assert bool((ph.backproject(plan, y) == first).all()), tune
    plan.set_tiles(-1, False)
    plan.set_bp_slices(2)
    assert plan.get_tiles()[0] >= 0
    plan.set_bp_slices(0)
    plan.set_tiles(3, False)
    assert plan.get_tiles() == (3, 0)
    assert ph.Plan(g, n_slices=4).get_tiles()[0] >= 0
    small = ph.Plan(g, n_slices=40)
    out = ph.backproject(small, y[:40])
    small.set_tiles(*small.get_tiles())
    assert bool((ph.backproject(small, y[:40]) == out).all())


def test_cp_primal_step_on_matrix_cores(dev, gen):
    """The fused Chambolle-Pock primal step of a plan of many slices (32 of 500 x 509) against the one-slice kernel."""
    g, og = pair(nx=500, ny=509, nb=510, K=7, axis=254.0, shifts=0.3)
    y = torch.from_numpy(gen.standard_normal((32, 7, 510)).astype(np.float32)).to(dev)
    res = []
    for per in (0, 1):
        plan = ph.Plan(g, n_slices=32)
        plan.set_bp_slices(per)
        res.append(ph.reconstruct_slices(plan, sino=y, method=ph.TV_CP, lam=0.05, n_iter=3, op_norm=80.0))
    assert rel(res[0], res[1].cpu().numpy()) <= TOL_PIPE and not torch.equal(res[0], res[1])
    for s in (0, 31):
        assert rel(res[0][s], oracle.cp_tv(y[s].double().cpu().numpy(), og, 0.05, 3, 80.0)) <= TOL_PIPE, s


@pytest.mark.parametrize("nb", [64, 65, 100, 128, 129, 250, 256, 257, 512, 513, 1000, 1024, 1025, 2047, 2048, 2049])
@pytest.mark.parametrize("K,scan", [(3, ph.SCAN_180), (37, ph.SCAN_180), (12, ph.SCAN_360_HALF)])
def test_fbp_filter_row_lengths(dev, gen, nb, K, scan):
    """The ramp filter over the row lengths where its transform changes (LDS passes below 65 and above 2048 bins, 16 / R
    row pairs per workgroup between): odd projection counts, a last workgroup that is not full, half acquisition."""
    half = scan == ph.SCAN_360_HALF
    g, og = pair(nx=8, ny=8, nb=nb, K=K, axis=0.9 * (nb - 1) if half else (nb - 1) / 2, scan=scan)
    S = 60 if nb <= 257 and K == 37 else 2       # enough pairs for the register filter of short rows
    y = gen.standard_normal((S, K, nb)).astype(np.float32)
    plan = ph.Plan(g, n_slices=S)
    out = ph.fbp_filter(plan, torch.from_numpy(y).to(dev))
    assert rel(out, oracle.fbp_filter(y, og)) <= TOL_OP
    if not half:
        again = torch.from_numpy(y).to(dev)
        ph.fbp_filter(plan, again, out=again)           # in place
        assert torch.equal(again, out)


def test_fbp_filter_uneven_row_lengths(dev, gen):
    """One plan over rows of every transform length of the register filter, and with one row length outside them."""
    for nbs in ([100, 256, 257, 600, 1500, 2048], [30, 256, 600], [700, 2100]):
        pairs = [pair(nx=8, ny=8, nb=nb, K=5 + i, axis=(nb - 1) / 2) for i, nb in enumerate(nbs)]
        plan = ph.Plan([q[0] for q in pairs], slice_geom=np.arange(len(nbs)))
        ys = [gen.standard_normal((5 + i, nb)).astype(np.float32) for i, nb in enumerate(nbs)]
        out = ph.fbp_filter(plan, torch.from_numpy(np.concatenate([y.ravel() for y in ys])).to(dev)).cpu().numpy()
        at = 0
        for y, (_, og) in zip(ys, pairs):
            assert rel(out[at:at + y.size], oracle.fbp_filter(y, og)) <= TOL_OP, y.shape
            at += y.size


@pytest.mark.parametrize("nb", [100, 200, 400, 900, 1800])
def test_fbp_from_raw_row_lengths(dev, nb):
    """Normalisation fused into the register filter's load, every transform length, three flats."""
    R, K = 3, 13
    g, og = pair(nx=24, ny=24, nb=nb, K=K, axis=(nb - 1) / 2 + 0.5)
    gen = np.random.default_rng(nb)
    flats = gen.uniform(30000, 40000, (3, R, nb)).astype(np.float32)
    pos = np.array([0.0, 5.5, 12.0])
    dark = gen.normal(100, 5, (R, nb)).astype(np.float32)
    raw = gen.uniform(2000, 30000, (K, R, nb)).astype(np.uint16)
    plan = ph.Plan(g, n_slices=R)
    t = [torch.from_numpy(a).to(dev) for a in (raw, flats, dark)]
    out = ph.reconstruct_slices(plan, raw=t[0], flats=t[1], flat_pos=pos, dark=t[2], method=ph.FBP)
    assert rel(out, oracle.fbp_raw(raw, flats, pos, dark, og)) <= TOL_PIPE


FP_KINDS = {"auto": ph.FP_AUTO, "blocks": ph.FP_BLOCKS, "staged": ph.FP_STAGED, "lines": ph.FP_LINES}


@pytest.mark.parametrize("case", list(CASES))
@pytest.mark.parametrize("kind", list(FP_KINDS))
def test_forward_project_parity(dev, gen, case, kind):
    g, og = pair(**CASES[case])
    plan = ph.Plan(g, n_slices=2)
    plan.set_fp_kernel(FP_KINDS[kind])
    assert plan.get_fp_kernel() == FP_KINDS[kind]
    x = gen.standard_normal((2, g.n_y, g.n_x)).astype(np.float32)
    out = ph.forward_project(plan, torch.from_numpy(x).to(dev))
    ref = oracle.forward_project(x, og)
    assert rel(out, ref) <= TOL_OP, (case, kind, rel(out, ref))


@pytest.mark.parametrize("case", ["odd_shift", "pix_0p7", "pix_1p6", "pix_0p4"])
@pytest.mark.parametrize("kind", list(FP_KINDS))
def test_adjoint_identity_gpu(dev, gen, case, kind):
    g, _ = pair(**CASES[case])
    plan = ph.Plan(g)
    plan.set_fp_kernel(FP_KINDS[kind])
    x = torch.from_numpy(gen.standard_normal((1, g.n_y, g.n_x)).astype(np.float32)).to(dev)
    y = torch.from_numpy(gen.standard_normal((1, g.n_angles, g.n_det)).astype(np.float32)).to(dev)
    ax = ph.forward_project(plan, x).double()
    lhs = float((ax * y.double()).sum())
    rhs = g.pixel_size ** 2 * float((x.double() * ph.backproject(plan, y).double()).sum())
    # rounding in <Ax, y> is bounded by |Ax| |y| (Cauchy-Schwarz), not by |<Ax, y>|, which a random draw
    # can make arbitrarily small through cancellation
    scale = float(ax.norm() * y.double().norm())
    assert abs(lhs - rhs) <= 1e-5 * scale, (case, kind, lhs, rhs, scale)


@pytest.mark.parametrize("ny,nx,nb,K,s,S", [
    (1, 1, 1, 2, 1.0, 1), (15, 17, 23, 8, 1.0, 1), (16, 64, 63, 12, 1.0, 2), (64, 16, 62, 12, 0.95, 1), (65, 81, 100, 24, 1.0, 3),
    (80, 79, 44, 24, 0.94, 1), (129, 128, 90, 40, 0.7, 2), (200, 203, 260, 36, 1.0, 1), (260, 256, 130, 36, 0.5, 2),
    (130, 1, 140, 12, 1.0, 1), (1, 130, 140, 12, 1.0, 1), (300, 300, 90, 30, 0.3, 1), (70, 70, 18, 200, 0.25, 2),
    (256, 256, 256, 400, 1.0, 1), (128, 128, 128, 700, 0.4, 9), (96, 96, 400, 16, 1.0, 1), (128, 128, 128, 42, 1.0, 5),
    (128, 128, 128, 43, 1.0, 5)])
def test_fp_frames(dev, gen, ny, nx, nb, K, s, S):
    """Frames of 64 positions: chunk and block edges, images wider and narrower than the detector, rows that are not
    16-byte aligned, an axis far from the middle, angles of every sign, 2, 4 and 8 wavefronts.  A bin sums at most
    some 1000 float32 products: 1e-6 of the norm, and the line kernel's result to twice that."""
    g, og = pair(nx=nx, ny=ny, nb=nb, K=K, axis=0.31 * (nb - 1), shifts=1.0, s=s, scan=ph.SCAN_360, jitter=0.2)
    x = gen.standard_normal((S, ny, nx)).astype(np.float32)
    flat = torch.empty(x.size + 1, device=dev)
    ref = oracle.forward_project(x, og)
    plan = ph.Plan(g, n_slices=S)
    for off in (0, 1):                          # a base of 16 and of 4 bytes' alignment
        t = flat[off:off + x.size].view(S, ny, nx)
        t.copy_(torch.from_numpy(x))
        out = ph.forward_project(plan, t)
        assert rel(out, ref) <= 1e-6
    plan.set_fp_kernel(ph.FP_LINES)
    assert rel(out, ph.forward_project(plan, t).cpu().numpy()) <= 2e-6


@pytest.mark.parametrize("ny,nx,nb,K,s,S", [
    (64, 63, 70, 20, 1.0, 5), (63, 63, 70, 20, 1.0, 5), (128, 100, 140, 300, 1.0, 5), (128, 100, 140, 800, 1.0, 5),
    (300, 301, 310, 70, 1.0, 15), (300, 301, 310, 70, 1.0, 16), (99, 90, 70, 300, 0.6, 4), (100, 90, 70, 300, 0.6, 4),
    (260, 256, 150, 40, 0.56, 17), (260, 256, 150, 31, 0.56, 17), (60, 50, 20, 30, 0.41, 70), (60, 50, 20, 30, 0.3, 70)])
def test_fp_either_side_of_the_frames_rule(dev, gen, ny, nx, nb, K, s, S):
    """Plans of several slices that the frames take and their neighbours that they do not: the oracle's projections, and
    the line kernel's in every slice."""
    g, og = pair(nx=nx, ny=ny, nb=nb, K=K, axis=0.48 * (nb - 1), s=s)
    x = gen.standard_normal((S, ny, nx)).astype(np.float32)
    xt = torch.from_numpy(x).to(dev)
    plan = ph.Plan(g, n_slices=S)
    out = ph.forward_project(plan, xt)
    plan.set_fp_kernel(ph.FP_LINES)
    assert rel(out, ph.forward_project(plan, xt).cpu().numpy()) <= 2 * TOL_OP
    for i in (0, S - 1):
        assert rel(out[i], oracle.forward_project(x[i:i + 1], og)[0]) <= TOL_OP, i


@pytest.mark.parametrize("s", [1.0, 0.95, 0.7, 0.5, 0.45, 0.3])
@pytest.mark.parametrize("value", [float("inf"), float("-inf"), float("nan")])
def test_fp_frames_non_finite_reach(dev, gen, s, value):
    """In the frames an infinite or NaN pixel reaches the bins that it touches, as itself, and no others; these hold the
    projection of the rest."""
    n, nb, K = 180, int(200 * s), 37
    g, og = pair(nx=n, ny=n - 7, nb=nb, K=K, axis=0.49 * nb, s=s, jitter=0.3, shifts=0.3)
    x = gen.uniform(0.1, 1.0, (1, n - 7, n)).astype(np.float32)
    rest = x.copy()
    hit = np.zeros((K, nb), bool)
    for iy, ix in [(5, 9), (90, 100), (172, 30), (60, 179)]:
        x[0, iy, ix], rest[0, iy, ix] = value, 0.0
        t = 0.49 * nb + g.axis_shift + s * (np.cos(g.angles) * (ix - (n - 1) / 2) + np.sin(g.angles) * (iy - (n - 8) / 2))
        d = np.abs(t[:, None] - np.arange(nb))
        assert np.abs(d - 1.0).min() > 1e-5 and np.abs(d).min() > 1e-5
        hit |= d < 1.0
    out = ph.forward_project(ph.Plan(g), torch.from_numpy(x).to(dev))[0].cpu().numpy()
    assert bool((np.isfinite(out) == ~hit).all())
    assert np.isnan(out[hit]).all() if np.isnan(value) else (out[hit] == value).all()
    clean = oracle.forward_project(rest, og)[0]
    assert np.abs(out - clean)[~hit].max() <= 1e-5 * np.abs(clean).max()


def test_fp_frames_uneven_and_non_finite(dev, gen):
    """Slices of their own sizes in one launch; an infinite or NaN pixel reaches the bins that it adds to, and none
    further than two bins from it (a lane's three sums hold |t - bin| <= 2; so do the staged kernel's candidates)."""
    geos = [pair(nx=50, ny=70, nb=64, K=20, axis=30.2), pair(nx=130, ny=90, nb=101, K=33, axis=49.7, s=0.8),
            pair(nx=9, ny=9, nb=300, K=7, axis=11.0)]
    plan = ph.Plan([q[0] for q in geos], slice_geom=[2, 0, 1, 0])
    x = torch.zeros(plan.img_elems, device=dev)
    for i, gi in enumerate([2, 0, 1, 0]):
        o, g = plan.slice_info(i).img_offset, geos[gi][0]
        x[o:o + g.n_x * g.n_y] = torch.from_numpy(gen.standard_normal(g.n_x * g.n_y).astype(np.float32)).to(dev)
    out = ph.forward_project(plan, x).flatten().cpu().numpy()
    for i, gi in enumerate([2, 0, 1, 0]):
        info, (g, og) = plan.slice_info(i), geos[gi]
        im = x[info.img_offset:info.img_offset + g.n_x * g.n_y].cpu().numpy().reshape(1, g.n_y, g.n_x)
        got = out[info.sino_offset:info.sino_offset + g.n_angles * g.n_det].reshape(1, g.n_angles, g.n_det)
        assert rel(got, oracle.forward_project(im, og)) <= 1e-6
    g, og = pair(nx=100, ny=100, nb=100, K=40, axis=49.5)
    im = torch.zeros(1, 100, 100)
    im[0, 31, 64] = float("inf")
    im[0, 70, 20] = float("nan")
    out = ph.forward_project(ph.Plan(g), im.to(dev))[0].cpu()
    bad = ~torch.isfinite(out).numpy()
    t = np.stack([49.5 + np.cos(g.angles) * (ix - 49.5) + np.sin(g.angles) * (iy - 49.5) for iy, ix in ((31, 64), (70, 20))])
    dist = np.abs(t[:, :, None] - np.arange(100)).min(0)
    assert bad[dist < 0.999].all() and not bad[dist > 2.001].any()


@pytest.mark.parametrize("s", [0.36, 0.3, 0.2])
def test_lines_projector_small_pixels(dev, gen, s):
    """The line kernel takes every candidate of a line, also where there are more than eight (below 0.354 bins)."""
    g, og = pair(nx=90, ny=80, nb=30, K=12, axis=14.2, s=s)
    plan = ph.Plan(g)
    plan.set_fp_kernel(ph.FP_LINES)
    x = gen.standard_normal((1, 80, 90)).astype(np.float32)
    assert rel(ph.forward_project(plan, torch.from_numpy(x).to(dev)), oracle.forward_project(x, og)) <= TOL_OP


def test_fp_kernel_override_rejects_bad_kind(dev):
    g, _ = pair(**CASES["tiny"])
    plan = ph.Plan(g)
    with pytest.raises(ph.PyhstError):
        plan.set_fp_kernel(4)
    assert plan.get_fp_kernel() == ph.FP_AUTO


FILTER_CASES = {
    "cfg1": dict(nx=256, ny=256, nb=256, K=180, axis=127.5),
    "odd": dict(nx=40, ny=40, nb=37, K=31, axis=17.5, jitter=0.4),
    "scan360": dict(nx=64, ny=64, nb=72, K=100, axis=36.4, scan=ph.SCAN_360),
    "half_right": dict(nx=96, ny=96, nb=59, K=180, axis=48.0, scan=ph.SCAN_360_HALF),
    "half_left": dict(nx=96, ny=96, nb=59, K=180, axis=10.0, scan=ph.SCAN_360_HALF, overlap=6.0),
    "long_rows": dict(nx=16, ny=16, nb=2500, K=4, axis=1249.5),
    # FFT length 4096 (the register-FFT filter): full rows, shorter rows, extended half-acquisition rows
    # on either side, odd projection counts (the last row pair has one row)
    "rows_2048_oddK": dict(nx=16, ny=16, nb=2048, K=5, axis=1023.5),
    "rows_1500": dict(nx=16, ny=16, nb=1500, K=4, axis=749.5, jitter=0.1),
    "half_right_p4096": dict(nx=32, ny=32, nb=600, K=7, axis=590.0, scan=ph.SCAN_360_HALF),
    "half_left_p4096": dict(nx=32, ny=32, nb=600, K=6, axis=9.0, scan=ph.SCAN_360_HALF, overlap=5.0),
}


DEGENERATE = {
    "one_pixel": dict(nx=1, ny=1, nb=1, K=2, axis=0.0),        # one pixel, one bin, two projections
    "one_row": dict(nx=9, ny=1, nb=5, K=3, axis=2.0),
    "one_col": dict(nx=1, ny=7, nb=4, K=3, axis=1.5),
    "two_angles": dict(nx=16, ny=16, nb=16, K=2, axis=7.5),    # the fewest projections a plan accepts
}


@pytest.mark.parametrize("case", list(DEGENERATE))
def test_degenerate_geometries(dev, gen, case):
    """The smallest plans the boundary accepts: backprojection (every tile shape, direct and persistent),
    projection (every projector kernel), ramp filter and the whole FBP against the oracle."""
    g, og = pair(**DEGENERATE[case])
    plan = ph.Plan(g, n_slices=2)
    y = gen.standard_normal((2, g.n_angles, g.n_det)).astype(np.float32)
    x = gen.standard_normal((2, g.n_y, g.n_x)).astype(np.float32)
    yt, xt = torch.from_numpy(y).to(dev), torch.from_numpy(x).to(dev)
    ref_bp, ref_fp = oracle.backproject(y, og), oracle.forward_project(x, og)
    for tile, pers in [(-1, False), (0, False), (3, True), (4, False), (5, False), (5, True)]:
        plan.set_tiles(tile, pers)
        assert rel(ph.backproject(plan, yt), ref_bp) <= TOL_OP, (case, tile, pers)
    plan.set_tiles(-1, False)
    for kind in FP_KINDS.values():
        plan.set_fp_kernel(kind)
        assert rel(ph.forward_project(plan, xt), ref_fp) <= TOL_OP, (case, kind)
    plan.set_fp_kernel(ph.FP_AUTO)
    assert rel(ph.fbp_filter(plan, yt), oracle.fbp_filter(y, og)) <= TOL_OP, case
    assert rel(ph.reconstruct_slices(plan, sino=yt, method=ph.FBP), oracle.fbp(y, og)) <= TOL_PIPE, case


@pytest.mark.parametrize("case", list(FILTER_CASES))
def test_fbp_filter_parity(dev, gen, case):
    g, og = pair(**FILTER_CASES[case])
    plan = ph.Plan(g, n_slices=2)
    p = gen.random((2, g.n_angles, g.n_det)).astype(np.float32)
    out = ph.fbp_filter(plan, torch.from_numpy(p).to(dev))
    ref = oracle.fbp_filter(p, og)
    assert out.shape == ref.shape
    assert rel(out, ref) <= TOL_OP, (case, rel(out, ref))


def test_fbp_filter_in_place(dev, gen):
    g, og = pair(**FILTER_CASES["odd"])
    plan = ph.Plan(g)
    p = gen.random((1, g.n_angles, g.n_det)).astype(np.float32)
    t = torch.from_numpy(p).to(dev)
    ph.fbp_filter(plan, t, out=t)
    assert rel(t, oracle.fbp_filter(p, og)) <= TOL_OP


def raw_case(R=3, N=96, K=90, nb=None, axis_offset=3.5, seed=7, n_flats=2):
    nb = nb or N
    ang = synth.uniform_angles(K)
    axis = (nb - 1) / 2 + axis_offset
    p = torch.stack([synth.ellipse_sinogram(synth.random_ellipses(synth.rng_for(9, 0, r), 8), ang, nb, axis, N)
                     for r in range(R)])
    raw, flats, fpos, dark, kap = synth.raw_acquisition(p, seed=seed)
    if n_flats == 3:   # a third flat acquired mid-scan
        flats = torch.cat([flats[:1], 0.5 * (flats[:1] + flats[1:]) * 1.01, flats[1:]])
        fpos = np.array([0.0, K / 2 + 0.5, K - 1.0])
    return ang, axis, raw, flats, fpos, dark


@pytest.mark.parametrize("n_flats", [2, 3])
def test_normalize_parity(dev, n_flats):
    ang, axis, raw, flats, fpos, dark = raw_case(n_flats=n_flats)
    g = ph.Geometry(96, 96, 96, ang, axis)
    plan = ph.Plan(g, n_slices=3)
    out = ph.normalize(plan, raw.to(dev), flats.to(dev), fpos, dark.to(dev))
    ref = oracle.normalize(raw.numpy().astype(np.float64), flats.numpy(), fpos, dark.numpy())
    assert rel(out, ref) <= TOL_OP


@pytest.mark.parametrize("graph", [False, True])
def test_fbp_from_raw_parity(dev, graph):
    ang, axis, raw, flats, fpos, dark = raw_case()
    g = ph.Geometry(96, 96, 96, ang, axis)
    og = oracle.Geom(96, 96, 96, ang, axis)
    plan = ph.Plan(g, n_slices=3)
    args = dict(raw=raw.to(dev), flats=flats.to(dev), flat_pos=fpos, dark=dark.to(dev), method=ph.FBP)
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        out = ph.reconstruct_slices(plan, use_graph=graph, **args)
    side.synchronize()
    ref = oracle.fbp_raw(raw.numpy().astype(np.float64), flats.numpy(), fpos, dark.numpy(), og)
    assert rel(out, ref) <= TOL_PIPE
    if graph:   # replays of the captured graph give the eager result every time
        eager = ph.reconstruct_slices(plan, use_graph=False, **args).clone()
        torch.cuda.synchronize()
        for _ in range(3):
            with torch.cuda.stream(side):
                again = ph.reconstruct_slices(plan, use_graph=True, **args)
            side.synchronize()
            assert torch.equal(again, eager)
            eager.add_(0.0)     # eager work between replays


def test_fbp_from_raw_parity_p4096(dev):
    """2048-bin rows from raw (normalisation fused into the register-FFT filter, FFT length 4096), an odd
    number of projections, two slices."""
    ang, axis, raw, flats, fpos, dark = raw_case(R=2, N=32, K=7, nb=2048)
    g = ph.Geometry(32, 32, 2048, ang, axis)
    og = oracle.Geom(32, 32, 2048, ang, axis)
    plan = ph.Plan(g, n_slices=2)
    out = ph.reconstruct_slices(plan, raw=raw.to(dev), flats=flats.to(dev), flat_pos=fpos, dark=dark.to(dev),
                                method=ph.FBP)
    ref = oracle.fbp_raw(raw.numpy().astype(np.float64), flats.numpy(), fpos, dark.numpy(), og)
    assert rel(out, ref) <= TOL_PIPE


@pytest.mark.parametrize("n,S,K,tile", [(256, 8, 9, 5), (256, 9, 9, 3), (256, 12, 90, 5), (256, 13, 90, 3), (500, 3, 90, 5)])
def test_bp_tile_rule_for_few_pairs(dev, gen, n, S, K, tile):
    """Up to three 32 x 32 tiles of one slice per compute unit (256 of them; two with few projections) take the angle
    groups, more of them pairs of slices; either side of the line holds the projector's transpose."""
    g, og = pair(nx=n, ny=n, nb=n, K=K, axis=0.49 * n)
    plan = ph.Plan(g, n_slices=S)
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        assert plan.get_tiles()[0] == tile
    y = gen.standard_normal((S, K, n)).astype(np.float32)
    out = ph.backproject(plan, torch.from_numpy(y).to(dev))
    at = [0, S // 2, S - 1]
    assert rel(out[at], oracle.backproject(y[at], og)) <= TOL_OP


@pytest.mark.parametrize("n,w,S,K,tile", [(1000, 1000, 7, 6, 0), (1023, 798, 9, 6, 1), (1650, 1650, 3, 6, 1), (530, 530, 13, 12, 3),
                                          (735, 735, 7, 12, 1), (852, 792, 5, 12, 3), (256, 256, 8, 8, 3)])
def test_bp_tile_rule_for_odd_slices(dev, gen, n, w, S, K, tile):
    """Tiles of plans where the odd last slice makes up the number of workgroups, or with next to no projections; a sampled
    slice, the last among them, holds the projector's transpose."""
    g, og = pair(nx=n, ny=w, nb=n, K=K, axis=0.49 * n)
    plan = ph.Plan(g, n_slices=S)
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        assert plan.get_tiles()[0] == tile
    y = gen.standard_normal((S, K, n)).astype(np.float32)
    out = ph.backproject(plan, torch.from_numpy(y).to(dev))
    for s in (0, S - 1):
        assert rel(out[s], oracle.backproject(y[s], og)) <= TOL_OP, s


@pytest.mark.parametrize("n,S,K", [(256, 8, 90), (256, 9, 30), (256, 12, 90), (500, 3, 120)])
def test_bp_two_slices_asked_for_with_few_pairs(dev, gen, n, S, K):
    """Where the automatic choice may take angle groups, two slices per workgroup are still what is run when they are asked
    for: the tile of one slice per workgroup, and its image bit for bit."""
    g, og = pair(nx=n, ny=n, nb=n, K=K, axis=0.49 * n)
    plan = ph.Plan(g, n_slices=S)
    y = torch.from_numpy(gen.standard_normal((S, K, n)).astype(np.float32)).to(dev)
    outs = []
    for per in (1, 2):
        plan.set_bp_slices(per)
        outs.append((plan.get_tiles()[0], ph.backproject(plan, y)))
    assert outs[0][0] == outs[1][0]
    assert bool((outs[0][1] == outs[1][1]).all())


def test_fbp_batch_equals_single(dev, gen):
    g, _ = pair(**CASES["odd_shift"])
    plan4 = ph.Plan(g, n_slices=4)
    plan1 = ph.Plan(g, n_slices=1)
    y = torch.from_numpy(gen.random((4, g.n_angles, g.n_det)).astype(np.float32)).to(dev)
    batch = ph.reconstruct_slices(plan4, sino=y, method=ph.FBP)
    for i in range(4):
        single = ph.reconstruct_slices(plan1, sino=y[i:i + 1].contiguous(), method=ph.FBP)
        assert torch.equal(batch[i], single[0])


@pytest.mark.parametrize("persistent", [False, True])
def test_uniform_plan_shared_by_two_streams(dev, gen, persistent):
    """A uniform plan may serve two streams at once when each call has its own buffers: FBP and TV-CP
    interleaved on two streams (graph and direct launches) equal the same calls made one at a time, also
    with the persistent backprojector (its work counter belongs to the stream)."""
    g, _ = pair(**CASES["odd_shift"])
    plan = ph.Plan(g, n_slices=2)
    plan.set_tiles(-1, persistent)
    y = [torch.from_numpy(gen.standard_normal((2, g.n_angles, g.n_det)).astype(np.float32)).to(dev) for _ in range(2)]
    kw = [dict(method=ph.FBP), dict(method=ph.TV_CP, lam=0.02, n_iter=15, op_norm=200.0)]   # 200 > |K| here
    ref = [ph.reconstruct_slices(plan, sino=y[i], **kw[i]) for i in range(2)]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    for st in streams:
        st.wait_stream(torch.cuda.current_stream())
    outs = []
    for rep in range(4):
        for i, st in enumerate(streams):
            with torch.cuda.stream(st):
                outs.append((i, ph.reconstruct_slices(plan, sino=y[i], use_graph=(rep + i) % 2 == 0, stream=st,
                                                      **kw[i])))
    torch.cuda.synchronize()
    for i, o in outs:
        assert torch.equal(o, ref[i]), i


def test_graph_cache_bound(dev, gen):
    """More distinct graph calls than the plan caches (64): the surplus run as plain launches, same result."""
    g, _ = pair(**CASES["tiny"])
    plan = ph.Plan(g)
    y = torch.from_numpy(gen.standard_normal((1, g.n_angles, g.n_det)).astype(np.float32)).to(dev)
    ref = ph.reconstruct_slices(plan, sino=y, method=ph.FBP)
    outs = [torch.empty_like(ref) for _ in range(70)]
    side = torch.cuda.Stream()   # graphs are captured on a created stream (the null stream cannot be)
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        for _ in range(2):
            for o in outs:
                ph.reconstruct_slices(plan, sino=y, method=ph.FBP, out=o, use_graph=True, stream=side)
    torch.cuda.synchronize()
    assert all(torch.equal(o, ref) for o in outs)


def test_uniform_plan_on_a_later_geometry(dev, gen):
    """A plan whose slices all use geometry 1 of two behaves as a plan of that geometry alone: the packed
    shapes, FBP, the projector and TV-CP use its sizes, not those of geometry 0."""
    g0, _ = pair(**CASES["wide_det"])
    g1, og1 = pair(**CASES["odd_shift"])
    both = ph.Plan([g0, g1], slice_geom=[1, 1])
    only = ph.Plan(g1, n_slices=2)
    assert both.uniform and both.sino_shape() == only.sino_shape() and both.img_shape() == only.img_shape()
    y = torch.from_numpy(gen.random((2, g1.n_angles, g1.n_det)).astype(np.float32)).to(dev)
    for kw in (dict(method=ph.FBP), dict(method=ph.TV_CP, lam=0.02, n_iter=5, op_norm=200.0)):
        assert torch.equal(ph.reconstruct_slices(both, sino=y, **kw), ph.reconstruct_slices(only, sino=y, **kw))
    x = ph.reconstruct_slices(only, sino=y, method=ph.FBP)
    assert torch.equal(ph.forward_project(both, x), ph.forward_project(only, x))
    assert rel(ph.reconstruct_slices(both, sino=y, method=ph.FBP)[1], oracle.fbp(y[1:].cpu().numpy(), og1)[0]) <= TOL_PIPE


def test_uneven_plan_matches_oracle(dev, gen):
    """One plan, slices of different sizes, angle counts and scan types (packed buffers)."""
    specs = [dict(nx=64, ny=64, nb=64, K=90, axis=31.5),
             dict(nx=96, ny=96, nb=59, K=180, axis=48.0, scan=ph.SCAN_360_HALF, shifts=0.5),
             dict(nx=48, ny=40, nb=70, K=31, axis=33.2, jitter=0.3)]
    pairs_ = [pair(**s, seed=i) for i, s in enumerate(specs)]
    sg = [0, 1, 2, 1, 0]
    plan = ph.Plan([p[0] for p in pairs_], slice_geom=sg)
    sinos = [gen.random((pairs_[i][0].n_angles, pairs_[i][0].n_det)).astype(np.float32) for i in sg]
    packed = torch.from_numpy(np.concatenate([s.ravel() for s in sinos])).to(dev)
    for persistent in (False, True):
        plan.set_tiles(-1, persistent)
        out = ph.reconstruct_slices(plan, sino=packed, method=ph.FBP).cpu().numpy()
        for i, gi in enumerate(sg):
            info = plan.slice_info(i)
            og = pairs_[gi][1]
            got = out[info.img_offset:info.img_offset + og.n_x * og.n_y].reshape(og.n_y, og.n_x)
            ref = oracle.fbp(sinos[i][None], og)[0]
            assert rel(got, ref) <= TOL_PIPE, (i, persistent, rel(got, ref))


@pytest.mark.parametrize("lam,n_inner", [(0.05, 40), (0.3, 100)])
def test_tv_prox_parity(dev, gen, lam, n_inner):
    g0 = (gen.standard_normal((2, 45, 61)) * 0.2 + 1.0).astype(np.float32)
    out = ph.tv_prox(torch.from_numpy(g0).to(dev), lam, n_inner)
    ref = oracle.tv_prox(g0, lam, n_inner)
    assert rel(out, ref) <= TOL_PIPE


@pytest.mark.parametrize("S,ny,nx,n_inner", [
    (1, 1, 1, 5), (3, 1, 70, 6), (2, 40, 1, 11), (1, 15, 52, 1), (2, 16, 53, 5), (1, 17, 54, 10), (3, 31, 106, 4),
    (1, 33, 107, 7), (2, 49, 59, 8), (1, 64, 62, 2), (1, 65, 61, 3), (2, 130, 200, 12), (1100, 40, 60, 5),
    (4096, 70, 54, 6)])
def test_tv_prox_strips(dev, S, ny, nx, n_inner):
    """Strips of 64 columns and segments of 16, 32 and 64 rows, with 1 to 5 steps in flight.  Every step is a
    contraction whose float32 rounding is a few 2^-24 of the values: 12 steps stay under 1e-6 of the norm."""
    gen = torch.Generator().manual_seed(S + 7 * ny + 31 * nx + n_inner)
    g0 = torch.randn(min(S, 3), ny, nx, generator=gen)
    g0 = torch.cat([g0, g0[:1].expand(max(S - 4, 0), ny, nx), g0[-1:].expand(int(S > 3), ny, nx)]).contiguous()
    t = g0.to(dev)
    out = ph.tv_prox(t, 0.3, n_inner)
    at = sorted({0, S // 2, S - 1} | set(range(min(S, 3))))
    ref = oracle.tv_prox(g0[at].numpy(), 0.3, n_inner)
    assert rel(out[at], ref) <= 1e-6
    assert torch.equal(ph.tv_prox(t, 0.3, n_inner, out=t), t) and rel(t[at], ref) <= 1e-6   # in place: another last step


def test_tv_prox_overflow_and_nan(dev):
    """A difference whose square overflows leaves no dual value there; a NaN reaches what its pixel's stencil reaches."""
    g0 = torch.zeros(1, 40, 80)
    g0[0, 20, 30], g0[0, 5, 60] = 1e25, float("nan")
    out = ph.tv_prox(g0.to(dev), 0.5, 4).cpu()[0]
    assert out[20, 30] == 1e25
    far = torch.ones(40, 80, dtype=torch.bool)
    far[0:11, 54:67] = False
    assert torch.isnan(out[5, 60]) and not torch.isnan(out[far]).any()


def test_tv_prox_in_place_and_identity(dev, gen):
    g0 = gen.standard_normal((1, 20, 20)).astype(np.float32)
    t = torch.from_numpy(g0).to(dev)
    assert torch.equal(ph.tv_prox(t, 0.0, 10), t)
    ph.tv_prox(t, 0.1, 30, out=t)
    assert rel(t, oracle.tv_prox(g0, 0.1, 30)) <= TOL_PIPE


@pytest.fixture(scope="module")
def cp_problem():
    N, K = 128, 32
    d = synth.cfg_tv_sparse(N=N, K=K, index=3)
    g = ph.Geometry(N, N, N, d["angles"], d["axis"])
    og = oracle.Geom(N, N, N, d["angles"], d["axis"])
    Lk = oracle.opnorm(og, synth.rng_for(3, 9, 0).standard_normal((N, N)), 200)
    return d, g, og, Lk


@pytest.mark.parametrize("k", [1, 10, 100])
def test_cp_iterates_parity(dev, cp_problem, k):
    d, g, og, Lk = cp_problem
    plan = ph.Plan(g)
    y = d["y"][None].contiguous().to(dev)
    x = ph.reconstruct_slices(plan, sino=y, method=ph.TV_CP, lam=0.01, n_iter=k, op_norm=Lk)
    ref = oracle.cp_tv(d["y"].numpy(), og, 0.01, k, Lk)
    assert rel(x[0], ref) <= TOL_PIPE, (k, rel(x[0], ref))


@pytest.mark.parametrize("kind", ["blocks", "staged", "lines"])
def test_cp_iterates_every_fp_kernel(dev, cp_problem, kind):
    d, g, og, Lk = cp_problem
    plan = ph.Plan(g)
    plan.set_fp_kernel(FP_KINDS[kind])
    y = d["y"][None].contiguous().to(dev)
    x = ph.reconstruct_slices(plan, sino=y, method=ph.TV_CP, lam=0.01, n_iter=10, op_norm=Lk)
    ref = oracle.cp_tv(d["y"].numpy(), og, 0.01, 10, Lk)
    assert rel(x[0], ref) <= TOL_PIPE, (kind, rel(x[0], ref))


def test_cp_energy_and_graph(dev, cp_problem):
    d, g, og, Lk = cp_problem
    plan = ph.Plan(g)
    y = d["y"][None].contiguous().to(dev)
    x, E = ph.reconstruct_slices(plan, sino=y, method=ph.TV_CP, lam=0.01, n_iter=20, op_norm=Lk, energy=True)
    xr, Er = oracle.cp_tv(d["y"].numpy(), og, 0.01, 20, Lk, energy=True)
    np.testing.assert_allclose(E, Er, rtol=1e-4)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    for _ in range(2):
        with torch.cuda.stream(side):
            xg = ph.reconstruct_slices(plan, sino=y, method=ph.TV_CP, lam=0.01, n_iter=20, op_norm=Lk,
                                       use_graph=True)
        side.synchronize()
        assert torch.equal(xg, x)


def test_cp_opnorm_estimate(dev, cp_problem):
    """op_norm <= 0: the GPU power iteration gives 1.02 |K| (a 2 % safety margin)."""
    d, g, og, Lk = cp_problem
    plan = ph.Plan(g)
    y = d["y"][None].contiguous().to(dev)
    x = ph.reconstruct_slices(plan, sino=y, method=ph.TV_CP, lam=0.01, n_iter=50, op_norm=0.0)
    ref = oracle.cp_tv(d["y"].numpy(), og, 0.01, 50, 1.02 * Lk)
    assert rel(x[0], ref) < 2e-3


def test_cp_identity_limit_matches_prox(dev, gen):
    """TV-CP on a full-angle noise-free disc recovers it (eq. (3) with small beta)."""
    N = 64
    g = ph.Geometry(N, N, N, synth.uniform_angles(96), (N - 1) / 2)
    og = oracle.Geom(N, N, N, g.angles, g.axis_pos)
    y = synth.ellipse_sinogram(synth.disc_params(0.5, 1.0), g.angles, N, g.axis_pos, N).float()
    Lk = oracle.opnorm(og, gen.standard_normal((N, N)), 100)
    x = ph.reconstruct_slices(ph.Plan(g), sino=y[None].contiguous().to(dev), method=ph.TV_CP, lam=0.02,
                              n_iter=300, op_norm=Lk)[0].cpu().numpy()
    yy, xx = np.mgrid[0:N, 0:N]
    inside = (xx - (N - 1) / 2) ** 2 + (yy - (N - 1) / 2) ** 2 < (0.4 * N / 2) ** 2
    assert abs(x[inside].mean() - 1.0) < 0.03


# --------------------------------------------------------------------------- ISTA / FISTA (section 3.1)
@pytest.fixture(scope="module")
def fista_problem(cp_problem):
    d, g, og, _ = cp_problem
    La = oracle.opnorm(og, synth.rng_for(3, 9, 2).standard_normal((og.n_y, og.n_x)), 200, with_grad=False) ** 2
    return d, g, og, La


@pytest.mark.parametrize("method", ["ista", "fista"])
@pytest.mark.parametrize("k,lam", [(1, 1.0), (10, 1.0), (100, 1.0), (100, 0.01)])
def test_fista_iterates_parity(dev, fista_problem, method, k, lam):
    d, g, og, La = fista_problem
    fast = method == "fista"
    y = d["y"][None].contiguous().to(dev)
    x = ph.reconstruct_slices(ph.Plan(g), sino=y, method=ph.FISTA if fast else ph.ISTA, lam=lam, n_iter=k,
                              op_norm=math.sqrt(La), n_inner=20)
    ref = oracle.fista_tv(d["y"].numpy(), og, lam, k, La, 20, fast=fast)
    assert rel(x[0], ref) <= TOL_PIPE, (method, k, lam, rel(x[0], ref))


@pytest.mark.parametrize("kind", ["blocks", "staged", "lines"])
def test_fista_iterates_every_fp_kernel(dev, fista_problem, kind):
    d, g, og, La = fista_problem
    plan = ph.Plan(g)
    plan.set_fp_kernel(FP_KINDS[kind])
    y = d["y"][None].contiguous().to(dev)
    x = ph.reconstruct_slices(plan, sino=y, method=ph.FISTA, lam=1.0, n_iter=10, op_norm=math.sqrt(La), n_inner=20)
    ref = oracle.fista_tv(d["y"].numpy(), og, 1.0, 10, La, 20, fast=True)
    assert rel(x[0], ref) <= TOL_PIPE, (kind, rel(x[0], ref))


def test_fista_energy_graph_and_opnorm(dev, fista_problem):
    d, g, og, La = fista_problem
    plan = ph.Plan(g)
    y = d["y"][None].contiguous().to(dev)
    x, E = ph.reconstruct_slices(plan, sino=y, method=ph.FISTA, lam=1.0, n_iter=30, op_norm=math.sqrt(La),
                                 n_inner=10, energy=True)
    xr, Er = oracle.fista_tv(d["y"].numpy(), og, 1.0, 30, La, 10, fast=True, energy=True)
    np.testing.assert_allclose(E, Er, rtol=1e-4)
    assert rel(x[0], xr) <= TOL_PIPE
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    for _ in range(3):
        with torch.cuda.stream(side):
            xg = ph.reconstruct_slices(plan, sino=y, method=ph.FISTA, lam=1.0, n_iter=30, op_norm=math.sqrt(La),
                                       n_inner=10, use_graph=True)
        side.synchronize()
        assert torch.equal(xg, x)
    # op_norm <= 0: 1.02 |A| from the GPU power iteration on A^T A
    ph.reconstruct_slices(plan, sino=y, method=ph.ISTA, lam=1.0, n_iter=1, op_norm=0.0, n_inner=10)
    assert abs(plan.last_op_norm / (1.02 * math.sqrt(La)) - 1) < 1e-3


def test_fista_beats_ista_and_recovers_disc(dev):
    """The paper's claim (section 3.1): FISTA converges faster than ISTA; both reach the disc."""
    N = 64
    g = ph.Geometry(N, N, N, synth.uniform_angles(48), (N - 1) / 2)
    y = synth.ellipse_sinogram(synth.disc_params(0.5, 1.0), g.angles, N, g.axis_pos, N).float()
    y = y[None].contiguous().to(dev)
    plan = ph.Plan(g)
    xf, Ef = ph.reconstruct_slices(plan, sino=y, method=ph.FISTA, lam=0.5, n_iter=150, n_inner=10, energy=True)
    xi, Ei = ph.reconstruct_slices(plan, sino=y, method=ph.ISTA, lam=0.5, n_iter=150, n_inner=10, energy=True)
    assert Ef[-1] < Ei[-1] and Ef[30] < Ei[30]
    yy, xx = np.mgrid[0:N, 0:N]
    inside = (xx - (N - 1) / 2) ** 2 + (yy - (N - 1) / 2) ** 2 < (0.4 * N / 2) ** 2
    assert abs(xf[0].cpu().numpy()[inside].mean() - 1.0) < 0.03


@pytest.mark.parametrize("S", [7, 11])
def test_fp_slice_pairs_equal_one_slice_kernel(dev, gen, S):
    """The automatic projector choice on a uniform plan of several slices takes two (7 slices of 256^2 x
    720) or four (11 slices) slices per workgroup (one staged segment and one set of hat weights for all);
    every value equals the one-slice staged kernel's bit for bit: a slice count that the group size does
    not divide (the last workgroup holds fewer), groups of up to four projections, the plain projection,
    the Chambolle-Pock dual update and the FISTA residual in the projector's epilogue."""
    N, K = 256, 720
    g, og = pair(nx=N, ny=N, nb=N, K=K, axis=128.2, shifts=0.3)
    x = torch.from_numpy(gen.standard_normal((S, N, N)).astype(np.float32)).to(dev)
    y = torch.from_numpy(gen.standard_normal((S, K, N)).astype(np.float32)).to(dev)
    res = {}
    for kind in (ph.FP_AUTO, ph.FP_STAGED):
        plan = ph.Plan(g, n_slices=S)
        plan.set_fp_kernel(kind)
        fp = ph.forward_project(plan, x)
        cp = ph.reconstruct_slices(plan, sino=y, method=ph.TV_CP, lam=0.01, n_iter=2, op_norm=400.0)
        fi = ph.reconstruct_slices(plan, sino=y, method=ph.FISTA, lam=0.5, n_iter=2, op_norm=400.0, n_inner=4)
        torch.cuda.synchronize()
        res[kind] = (fp, cp, fi)
    for a, b in zip(res[ph.FP_AUTO], res[ph.FP_STAGED]):
        assert torch.equal(a, b)


def test_fp_groups_of_four_parity(dev, gen):
    """A plan big enough for the staged projector's groups of four (8 slices x 256^2 x 720 angles with
    axis shifts: about 5800 workgroups, at least 16 per CU): the plain projection of every slice, and
    two Chambolle-Pock iterations (dual update fused into the projector) and two FISTA iterations
    (residual in the projector's epilogue) of the first two slices, against the oracle."""
    import test_kernel_index_replay as rp
    N, K, S = 256, 720, 8
    g, og = pair(nx=N, ny=N, nb=N, K=K, axis=128.2, shifts=0.3)
    # the plan's grouping rule, replayed: groups of up to four and enough workgroups to keep them
    P = [rp._proj(k, th, 1.0, N, N, og.axis, og.shifts[k]) for k, th in enumerate(og.angles)]
    groups = rp.staged_groups(P, N, N, N, 3, cap=4)
    assert max(len(q) for q in groups) == 4 and S * (N // 64) * len(groups) >= 16 * 256
    plan = ph.Plan(g, n_slices=S)
    x = gen.standard_normal((S, N, N)).astype(np.float32)
    out = ph.forward_project(plan, torch.from_numpy(x).to(dev))
    assert rel(out, oracle.forward_project(x, og)) <= TOL_OP
    y = gen.standard_normal((S, K, N)).astype(np.float32)
    xs = ph.reconstruct_slices(plan, sino=torch.from_numpy(y).to(dev), method=ph.TV_CP, lam=0.01, n_iter=2,
                               op_norm=400.0)
    for s in range(2):
        assert rel(xs[s], oracle.cp_tv(y[s], og, 0.01, 2, 400.0)) <= TOL_PIPE, s
    # FISTA: the residual A x - y computed in the projector's epilogue
    xf = ph.reconstruct_slices(plan, sino=torch.from_numpy(y).to(dev), method=ph.FISTA, lam=0.5, n_iter=2,
                               op_norm=400.0, n_inner=4)
    for s in range(2):
        assert rel(xf[s], oracle.fista_tv(y[s], og, 0.5, 2, 400.0 ** 2, 4, fast=True)) <= TOL_PIPE, s
