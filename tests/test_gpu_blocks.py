"""Edges of the kernels' work splits on the GPU: the list of near traces and
the trace blocks of migration, its kept source legs and trace parts, the bin
search, the moveout's lag blocks and depth parts, the filter's rows and the
stream kernels, each at the sizes where a split begins or ends, against the
FP64 oracle or float64.

Migration's tolerance is the parity bar of band-limited traces, 1e-5 relative
L2; the filter's 1e-6 of sum |h| max |x| (65 float32 roundings at most); the dot
product is a float64 sum of exact products, 1e-12 of the sum of magnitudes."""
import dataclasses

import numpy as np
import pytest
import torch

from oracle import trace_filter as oracle_filter
from paper_1204_1225_amd import survey
from test_gpu_cig import check_moveout

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ops():
    from paper_1204_1225_amd import _lib, ops

    _lib.load()
    return ops


def rel_l2(a, b):
    return float(np.linalg.norm(a.astype(np.float64) - b) / max(np.linalg.norm(b), 1e-300))


def shot_order(p, run):
    """The problem with its traces in runs of `run` that share a source (bins kept)."""
    src = p.src.copy()
    for j in range(p.n_traces):
        src[j] = src[j - j % run]
    return dataclasses.replace(p, src=src)


# traces, samples, nx, ny, nz, bins, run of equal sources, t_first, weight
CASES = [
    (1, 200, 1, 1, 1, 1, 1, 0.0, survey.WEIGHT_COSCOS),        # a single pair
    (63, 300, 5, 1, 15, 2, 3, 0.0, survey.WEIGHT_UNIT),        # one partial slot, a partial wavefront of bins
    (65, 300, 17, 3, 33, 3, 16, 0.1, survey.WEIGHT_COSCOS),    # one column, one depth past a tile
    (1100, 250, 4, 4, 140, 1, 17, 0.0, survey.WEIGHT_COSCOS),  # more near traces than the list holds
    (4097, 64, 16, 1, 32, 70, 2, 0.0, survey.WEIGHT_COSCOS),   # the bin search's second step, empty bins
    (300, 1500, 33, 2, 257, 1, 300, 0.0, survey.WEIGHT_COSCOS),  # windows longer than one staging step
]


@pytest.mark.parametrize("case", CASES)
@pytest.mark.parametrize("prec", ["fp32", "extended"])
def test_migrate_edges(ops, oracle_lib, case, prec):
    n, n_t, nx, ny, nz, bins, run, t_first, weight = case
    p = shot_order(survey.make_random(n + nz, n, n_t, nx, ny, nz, bins, t_first=t_first, weight=weight), run)
    dp = ops.to_device(p, prec=prec)
    ref = oracle_lib.migrate(p)
    first = None
    for tile in [-1] + list(range(ops.tile_count(0))):
        img = ops.migrate(dp, tile=tile)
        if not np.any(ref):
            assert not torch.any(img), tile
            continue
        assert rel_l2(img.cpu().numpy(), ref) <= 1e-5, (tile, prec)
        if 0 <= tile < 7:  # tiles without trace parts add a point's pairs in trace order: the same bits
            first = img if first is None else first
            assert torch.equal(img, first), tile


def test_table_pairs_at_the_aperture_edge(ops, oracle_lib):
    # amplitude tables and depth slots that only some columns of a group reach:
    # every tile without trace parts gives the same bits, all within 1e-5
    p = survey.make_random(11, 120, 400, 29, 5, 150, 3, aperture_deg=35.0)
    p = survey.with_curved_ray_table(shot_order(p, 6), 10.0, amplitude=True)
    ref = oracle_lib.migrate(p)
    dp = ops.to_device(p)
    a = ops.migrate(dp, tile=0)
    for tile in range(ops.tile_count(0)):
        img = ops.migrate(dp, tile=tile)
        assert rel_l2(img.cpu().numpy(), ref) <= 1e-5, tile
        assert tile >= 7 or torch.equal(img, a), tile


# bins, ny, nx, nz, lags, window
@pytest.mark.parametrize("shape", [(3, 1, 3, 33, 0, None), (16, 1, 4, 100, 4, (7, 90)), (17, 2, 2, 63, 12, None),
                                   (40, 1, 2, 64, 20, (0, 1)), (300, 1, 1, 24, 3, None), (2, 1, 2, 30, 40, None)])
def test_moveout_splits(ops, shape):
    nb, ny, nx, nz, lag, win = shape
    rng = np.random.default_rng(nb + nz)
    base = survey.bandlimited_noise(rng, ny * nx, nz + 8, 0.004)
    img = np.stack([np.roll(base, b % 3, axis=1)[:, :nz] for b in range(nb)]).reshape(nb, ny, nx, nz)
    img = (img + 0.2 * rng.standard_normal(img.shape)).astype(np.float32)
    off = np.linspace(10.0, 900.0, nb).astype(np.float32)
    z_lo, z_hi = win or (0, nz)
    got = ops.cig_moveout(torch.from_numpy(img).cuda(), torch.from_numpy(off).cuda(), lag, z_lo, z_hi)
    if lag == 0:  # one lag: no runner-up to compare with
        S = img.astype(np.float64).sum(0)
        C = (S * img.astype(np.float64))[..., z_lo:z_hi].sum(-1)
        assert not torch.any(got[1])
        assert np.abs(got[2].cpu().numpy() - C).max() <= 1e-6 * np.abs(C).max()
        return
    check_moveout(img, off, lag, z_lo, z_hi, got)


# records of 40 900 samples leave room for the tight rows only
@pytest.mark.parametrize("n,n_t,K,center,stride", [(1, 1, 1, 0, 1), (5, 7, 3, 1, 8), (4, 8, 65, 32, 8),
                                                   (9, 1499, 66, 0, 1500), (3, 1503, 67, 66, 1503),
                                                   (2, 5000, 64, 20, 5000), (2, 40900, 5, 2, 40900)])
@pytest.mark.parametrize("adjoint", [False, True])
def test_filter_splits(ops, n, n_t, K, center, stride, adjoint):
    rng = np.random.default_rng(n_t + K)
    x = rng.standard_normal((n, n_t)).astype(np.float32)
    h = rng.standard_normal(K).astype(np.float32)
    buf = torch.zeros((n, stride), device="cuda")
    buf[:, :n_t] = torch.from_numpy(x).cuda()
    t = buf[:, :n_t]
    ref = (oracle_filter.adjoint if adjoint else oracle_filter.forward)(x, h, center)
    tol = 1e-6 * float(np.abs(h).sum()) * float(np.abs(x).max())
    got = ops.trace_filter(t, torch.from_numpy(h).cuda(), center, adjoint=adjoint)
    assert np.abs(got.cpu().numpy() - ref).max() <= tol
    ops.trace_filter(t, torch.from_numpy(h).cuda(), center, adjoint=adjoint, out=t)  # in place
    assert torch.equal(t, got)


def test_filter_infinity_stays_within_its_taps(ops):
    x = torch.zeros((1, 200), device="cuda")
    x[0, 100] = float("inf")
    h = torch.ones(5, device="cuda")
    y = ops.trace_filter(x, h, 2)[0].cpu().numpy()
    assert np.isinf(y[98:103]).all() and (y[:98] == 0).all() and (y[103:] == 0).all()


@pytest.mark.parametrize("n", [0, 1, 3, 4, 5, 1023, 4 * 4 * 256 * 3 + 7, 1 << 21])
@pytest.mark.parametrize("shift", [0, 1])
def test_streams(ops, n, shift):
    g = torch.Generator(device="cuda").manual_seed(n + shift)
    a = torch.randn(n + shift, generator=g, device="cuda")[shift:]
    b = torch.randn(n + shift, generator=g, device="cuda")[shift:]
    ref = float((a.double() * b.double()).sum())
    size = float((a.double() * b.double()).abs().sum())
    assert abs(float(ops.dot_f64(a, b)) - ref) <= 1e-12 * size
    y = b.clone()[:] if shift == 0 else torch.cat([b[:1], b])[1:]
    ops.axpby(2.5, a, -0.5, y)
    ref_y = torch.addcmul(-0.5 * b, a, torch.full_like(a, 2.5))
    assert n == 0 or float((y - ref_y).abs().max()) <= 2.0 ** -22 * 10.0
    y.fill_(float("nan"))
    ops.axpby(3.0, a, 0.0, y)
    assert torch.equal(y, 3.0 * a)


# windows of one position up to several staging steps of 256, 16-bit rows at odd samples
@pytest.mark.parametrize("n_t,dtype", [(1, "f32"), (3, "f32"), (254, "bf16"), (257, "f16"), (1031, "f32"), (1500, "bf16")])
def test_anti_alias_windows(ops, oracle_lib, n_t, dtype):
    p = survey.make_random(n_t, 70, n_t, 19, 3, 70, 2, weight=survey.WEIGHT_UNIT)
    p = dataclasses.replace(p, aa=(12.0, 12.0, 16))
    dp = ops.to_device(p, dtype=dtype)
    if dtype != "f32":
        p = dataclasses.replace(p, data=survey.quantise(p.data, dtype)[2])
    ref = oracle_lib.migrate(p)
    for tile in [-1] + list(range(ops.tile_count(0))):
        assert rel_l2(ops.migrate(dp, tile=tile).cpu().numpy(), ref) <= 1e-5, tile


# A record that most pairs outlast holds the first samples of a longer one: the same
# taps in another order, so each sample within two roundings (and the anti-alias
# kernel's double suffix sums, float64, within 1e-9 of the long record's largest).
@pytest.mark.parametrize("n_t,t_first,weight", [(1, 0.0, survey.WEIGHT_UNIT), (60, 0.0, survey.WEIGHT_COSCOS),
                                                (130, 0.35, survey.WEIGHT_COSCOS), (64, 0.5, survey.WEIGHT_UNIT)])
@pytest.mark.parametrize("kind", ["fp32", "extended", "aa", "table", "ltable"])
@pytest.mark.parametrize("spread", [40.0, 900.0])
def test_adjoint_pairs_past_the_record(ops, n_t, t_first, weight, kind, spread):
    p = survey.make_random(n_t + int(spread), 45, n_t, 37, 6, 140, 2, t_first=t_first, weight=weight, spread=spread)
    if kind == "aa":
        p = dataclasses.replace(p, aa=(12.0, 12.0, 8))
    elif kind == "table":
        p = survey.with_curved_ray_table(p, 10.0, amplitude=True)
    elif kind == "ltable":
        p = survey.with_lateral_tables(p, lambda x, y: 1500.0 + 0.05 * x, 0.5, -300.0, 800.0, 700.0, 700.0, 4, 4, dh=20.0)
    prec = "extended" if kind == "extended" else "fp32"
    m = torch.from_numpy(survey.random_image(p, n_t)).cuda()
    long = ops.to_device(dataclasses.replace(p, n_t=n_t + 900, data=None), prec=prec)
    ref = ops.demigrate(long, m, tile=0).cpu().numpy().astype(np.float64)
    largest, ref = np.abs(ref).max(), ref[:, :n_t]
    dp = ops.to_device(p, prec=prec)
    for tile in [-1] + list(range(ops.tile_count(1))):
        d = ops.demigrate(dp, m, tile=tile).cpu().numpy()
        assert np.all(np.abs(d - ref) <= 2.0 ** -22 * np.abs(ref) + 1e-9 * largest), tile


# four float64 rows beside the small tables: within the shape's budget, up to and past two and one
# workgroups per CU, up to the last record of which four fit, and where fewer do
@pytest.mark.parametrize("n_t", [1500, 2530, 2560, 5090, 5110, 10300])
@pytest.mark.parametrize("kind", ["fp32", "extended", "aa", "table"])
def test_adjoint_rows_of_long_records(ops, oracle_lib, n_t, kind):
    p = survey.make_random(n_t, 13, n_t, 9, 2, 40, 2, weight=survey.WEIGHT_UNIT, dt=0.0004)
    if kind == "aa":
        p = dataclasses.replace(p, aa=(12.0, 12.0, 8))
    elif kind == "table":
        p = survey.with_curved_ray_table(p, 10.0)
    dp = ops.to_device(p, prec="extended" if kind == "extended" else "fp32")
    m = survey.random_image(p, 3)
    ref = ops.demigrate(dp, torch.from_numpy(m).cuda(), tile=1).cpu().numpy().astype(np.float64)
    # the same taps in another order, float64: two roundings, 1e-9 for the anti-alias sums
    for tile in [-1] + list(range(ops.tile_count(1))):
        d = ops.demigrate(dp, torch.from_numpy(m).cuda(), tile=tile).cpu().numpy()
        assert np.all(np.abs(d - ref) <= 2.0 ** -22 * np.abs(ref) + 1e-9 * np.abs(ref).max()), tile
    # against the oracle: a float32 time of up to 10 300 samples is good to 3 x 2^-24 of itself, 2e-3 samples
    data = survey.random_data(p, 4)
    lhs = float(np.vdot(oracle_lib.migrate(dataclasses.replace(p, data=data)), m))
    rhs = float(np.vdot(data.astype(np.float64), ref))
    assert abs(lhs - rhs) <= 2e-3 * np.linalg.norm(data.astype(np.float64)) * np.linalg.norm(ref)


# An aperture value that is NaN admits no pair (h^2 <= NaN is false), in both directions, also
# where the record's end bounds the aperture or the slot's other depths are all inside: as -1 does.  The same taps in another
# order: two roundings, 1e-9 of the largest for the anti-alias sums.
@pytest.mark.parametrize("kind", ["fp32", "extended", "aa"])
@pytest.mark.parametrize("flat", [False, True])  # s2 = 0 at those depths: no bound from the record's end
def test_nan_aperture_admits_no_pair(ops, kind, flat):
    p = survey.make_random(5, 45, 120, 21, 4, 90, 2, weight=survey.WEIGHT_UNIT)
    deep = np.arange(p.nz) % 3 == 1
    if flat:
        p = dataclasses.replace(p, s2=np.where(deep, 0.0, p.s2))
    if kind == "aa":
        p = dataclasses.replace(p, aa=(12.0, 12.0, 8))
    prec = "extended" if kind == "extended" else "fp32"
    m = torch.from_numpy(survey.random_image(p, 6)).cuda()
    none = ops.to_device(dataclasses.replace(p, r2=np.where(deep, -1.0, p.r2)), prec=prec)
    nan = ops.to_device(dataclasses.replace(p, r2=np.where(deep, np.nan, p.r2)), prec=prec)
    ref = ops.demigrate(none, m).cpu().numpy().astype(np.float64)
    assert np.any(ref)
    for tile in [-1] + list(range(ops.tile_count(1))):
        d = ops.demigrate(nan, m, tile=tile).cpu().numpy()
        assert np.all(np.abs(d - ref) <= 2.0 ** -22 * np.abs(ref) + 1e-9 * np.abs(ref).max()), tile
    for tile in [-1] + list(range(ops.tile_count(0))):
        img = ops.migrate(nan, tile=tile)
        assert torch.equal(img, ops.migrate(none, tile=tile)) and torch.any(img), tile


# An infinite image value reaches the two samples around its pairs' times and no other: the
# adjoint of one infinite point is non-finite there only, everything else as with a 0 in its place
# (another summation order: two roundings).  A time within 2^-18 of a sample may count as that
# sample, so a pair's two samples are those of the times a little to either side.
@pytest.mark.parametrize("weight", [survey.WEIGHT_UNIT, survey.WEIGHT_COSCOS])
@pytest.mark.parametrize("t_first", [0.0, 0.1])
def test_adjoint_infinity_stays_within_its_taps(ops, weight, t_first):
    p = survey.make_random(8, 37, 260, 15, 3, 70, 1, weight=weight, t_first=t_first, spread=100.0)
    dp = ops.to_device(p)
    m = survey.random_image(p, 9)
    points = [(0, 1, 7, iz) for iz in range(20, 52)]  # both slots of every depth pair
    hit = 0
    for b, iy, ix, iz in points:
        m0, m1 = m.copy(), m.copy()
        m0[b, iy, ix, iz], m1[b, iy, ix, iz] = 0.0, np.inf
        h2 = [((p.x[ix] - q[:, 0]) ** 2 + (p.y[iy] - q[:, 1]) ** 2).astype(np.float64) for q in (p.src, p.rec)]
        u = (sum(np.sqrt(p.t0sq[iz] + p.s2[iz] * h) for h in h2) - t_first) / p.dt
        inside = np.maximum(*h2) <= p.r2[iz] * (1.0 + 1e-5)
        may = np.zeros((p.n_traces, p.n_t), bool)
        for j in np.flatnonzero(inside):
            for i in {int(np.floor(u[j] * (1.0 + e))) + k for e in (-1e-6, 1e-6) for k in (0, 1)}:
                if 0 <= i < p.n_t:
                    may[j, i] = True
        ref = ops.demigrate(dp, torch.from_numpy(m0).cuda()).cpu().numpy().astype(np.float64)
        d = ops.demigrate(dp, torch.from_numpy(m1).cuda()).cpu().numpy()
        assert not np.any(~np.isfinite(d) & ~may), iz
        ok = np.isfinite(d)
        assert np.all(np.abs(d - ref)[ok] <= 2.0 ** -22 * np.abs(ref[ok]) + 1e-9 * np.abs(ref).max()), iz
        hit += int(np.sum(~ok))
    assert hit > 100


# Depths that no lag of the window reaches do not matter, whatever they hold (lags of one to
# five blocks, windows that end inside a block's turn).
@pytest.mark.parametrize("lag", [1, 4, 6, 12, 20, 40])
@pytest.mark.parametrize("bins", [2, 16, 40])
def test_moveout_window_shuts_out_other_depths(ops, lag, bins):
    rng = np.random.default_rng(lag + bins)
    nz, z_lo, z_hi = 200, 50, 90 + lag % 3
    img = rng.standard_normal((bins, 1, 3, nz)).astype(np.float32)
    out = np.r_[0:max(z_lo - lag, 0), z_hi + lag:nz]
    off = torch.linspace(10.0, 900.0, bins, device="cuda")
    img[..., out] = 0.0
    ref = ops.cig_moveout(torch.from_numpy(img).cuda(), off, lag, z_lo, z_hi)
    for v in (np.inf, np.nan):
        img[..., out] = v
        got = ops.cig_moveout(torch.from_numpy(img).cuda(), off, lag, z_lo, z_hi)
        for a, b in zip(got[1:], ref[1:]):
            assert torch.equal(a, b) and torch.isfinite(a).all(), v


# Records whose trace block would take the whole of a workgroup's LDS: the batch kernel keeps a
# variable of its own there.  One batch per tile, the same bits as the single launch.
@pytest.mark.parametrize("n_t", [19764, 19796, 19956])
def test_batches_of_the_longest_records(ops, n_t):
    p = survey.make_random(n_t, 20, n_t, 9, 1, 40, 1, weight=survey.WEIGHT_UNIT, dt=0.0002, spread=50.0)
    dp = ops.to_device(p)
    for tile in [-1, 1 + 64 * 3] + list(range(ops.tile_count(0))):
        img = torch.full(dp.image_shape, float("nan"), device="cuda")
        b = ops.Batch([dp], [img], tile=tile)
        b.run()
        torch.cuda.synchronize()
        b.close()
        ref = ops.migrate(dp, tile=tile)
        assert bool(torch.equal(img, ref)) and bool(torch.any(img)), tile


# Traces whose sources repeat (a kept source leg) or do not (both legs of every pair), and a list
# where half do: the same bits on every tile without trace parts, 16-bit staging included, all
# within the parity bar of the oracle.
@pytest.mark.parametrize("run", [1, 2, 5])
@pytest.mark.parametrize("kind", ["fp32", "extended", "table", "ltable"])
@pytest.mark.parametrize("dtype,t_first", [("f32", 0.1), ("bf16", 0.0), ("f16", 0.1)])
def test_repeated_and_single_sources(ops, oracle_lib, run, kind, dtype, t_first):
    p = shot_order(survey.make_random(run + 3, 130, 300, 21, 3, 75, 3, t_first=t_first, spread=200.0), run)
    if kind == "table":
        p = survey.with_curved_ray_table(p, 10.0, amplitude=True)
    elif kind == "ltable":
        p = survey.with_lateral_tables(p, lambda x, y: 1500.0 + 0.05 * x, 0.5, 600.0, 1500.0, 400.0, 400.0, 4, 4, dh=20.0)
    dp = ops.to_device(p, dtype=dtype, prec="extended" if kind == "extended" else "fp32")
    if dtype != "f32":
        p = dataclasses.replace(p, data=survey.quantise(p.data, dtype)[2])
    ref = oracle_lib.migrate(p)
    assert np.any(ref)
    first = ops.migrate(dp, tile=0)
    for tile in range(ops.tile_count(0)):
        img = ops.migrate(dp, tile=tile)
        assert rel_l2(img.cpu().numpy(), ref) <= 1e-5, tile
        assert tile >= 7 or bool(torch.equal(img, first)), tile
        if dtype != "f32" and kind != "extended":
            assert rel_l2(ops.migrate(dp, tile=tile + 256).cpu().numpy(), ref) <= 1e-5, tile


# From 4096 traces on a wavefront takes a trace, below a workgroup: the same sums.
@pytest.mark.parametrize("n_t,K", [(70, 9), (601, 65)])
@pytest.mark.parametrize("adjoint", [False, True])
def test_filter_of_few_and_many_traces(ops, n_t, K, adjoint):
    rng = np.random.default_rng(K)
    x = rng.standard_normal((4097, n_t)).astype(np.float32)
    h = rng.standard_normal(K).astype(np.float32)
    ref = (oracle_filter.adjoint if adjoint else oracle_filter.forward)(x, h, K // 3)
    t, taps = torch.from_numpy(x).cuda(), torch.from_numpy(h).cuda()
    many = ops.trace_filter(t, taps, K // 3, adjoint=adjoint)
    assert np.abs(many.cpu().numpy() - ref).max() <= 1e-6 * float(np.abs(h).sum()) * float(np.abs(x).max())
    assert torch.equal(ops.trace_filter(t[:4095], taps, K // 3, adjoint=adjoint), many[:4095])


# Adjoints of long records against the oracle, the pairs spread over the whole record (rows of
# four, two and one workgroups per CU, and records of which fewer than four rows fit).  A float32
# time is good to 3 x 2^-24 of itself, d samples at the record's end: each tap is off by at most d
# of its weight, a relative L2 error of at most 2 d on taps that do not cancel; 4 d leaves room for
# those that do.  A float32 table time has its leg length's rounding, 2^-24 of the part that grows
# with it: within the same bound.  Extended times are good to 1e-9 samples: the parity bar.
@pytest.mark.parametrize("n_t", [1500, 2530, 2560, 5090, 5110, 10300])
@pytest.mark.parametrize("kind", ["fp32", "extended", "aa", "table"])
def test_adjoint_of_long_records_against_the_oracle(ops, oracle_lib, n_t, kind):
    p = survey.make_random(n_t, 13, n_t, 9, 2, 70, 2, weight=survey.WEIGHT_UNIT, dt=1.25 / n_t, dz=15.0, spread=50.0)
    if kind == "aa":
        p = dataclasses.replace(p, aa=(12.0, 12.0, 8))
    elif kind == "table":
        p = survey.with_curved_ray_table(p, 10.0)
    m = survey.random_image(p, 3)
    ref = oracle_lib.demigrate(p, m)
    assert np.count_nonzero(ref) > 0.05 * ref.size and np.any(ref[:, -n_t // 10:]) and np.any(ref[:, :n_t // 5])
    bar = 4 * 3 * 2.0 ** -24 * n_t if kind != "extended" else 1e-5
    dp = ops.to_device(p, prec="extended" if kind == "extended" else "fp32")
    for tile in [-1] + list(range(ops.tile_count(1))):
        d = ops.demigrate(dp, torch.from_numpy(m).cuda(), tile=tile).cpu().numpy()
        assert rel_l2(d, ref) <= bar, (tile, rel_l2(d, ref), bar)


# One pair and records of one to three samples, its time 0.3 samples after the first: every lane,
# slot and window edge of the kernels at its smallest.  The time is a few samples long before
# t_first is taken off, good to 1e-6 samples in float32.
@pytest.mark.parametrize("n_t", [1, 2, 3])
@pytest.mark.parametrize("kind", ["fp32", "extended", "aa", "table"])
@pytest.mark.parametrize("weight", [survey.WEIGHT_UNIT, survey.WEIGHT_COSCOS])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_a_single_pair(ops, oracle_lib, n_t, kind, weight, dtype):
    p = survey.make_random(1, 1, n_t, 1, 1, 1, 1, weight=weight)
    x = float(p.x[0])
    src, rec = np.array([[x - 3.0, 0.0]], np.float32), np.array([[x + 4.0, 0.0]], np.float32)
    T = sum(float(np.sqrt(p.t0sq[0] + p.s2[0] * h * h)) for h in (3.0, 4.0))
    data = np.array([[1.5, -0.75, 0.5]], np.float32)[:, :n_t]
    p = dataclasses.replace(p, src=src, rec=rec, bin=np.zeros(1, np.int32), t_first=T - 0.3 * p.dt, data=data)
    if kind == "aa":
        p = dataclasses.replace(p, aa=(12.0, 0.0, 16))
    elif kind == "table":
        p = survey.with_curved_ray_table(dataclasses.replace(p, weight=survey.WEIGHT_UNIT), 10.0,
                                         amplitude=weight == survey.WEIGHT_COSCOS)
    dp = ops.to_device(p, dtype=dtype, prec="extended" if kind == "extended" else "fp32")
    m = np.full(p.image_shape, 2.0, np.float32)
    if dtype != "f32":
        p = dataclasses.replace(p, data=survey.quantise(p.data, dtype)[2])
    ref, ref_d = oracle_lib.migrate(p), oracle_lib.demigrate(p, m)
    assert np.any(ref) and np.any(ref_d)
    for tile in [-1] + list(range(ops.tile_count(0))):
        assert rel_l2(ops.migrate(dp, tile=tile).cpu().numpy(), ref) <= 1e-5, tile
    for tile in [-1] + list(range(ops.tile_count(1))):
        d = ops.demigrate(dp, torch.from_numpy(m).cuda(), tile=tile).cpu().numpy()
        assert rel_l2(d, ref_d) <= 1e-5, tile


# Nothing to add leaves zeros, whatever the output memory held.
def test_empty_problems_overwrite_nan(ops):
    p = survey.make_random(2, 6, 50, 5, 3, 7, 2)
    empty = ops.to_device(p.subset(np.zeros(0, np.int64)))
    img = torch.full(empty.image_shape, float("nan"), device="cuda")
    assert not torch.any(ops.migrate(empty, data=torch.zeros((0, 50), device="cuda"), dtype="f32", image=img))
    dp = ops.to_device(dataclasses.replace(p, x=p.x[:0]))
    out = torch.full((6, 50), float("inf"), device="cuda")
    assert not torch.any(ops.demigrate(dp, torch.zeros(dp.image_shape, device="cuda"), out=out))
