"""GPU gather and scatter lanes: windows that start at any sample, flagged samples inside a lane,
and runs of every length, against the FP64 oracle.

A lane holds 8 consecutive samples.  Cases: one to nine samples per pixel (a lane then sees one to
eight pixels, and a wavefront completes up to 512 runs, eight times the 64 that its list holds);
many flags (lanes that begin, end or consist of flagged samples) with NaN weights at the flagged
samples, whose values are nowhere used; odd detector lengths and intervals, so that windows start
at every alignment; bands short enough for the scatter's last list to reach past the window.

Tolerances: P x within one FP32 ulp; P^T u 1e-12 relative; A x and b of the mixed-precision
products relative L2 3e-6 (FP32 time domain and transform); of FP64 plans 1e-12 of the norm of
|P|^T |N^-1| |P| |x|, whose elements bound the sums that form each result.
"""

import dataclasses

import numpy as np
import pytest

import oracle as O
import synth

pytestmark = pytest.mark.gpu


def _dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


def _rel(a, b):
    return np.linalg.norm(np.asarray(a, np.float64) - b) / np.linalg.norm(b)


def _problem(dwell, lam, flag_frac, n_dets=3, per_det=30011, interval=9001, side=20):
    prob = synth.make_ground(cfg_id=700 + 10 * dwell + n_dets, n_dets=n_dets,
                             samples_per_det=per_det, interval=interval, side=side, dwell=dwell,
                             lam=lam, flag_frac=flag_frac)
    ref = O.plan_from_problem(prob)
    skip = prob.pix < 0
    gpu = dataclasses.replace(prob, wq=np.where(skip, np.float32("nan"), prob.wq),
                              wu=np.where(skip, np.float32("nan"), prob.wu))
    return gpu, ref


@pytest.mark.parametrize("dwell", [1, 2, 4, 7, 9])
@pytest.mark.parametrize("flag_frac", [0.02, 0.6])
def test_lanes_scan_and_bin(gpu_lib, dwell, flag_frac):
    prob, ref = _problem(dwell, 40, flag_frac)
    plan = gpu_lib.Plan.from_problem(prob)
    g = np.random.default_rng(dwell)
    x = g.standard_normal((ref.n_kept, 3))
    import torch
    for shift in (0, 1, 3):  # time streams at any float address
        t = torch.empty(prob.n_samples + 4, device="cuda")[shift:shift + prob.n_samples]
        got = plan.unpoint(_dev(x), t=t).cpu().numpy()
        want = O.unpoint(ref, x)
        assert np.all(np.abs(got - want) <= 2.0 ** -23 * np.abs(want) + 1e-30)
        u = g.standard_normal(prob.n_samples + 4).astype(np.float32)
        du = _dev(u)[shift:shift + prob.n_samples]
        y = plan.point(du).cpu().numpy()
        assert _rel(y, O.point(ref, u[shift:shift + prob.n_samples].astype(np.float64))) <= 1e-12


# every product kernel: LDS (one wavefront per segment .. 16), register, long; and bands so short
# that a wavefront's outputs start within 256 samples of the window's end
PRODUCTS = [(300, 0), (40, 2048), (1, 2048), (85, 2048), (900, 0), (85, 4096), (2000, 0),
            (200, 8192), (3000, 0), (5000, 0), (8192, 0), (9000, 0), (12001, 65536),
            (20001, 131072)]


@pytest.mark.parametrize("dwell,flag_frac", [(1, 0.02), (3, 0.3), (7, 0.02)])
@pytest.mark.parametrize("lam,fft_size", PRODUCTS)
def test_lanes_system_product(gpu_lib, lam, fft_size, dwell, flag_frac):
    prob, ref = _problem(dwell, lam, flag_frac, n_dets=2, per_det=60013, interval=20011)
    plan = gpu_lib.Plan.from_problem(prob, toeplitz_algo=gpu_lib.TOEPLITZ_FFT, fft_size=fft_size)
    x = np.random.default_rng(lam).standard_normal((ref.n_kept, 3))
    assert _rel(plan.apply_A(_dev(x)).cpu().numpy(), O.apply_A(ref, x)) <= 3e-6
    n = prob.n_samples
    d = np.concatenate([np.zeros(1, np.float32), prob.d[0]])
    b = plan.rhs(_dev(d)[1:1 + n]).cpu().numpy()  # data at an odd float address
    assert _rel(b, O.rhs(ref, prob.d[0])) <= 3e-6


@pytest.mark.parametrize("dwell,flag_frac", [(1, 0.02), (3, 0.3), (7, 0.02)])
@pytest.mark.parametrize("lam", [12, 600, 1025, 4096, 8192, 20001])
def test_lanes_fp64_product(gpu_lib, lam, dwell, flag_frac):
    prob, ref = _problem(dwell, lam, flag_frac, n_dets=2, per_det=60013, interval=20011)
    plan = gpu_lib.Plan.from_problem(prob, precision=gpu_lib.PRECISION_FP64)
    x = np.random.default_rng(lam).standard_normal((ref.n_kept, 3))
    absref = dataclasses.replace(ref, bands=[np.abs(b) for b in ref.bands],
                                 wq=np.abs(ref.wq), wu=np.abs(ref.wu))
    scale = np.linalg.norm(O.apply_A(absref, np.abs(x)))
    got = plan.apply_A(_dev(x)).cpu().numpy()
    assert np.linalg.norm(got - O.apply_A(ref, x)) <= 1e-12 * scale


@pytest.mark.parametrize("n,lam", [(2048, 1), (2048, 301), (2048, 600), (4096, 1023), (4096, 1025),
                                   (8192, 999), (8192, 2500), (16384, 4095), (16384, 4096),
                                   (32768, 1), (32768, 8191), (32768, 8193)])
def test_lanes_fp64_segments(gpu_lib, n, lam):
    """FP64 segments of every size with more and with at most N / 2 outputs, even and odd bands."""
    prob, ref = _problem(3, lam, 0.02, n_dets=2, per_det=60013, interval=40011)
    plan = gpu_lib.Plan.from_problem(prob, precision=gpu_lib.PRECISION_FP64,
                                     toeplitz_algo=gpu_lib.TOEPLITZ_FFT, fft_size=n)
    x = np.random.default_rng(lam).standard_normal((ref.n_kept, 3))
    absref = dataclasses.replace(ref, bands=[np.abs(b) for b in ref.bands],
                                 wq=np.abs(ref.wq), wu=np.abs(ref.wu))
    got = plan.apply_A(_dev(x)).cpu().numpy()
    scale = np.linalg.norm(O.apply_A(absref, np.abs(x)))
    assert np.linalg.norm(got - O.apply_A(ref, x)) <= 1e-12 * scale
    b = plan.rhs(_dev(prob.d[0])).cpu().numpy()
    d = np.abs(np.where(prob.pix >= 0, prob.d[0], 0.0))
    assert np.linalg.norm(b - O.rhs(ref, prob.d[0])) <= 1e-12 * np.linalg.norm(O.rhs(absref, d))


@pytest.mark.parametrize("unfused", [False, True])
@pytest.mark.parametrize("lam", [1, 6, 7, 8, 9, 15, 16, 17, 32, 33, 500, 4096])
def test_lanes_direct_product(gpu_lib, lam, unfused):
    """Direct products around the rounds of eight lags, with blocks shorter than the band, samples
    outside every block, ragged tiles and flags; two columns in one launch."""
    prob = synth.make_random_small(seed=40, n_samples=13007, n_pix=60, n_dets=4, lam_max=4,
                                   flag_frac=0.1, gap_frac=0.3, dwell=5)
    k = np.arange(lam + 1)
    c = -0.3 * np.exp(-k / (1.0 + lam / 4.0)) / (1.0 + lam / 8.0)
    c[0] = 1.0 + 2.0 * np.abs(c[1:]).sum()
    bands = [c.astype(np.float32)] + [(c[: max(1, lam // 2)] * 1.5).astype(np.float32)] * (
        len(prob.bands) - 1)
    prob = dataclasses.replace(prob, bands=bands)
    ref = O.plan_from_problem(prob)
    plan = gpu_lib.Plan.from_problem(prob, toeplitz_algo=gpu_lib.TOEPLITZ_DIRECT,
                                     flags=gpu_lib.FLAG_UNFUSED if unfused else 0)
    x = np.random.default_rng(lam).standard_normal((2, ref.n_kept, 3))
    y = plan.apply_A(_dev(x)).cpu().numpy()
    for j in range(2):
        assert _rel(y[j], O.apply_A(ref, x[j])) <= 3e-6
    assert _rel(plan.rhs(_dev(prob.d[0])).cpu().numpy(), O.rhs(ref, prob.d[0])) <= 3e-6
    t = np.random.default_rng(1).standard_normal(prob.n_samples).astype(np.float32)
    u = plan.noise_weight(_dev(t)).cpu().numpy()
    assert _rel(u, O.noise_weight(t.astype(np.float64), ref)) <= 2e-6


@pytest.mark.parametrize("lam", [8192, 8193, 12000, 15000])
def test_lanes_register_noise_weight(gpu_lib, lam):
    """u = N^-1 t by the register transform: whole and partial segments (a block shorter than the
    band, odd block lengths, odd bands), samples outside every block, streams at odd addresses.
    FP32 transform of 2^15 samples: relative L2 2e-6."""
    prob, ref = _problem(3, lam, 0.02, n_dets=2, per_det=60013, interval=40011)
    plan = gpu_lib.Plan.from_problem(prob, toeplitz_algo=gpu_lib.TOEPLITZ_FFT, fft_size=32768)
    import torch
    n = prob.n_samples
    t = np.random.default_rng(lam).standard_normal(n + 1).astype(np.float32)
    for shift in (0, 1):
        out = torch.full((n + 4,), 7.0, device="cuda")
        u = plan.noise_weight(_dev(t)[shift:shift + n], u=out[1 + shift:1 + shift + n]).cpu().numpy()
        assert _rel(u, O.noise_weight(t[shift:shift + n].astype(np.float64), ref)) <= 2e-6
        rest = torch.cat([out[:1 + shift], out[1 + shift + n:]]).cpu().numpy()
        assert np.all(rest == 7.0)


@pytest.mark.parametrize("flag_frac", [0.0, 0.02])
@pytest.mark.parametrize("baseline,n_poly", [(60, 1), (500, 3), (1024, 3), (1025, 2), (4096, 4),
                                             (4097, 3), (8192, 3), (8193, 8), (20011, 3)])
def test_lanes_template_product(gpu_lib, baseline, n_poly, flag_frac):
    """Template products around the rules of workgroup size and held steps, with samples outside
    every baseline (diagonal tiles) and runs of two samples (more runs than a list holds).  FP64
    throughout: 1e-11 of the product with every factor replaced by its magnitude, which bounds
    the sums that form each element."""
    prob = synth.make_templates(cfg_id=800 + n_poly, n_dets=3, samples_per_det=60033,
                                interval=20011, side=20, dwell=2, baseline=baseline,
                                n_poly=n_poly, cover=0.9, flag_frac=flag_frac)
    m = prob.meta
    tp = O.template_plan_from_problem(prob)
    plan = gpu_lib.Plan.from_problem(prob, n_poly=n_poly, base_start=m["base_start"],
                                     base_len=m["base_len"])
    x = np.random.default_rng(n_poly).standard_normal((tp.plan.n_kept, 3))

    def magnitude(t):
        fit = np.zeros_like(t)
        for i, (s, L) in enumerate(zip(tp.base_start, tp.base_len)):
            T = O.legendre_templates(int(L), n_poly)
            fit[s:s + L] = np.abs(T) @ (np.abs(tp.Kinv[i]) @ (np.abs(T).T @ np.abs(
                tp.w[s:s + L] * t[s:s + L])))
        a = tp.w * (np.abs(t) + fit)
        p = dataclasses.replace(tp.plan, wq=np.abs(tp.plan.wq), wu=np.abs(tp.plan.wu))
        return O.point(p, a)

    err = np.abs(plan.apply_A(_dev(x)).cpu().numpy() - O.template_apply_A(tp, x))
    assert np.all(err <= 1e-11 * magnitude(O.unpoint(tp.plan, x)) + 1e-300)
    err = np.abs(plan.rhs(_dev(prob.d[0])).cpu().numpy() - O.template_rhs(tp, prob.d[0]))
    d = np.where(tp.plan.lpix >= 0, prob.d[0], 0.0)
    assert np.all(err <= 1e-11 * magnitude(d) + 1e-300)


@pytest.mark.parametrize("dwell,flag_frac", [(1, 0.02), (3, 0.6), (8, 0.0)])
def test_lanes_diagonal_product(gpu_lib, dwell, flag_frac):
    """Diagonal weights: FP64 throughout, 1e-12 relative."""
    prob, ref = _problem(dwell, 0, flag_frac)
    plan = gpu_lib.Plan.from_problem(prob)
    x = np.random.default_rng(dwell).standard_normal((ref.n_kept, 3))
    assert _rel(plan.apply_A(_dev(x)).cpu().numpy(), O.apply_A(ref, x)) <= 1e-12
    assert _rel(plan.rhs(_dev(prob.d[0])).cpu().numpy(), O.rhs(ref, prob.d[0])) <= 1e-12


@pytest.mark.parametrize("lam", [1, 7, 8, 9, 32, 33, 500, 4096])
def test_lanes_fp64_direct_product(gpu_lib, lam):
    """FP64 direct products around the rounds of eight lags (and a window beyond 64 KiB of LDS),
    with blocks shorter than the band, samples outside every block, ragged tiles and flags."""
    prob = synth.make_random_small(seed=41, n_samples=13007, n_pix=60, n_dets=4, lam_max=4,
                                   flag_frac=0.1, gap_frac=0.3, dwell=5)
    k = np.arange(lam + 1)
    c = -0.3 * np.exp(-k / (1.0 + lam / 4.0)) / (1.0 + lam / 8.0)
    c[0] = 1.0 + 2.0 * np.abs(c[1:]).sum()
    bands = [c.astype(np.float32)] + [(c[: max(1, lam // 2)] * 1.5).astype(np.float32)] * (
        len(prob.bands) - 1)
    prob = dataclasses.replace(prob, bands=bands)
    ref = O.plan_from_problem(prob)
    plan = gpu_lib.Plan.from_problem(prob, toeplitz_algo=gpu_lib.TOEPLITZ_DIRECT,
                                     precision=gpu_lib.PRECISION_FP64)
    absref = dataclasses.replace(ref, bands=[np.abs(b) for b in ref.bands],
                                 wq=np.abs(ref.wq), wu=np.abs(ref.wu))
    x = np.random.default_rng(lam).standard_normal((ref.n_kept, 3))
    got = plan.apply_A(_dev(x)).cpu().numpy()
    scale = np.linalg.norm(O.apply_A(absref, np.abs(x)))
    assert np.linalg.norm(got - O.apply_A(ref, x)) <= 1e-12 * scale
    b = plan.rhs(_dev(prob.d[0])).cpu().numpy()
    d = np.abs(np.where(prob.pix >= 0, prob.d[0], 0.0))
    assert np.linalg.norm(b - O.rhs(ref, prob.d[0])) <= 1e-12 * np.linalg.norm(O.rhs(absref, d))


@pytest.mark.parametrize("lam", [1, 32])
def test_direct_plans_report_their_product(gpu_lib, lam):
    """mm_plan_info.fused of direct plans: 4 for the fused product, 0 for the three kernels, and 0
    for diagonal weights, which take neither."""
    prob, _ = _problem(3, lam, 0.02, n_dets=2, per_det=5003, interval=2001)
    for flags, fused in ((0, 4), (gpu_lib.FLAG_UNFUSED, 0)):
        plan = gpu_lib.Plan.from_problem(prob, flags=flags)
        assert plan.info["toeplitz_algo"] == gpu_lib.TOEPLITZ_DIRECT
        assert plan.info["fused"] == fused, plan.info
        plan.set_timing(True)
        plan.apply_A(_dev(np.ones((plan.n_kept, 3))))
        # un-pointing, Toeplitz product, pointing: the launches that the flag selects
        assert [plan.kernel_time(k)[1] for k in range(3)] == ([0, 1, 0] if fused else [1, 1, 1])
    diag, _ = _problem(3, 0, 0.02, n_dets=2, per_det=5003, interval=2001)
    assert gpu_lib.Plan.from_problem(diag).info["fused"] == 0


@pytest.mark.parametrize("lam", [8192, 8193, 12000])
def test_lanes_register_noise_weight_short_blocks_and_gaps(gpu_lib, lam):
    """The register transform on blocks shorter than the band, next to samples outside every block
    (copied by the same call) and to blocks of one and several segments at odd starts.  FP32
    transform of 2^15 samples: relative L2 2e-6; samples outside every block exactly."""
    import torch
    n = 90_007
    start = np.array([3, 5_100, 46_007, 46_010, 89_000], np.int64)
    length = np.array([5_001, 40_011, 1, 30_000, 1_006], np.int64)
    prob, _ = _problem(3, lam, 0.0, n_dets=1, per_det=n, interval=n)
    prob = dataclasses.replace(prob, blk_start=start, blk_len=length,
                               blk_band=np.zeros(len(start), np.int32))
    ref = O.plan_from_problem(prob)
    plan = gpu_lib.Plan.from_problem(prob, toeplitz_algo=gpu_lib.TOEPLITZ_FFT, fft_size=32768)
    assert plan.info["fused"] == 2, plan.info
    outside = np.ones(n, bool)
    for s, m in zip(start, length):
        outside[s:s + m] = False
    t = np.random.default_rng(lam).standard_normal(n + 1).astype(np.float32)
    for shift in (0, 1):
        out = torch.full((n + 4,), 7.0, device="cuda")
        ts = t[shift:shift + n]
        u = plan.noise_weight(_dev(t)[shift:shift + n], u=out[1 + shift:1 + shift + n]).cpu().numpy()
        want = O.noise_weight(ts.astype(np.float64), ref)
        assert np.array_equal(u[outside], ts[outside])
        for s, m in zip(start, length):
            assert _rel(u[s:s + m], want[s:s + m]) <= 2e-6
        rest = torch.cat([out[:1 + shift], out[1 + shift + n:]]).cpu().numpy()
        assert np.all(rest == 7.0)


@pytest.mark.parametrize("n,lam", [(65536, 1), (65536, 3), (65536, 12000), (131072, 2),
                                   (131072, 16385)])
def test_lanes_fp64_long_segments(gpu_lib, n, lam):
    """The scatter of long FP64 segments: even and odd bands, and bands so short that the last
    lane's outputs end at the segment's last point."""
    prob, ref = _problem(3, lam, 0.02, n_dets=2, per_det=150013, interval=140011)
    plan = gpu_lib.Plan.from_problem(prob, precision=gpu_lib.PRECISION_FP64,
                                     toeplitz_algo=gpu_lib.TOEPLITZ_FFT, fft_size=n)
    x = np.random.default_rng(lam).standard_normal((ref.n_kept, 3))
    absref = dataclasses.replace(ref, bands=[np.abs(b) for b in ref.bands],
                                 wq=np.abs(ref.wq), wu=np.abs(ref.wu))
    got = plan.apply_A(_dev(x)).cpu().numpy()
    scale = np.linalg.norm(O.apply_A(absref, np.abs(x)))
    assert np.linalg.norm(got - O.apply_A(ref, x)) <= 1e-12 * scale


@pytest.mark.parametrize("lam", [8192, 9001])
def test_register_noise_weight_is_as_accurate_as_the_lds_one(gpu_lib, lam):
    """u = N^-1 t of 2^15-sample segments by the register transform is no further from FP64 than by
    the LDS transform.  Both errors are sums over 2^21 samples, whose ratio scatters by about 0.1 %
    from one draw of rounding errors to another: 0.3 % is allowed for."""
    prob, ref = _problem(8, lam, 0.0, n_dets=8, per_det=1 << 18, interval=1 << 16, side=32)
    t = np.random.default_rng(lam).standard_normal(prob.n_samples).astype(np.float32)
    want = O.noise_weight(t.astype(np.float64), ref, "fft")
    err = []
    for flags, fused in ((0, 2), (gpu_lib.FLAG_LDS_FFT, 1)):
        plan = gpu_lib.Plan.from_problem(prob, flags=flags)
        assert plan.info["fused"] == fused
        err.append(_rel(plan.noise_weight(_dev(t)).cpu().numpy(), want))
    assert err[0] <= 1.003 * err[1], err
