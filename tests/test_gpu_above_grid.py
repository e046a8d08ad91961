"""Split-precision kernels for lags above the lag-resolved grid's (4 segments): the 256-point and the
256- to 1024-point spectra + pair-sum kernels and the resampler's two weighted series, at lags 5 and
6, against the oracle (split 1e-4, FP64 1e-10 of max(|rho|, 1)).  Each case states the kernel that has to
run: the grid reports transform length 0, and the slot of the kernel counts the launches.

The cases follow the forms: 1 to 4 detectors (segments a step, wavefronts a workgroup), pairs within,
across and both, runs of empty segments longer and shorter than the lag, chunks shorter than the lag
with their halo and chunks longer than the series, last steps that are part filled, classes of more
than 256 bins (eight columns a lane), both weights, and per-sample antenna functions with every
node rule of the time base that the bands reach."""

import numpy as np
import pytest

import oracle
import synth
from conftest import small_config

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ccr():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1712_06515_amd import ccr as mod
    mod.load_library()
    return mod


CASES = {
    # (kernel slot, segment FFT, detectors, lag, pair kinds, weight, per-sample, T_short, f_band, segments,
    #  chunk, gaps)
    "sp_q1_lag5_same": ("spectra_pairs", 256, 1, 5, 2, 0, False, 400.0, 0.05, 23, 256, 0.2),
    "sp_q2_lag6_both": ("spectra_pairs", 256, 2, 6, 3, 0, False, 400.0, 0.02, 23, 4, 0.2),
    "sp_q2_lag5_cross": ("spectra_pairs", 256, 2, 5, 1, 0, False, 400.0, 0.03, 30, 256, 0.4),
    "sp_q3_lag5_both": ("spectra_pairs", 256, 3, 5, 3, 0, False, 400.0, 0.03, 23, 7, 0.2),
    "sp_q4_lag5_both": ("spectra_pairs", 256, 4, 5, 3, 0, False, 400.0, 0.02, 21, 256, 0.2),
    "wide256_q3_lag5_circ": ("spectra_wide", 256, 3, 5, 3, 1, False, 400.0, 0.04, 26, 5, 0.3),
    "wide256_q2_lag6_many_bins": ("spectra_wide", 256, 2, 6, 3, 0, False, 400.0, 0.1, 26, 256, 0.3),
    "wide512_q2_lag5_both": ("spectra_wide", 512, 2, 5, 3, 0, False, 1000.0, 0.06, 26, 7, 0.3),
    "wide512_q4_lag5_circ": ("spectra_wide", 512, 4, 5, 3, 1, False, 1000.0, 0.04, 24, 6, 0.3),
    "wide1024_q1_lag6_same": ("spectra_wide", 1024, 1, 6, 2, 0, False, 2000.0, 0.06, 30, 7, 0.3),
    "wide1024_q2_lag5_both": ("spectra_wide", 1024, 2, 5, 3, 0, False, 2000.0, 0.06, 30, 3, 0.4),
    "wide1024_q3_lag5_cross": ("spectra_wide", 1024, 3, 5, 1, 1, False, 2000.0, 0.04, 22, 256, 0.2),
    "wide1024_q1_wide_classes": ("spectra_wide", 1024, 1, 5, 2, 0, False, 1000.0, 0.3, 26, 7, 0.3),
    "ps256_q2_lag5": ("spectra_wide", 256, 2, 5, 3, 0, True, 400.0, 0.04, 23, 5, 0.2),
    "ps256_q4_lag5_cross": ("spectra_wide", 256, 4, 5, 1, 1, True, 400.0, 0.02, 20, 256, 0.2),
    "ps1024_q2_lag6": ("spectra_wide", 1024, 2, 6, 3, 0, True, 2000.0, 0.05, 26, 4, 0.3),
    "ps1024_q1_lag5_circ": ("spectra_wide", 1024, 1, 5, 2, 1, True, 2000.0, 0.06, 26, 256, 0.2),
}


@pytest.mark.parametrize("case", sorted(CASES))
def test_lags_above_the_grid(ccr, case):
    slot, ns, q, R, pairs, weight, ps, ts, fb, n_seg, kc, gaps = CASES[case]
    cfg = small_config(q=q, n_seg=n_seg, t_short=ts, f_min=400.0, f_band=fb, max_lag=R, pairs=pairs, a_p_max=2.0,
                       gap_fraction=gaps,
                       templates=dict(a_p=(1.0, 2.0, 2), t_asc=(-200.0, 200.0, 2), period=[68023.70]),
                       injections=[dict(f0=400.0 + 0.45 * fb, a_p=1.3, t_asc_off=0.0, period=68023.7, h0=0.3,
                                        cosi=0.7, psi=0.4, phi0=2.0)])
    cfg["band"]["weight"] = weight
    ds = synth.make_dataset(cfg, sigma_wander=0.2, per_sample_antenna=ps)
    ref = oracle.Oracle(ds).rho(ds.templates)
    err = lambda r: float(np.max(np.abs(r - ref) / np.maximum(np.abs(ref), 1.0)))
    with ccr.Context(ds.sky, device=0) as ctx:
        ctx.set_option("timing", 1)
        ctx.set_option("k_chunk", kc)
        bid = ctx.load(ds)
        info = ctx.band_info(bid)
        print(f"{case} N_K {info['n_k']} N_FFT {info['n_fft']} n_s {info['n_s']} bins {info['n_f']}", flush=True)
        assert info["n_s"] == ns, info
        ctx.kernel_times(reset=True)
        r32 = ctx.compute_rho(bid, prec=ccr.PREC_SPLIT, out_fp64=False)
        kt = ctx.kernel_times(reset=True)
        assert ctx.get_option("grid_ns") == 0
        assert {k for k in ("spectra", "pairs", "spectra_pairs", "spectra_wide") if kt[k][1]} == {slot}, kt
        ctx.set_option("template_batch", 1)
        r32b = ctx.compute_rho(bid, prec=ccr.PREC_SPLIT, out_fp64=False)
        r64 = ctx.compute_rho(bid, prec=ccr.PREC_FP64)
        if slot == "spectra_pairs":  # the other kernel takes these bands too
            ctx.set_option("spectra_kernel", 1)
            ctx.kernel_times(reset=True)
            other = ctx.compute_rho(bid, prec=ccr.PREC_SPLIT, out_fp64=False)
            kt = ctx.kernel_times(reset=True)
            assert kt["spectra_wide"][1] > 0 and kt["spectra_pairs"][1] == 0 and kt["spectra"][1] == 0, kt
            assert err(other) < 1e-4
    print(f"  split {err(r32):.2e} fp64 {err(r64):.2e} max|rho| {np.abs(ref).max():.2f}", flush=True)
    assert err(r32) < 1e-4 and err(r64) < 1e-10
    assert np.array_equal(r32, r32b)


@pytest.mark.parametrize("q,pairs", [(1, 2), (2, 3)])
def test_one_template_alone_and_in_a_list(ccr, q, pairs):
    """The 256-point kernel sums the pair terms of up to 4 / Q segments in FP32; which segments share a
    sum follows from where chunks start, so the chunks do not depend on the number of templates."""
    cfg = small_config(q=q, n_seg=1500, t_short=400.0, f_min=400.0, f_band=0.03, max_lag=5, pairs=pairs, a_p_max=2.0,
                       gap_fraction=0.2, templates=dict(a_p=(1.0, 2.0, 16), t_asc=(-200.0, 200.0, 16), period=[68023.70]))
    ds = synth.make_dataset(cfg)
    with ccr.Context(ds.sky, device=0) as ctx:
        ctx.set_option("timing", 1)
        bid = ctx.load(ds)
        many = ctx.compute_rho(bid, prec=ccr.PREC_SPLIT)
        assert ctx.kernel_times()["spectra_pairs"][1] > 0 and ctx.get_option("grid_ns") == 0
        for t in (0, 200):
            ctx.set_templates(bid, ds.templates[t:t + 1])
            alone = ctx.compute_rho(bid, prec=ccr.PREC_SPLIT)[0]
            differ = int(np.count_nonzero(alone != many[t]))
            assert differ == 0
