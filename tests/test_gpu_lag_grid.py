"""Spectra and pair sums on the lag-resolved frequency grid, and every ordered pair from the folded
series, against the oracle.

The kernel's transform length, number of classes, folded rows, kept columns and interpolation
taps follow from N_K, the band and the lag, so the cases sit at the edges of those choices: N_K
at and just past 256, 512 and 1024 samples, 2048 (four and two folded rows), a band that fills the
grid (indices wrap), output bins that are grid points (one tap), repeated output bins; chunks
shorter than a step of four segments, than the lag and than the series; pairs within one
detector (one problem a detector) and across detectors only (one problem a pair), both weights,
per-sample antenna functions, up to 5 detectors, gaps.  Tolerances are the library's stated
1e-10 (FP64) and 1e-4 (split) of max(|rho|, 1)."""

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
    # (detectors, max lag, pair kinds, weight, per-sample, N_K, T_short, f_band, segments, k_chunk, gaps)
    "nk256_lag1": (2, 1, 3, 0, False, 256, 400.0, 0.1, 21, 5, 0.2),
    "nk257_lag2": (2, 2, 3, 0, False, 257, 400.0, 0.1, 18, 7, 0.2),
    "nk512_lag3": (2, 3, 3, 0, False, 512, 900.0, 0.1, 18, 1, 0.1),
    "nk513_lag4": (2, 4, 3, 0, False, 513, 900.0, 0.1, 18, 3, 0.2),
    "nk1024_lag4": (2, 4, 3, 0, False, 1024, 1500.0, 0.2, 14, 256, 0.1),
    "nk1025_lag1": (2, 1, 3, 1, False, 1025, 1500.0, 0.2, 13, 4, 0.1),
    "nk2048_lag2": (2, 2, 3, 0, False, 2048, 1700.0, 0.3, 9, 6, 0.0),
    "wrap_lag1": (2, 1, 3, 0, False, 0, 400.0, 0.45, 17, 6, 0.2),
    "lag0_circ": (3, 0, 3, 1, False, 300, 400.0, 0.2, 15, 4, 0.2),
    "same_q3": (3, 3, 2, 0, False, 0, 900.0, 0.2, 19, 6, 0.3),
    "cross_q2": (2, 3, 1, 0, False, 0, 900.0, 0.2, 19, 5, 0.3),
    "cross_q4_circ": (4, 2, 1, 1, False, 0, 1500.0, 0.3, 11, 4, 0.2),
    "both_q5": (5, 1, 3, 0, False, 0, 400.0, 0.2, 13, 6, 0.2),
    "ps_q3_lag1": (3, 1, 3, 0, True, 0, 1500.0, 0.3, 11, 5, 0.2),
    "ps_cross_q3_circ": (3, 2, 1, 1, True, 300, 400.0, 0.1, 15, 5, 0.2),
    "ps_same_q2_lag4": (2, 4, 2, 0, True, 700, 900.0, 0.2, 17, 8, 0.2),
    "ps_lag0": (2, 0, 1, 1, True, 1100, 1500.0, 0.2, 10, 3, 0.2),
    # every ordered pair: series folded onto N_FFT samples many times, less than once, on 2048-point
    # classes, with both weightings of several detectors
    "all_fold_many": (2, 0, 4, 0, False, 0, 400.0, 0.1, 60, 256, 0.2),
    "all_fold_less_than_once": (2, 4, 4, 0, False, 0, 400.0, 0.1, 3, 256, 0.0),
    "all_nk1100_circ": (2, 1, 4, 1, False, 1100, 1500.0, 0.2, 9, 256, 0.2),
    "all_ps_q3_circ": (3, 1, 4, 1, True, 300, 400.0, 0.1, 15, 256, 0.2),
    "mu_repeated_bins": (2, 1, 3, 0, False, 200, 400.0, 0.1, 15, 6, 0.2),
}


@pytest.mark.parametrize("case", sorted(CASES))
def test_lag_grid(ccr, case):
    q, R, pairs, weight, ps, n_k, ts, fb, n_seg, kc, gaps = CASES[case]
    cfg = small_config(q=q, n_seg=n_seg, t_short=ts, f_min=100.0, f_band=fb, max_lag=R, pairs=pairs, a_p_max=2.0,
                       gap_fraction=gaps, mu_f=0.02 if case.startswith("mu_") else 0.1,
                       n_fft_override=256 if case.startswith("mu_") else 0,
                       templates=dict(a_p=(1.0, 2.0, 2), t_asc=(-200.0, 200.0, 1), period=[68023.70]),
                       injections=[dict(f0=100.0 + 0.45 * fb, a_p=1.3, t_asc_off=0.0, period=68023.7, h0=0.3,
                                        cosi=0.7, psi=0.4, phi0=2.0)])
    if n_k:
        cfg["n_k"] = n_k
    cfg["band"]["weight"] = weight
    ds = synth.make_dataset(cfg, sigma_wander=0.2, per_sample_antenna=ps)
    ref = oracle.Oracle(ds).rho(ds.templates)
    err = lambda r: float(np.max(np.abs(r - ref) / np.maximum(np.abs(ref), 1.0)))
    with ccr.Context(ds.sky, device=0) as ctx:
        ctx.set_option("timing", 1)
        ctx.set_option("k_chunk", kc)
        bid = ctx.load(ds)
        info = ctx.band_info(bid)
        for prec in (ccr.PREC_SPLIT, ccr.PREC_FP64):
            print(f"{case} prec {prec} N_K {info['n_k']} N_FFT {info['n_fft']} bins {info['n_f']}", flush=True)
            ctx.kernel_times(reset=True)
            r = ctx.compute_rho(bid, prec=prec, out_fp64=prec == ccr.PREC_FP64)
            kt = ctx.kernel_times(reset=True)
            e = err(r)
            print(f"  error {e:.2e}, max|rho| {np.abs(ref).max():.2f}", flush=True)
            assert kt["spectra"][1] == 0 and kt["pairs"][1] == 0, kt  # not the general path
            assert e < (1e-10 if prec == ccr.PREC_FP64 else 1e-4)


def test_fixed_workspace_limit(ccr):
    """The call without allocations refuses the same bands whichever kernel they would take: 14 days
    in FP64 with 7413 bins, whose spectra (2 x 840 x 7413 complex, 199 MB) and series (23 MB) fit
    one template's fixed workspace, are taken, 21 days (298 MB and 35 MB) are not."""
    import torch
    for n_seg, fits in ((840, True), (1260, False)):
        cfg = small_config(q=2, n_seg=n_seg, t_short=1440.0, f_min=399.875, f_band=0.25, max_lag=4, pairs=3, a_p_max=2.0,
                           gap_fraction=0.0, templates=dict(a_p=(1.0, 1.0, 1), t_asc=(0.0, 0.0, 1), period=[68023.70]),
                           injections=[])
        ds = synth.make_dataset(cfg)
        with ccr.Context(ds.sky, device=0) as ctx:
            bid = ctx.load(ds)
            info = ctx.band_info(bid)
            need = 16 * 2 * n_seg * (info["n_f"] + info["n_k"])
            assert (need < 240 << 20) == fits and (need > 260 << 20) == (not fits), need
            out = torch.zeros((len(ds.templates), info["n_f"]), dtype=torch.float64, device="cuda")
            if fits:
                ctx.compute_rho_noalloc(bid, prec=ccr.PREC_FP64, out_fp64=True, outputs=[out.data_ptr()])
                torch.cuda.synchronize()
                ref = ctx.compute_rho(bid, prec=ccr.PREC_FP64, out_fp64=True)
                # the same kernels with other chunks: FP64 sums in another order
                assert float(np.max(np.abs(out.cpu().numpy() - ref))) < 1e-10 * max(1.0, float(np.abs(ref).max()))
            else:
                with pytest.raises(ccr.CcrError):
                    ctx.compute_rho_noalloc(bid, prec=ccr.PREC_FP64, out_fp64=True, outputs=[out.data_ptr()])
