"""The forms of the lag-resolved grid that its plan chooses by size, each shown to be taken.

Against the oracle, in both precisions: a grid whose every point is kept (indices wrap, and a bin's
taps reach round it), also in the registers of the same-time kernel; 1024-point classes with one row
folded, at the largest N_K two of them hold (1.05 (2 N_K - 1) <= 2048) and next to it; bins that are
grid points (one tap); a chunk that is the whole series (a single partial a template).  Tolerances are
the library's stated 1e-10 (FP64) and 1e-4 (split) of max(|rho|, 1)."""

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
    # (detectors, lag, weight, N_K, f_min, T_short, f_band, N_FFT override, segments, chunk),
    # expected (transform length, classes, every point kept, taps) in split precision and in FP64
    "wrap_lag1": ((2, 1, 0, 122, 50.0, 300.0, 0.25, 0, 19, 6), (256, 1, 1, 240), (256, 1, 1, 406)),
    "wrap_lag0": ((3, 0, 0, 122, 50.0, 300.0, 0.25, 0, 37, 7), (256, 1, 1, 240), (256, 1, 1, 406)),
    "wrap_lag0_circ": ((2, 0, 1, 122, 50.0, 300.0, 0.25, 0, 33, 256), (256, 1, 1, 240), (256, 1, 1, 406)),
    "one_fold_975": ((2, 4, 0, 975, 100.0, 1440.0, 0.25, 0, 14, 5), (1024, 2, 0, None), (512, 4, 0, None)),
    "one_fold_870_one_chunk": ((2, 3, 0, 870, 100.0, 1440.0, 0.25, 0, 14, 256), (1024, 2, 0, None), (512, 4, 0, None)),
    "grid_points": ((2, 1, 0, 200, 100.0, 400.0, 0.1, 256, 15, 6), (256, 1, None, 1), (256, 1, None, 1)),
    "same_time_grid_points": ((2, 0, 0, 200, 100.0, 400.0, 0.1, 256, 35, 256), (256, 1, None, 1), (256, 1, None, 1)),
}


@pytest.mark.parametrize("case", sorted(CASES))
def test_planned_form(ccr, case):
    (q, R, weight, n_k, f0, ts, fb, nfft, n_seg, kc), split, fp64 = CASES[case]
    cfg = small_config(q=q, n_seg=n_seg, t_short=ts, f_min=f0, f_band=fb, max_lag=R, a_p_max=1.5, gap_fraction=0.2,
                       n_fft_override=nfft, mu_f=0.02 if nfft else 0.1,
                       templates=dict(a_p=(1.0, 1.5, 2), t_asc=(-200.0, 200.0, 1), period=[68023.70]),
                       injections=[dict(f0=f0 + 0.45 * fb, a_p=1.3, t_asc_off=0.0, period=68023.7, h0=0.3,
                                        cosi=0.7, psi=0.4, phi0=2.0)])
    cfg["n_k"] = n_k
    cfg["band"]["weight"] = weight
    ds = synth.make_dataset(cfg, sigma_wander=0.2)
    ref = oracle.Oracle(ds).rho(ds.templates)
    with ccr.Context(ds.sky, device=0) as ctx:
        ctx.set_option("k_chunk", kc)
        bid = ctx.load(ds)
        for prec, expect in ((ccr.PREC_SPLIT, split), (ccr.PREC_FP64, fp64)):
            print(f"{case} precision {prec}", flush=True)
            r = ctx.compute_rho(bid, prec=prec, out_fp64=prec == ccr.PREC_FP64)
            grid = tuple(ctx.get_option(f"grid_{k}") for k in ("ns", "classes", "wrap", "taps"))
            err = float(np.max(np.abs(r - ref) / np.maximum(np.abs(ref), 1.0)))
            print(f"  grid {grid}, error {err:.2e}, max|rho| {np.abs(ref).max():.2f}", flush=True)
            assert err < (1e-10 if prec == ccr.PREC_FP64 else 1e-4)
            assert all(e is None or g == e for g, e in zip(grid, expect)), (grid, expect)


def test_single_partials_beside_chunks(ccr):
    """Bands of one kernel in one call, the first, the middle and the last with a single chunk (nothing to
    add up) and others with several, give what each gives alone."""
    kw = dict(t_short=400.0, f_min=100.0, f_band=0.1, max_lag=1, a_p_max=2.0)
    dss = [synth.make_dataset(small_config(n_seg=n, seed=n, **kw)) for n in (6, 31, 5, 4, 17, 3)]
    with ccr.Context(dss[0].sky, device=0) as ctx:
        ctx.set_option("k_chunk", 6)
        ids = [ctx.load(ds) for ds in dss]
        for prec in (ccr.PREC_FP64, ccr.PREC_SPLIT):
            print(f"precision {prec}", flush=True)
            together = ctx.compute_rho(ids, prec=prec)
            for i, r, ds in zip(ids, together, dss):
                assert np.array_equal(r, ctx.compute_rho(i, prec=prec))
                if prec == ccr.PREC_FP64:
                    ref = oracle.Oracle(ds).rho(ds.templates)
                    assert float(np.max(np.abs(r - ref) / np.maximum(np.abs(ref), 1.0))) < 1e-10
