"""FP64 resampling of the default interpolation (8 taps each side, tap-indexed window) against the
oracle: one workgroup stages a segment for up to four templates and shares its 64-sample passes
among four wavefronts, so the cases are template counts around the tile, N_K around a pass and
at its largest, gaps and a series whose first and last windows leave the data.  Tolerance: the
library's FP64 bound, 1e-10 of max(|rho|, 1).  Templates whose delays differ by more samples than
the staged window holds (every sample then reads its taps from global memory) are compared with
the same templates one at a time, which the window holds: the two paths share the time base and
differ in the rounding of the interpolation, a few 1e-16 a sample, so 1e-12 of max(|rho|, 1)."""

import numpy as np
import pytest

import oracle
import synth
from conftest import small_config

pytestmark = pytest.mark.gpu
P0 = 68023.70


@pytest.fixture(scope="module")
def ccr():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1712_06515_amd import ccr as mod
    mod.load_library()
    return mod


CASES = {
    # (N_K or 0, T_short, f_band, segments, templates, largest a_p of the templates)
    "one_template": (0, 120.0, 0.4, 6, 1, 1.5),
    "nk128_five": (128, 120.0, 0.4, 6, 5, 1.5),
    "nk129_four": (129, 120.0, 0.4, 6, 4, 1.5),
    "nk2048_three": (2048, 1500.0, 0.3, 3, 3, 1.5),
}


@pytest.mark.parametrize("case", sorted(CASES))
def test_resample64(ccr, case):
    n_k, ts, fb, n_seg, n_t, ap = CASES[case]
    cfg = small_config(q=2, n_seg=n_seg, t_short=ts, f_band=fb, gap_fraction=0.2)
    if n_k:
        cfg["n_k"] = n_k
    ds = synth.make_dataset(cfg)
    i = np.arange(n_t)
    ds.templates = np.stack([ap * (i + 1) / n_t, 5000.0 + P0 * (0.25 + 0.5 * (i % 2)), np.full(n_t, P0)], axis=1)
    ref = oracle.Oracle(ds).rho(ds.templates)
    with ccr.Context(ds.sky, device=0) as ctx:
        bid = ctx.load(ds)
        r = ctx.compute_rho(bid, prec=ccr.PREC_FP64)
        err = float(np.max(np.abs(r - ref) / np.maximum(np.abs(ref), 1.0)))
        print(f"{case}: error {err:.2e}, max|rho| {np.abs(ref).max():.2f}", flush=True)
        assert np.any(ref != 0.0)
        assert err < 1e-10


def test_resample64_wide_delays(ccr):
    cfg = small_config(q=2, n_seg=30, t_short=240.0, f_band=0.3, gap_fraction=0.2)
    cfg["n_k"] = 256
    ds = synth.make_dataset(cfg)
    i = np.arange(6)
    ds.templates = np.stack([250.0 * (i + 1), 5000.0 + P0 * (0.25 + 0.5 * (i % 2)), np.full(6, P0)], axis=1)
    with ccr.Context(ds.sky, device=0) as ctx:
        bid = ctx.load(ds)
        together = ctx.compute_rho(bid, prec=ccr.PREC_FP64)
        ctx.set_option("template_batch", 1)
        alone = ctx.compute_rho(bid, prec=ccr.PREC_FP64)
    assert np.abs(alone).max() > 1.0
    assert np.max(np.abs(together - alone) / np.maximum(np.abs(alone), 1.0)) < 1e-12
