"""Same-time pair sums of 256-point grids (spectra held in registers) against the oracle.

The kernel's forms follow from N_K (8, 12 or 16 input rows of 16 samples), the kept outputs (6 or 16
a lane) and the detectors (2, 3, or a loop), so N_K sits at and next to 128, 192 and 256, bands are
narrow and wide, and segment lists end inside a wavefront's four, a workgroup's sixteen and a chunk.
A split result is within 1e-4 of max(|rho|, 1), the library's stated accuracy."""

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
    # (detectors, pair kinds, weight, N_K, T_short, f_band, segments, k_chunk, gaps)
    "q2_nk127": (2, 3, 0, 127, 400.0, 0.05, 37, 256, 0.2),
    "q2_nk128_circ": (2, 1, 1, 128, 400.0, 0.05, 16, 256, 0.0),
    "q2_nk129": (2, 3, 0, 129, 400.0, 0.1, 5, 256, 0.0),
    "q2_nk192": (2, 3, 0, 192, 400.0, 0.1, 50, 17, 0.3),
    "q3_nk193": (3, 3, 0, 193, 400.0, 0.1, 33, 20, 0.3),
    "q3_nk256_wide": (3, 1, 0, 256, 400.0, 0.3, 21, 1, 0.2),
    "q3_nk160_circ": (3, 3, 1, 160, 400.0, 0.2, 70, 256, 0.3),
    "q4_nk131": (4, 3, 0, 131, 400.0, 0.1, 19, 6, 0.3),
    "q5_nk250_circ": (5, 1, 1, 250, 400.0, 0.3, 17, 256, 0.3),
    "q2_one_segment": (2, 3, 0, 150, 400.0, 0.1, 1, 256, 0.0),
    "q2_within_only": (2, 2, 0, 150, 400.0, 0.1, 9, 4, 0.0),
}


@pytest.mark.parametrize("case", sorted(CASES))
def test_same_time(ccr, case):
    q, pairs, weight, n_k, ts, fb, n_seg, kc, gaps = CASES[case]
    cfg = small_config(q=q, n_seg=n_seg, t_short=ts, f_min=100.0, f_band=fb, max_lag=0, pairs=pairs, a_p_max=2.0,
                       gap_fraction=gaps, templates=dict(a_p=(1.0, 2.0, 2), t_asc=(-200.0, 200.0, 1), period=[68023.70]),
                       injections=[dict(f0=100.0 + 0.45 * fb, a_p=1.3, t_asc_off=0.0, period=68023.7, h0=0.3,
                                        cosi=0.7, psi=0.4, phi0=2.0)])
    cfg["n_k"] = n_k
    cfg["band"]["weight"] = weight
    ds = synth.make_dataset(cfg, sigma_wander=0.2)
    ref = oracle.Oracle(ds).rho(ds.templates)
    with ccr.Context(ds.sky, device=0) as ctx:
        ctx.set_option("k_chunk", kc)
        bid = ctx.load(ds)
        info = ctx.band_info(bid)
        print(f"{case} N_K {info['n_k']} N_FFT {info['n_fft']} bins {info['n_f']}", flush=True)
        r = ctx.compute_rho(bid, prec=ccr.PREC_SPLIT)
        e = float(np.max(np.abs(r - ref) / np.maximum(np.abs(ref), 1.0)))
        grid = ctx.get_option("grid_ns"), ctx.get_option("grid_classes")
        print(f"  grid {grid[0]} x {grid[1]}, error {e:.2e}, max|rho| {np.abs(ref).max():.2f}", flush=True)
        assert grid[0] == 256
        assert e < 1e-4
