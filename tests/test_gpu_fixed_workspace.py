"""The call without allocations against the ordinary one at the limits of its fixed device array.

Both entry points take the same kernels, chunks and summation order for the same options, so FP64 rho
(and split rho: the same launches) is bitwise equal also where the grid's chunk partials or the folded
series of every ordered pair would not fit the array."""

import numpy as np
import pytest

import synth
from conftest import small_config

pytestmark = pytest.mark.gpu

ARRAY = 255 << 20  # workspace bytes of the fixed array


@pytest.fixture(scope="module")
def ccr():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1712_06515_amd import ccr as mod
    mod.load_library()
    return mod


def both(ccr, ctx, bid, prec):
    import torch
    fp64 = prec == ccr.PREC_FP64
    info = ctx.band_info(bid)
    ref = ctx.compute_rho(bid, prec=prec, out_fp64=fp64)
    out = torch.full((info["n_templates"], info["n_f"]), float("nan"), dtype=torch.float64 if fp64 else torch.float32,
                     device="cuda")
    torch.cuda.synchronize()
    ctx.compute_rho_noalloc(bid, [out.data_ptr()], prec=prec, out_fp64=fp64)
    ctx.sync()
    return out.cpu().numpy(), ref


def test_chunk_partials_over_the_array(ccr):
    """Pairs across four detectors at lags up to 4 with chunks of one segment: 6 detector pairs x 9
    sums x 16000 chunks of grid partials exceed the array, the spectra at the output bins do not."""
    cfg = small_config(q=4, n_seg=16000, f_band=0.02, max_lag=4, pairs=1, gap_fraction=0.1,
                       templates=dict(a_p=(1.0, 1.4, 2), t_asc=(0.0, 0.0, 1), period=[68023.70]))
    ds = synth.make_dataset(cfg)
    with ccr.Context(ds.sky, device=0) as ctx:
        ctx.set_option("k_chunk", 1)
        bid = ctx.load(ds)
        info = ctx.band_info(bid)
        assert 16 * 4 * 16000 * (info["n_k"] + info["n_f"]) < ARRAY
        for prec in (ccr.PREC_FP64, ccr.PREC_SPLIT):
            print(f"chunks of one segment, precision {prec}", flush=True)
            got, ref = both(ccr, ctx, bid, prec)
            assert np.all(np.isfinite(ref)) and np.abs(ref).max() > 0.5
            same = np.array_equal(got, ref)
            assert same


def test_folded_series_over_the_array(ccr):
    """Every ordered pair with N_FFT = 2^20: one template's series (223 MiB) leaves no room for its
    folded form (32 MiB), while its spectra at the output bins fit."""
    cfg = small_config(q=2, n_seg=28500, t_short=120.0, f_band=0.08, max_lag=0, pairs=4, n_fft_override=1 << 20,
                       templates=dict(a_p=(1.0, 1.0, 1), t_asc=(0.0, 0.0, 1), period=[68023.70]))
    cfg["n_k"] = 256
    ds = synth.make_dataset(cfg, signal=False)
    with ccr.Context(ds.sky, device=0) as ctx:
        bid = ctx.load(ds)
        info = ctx.band_info(bid)
        series = 16 * 2 * 28500 * 256
        assert series + 16 * 2 * 28500 * info["n_f"] + (8 << 20) < ARRAY < series + 32 * info["n_fft"] + (2 << 20)
        print(f"folded series, {info['n_f']} bins", flush=True)
        got, ref = both(ccr, ctx, bid, ccr.PREC_FP64)
        assert np.all(np.isfinite(ref)) and np.abs(ref).max() > 0.5
        same = np.array_equal(got, ref)
        assert same
