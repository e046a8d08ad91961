"""What a context reports about its last call."""

import numpy as np
import pytest

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


def test_grid_after_replay(ccr):
    """grid_ns and grid_classes name the last call's grid also when that call replayed a graph."""
    import torch
    a = synth.make_dataset(small_config(n_seg=12, t_short=400.0, f_min=100.0, f_band=0.1, max_lag=1))
    b = synth.make_dataset(small_config(n_seg=9, t_short=1440.0, f_min=399.875, f_band=0.25, max_lag=4, a_p_max=2.0))
    with ccr.Context(a.sky, device=0) as ctx:
        ids = [ctx.load(a), ctx.load(b)]
        outs = [torch.empty((ctx.band_info(i)["n_templates"], ctx.band_info(i)["n_f"]), dtype=torch.float32, device="cuda")
                for i in ids]
        ctx.set_option("graph", 1)
        grids = {}
        for rep in range(3):
            for k in (0, 1):
                ctx.compute_rho(ids[k], prec=ccr.PREC_SPLIT, out_fp64=False, outputs=[outs[k].data_ptr()])
                ctx.sync()
                g = ctx.get_option("grid_ns"), ctx.get_option("grid_classes")
                assert grids.setdefault(k, g) == g
        assert grids[0][0] == 256 and grids[1][0] == 1024
        # the stage outputs plan a call of their own, which is no compute call
        ctx.resample_series(ids[0], 0, 0, prec=ccr.PREC_SPLIT)
        assert (ctx.get_option("grid_ns"), ctx.get_option("grid_classes")) == grids[1]
        # fused: not on the grid
        ctx.set_option("graph", 0)
        ctx.set_option("fused", 1)
        ctx.set_option("timing", 1)
        ctx.compute_rho(ids[0], prec=ccr.PREC_SPLIT)
        assert ctx.kernel_times()["fused"][1] > 0
        assert ctx.get_option("grid_ns") == 0 and ctx.get_option("grid_classes") == 0


def test_time_slots_of_bands_sharing_a_kernel(ccr):
    """Slot 6 counts 256-point bands with the Gamma^ave weight that the 256-point kernel of higher lags
    holds (up to 4 detectors), slot 7 every other band, also where one call's bands run on the same grid
    kernel."""
    kw = dict(n_seg=12, t_short=400.0, f_min=400.0, f_band=0.06, max_lag=1, a_p_max=2.0)
    dss = [synth.make_dataset(small_config(q=q, **kw)) for q in (2, 5)]
    with ccr.Context(dss[0].sky, device=0) as ctx:
        ctx.set_option("timing", 1)
        ids = [ctx.load(ds) for ds in dss]
        alone, grids = [], []
        for i in ids:
            ctx.kernel_times(reset=True)
            ctx.compute_rho(i, prec=ccr.PREC_SPLIT)
            kt = ctx.kernel_times(reset=True)
            alone.append((kt["spectra_pairs"][1], kt["spectra_wide"][1]))
            grids.append((ctx.get_option("grid_ns"), ctx.get_option("grid_classes")))
        assert alone == [(1, 0), (0, 1)] and grids[0] == grids[1] and grids[0][0] == 256
        for order in (ids, ids[::-1]):
            ctx.kernel_times(reset=True)
            ctx.compute_rho(order, prec=ccr.PREC_SPLIT)
            kt = ctx.kernel_times(reset=True)
            assert kt["spectra_pairs"][1] == 1 and kt["spectra_wide"][1] == 1, kt


def test_tuner_tries_the_bands_own_chunks(ccr):
    """Few templates of a short series: the untuned call takes chunks of 16 segments, below every
    length of the tuner's ladder, so the tuner times that shape too and reports when it keeps it."""
    ds = synth.make_dataset(small_config(n_seg=480, t_short=360.0, f_min=99.875, f_band=0.25, max_lag=1))
    with ccr.Context(ds.sky, device=0) as ctx:
        bid = ctx.load(ds, templates=ds.templates[:1])
        base = ctx.compute_rho(bid, prec=ccr.PREC_FP64)
        assert ctx.get_option("tuned_own_chunks") == 0
        ctx.set_option("autotune", 1)
        tuned = ctx.compute_rho(bid, prec=ccr.PREC_FP64)
        assert ctx.get_option("tuned_k_chunk") in (32, 64, 128, 256, 512, 1024)
        assert np.max(np.abs(tuned - base)) < 1e-12 * max(1.0, np.abs(base).max())
        # 16-segment chunks against the shortest of the ladder: twice the workgroups, half the steps a
        # workgroup, on a GPU that neither fills
        assert ctx.get_option("tuned_own_chunks") == 1
        assert np.array_equal(tuned, base)
