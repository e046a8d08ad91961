"""What the sums of the lag-resolved grid keep of the kernels before it, in split precision.

- Products of a segment are summed in FP32, segments in FP64: the sum over all segments is the sum of the
  parts, each with every other segment's weights set to zero, to FP64 rounding; so a template's rho
  (FP32 output) has the same bits alone and in a list, whatever chunks of segments the list gives.
- 256-point bands, Gamma^ave: a pair's weight enters rounded to FP32 once (2^-24), not as products of
  rounded factors.
- Data scaled by a power of two with its noise variance gives the same bits: no weight or product of
  spectra leaves the range of FP32 before rho itself would."""

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


def dataset(n_k, ts=400.0, fb=0.1, weight=0, f_min=100.0, **kw):
    cfg = small_config(t_short=ts, f_min=f_min, f_band=fb, a_p_max=2.0, **kw)
    cfg["n_k"] = n_k
    cfg["band"]["weight"] = weight
    return synth.make_dataset(cfg, sigma_wander=0.2)


LISTS = {
    # (detectors, lag, N_K, T_short): same-time pairs in registers, 256-, 512- and 1024-point classes
    "q2_lag0_nk179": (2, 0, 179, 400.0),
    "q3_lag1_nk179": (3, 1, 179, 400.0),
    "q2_lag3_nk500": (2, 3, 500, 900.0),
    "q2_lag4_nk870": (2, 4, 870, 1440.0),
}


@pytest.mark.parametrize("case", sorted(LISTS))
def test_one_template_alone_and_in_a_list(ccr, case):
    q, R, n_k, ts = LISTS[case]
    ds = dataset(n_k, ts=ts, q=q, n_seg=1500, max_lag=R, gap_fraction=0.2,
                 templates=dict(a_p=(1.0, 2.0, 8), t_asc=(-200.0, 200.0, 8), period=[68023.70]))
    with ccr.Context(ds.sky, device=0) as ctx:
        bid = ctx.load(ds)
        print(case, flush=True)
        many = ctx.compute_rho(bid, prec=ccr.PREC_SPLIT, out_fp64=False)
        assert ctx.get_option("grid_ns") > 0
        for t in (0, 51):
            ctx.set_templates(bid, ds.templates[t:t + 1])
            alone = ctx.compute_rho(bid, prec=ccr.PREC_SPLIT, out_fp64=False)[0]
            differ = int(np.count_nonzero(alone != many[t]))
            assert differ == 0


ADDITIVE = {
    # (detectors, lag, pair kinds, weight, N_K, T_short)
    "q2_lag0_nk500": (2, 0, 1, 0, 500, 900.0),
    "q2_lag1_nk179": (2, 1, 3, 0, 179, 400.0),
    "q3_lag1_nk179_circ": (3, 1, 3, 1, 179, 400.0),
    "q2_lag4_nk870": (2, 4, 3, 0, 870, 1440.0),
    "q3_lag2_nk500_cross": (3, 2, 1, 0, 500, 900.0),
}


@pytest.mark.parametrize("case", sorted(ADDITIVE))
def test_segments_add_in_fp64(ccr, case):
    q, R, pairs, weight, n_k, ts = ADDITIVE[case]
    n_seg = 12
    ds = dataset(n_k, ts=ts, weight=weight, q=q, n_seg=n_seg, max_lag=R, pairs=pairs)
    with ccr.Context(ds.sky, device=0) as ctx:
        bid = ctx.load(ds)

        def total(keep):
            for X in range(q):
                k = np.isin(np.arange(n_seg), keep)
                ctx.set_weights(bid, X, np.where(k, ds.a[X], 0.0), np.where(k, ds.b[X], 0.0), ds.noise_var[X])
            ctx.set_templates(bid, ds.templates)
            norm = ctx.band_info(bid)["norm"]
            return norm * ctx.compute_rho(bid, prec=ccr.PREC_SPLIT) if norm > 0 else 0.0

        print(case, flush=True)
        whole = total(range(n_seg))
        # pairs of later segment K: those of the segments K - R .. K less those of K - R .. K - 1
        parts = 0.0
        for K in range(n_seg):
            parts = parts + total(range(max(0, K - R), K + 1)) - total(range(max(0, K - R), K))
    # FP64 rounding of at most 2 n_seg sums of these magnitudes, and of the interpolation's ~400 taps
    assert np.abs(whole - parts).max() <= 1e-13 * np.abs(whole).max()


def weights_rounded_badly(n_k):
    """(hat a_K, hat a_L) with sigma = 1, b = 0 whose FP32 factors' FP32 product is furthest from the pair
    weight among 20000 draws, and that distance (relative)."""
    rng = np.random.default_rng(3)
    a = rng.uniform(0.5, 1.0, (20000, 2))
    f = (a / np.sqrt(n_k)).astype(np.float32)
    w = a[:, 0] * a[:, 1] / n_k
    e = np.abs((f[:, 0] * f[:, 1]).astype(np.float64) / w - 1.0)
    i = int(np.argmax(e))
    return a[i], float(e[i])


PAIR_WEIGHT = {
    # (detectors, lag, the two (detector, segment) entries of the one pair, N_K); away from the ends,
    # whose segments the Earth's orbit moves out of the data
    "q2_lag0": (2, 0, (0, 4), (1, 4), 179),
    "q3_lag0_first_third": (3, 0, (0, 3), (2, 3), 256),
    "q4_lag0_second_fourth": (4, 0, (1, 4), (3, 4), 100),
    # lags: N_K as planned at 400 Hz (distinct bins), 256- and 512-point classes
    "q1_lag1": (1, 1, (0, 3), (0, 4), 0),
    "q2_lag2": (2, 2, (0, 3), (1, 5), 0),
    "q1_lag4_512_points": (1, 4, (0, 2), (0, 6), 0),
    "q3_lag1_across_only": (3, 1, (0, 3), (2, 4), 0),
}


@pytest.mark.parametrize("case", sorted(PAIR_WEIGHT))
def test_pair_weight_rounded_once(ccr, case):
    """One pair carries all the weight, so the unnormalised sum is its weight times a product of spectra
    that no weight enters: two sets of weights differ by the ratio of the pair weights, up to one rounding
    (2^-24; the reference weight and its factors are powers of two) and, averaged over ~1e4 bins and
    templates, 1e-9 of the products' own rounding."""
    q, R, (X, K), (Y, L), n_k = PAIR_WEIGHT[case]
    n_seg = 9
    ds = dataset(n_k, fb=0.02 if "512" in case else (0.05 if n_k < 150 else 0.1), f_min=100.0 if n_k else 400.0, q=q, n_seg=n_seg, max_lag=R,
                 pairs=2 if q == 1 else (1 if case.endswith("only") else 3),
                 templates=dict(a_p=(1.0, 2.0, 16), t_asc=(-900.0, 900.0, 16), period=[68023.70]))
    n_k = ds.n_k
    bad, off = weights_rounded_badly(n_k)
    assert off > 1.1e-7
    with ccr.Context(ds.sky, device=0) as ctx:
        bid = ctx.load(ds)

        def unnormalised(ak, al):
            a = np.zeros((q, n_seg))
            a[X, K], a[Y, L] = ak, al
            for d in range(q):
                ctx.set_weights(bid, d, a[d], np.zeros(n_seg), np.ones(n_seg))
            ctx.set_templates(bid, ds.templates)
            return ctx.band_info(bid)["norm"] * ctx.compute_rho(bid, prec=ccr.PREC_SPLIT)

        print(case, flush=True)
        s_ref = unnormalised(np.sqrt(n_k) / 16.0, np.sqrt(n_k) / 16.0)
        s_bad = unnormalised(bad[0], bad[1])
        assert ctx.get_option("grid_ns") == (512 if "512" in case else 256)
    ratio = float((s_bad * s_ref).sum() / (s_ref * s_ref).sum()) / (bad[0] * bad[1] / n_k * 256.0) - 1.0
    print(f"  pair weight off by {ratio:.2e}, products of rounded factors by {off:.2e}", flush=True)
    assert abs(ratio) <= 2.0**-24 + 2e-9


SCALED = {"lag0_circ": (0, 1), "lag0_ave": (0, 0), "lag1_ave": (1, 0), "lag1_circ": (1, 1)}


@pytest.mark.parametrize("case", sorted(SCALED))
@pytest.mark.parametrize("q", [2, 3, 5])
def test_power_of_two_scaled_data(ccr, case, q):
    R, weight = SCALED[case]
    ds = dataset(179, weight=weight, q=q, n_seg=20, max_lag=R, gap_fraction=0.2)
    with ccr.Context(ds.sky, device=0) as ctx:
        out = []
        for e in (0, -40, 40):
            print(case, q, e, flush=True)
            bid = ctx.load(ds)
            for X in range(q):
                ctx.set_data(bid, X, ds.sites[X], ds.t0, ds.dt, ds.x[X] * np.float32(2.0**e), ds.f_het, ds.valid[X])
                ctx.set_weights(bid, X, ds.a[X], ds.b[X], ds.noise_var[X] * 2.0**(2 * e))
            ctx.set_templates(bid, ds.templates)
            out.append(ctx.compute_rho(bid, prec=ccr.PREC_SPLIT))
    assert np.abs(out[0]).max() > 1.0
    differ = [int(np.count_nonzero(out[0] != o)) for o in out[1:]]
    assert differ == [0, 0]


@pytest.mark.parametrize("weight", [0, 1])
def test_detectors_add_in_fp64_at_lag_0(ccr, weight):
    """One segment's weight, output bins that are grid points, pairs at lag 0 only: the unnormalised sum is
    the FP64 sum of the FP32 products of detectors 1 and 2 with those before them, so most values need
    more than 24 bits (a sum in FP32 would need 24 in every bin)."""
    q, n_k, n_seg = 3, 500, 7
    ds = dataset(n_k, ts=900.0, fb=0.1, weight=weight, q=q, n_seg=n_seg, max_lag=0, mu_f=0.02, n_fft_override=512)
    with ccr.Context(ds.sky, device=0) as ctx:
        bid = ctx.load(ds)
        for X in range(q):
            only = np.arange(n_seg) == 3
            ctx.set_weights(bid, X, np.where(only, ds.a[X], 0.0), np.where(only, ds.b[X], 0.0), ds.noise_var[X])
        ctx.set_templates(bid, ds.templates)
        s = ctx.compute_rho(bid, prec=ccr.PREC_SPLIT) * (ctx.band_info(bid)["norm"] / np.sqrt(2.0))
        assert (ctx.get_option("grid_ns"), ctx.get_option("grid_taps")) == (512, 1)
    # within FP64 rounding of the normalisation of a 24-bit number
    short = np.abs(s.astype(np.float32).astype(np.float64) / s - 1.0) < 1e-14
    print(f"weight {weight}: {short.mean():.2f} of {s.size} sums have 24 bits", flush=True)
    assert short.mean() < 0.5
