"""Roots of unity of the SFT front end, and its largest tiles.

Two bins half the transform apart cancel at every odd output, w^(l j) + w^((l + N'/2) j) = 0, so what is
left there is the rounding of the two roots, which the FP32 output shows in full.  A root rounded to
FP64 is off by at most 2^-54 in each component, two of them by an rms of at most 2^-54 sqrt(4) = 2^-53;
roots taken from angles rounded to FP64 (2 m / N' below 2: up to 2^-53 of a half turn) have twice that."""

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ccr():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1712_06515_amd import ccr as mod
    mod.load_library()
    return mod


@pytest.mark.parametrize("n_out", [122, 870, 1802, 3042])
def test_opposite_roots_cancel(ccr, n_out):
    n_sft = 64
    t_sft, f_het = 1024.0, 100.0
    k_first = int(f_het * t_sft) - n_out // 2
    z = np.zeros((n_sft, n_out), dtype=np.complex64)
    m = (np.arange(n_sft) * (n_out // 2)) // n_sft
    z[np.arange(n_sft), m] = 1.0
    z[np.arange(n_sft), m + n_out // 2] = 1.0
    from synth import default_sky
    with ccr.Context(default_sky(), device=0) as ctx:
        x, _ = ctx.sft_series(z, t_sft, 0.0, k_first, f_het, n_out)
    x = x.reshape(n_sft, n_out).astype(np.complex128) * t_sft
    rms = float(np.sqrt(np.mean(np.abs(x[:, 1::2]) ** 2)))
    print(f"{n_out} outputs: what is left of two cancelling roots {rms:.2e} rms, even outputs {np.abs(x[:, 0::2]).mean():.3f}")
    assert np.abs(np.abs(x[:, 0::2]) - 2.0).max() < 1e-6
    assert rms <= 2.0**-53


# 4096 and 3041 outputs in 64-SFT tiles (RT = 4) take 66 to 82 KB of LDS; 256 tiles and one short one
@pytest.mark.parametrize("n_sft,n_out", [(257, 4096), (385, 3041)])
def test_largest_tiles(ccr, n_sft, n_out):
    rng = np.random.default_rng(12)
    t_sft, f_het = 1800.0, 250.0003
    k_first = int(round(f_het * t_sft)) - n_out // 2 - 3
    z = (rng.standard_normal((n_sft, n_out + 7)) + 1j * rng.standard_normal((n_sft, n_out + 7))).astype(np.complex64)
    valid = (rng.random(n_sft) < 0.9).astype(np.uint8)
    valid[[0, 63, 64, n_sft - 1]] = 1
    assert ((n_out + 63) // 64) * ((n_sft + 63) // 64) >= 256
    from synth import default_sky
    with ccr.Context(default_sky(), device=0) as ctx:
        print(f"{n_sft} SFTs x {n_out}", flush=True)
        x, v = ctx.sft_series(z, t_sft, 321.5, k_first, f_het, n_out, sft_valid=valid)
    rows = [0, 1, 63, 64, 200, n_sft - 1]
    for K in rows:
        ref = oracle.sft_series(z[K:K + 1], t_sft, 321.5 + K * t_sft, k_first, f_het, n_out, sft_valid=valid[K:K + 1])
        assert np.abs(x[K * n_out:(K + 1) * n_out] - ref).max() < 2e-6 * max(1e-3, np.abs(x).max())
    assert np.array_equal(v, np.repeat(valid, n_out))
