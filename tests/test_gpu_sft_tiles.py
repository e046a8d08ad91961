"""SFT front end on the matrix units: calls long enough for 64-SFT tiles (RT = 4) and the longest
shorter ones (RT = 1), with a last tile of one SFT and one output column past the 64-output tile,
missing SFTs, against the oracle's direct transform (2e-6 of the largest sample: FP32 output)."""

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


# (SFTs, outputs): 2 column tiles x 129 row tiles (RT = 4); 2 x 127 (RT = 1); one column tile of
# one output x 256 (RT = 4)
@pytest.mark.parametrize("n_sft,n_out", [(8193, 65), (8128, 65), (16384, 1)])
def test_sft_tiles(ccr, n_sft, n_out):
    rng = np.random.default_rng(11)
    t_sft, f_het = 600.0, 100.0371
    k_first = int(round(f_het * t_sft)) - n_out // 2 - 3
    z = (rng.standard_normal((n_sft, n_out + 7)) + 1j * rng.standard_normal((n_sft, n_out + 7))).astype(np.complex64)
    valid = (rng.random(n_sft) < 0.9).astype(np.uint8)
    from synth import default_sky
    with ccr.Context(default_sky(), device=0) as ctx:
        x, v = ctx.sft_series(z, t_sft, 321.5, k_first, f_het, n_out, sft_valid=valid)
    ref = oracle.sft_series(z, t_sft, 321.5, k_first, f_het, n_out, sft_valid=valid)
    scale = np.abs(ref).max()
    err = np.abs(x - ref).max() / scale
    print(f"{n_sft} SFTs x {n_out}: {err:.2e}", flush=True)
    assert err < 2e-6
    assert np.array_equal(v, np.repeat(valid, n_out))
