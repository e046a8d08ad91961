"""Bands of one call without allocations: 2000 fit the tables of the fixed array (2016 is its limit)."""

import numpy as np
import pytest

import synth
from conftest import small_config

pytestmark = pytest.mark.gpu


def test_two_thousand_bands():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1712_06515_amd import ccr
    ds = synth.make_dataset(small_config(n_seg=6, f_band=0.1))
    with ccr.Context(ds.sky, device=0) as ctx:
        bid = ctx.load(ds, templates=ds.templates[:1])
        info = ctx.band_info(bid)
        ref = ctx.compute_rho(bid, prec=ccr.PREC_FP64)
        n = 2000
        out = torch.full((n, 1, info["n_f"]), float("nan"), dtype=torch.float64, device="cuda")
        torch.cuda.synchronize()
        ctx.compute_rho_noalloc([bid] * n, [out[i].data_ptr() for i in range(n)], prec=ccr.PREC_FP64)
        ctx.sync()
        assert np.array_equal(out.cpu().numpy(), np.broadcast_to(ref, (n,) + ref.shape))
        # the array's limit itself is still an error, not an overrun
        m = 4000
        with pytest.raises(ccr.CcrError) as e:
            ctx.compute_rho_noalloc([bid] * m, [out[i % n].data_ptr() for i in range(m)], prec=ccr.PREC_FP64)
        assert e.value.status == ccr.ERANGE
