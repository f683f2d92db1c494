"""Filters with |a1| >= 1, which a descriptor may hold: a filter that grows and is not
excited stays at zero, whatever the block length and the split.
"""
import dataclasses

import numpy as np
import pytest

import oracle
from paper_1702_02256_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kw", [{}, {"time_chunks": 2}, {"time_chunks": 8}, {"time_chunks": -1},
                                {"time_chunks": 2, "filters_per_lane": 2, "waves_per_group": 1}])
@pytest.mark.parametrize("growth", [1.0, 1.5, 2.0])
def test_growing_filters_at_rest(growth, kw):
    import torch
    from paper_1702_02256_amd import spiir as S
    tb = W.random_bank(91, np.array([[128], [40]], np.int32), 4096, [200])
    a1, b0 = tb.a1.copy(), tb.b0.copy()
    a1[5] = growth * np.exp(0.3j)
    b0[5] = 0
    tb = dataclasses.replace(tb, a1=a1, b0=b0)
    x = W.noise_stream(92, 4 * 4096)
    xt = torch.from_numpy(x.astype(np.float32)).cuda()
    bank = S.Bank(tb, 4096, **kw)
    z = torch.zeros((2, len(x)), dtype=torch.complex64, device="cuda")
    pos = 0
    for n in (4096, 64, 4032, 4096, 4096):
        bank.process_block(xt[pos:pos + n], z[:, pos:pos + n])
        pos += n
    torch.cuda.synchronize()
    rc = bank.status()[0]
    bank.destroy()
    zr = oracle.run_stream(tb, x)
    zg = z.cpu().numpy()
    assert rc == S.SPIIR_OK and np.isfinite(zg).all()
    err = np.max(np.abs(zg - zr), axis=1) / np.max(np.abs(zr), axis=1)
    assert err.max() <= 1e-5, err
