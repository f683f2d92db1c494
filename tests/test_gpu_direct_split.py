"""Single-rate banks split in time, whose end-state pass reads the block itself and
appends it to the input ring: where blocks begin changes no bit.
"""
import numpy as np
import pytest

import oracle
from paper_1702_02256_amd import workloads as W

pytestmark = pytest.mark.gpu
CUTS = [[6000, 4096, 904], [1, 63, 256, 512, 77, 5091, 2500, 2500], [500] * 22, [37, 219] * 42 + [248]]


@pytest.mark.parametrize("kw", [{}, {"time_chunks": 8}, {"time_chunks": 4, "filters_per_lane": 2, "waves_per_group": 2},
                                {"time_chunks": 64, "precision": "fp32_compensated"}])
def test_where_blocks_begin_changes_no_bit(kw):
    import torch
    from paper_1702_02256_amd import spiir as S
    tb = W.random_bank(31, np.array([[40], [90]], np.int32), 2048, [500])
    x = W.noise_stream(33, 11000)
    xt = torch.from_numpy(x.astype(np.float32)).cuda()
    bank = S.Bank(tb, 6000, **kw)
    zr = oracle.run_stream(tb, x)
    ref = None
    for cuts in CUTS:
        assert sum(cuts) == 11000
        print(f"single rate, split {kw}: blocks {cuts[:6]}", flush=True)
        z = torch.zeros((2, 11000), dtype=torch.complex64, device="cuda")
        pos = 0
        for n in cuts:
            bank.process_block(xt[pos:pos + n], z[:, pos:pos + n])
            pos += n
        torch.cuda.synchronize()
        assert bank.samples_done == 11000
        bank.reset()
        got = z.cpu().numpy()
        err = np.max(np.abs(got - zr), axis=1) / np.max(np.abs(zr), axis=1)
        assert err.max() <= 1e-5, err
        ref = got if ref is None else ref
        assert np.array_equal(got.view(np.uint64), ref.view(np.uint64)), cuts[:6]
    bank.destroy()
