"""Single-rate banks on both sides of the number of workgroups from which a call is
staged: z written by the filter kernel against z that goes through the workspace (a
call with peaks), the same bits, and the oracle.
"""
import numpy as np
import pytest

import oracle
from paper_1702_02256_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("templates", [340, 341, 700])
def test_z_with_and_without_the_workspace(templates):
    import torch
    from paper_1702_02256_amd import spiir as S
    tb = W.random_bank(41, np.full((templates, 1), 256, np.int32), 2048, [300])
    blocks = [512, 1, 63, 5000, 500]
    x = W.noise_stream(42, sum(blocks))
    xt = torch.from_numpy(x.astype(np.float32)).cuda()
    banks = [S.Bank(tb, 5000, filters_per_lane=4, waves_per_group=1) for _ in range(2)]
    assert banks[0].plan["n_groups"] == templates
    z = [torch.zeros((templates, sum(blocks)), dtype=torch.complex64, device="cuda") for _ in range(2)]
    peaks = S.peaks_empty(templates)
    pos = 0
    for n in blocks:
        banks[0].process_block(xt[pos:pos + n], z[0][:, pos:pos + n])
        banks[1].process_peaks(xt[pos:pos + n], z[1][:, pos:pos + n], peaks, 1.0)
        pos += n
    torch.cuda.synchronize()
    assert torch.equal(torch.view_as_real(z[0]), torch.view_as_real(z[1]))
    assert banks[0].samples_done == sum(blocks) and banks[0].save_state() == banks[1].save_state()
    some = [0, 170, templates - 1]
    zr = oracle.run_stream(tb.subset(some), x)
    err = np.max(np.abs(z[0][some].cpu().numpy() - zr), axis=1) / np.max(np.abs(zr), axis=1)
    assert err.max() <= 1e-5, err
    for b in banks:
        b.destroy()
