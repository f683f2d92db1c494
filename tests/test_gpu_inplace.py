"""A block filtered in place: z written over the memory that x was read from."""
import numpy as np
import pytest

from paper_1702_02256_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kw", [{}, {"time_chunks": 8}, {"filters_per_lane": 4, "waves_per_group": 8}])
@pytest.mark.parametrize("bands,templates", [(1, 1), (1, 40), (2, 3)])
def test_in_place(bands, templates, kw):
    import torch
    from paper_1702_02256_amd import spiir as S
    n = 2048
    tb = W.random_bank(71, np.full((templates, bands), 130, np.int32), 2048, [300, 100][:bands])
    x = torch.from_numpy(W.noise_stream(72, 3 * n).astype(np.float32)).cuda()
    apart, inside = S.Bank(tb, n, **kw), S.Bank(tb, n, **kw)
    z = torch.empty((templates, n), dtype=torch.complex64, device="cuda")
    both = torch.empty_like(z)
    floats = torch.view_as_real(both).reshape(-1)
    for i, at in enumerate((0, n // 2 + 3, floats.numel() - n)):  # x at the start, in the middle, at the end of z
        block = x[i * n:(i + 1) * n]
        apart.process_block(block, z)
        floats[at:at + n] = block
        inside.process_block(floats[at:at + n], both)
        torch.cuda.synchronize()
        assert torch.equal(torch.view_as_real(z), torch.view_as_real(both)), at
    apart.destroy()
    inside.destroy()
