"""The number of chunks a split asked for in P is run in: seen in the footprint (the
split's arrays), and the results against the oracle on both sides of each line.
"""
import numpy as np
import pytest

import oracle
from paper_1702_02256_amd import spiir as S
from paper_1702_02256_amd import workloads as W

SHAPE = {"filters_per_lane": 4, "waves_per_group": 4}
# bands, max_block, P asked for -> P run
CASES = [(3, 256, 32, 1), (3, 260, 32, 32), (1, 2048, 2, 1), (3, 4096, 2, 1), (3, 1024, 4, 4),
         (3, 2044, 4, 4), (3, 2048, 4, 8), (3, 512, 4, 4), (3, 4096, 16, 16)]


def _tables(bands):
    nf = np.full((3, bands), 40, np.int32)
    return W.random_bank(61, nf, 2048, [700 >> h for h in range(bands)])


@pytest.mark.parametrize("bands,mb,P,run", CASES)
def test_plan(bands, mb, P, run):
    tb = _tables(bands)
    p = S.spiir_plan(tb, mb, time_chunks=P, **SHAPE)
    assert p["time_chunks"] == P
    whole = S.spiir_plan(tb, mb, time_chunks=1, **SHAPE)
    rows = 2 + 2 * (run + 1) + 6 if run > 1 else 0  # arrays of n_slots complex values
    assert p["footprint"] == whole["footprint"] + rows * 8 * p["filter_slots"]
    # a shape the pipelined kernel cannot take keeps P
    two = {"filters_per_lane": 2, "waves_per_group": 4}
    q = S.spiir_plan(tb, mb, time_chunks=P, **two)
    assert q["footprint"] == (S.spiir_plan(tb, mb, time_chunks=1, **two)["footprint"]
                              + (8 + 2 * (P + 1)) * 8 * q["filter_slots"])


@pytest.mark.gpu
@pytest.mark.parametrize("bands,mb,P,run", CASES)
def test_results(bands, mb, P, run):
    import torch
    tb = _tables(bands)
    blocks = [mb, mb // 2 // 4 * 4, 4, mb]
    x = W.noise_stream(62, sum(blocks))
    print(f"P={P} run {run}: {bands} bands, blocks {blocks}", flush=True)
    bank = S.Bank(tb, mb, time_chunks=P, **SHAPE)
    xt = torch.from_numpy(x.astype(np.float32)).cuda()
    z = torch.zeros((3, sum(blocks)), dtype=torch.complex64, device="cuda")
    pos = 0
    for n in blocks:
        bank.process_block(xt[pos:pos + n], z[:, pos:pos + n])
        pos += n
    torch.cuda.synchronize()
    assert bank.status()[0] == 0
    bank.destroy()
    zr = oracle.run_stream(tb, x)
    e = np.max(np.abs(z.cpu().numpy() - zr), axis=1) / np.max(np.abs(zr), axis=1)
    assert e.max() <= 1e-5, e.max()
