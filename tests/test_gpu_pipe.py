"""The pipelined filter kernel against k_filter, bit for bit.

Which of the two a launch takes depends on how full the device is, so a small
bank alone runs the pipelined kernel (4, 2 or 1 threads per lane) and k_filter
in one launch with enough other work of its shape.  Both run the same
recurrences and the same order of every sum, so the bank's outputs and
states have to be the same bits whatever shares its launch.
"""
import numpy as np
import pytest

import oracle
from paper_1702_02256_amd import workloads as W

pytestmark = pytest.mark.gpu
N = 512

# (filters per segment, bands, delays) of the small bank
BANKS = {
    "one segment": (np.array([[128]]), [300]),                     # 32 lanes: 4 threads per lane
    "one filter": (np.array([[1]]), [0]),
    "tails": (np.array([[130, 3], [7, 61], [64, 0]]), [900, 100]),  # runs that end inside a 16-lane group
    "full groups": (np.array([[512], [512], [256]]), [1000]),       # every group one run
    "long segment": (np.array([[2100], [90]]), [77]),               # pieces in several workgroups, over 8 runs
    "many pieces": (np.full((70, 1), 5), [40]),                     # more level-2 tasks than threads
}
# workgroups of 256 lanes that share the launch: alone, over one per compute
# unit (one thread per lane), over two (k_filter)
FILL = (0, 300, 600)


def _run(bank, x, blocks, filler):
    import torch
    from paper_1702_02256_amd import spiir as S
    z = torch.zeros((bank.n_templates, sum(blocks)), dtype=torch.complex64, device="cuda")
    pos = 0
    for n in blocks:
        req = [(bank, x[pos:pos + n], z[:, pos:pos + n])]
        if filler is not None:
            zf = torch.empty((filler.n_templates, n), dtype=torch.complex64, device="cuda")
            req.append((filler, x[pos:pos + n], zf))
        S.spiir_process_batch(req)
        pos += n
    torch.cuda.synchronize()
    state = bank.save_state()
    bank.reset()
    return z.cpu().numpy(), state


@pytest.fixture(scope="module")
def fillers():
    from paper_1702_02256_amd import spiir as S
    out = {0: None}
    for n_wg in FILL[1:]:
        tb = W.random_bank(7, np.full((n_wg, 1), 1024), 4096, [20])
        out[n_wg] = {p: S.Bank(tb, N, precision=p, filters_per_lane=4, waves_per_group=4)
                     for p in ("fp32", "fp32_compensated")}
    yield out
    for f in out.values():
        for b in (f or {}).values():
            b.destroy()


@pytest.mark.parametrize("precision", ["fp32", "fp32_compensated"])
@pytest.mark.parametrize("name", list(BANKS))
def test_same_bits_whatever_shares_the_launch(fillers, name, precision):
    import torch
    from paper_1702_02256_amd import spiir as S
    nf, dmax = BANKS[name]
    H = nf.shape[1]
    tb = W.random_bank(11, nf.astype(np.int32), 4096, dmax)
    x = W.noise_stream(12, 4 * N)
    xt = torch.from_numpy(x.astype(np.float32)).cuda()
    blocks = [N, 2, 38, 16, 120, N, 200] if H > 1 else [N, 1, 37, 17, 121, N, 199]
    for kw in ({}, {"window_copies": 1, "carry_chunk": 16}, {"time_chunks": 4}):
        bank = S.Bank(tb, N, precision=precision, filters_per_lane=4, waves_per_group=4, **kw)
        ref = None
        for n_wg in FILL:
            print(f"{name}, {precision}, {kw}: {n_wg} workgroups beside it", flush=True)
            filler = fillers[n_wg][precision] if n_wg else None
            if filler is not None:
                filler.reset()
            got = _run(bank, xt, blocks, filler)
            if ref is None:
                ref = got
                zr = oracle.run_stream(tb, x[:sum(blocks)])
                err = np.max(np.abs(got[0] - zr), axis=1) / np.maximum(np.max(np.abs(zr), axis=1), 1e-300)
                assert err.max() <= 1e-5, err
            assert np.array_equal(got[0], ref[0]), (name, kw, n_wg)
            assert got[1] == ref[1], (name, kw, n_wg)
        bank.destroy()
