"""Single-rate banks take one launch: the filter kernel reads the block itself,
appends it to the input ring, advances the clock and, where every template is
one piece, writes z.  The pieces of that path against the staged one (the same
filters as band 0 of a two-band bank whose lower band is empty, which carries
zeros up) and the oracle, over blocks from one sample to several launches.
"""
import dataclasses

import numpy as np
import pytest

import oracle
from paper_1702_02256_amd import workloads as W

pytestmark = pytest.mark.gpu


def _stream(bank, x, blocks, graph=False, odd=0):
    import torch
    from paper_1702_02256_amd import spiir as S
    T, total = bank.n_templates, sum(blocks)
    z = torch.zeros((T, total + odd), dtype=torch.complex64, device="cuda")[:, :total]
    pos = 0
    for i, n in enumerate(blocks):
        if graph and i % 2:
            buf, out = x[pos:pos + n].clone(), torch.zeros((T, n), dtype=torch.complex64, device="cuda")
            g = S.Graph([(bank, buf, out)])
            g.launch()
            z[:, pos:pos + n] = out
            g.destroy()
        else:
            bank.process_block(x[pos:pos + n], z[:, pos:pos + n])
        pos += n
    torch.cuda.synchronize()
    assert bank.status()[0] == 0 and bank.samples_done == total
    return z.cpu().numpy()


@pytest.mark.parametrize("nf,dmax,kw", [
    ([128], 2047, {}),                                   # one piece: z from the filter kernel
    ([301] * 9, 4095, {"precision": "fp32_compensated"}),  # pieces over two workgroups: workspace and up-add
    ([5, 0, 70], 63, {}),                                # a template without filters
    ([512] * 4, 4095, {"filters_per_lane": 4, "waves_per_group": 8}),
    ([64, 64], 16383, {"window_copies": 1}),             # history far longer than a block
    ([40, 90], 500, {"time_chunks": 8}),                 # chunks, some of them empty
    ([33], 100, {"filters_per_lane": 1}),
])
def test_one_launch_path(nf, dmax, kw):
    import torch
    from paper_1702_02256_amd import spiir as S
    tb = W.random_bank(31, np.array(nf, np.int32)[:, None], 2048, [dmax])
    staged = dataclasses.replace(tb, n_filters=np.stack([np.array(nf, np.int32), np.zeros(len(nf), np.int32)], 1),
                                 h_down=W.down_taps(32), h_up=W.up_taps(32))
    blocks = [2, 64, 1000, 126, 256, 6000, 510, 258]
    x = W.noise_stream(32, sum(blocks))
    xt = torch.from_numpy(x.astype(np.float32)).cuda()
    print(f"single-rate {nf} delays to {dmax} {kw}", flush=True)
    ref_bank = S.Bank(staged, 6000, **kw)
    ref = _stream(ref_bank, xt, blocks)
    bank = S.Bank(tb, 6000, **kw)
    got = _stream(bank, xt, blocks)
    zr = oracle.run_stream(tb, x)
    err = np.max(np.abs(got - zr), axis=1) / np.maximum(np.max(np.abs(zr), axis=1), 1e-300)
    assert err.max() <= 1e-5, err
    assert np.array_equal(got, ref)
    # odd blocks, odd row strides, recorded and eager calls in turn; a checkpoint in between
    bank.reset()
    again = _stream(bank, xt, blocks, graph=True, odd=1)
    assert np.array_equal(again, got)
    blob = bank.save_state()
    assert len(blob) == bank.state_size()
    bank.load_state(blob)
    tail = xt[:77]
    za = torch.zeros((len(nf), 77), dtype=torch.complex64, device="cuda")
    zb = torch.zeros_like(za)
    bank.process_block(tail, za)
    bank.load_state(blob)
    for a, b in ((0, 1), (1, 40), (40, 77)):
        bank.process_block(tail[a:b], zb[:, a:b])
    torch.cuda.synchronize()
    # (a time split's rounding depends on where blocks begin)
    same = np.allclose if "time_chunks" in kw else np.array_equal
    assert same(za.cpu().numpy(), zb.cpu().numpy())
    bank.destroy()
    ref_bank.destroy()
