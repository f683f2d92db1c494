"""What a time split carries from block to block: where blocks begin changes no
bit (small banks are split without being asked), and states move between banks
that are split differently or not at all.
"""
import struct

import numpy as np
import pytest

import oracle
from paper_1702_02256_amd import workloads as W

pytestmark = pytest.mark.gpu
MB = 4096


def _bank(**kw):
    from paper_1702_02256_amd import spiir as S
    nf = np.array([[130, 20, 0], [9, 77, 40]], np.int32)
    tb = W.random_bank(51, nf, 4096, [2047, 300, 500])
    return tb, S.Bank(tb, MB, **kw)


def _run(bank, x, blocks):
    import torch
    z = torch.zeros((bank.n_templates, sum(blocks)), dtype=torch.complex64, device="cuda")
    pos = 0
    for n in blocks:
        bank.process_block(x[pos:pos + n], z[:, pos:pos + n])
        pos += n
    torch.cuda.synchronize()
    assert bank.status()[0] == 0
    return z.cpu().numpy()


def _x(n):
    import torch
    x = W.noise_stream(52, n)
    return x, torch.from_numpy(x.astype(np.float32)).cuda()


def _err(z, zr):
    return np.max(np.max(np.abs(z - zr), axis=1) / np.max(np.abs(zr), axis=1))


# cuts on and off chunk boundaries, blocks inside one chunk, of one step, of all
CUTS = [[4096, 4096, 1808], [4, 252, 256, 512, 3072, 4096, 8, 1800],
        [1000, 100, 60, 500, 36, 2300, 2048, 52, 1948, 1956], [256] * 39 + [16]]


@pytest.mark.parametrize("kw", [{}, {"time_chunks": 8}, {"time_chunks": 64}, {"time_chunks": -1},
                                {"time_chunks": 4, "filters_per_lane": 2}, {"carry_chunk": 256}])
def test_where_blocks_begin_changes_no_bit(kw):
    _, bank = _bank(**kw)
    x, xt = _x(10000)
    ref = None
    for cuts in CUTS:
        assert sum(cuts) == 10000
        print(f"time split {kw}: blocks {cuts[:8]}", flush=True)
        z = _run(bank, xt, cuts)
        if ref is None:
            ref = z
            e = _err(z, oracle.run_stream(_bank()[0], x))
            assert e <= 1e-5, e
        assert np.array_equal(z.view(np.uint64), ref.view(np.uint64)), cuts
        bank.reset()
    bank.destroy()


@pytest.mark.parametrize("done", [4096, 5000])  # on a chunk boundary, inside a chunk
def test_states_move_between_splits(done):
    from paper_1702_02256_amd import spiir as S
    shape = {"filters_per_lane": 4, "waves_per_group": 4}
    tb, small = _bank()  # split by the library
    _, plain = _bank(**shape)
    _, eight = _bank(time_chunks=8, **shape)
    x, xt = _x(10000)
    zr = oracle.run_stream(tb, x)
    head = [4096] + ([done - 4096] if done > 4096 else [])
    blobs = {}
    for name, b in (("small", small), ("plain", plain), ("eight", eight)):
        _run(b, xt, head)
        blobs[name] = b.save_state()
        assert len(blobs[name]) == b.state_size()
    assert len(blobs["plain"]) < len(blobs["small"])
    # a state without the split's part, as banks wrote it that had none
    old = bytearray(blobs["small"][:len(blobs["plain"])])
    struct.pack_into("<I", old, 4, 3)
    blobs["old"] = bytes(old)
    for target, b in (("small", small), ("plain", plain), ("eight", eight)):
        for source, blob in blobs.items():
            b.load_state(blob)
            assert b.samples_done == done
            z = _run(b, xt[done:], [10000 - done - 1000 if done == 5000 else 4096, 1000])
            e = _err(z, zr[:, done:done + z.shape[1]])
            print(f"state of {source} into {target} at {done}: {e:.2e}", flush=True)
            assert e <= 1e-5
        with pytest.raises(S.SpiirError):
            b.load_state(blobs["small"][:-8])
        b.destroy()
