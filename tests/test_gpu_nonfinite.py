"""Non-finite samples and states: the same results whichever filter kernel a
launch takes, and a restored state that recovers the bank.

A bank's workgroups end in lanes that hold no filter.  The pipelined kernel leaves
whole waves of them out, k_filter launches them; which of the two runs depends on
what else is in the batch (see test_gpu_pipe.py).
"""
import numpy as np
import pytest

from paper_1702_02256_amd import workloads as W

pytestmark = pytest.mark.gpu
N = 512
SHAPE = {"filters_per_lane": 4, "waves_per_group": 4}
FILL = (0, 300, 600)  # workgroups beside the bank: pipelined (4 or 2, then 1 thread per lane), k_filter

# filters per segment: one wave of which half is used; two waves of four, the
# second partly used; three full waves
BANKS = {"half a wave": [[128]], "a wave and a quarter": [[300], [5]], "three waves": [[512], [256]],
         "two bands": [[130, 3], [7, 61]]}


def _tables(name):
    nf = np.array(BANKS[name], np.int32)
    return W.random_bank(81, nf, 2048, [300, 100][:nf.shape[1]])


@pytest.fixture(scope="module")
def fillers():
    from paper_1702_02256_amd import spiir as S
    out = {}
    for n in FILL[1:]:
        out[n] = S.Bank(W.random_bank(7, np.full((n, 1), 1024), 4096, [20]), N, **SHAPE)
    yield out
    for b in out.values():
        b.destroy()


def _run(bank, x, blocks, filler=None):
    import torch
    from paper_1702_02256_amd import spiir as S
    z = torch.zeros((bank.n_templates, sum(blocks)), dtype=torch.complex64, device="cuda")
    pos = 0
    for n in blocks:
        req = [(bank, x[pos:pos + n], z[:, pos:pos + n])]
        if filler is not None:
            filler.reset()
            req.append((filler, torch.zeros(n, device="cuda"),
                        torch.empty((filler.n_templates, n), dtype=torch.complex64, device="cuda")))
        S.spiir_process_batch(req)
        pos += n
    torch.cuda.synchronize()
    return z.cpu().numpy()


def _bits(a):
    """The values' bits, every NaN the same one."""
    v = np.ascontiguousarray(a).view(np.float32).copy()
    v[np.isnan(v)] = np.float32(np.nan)
    return v.view(np.uint32)


def _stream(n, at, value):
    import torch
    x = W.noise_stream(82, n).astype(np.float32)
    if at is not None:
        x[at] = value
    return torch.from_numpy(x).cuda()


@pytest.mark.parametrize("value", [np.nan, np.inf, -np.inf])
@pytest.mark.parametrize("name", list(BANKS))
def test_same_bits_whatever_shares_the_launch(fillers, name, value):
    from paper_1702_02256_amd import spiir as S
    tb = _tables(name)
    x = _stream(3 * N, N + 100, value)
    # a split bank's blocks of 128 samples run both recurrences in one workgroup
    for kw, blocks in (({}, [N, N, N]), ({"time_chunks": 4}, [N, N, N]), ({"time_chunks": 4}, [128] * 12)):
        bank = S.Bank(tb, N, **SHAPE, **kw)
        ref = None
        for n_wg in FILL:
            print(f"{name}, {value}, {kw}: {n_wg} workgroups beside it", flush=True)
            bank.reset()
            z = _run(bank, x, blocks, fillers.get(n_wg))
            state = np.frombuffer(bank.save_state(), np.uint8)[128:]
            rc, flags = bank.status()
            assert rc == S.SPIIR_ENONFINITE and flags.all()
            got = (_bits(z), _bits(state), flags)
            ref = ref or got
            for a, b in zip(got, ref):
                assert np.array_equal(a, b), (name, kw, n_wg)
        bank.destroy()


@pytest.mark.parametrize("kw", [{}, {"time_chunks": 4}])
@pytest.mark.parametrize("name", list(BANKS))
def test_a_restored_state_recovers_the_bank(fillers, name, kw):
    """A good state restored after a NaN block, and the bank run alone and in a
    full batch again: the same bits as a new bank with that state."""
    from paper_1702_02256_amd import spiir as S
    tb = _tables(name)
    bank, fresh = (S.Bank(tb, N, **SHAPE, **kw) for _ in range(2))
    _run(bank, _stream(N, None, 0), [N])
    blob = bank.save_state()
    _run(bank, _stream(N, 0, np.nan), [N], fillers[600])
    x = _stream(4 * N, None, 0)
    out = []
    for b in (bank, fresh):
        b.load_state(blob)
        z = [_run(b, x[:N], [N]), _run(b, x[N:2 * N], [N], fillers[600]), _run(b, x[2 * N:], [N, 37 * 2, N - 74])]
        assert b.status()[0] == S.SPIIR_OK
        out.append(np.concatenate(z, axis=1))
        b.destroy()
    assert np.isfinite(out[0]).all()
    assert np.array_equal(_bits(out[0]), _bits(out[1]))
