"""The number of chunks a split is run in where it follows from the bank's work: both
sides of each line, and the results of one bank on either side; a split that is turned
off.
"""
import numpy as np
import pytest

import oracle
from paper_1702_02256_amd import spiir as S
from paper_1702_02256_amd import workloads as W

SHAPE = {"filters_per_lane": 4, "waves_per_group": 4}

# workgroups (single rate, one per template of 1024 filters), max_block, P asked for -> P run
CASES = [(256, 2048, 2, 1), (257, 2048, 2, 8), (257, 2044, 2, 1),
         (160, 2048, 4, 8), (161, 2048, 4, 4), (161, 2044, 4, 4),
         (64, 1023, 4, 4), (65, 1023, 4, 1), (65, 1024, 4, 4)]


def _tables(n):
    return W.random_bank(63, np.full((n, 1), 1024, np.int32), 2048, [700])


@pytest.mark.parametrize("groups,mb,P,run", CASES)
def test_chunks_run(groups, mb, P, run):
    tb = _tables(groups)
    p = S.spiir_plan(tb, mb, time_chunks=P, **SHAPE)
    assert p["n_groups"] == groups and p["time_chunks"] == P
    assert S.spiir_chunks_run(tb, mb, time_chunks=P, **SHAPE) == run
    # two bands: a split in two never becomes one in eight
    if P == 2:
        tb2 = W.random_bank(64, np.full((groups, 2), 1024, np.int32), 2048, [700, 300])
        assert S.spiir_chunks_run(tb2, mb // 4 * 4, time_chunks=P, **SHAPE) == 1


@pytest.mark.parametrize("T,mb,run", [(1, 4096, 16), (1, 512, 8), (1, 508, 1), (40, 4096, 16), (45, 4096, 1),
                                      (90, 4096, 1)])
def test_chunks_of_small_banks(T, mb, run):
    nf = np.random.default_rng(1).integers(40, 301, size=(90, 5)).astype(np.int32)[:T]
    tb = W.random_bank(65, nf, 4096, [2047 >> h for h in range(5)])
    mb = mb // 16 * 16
    run = run if mb >= 512 else 1
    assert S.spiir_chunks_run(tb, mb) == run
    # turned off, or the shape chosen by the caller
    plan = S.spiir_plan(tb, mb)
    shape = {"filters_per_lane": plan["filters_per_lane"], "waves_per_group": plan["lanes_per_group"] // 64}
    for kw in ({"time_chunks": 1}, shape, {"time_chunks": 1, **shape}):
        assert S.spiir_chunks_run(tb, mb, **kw) == 1
        assert S.spiir_plan(tb, mb, **kw)["footprint"] <= plan["footprint"]
    with pytest.raises(S.SpiirError):
        S.spiir_chunks_run(tb, mb, time_chunks=3)


def _run(tb, blocks, **kw):
    import torch
    x = W.noise_stream(66, sum(blocks))
    xt = torch.from_numpy(x.astype(np.float32)).cuda()
    bank = S.Bank(tb, max(blocks), **kw)
    z = torch.zeros((tb.n_filters.shape[0], sum(blocks)), dtype=torch.complex64, device="cuda")
    pos = 0
    for n in blocks:
        bank.process_block(xt[pos:pos + n], z[:, pos:pos + n])
        pos += n
    torch.cuda.synchronize()
    assert bank.status()[0] == 0
    state = bank.save_state()
    bank.destroy()
    return x, z, state


@pytest.mark.gpu
@pytest.mark.parametrize("groups,mb,P,run", [c for c in CASES if (c[0], c[1]) in
                                             ((257, 2048), (161, 2048), (65, 1023), (64, 1023))])
def test_results(groups, mb, P, run):
    tb = _tables(groups)
    blocks = [mb, mb // 2, 3, mb]
    print(f"P={P} run {run}: {groups} workgroups, blocks {blocks}", flush=True)
    x, z, _ = _run(tb, blocks, time_chunks=P, **SHAPE)
    _, ref, _ = _run(tb, blocks, **SHAPE)
    top = ref.abs().amax(1)
    assert ((z - ref).abs().amax(1) / top).max().item() <= 1e-5
    some = [0, groups // 2, groups - 1]
    zr = oracle.run_stream(tb.subset(some), x)
    e = np.max(np.abs(z[some].cpu().numpy() - zr), axis=1) / np.max(np.abs(zr), axis=1)
    assert e.max() <= 1e-5, e.max()


@pytest.mark.gpu
def test_turned_off_is_the_whole_bank():
    """time_chunks = 1 of a bank that the library would split: the bits and the state
    of the bank whose shape the caller gives."""
    import torch
    nf = np.array([[130, 20, 0], [9, 77, 40]], np.int32)
    tb = W.random_bank(51, nf, 4096, [2047, 300, 500])
    blocks = [4096, 1000, 64, 4096]
    plan = S.spiir_plan(tb, 4096)
    shape = {"filters_per_lane": plan["filters_per_lane"], "waves_per_group": plan["lanes_per_group"] // 64}
    _, za, sa = _run(tb, blocks, time_chunks=1)
    _, zb, sb = _run(tb, blocks, **shape)
    assert torch.equal(torch.view_as_real(za), torch.view_as_real(zb)) and sa == sb
    # a state of the split bank is taken
    _, _, split = _run(tb, blocks)
    assert len(split) > len(sa)
    bank = S.Bank(tb, 4096, time_chunks=1)
    bank.load_state(split)
    assert bank.samples_done == sum(blocks)
    bank.destroy()
