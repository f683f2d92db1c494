"""What the host library launches and keeps, on the CPU (tests/hoststub.py)."""
import ctypes as C
import dataclasses

import numpy as np
import pytest

import hoststub
from paper_1702_02256_amd import spiir as S
from paper_1702_02256_amd import workloads as W

SHAPE = {"filters_per_lane": 4, "waves_per_group": 4}


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    s = hoststub.Stub(hoststub.build(tmp_path_factory.mktemp("stub")))
    with s.active():
        yield s


def _tables(T, H=1, M=128, seed=3):
    return W.random_bank(seed, np.full((T, H), M, np.int32), 4096, [200 >> h for h in range(H)])


def _io(bank, n):
    return np.zeros(n, np.float32), np.zeros((bank.n_templates, n), np.complex64)


def test_a_restored_state_clears_the_chunk_end_states(stub):
    # k_chain reads the end states of lanes that the next launch may leave out
    bank = stub.bank(_tables(2), 4096, time_chunks=8, **SHAPE)
    x, z = _io(bank, 4096)
    dev = stub.process([(bank, x, z)])[0].req[0].bank
    ends, pending = stub.end_states(dev)
    pending = np.ctypeslib.as_array(pending, (2 * bank.plan["filter_slots"],))
    assert not ends.any() and not pending.any()
    blob = bank.save_state(stream=0)
    ends[:] = np.nan
    pending[:] = np.nan
    bank.load_state(blob, stream=0)
    assert not ends.any() and not pending.any()
    bank.destroy()


@pytest.mark.parametrize("F", [4, 2])
@pytest.mark.parametrize("growth,lc,whole", [(0.9999, 256, False), (1.01, 512, False), (1.42, 256, True),
                                             (1.0, 2048, False), (1.05, 2048, True), (1e200, 64, True)])
def test_banks_whose_chain_overflows_run_whole(growth, lc, whole, F):
    # a1^lc beyond FP32 would turn a state of zero into NaN: such banks are not cut
    tb = _tables(2)
    a1 = tb.a1.copy()
    a1[7] = growth
    tb = dataclasses.replace(tb, a1=a1)
    shape = {"filters_per_lane": F, "waves_per_group": 4}
    P = 4096 // lc if F == 2 or lc < 2048 else 1
    asked = S.spiir_plan(tb, 4096, time_chunks=4096 // lc, **shape)
    plain = S.spiir_plan(tb, 4096, **shape)
    rows = 0 if whole or P == 1 else 2 + 2 * (P + 1) + 6
    assert asked["footprint"] == plain["footprint"] + rows * 8 * asked["filter_slots"]
    assert asked["time_chunks"] == 4096 // lc
    # not asked for: only where every filter decays
    own = S.spiir_plan(tb, 4096)
    plain = S.spiir_plan(tb, 4096, **SHAPE)
    assert (own["footprint"] > plain["footprint"]) == (growth < 1.0)


def test_a_block_filtered_in_place_keeps_the_pass_that_writes_z(stub):
    # the filter launch reads x in every workgroup, so it must not write z over it
    n = 1000
    bank = stub.bank(_tables(3), n, **SHAPE)
    other = stub.bank(_tables(2, seed=4), n, **SHAPE)
    staged = stub.bank(_tables(2, H=2, seed=5), n, **SHAPE)
    buf = np.zeros(40 * n, np.float32)  # z of `bank`: floats [2n, 8n)
    z = buf[2 * n:8 * n].view(np.complex64).reshape(3, n)

    def direct(requests):
        filters = [l for l in stub.process(requests) if l.kind in ("filter", "pipe")]
        last = [r for l in stub.launches() if l.kind == "upadd" for r in l.req]
        got = [r.z_direct for r in filters[0].req]
        assert [r.T for r in filters[0].req] == [0 if d else b.n_templates for d, (b, _, _) in zip(got, requests)]
        assert bool(last) == (0 in got)
        return got

    for at, apart in ((0, 1), (n, 1), (n + 1, 0), (2 * n, 0), (5 * n, 0), (8 * n - 1, 0), (8 * n, 1)):
        assert direct([(bank, buf[at:at + n], z)]) == [apart], at
    # another request's x in the same launch; a staged request has read its own before
    free = buf[10 * n:].view(np.complex64)
    zo = free[:2 * n].reshape(2, n)
    assert direct([(bank, buf[:n], z), (other, buf[3 * n:4 * n], zo)]) == [0, 1]
    assert direct([(bank, buf[:n], z), (other, buf[9 * n:10 * n], zo)]) == [1, 1]
    # rows with a stride: the gaps count as z
    wide = free[:9 * n].reshape(3, 3 * n)[:, :n]
    assert direct([(bank, buf[10 * n + 4 * n:10 * n + 5 * n], wide)]) == [0]
    launches = stub.process([(bank, buf[:n], z), (staged, buf[3 * n:4 * n], zo)])
    assert [l.kind for l in launches][0] == "stage"
    assert [r.z_direct for r in [l for l in launches if l.kind in ("filter", "pipe")][0].req] == [1, 0]
    for b in (bank, other, staged):
        b.destroy()


@pytest.mark.parametrize("n", [0, 1, 127, 128])
def test_a_blob_without_a_header_is_refused(stub, monkeypatch, n):
    # the library reads the header before it knows the length
    bank = stub.bank(_tables(1), 512, **SHAPE)
    called = []
    real = stub.lib.spiir_load_state
    monkeypatch.setattr(stub.lib, "spiir_load_state", lambda h, buf, s: called.append(len(buf)) or real(h, buf, s))
    with pytest.raises(S.SpiirError):
        bank.load_state(bytes(n), stream=0)
    assert called == ([128] if n == 128 else [])
    bank.destroy()


@pytest.mark.parametrize("H", [1, 2])
def test_profiled_calls_reuse_their_events(stub, H):
    # every event taken for a call comes back, also where a kind of kernel is not launched
    bank = stub.bank(_tables(2, H), 4096, **SHAPE)
    x, z = _io(bank, 4096)
    lib, counts = stub.lib, []
    for _ in range(4):
        assert lib.spiir_profile_enable(1) == S.SPIIR_OK
        for _ in range(5):
            stub.process([(bank, x, z)])
        data = S.ProfileData()
        assert lib.spiir_profile_read(C.byref(data)) == S.SPIIR_OK
        assert list(data.launches) == ([0, 5, 0] if H == 1 else [5, 5, 5])
        counts.append(stub.events())
    lib.spiir_profile_enable(0)
    assert len(set(counts)) == 1, counts
    bank.destroy()


def test_short_blocks_of_split_banks_take_the_cheaper_route(stub):
    # (templates, banks in the batch, n) -> one launch of both runs, or three launches
    routes = [(1, 1, 256, 1), (1, 1, 512, 1), (40, 1, 256, 1), (40, 1, 320, 0), (40, 1, 512, 0), (40, 4, 512, 0),
              (20, 16, 512, 1), (4, 1, 512, 0), (40, 16, 512, 1), (40, 16, 528, 0), (1, 1, 4096, 0)]
    nf = np.random.default_rng(1).integers(40, 301, size=(40, 5)).astype(np.int32)
    full = W.random_bank(6, nf, 4096, [2047 >> h for h in range(5)])
    for T, nb, n, one in routes:
        tb = full.subset(list(range(T))) if T < 40 else full
        banks = [stub.bank(tb, 4096) for _ in range(nb)]
        launches = stub.process([(b, *_io(b, n)) for b in banks])
        kinds = [l.kind for l in launches]
        assert ("chain" in kinds) == (not one), (T, nb, n, kinds)
        assert all(r.dual == one for l in launches if l.kind == "pipe" for r in l.req), (T, nb, n)
        for b in banks:
            b.destroy()
    # chunks of 512 samples that were asked for
    bank = stub.bank(full, 4096, time_chunks=8)
    for n, one in ((512, 1), (528, 0), (1024, 0)):
        assert ("chain" in [l.kind for l in stub.process([(bank, *_io(bank, n))])]) == (not one), n
    bank.destroy()


@pytest.mark.parametrize("T,H,M,P", [(160, 3, 64, 32), (512, 1, 300, 4)])
def test_automatic_split_is_the_same_for_both_sums(T, H, M, P):
    # four filters per lane leave four waves per SIMD with either sum; short delays,
    # so that the LDS does not decide
    tb = W.random_bank(7, np.full((T, H), M, np.int32), 4096, [20 >> h for h in range(H)])
    for precision in ("fp32", "fp32_compensated"):
        assert S.spiir_plan(tb, 512, precision=precision, time_chunks=S.TIME_CHUNKS_AUTO)["time_chunks"] == P


@pytest.mark.parametrize("groups,direct", [(340, 1), (341, 0)])
def test_many_workgroups_are_staged(stub, groups, direct):
    bank = stub.bank(_tables(groups, M=256), 512, filters_per_lane=4, waves_per_group=1)
    assert bank.plan["n_groups"] == groups
    launches = stub.process([(bank, *_io(bank, 512))])
    assert [l.kind for l in launches] == ([] if direct else ["stage"]) + [launches[-1].kind]
    r = launches[-1].req[0]
    assert (r.direct, r.z_direct, r.T) == (direct, 1, 0)
    bank.destroy()


@pytest.mark.parametrize("groups,n,kind", [(256, 256, "pipe"), (257, 256, "filter"), (257, 512, "pipe")])
def test_short_runs_of_compensated_small_groups(stub, groups, n, kind):
    # four threads per lane and the compensated sum: one group of 128 lanes per compute unit
    tb = _tables(groups, M=512)
    for precision, want in (("fp32_compensated", kind), ("fp32", "pipe")):
        bank = stub.bank(tb, 512, filters_per_lane=4, waves_per_group=2, precision=precision)
        launches = stub.process([(bank, *_io(bank, n))])
        assert bank.plan["n_groups"] == groups and [l.kind for l in launches] == [want]
        bank.destroy()
