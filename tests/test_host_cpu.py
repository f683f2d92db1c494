"""What the host library launches and keeps, on the CPU (tests/hoststub.py)."""
import numpy as np
import pytest

import hoststub
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
