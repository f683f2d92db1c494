"""Builds and loads the host library with tests/c/host_stub.cpp in the place of
the HIP runtime and the kernels, so that what the host decides and keeps
(launches, events, states) is seen on the CPU.
"""
import contextlib
import ctypes as C
import os
import subprocess
from types import SimpleNamespace

import numpy as np

from paper_1702_02256_amd import _build
from paper_1702_02256_amd import spiir as S

HERE = os.path.dirname(os.path.abspath(__file__))
KINDS = ("stage", "filter", "local", "pipe", "mfma", "chain", "upadd")


def build(folder) -> str:
    out = os.path.join(str(folder), "libspiir_stub.so")
    cmd = ["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-Wl,-Bsymbolic", "-w", "-D__HIP_PLATFORM_AMD__",
           "-I", os.path.join(_build.ROCM, "include"), "-I", _build.INCLUDE, "-I", _build.CSRC,
           os.path.join(_build.CSRC, "spiir_host.cpp"), os.path.join(HERE, "c", "host_stub.cpp"), "-o", out]
    subprocess.run(cmd, check=True)
    return out


class Stub:
    """The stub library's record; `active()` puts it in the place of the GPU library."""

    def __init__(self, path):
        self.path = path
        self.lib = None

    @contextlib.contextmanager
    def active(self):
        kept, kept_path, kept_first = S._lib, S.LIB_PATH, S._torch_hip_first
        S._lib, S.LIB_PATH, S._torch_hip_first = self.lib, self.path, lambda: None
        try:
            self.lib = S.load_library()
            self.lib.stub_request.restype = C.c_void_p
            self.lib.stub_uend.restype = self.lib.stub_euend.restype = C.POINTER(C.c_float)
            yield self
        finally:
            S._lib, S.LIB_PATH, S._torch_hip_first = kept, kept_path, kept_first

    def events(self) -> int:
        return self.lib.stub_events()

    def bank(self, tables, max_block, **kw):
        return S.Bank(tables, max_block, stream=0, **kw)

    def process(self, requests, peaks=None):
        """One batch of (bank, x, z) numpy arrays (z may have a row stride); its launches."""
        arr = (S.Request * len(requests))()
        for i, (bank, x, z) in enumerate(requests):
            arr[i] = S.Request(bank._h, x.ctypes.data, len(x), z.ctypes.data, z.strides[0] // 8, None)
        self.lib.stub_clear()
        if peaks is None:
            rc = self.lib.spiir_process_batch(len(requests), arr, None)
        else:
            ptrs = (C.c_void_p * len(peaks))(*[p.ctypes.data for p in peaks])
            rc = self.lib.spiir_process_batch_peaks(len(requests), arr, ptrs, 1.0, None)
        assert rc == S.SPIIR_OK, rc
        return self.launches()

    def launches(self):
        out = []
        for i in range(self.lib.stub_launches()):
            v = (C.c_int32 * 6)()
            self.lib.stub_launch(i, v)
            reqs = []
            for k in range(v[5]):
                r = (C.c_int32 * 6)()
                bd = self.lib.stub_request(i, k, r)
                reqs.append(SimpleNamespace(n=r[0], nchunk=r[1], dual=r[2], direct=r[3], z_direct=r[4], T=r[5], bank=bd))
            out.append(SimpleNamespace(kind=KINDS[v[0]], X=v[1], mode=v[2], groups=v[3], lanes=v[4], req=reqs))
        return out

    def end_states(self, bank_dev):
        """The chunk end states (uend) and pending corrections (euend) of a bank, as float32 arrays."""
        n = C.c_int64()
        u = self.lib.stub_uend(C.c_void_p(bank_dev), C.byref(n))
        rows = np.ctypeslib.as_array(u, (n.value,))
        return rows, self.lib.stub_euend(C.c_void_p(bank_dev))
