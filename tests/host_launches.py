"""The library on a HIP runtime that does nothing (hip_stub.c): which kernels a
call launches, with how many threads, and what a failing HIP call leaves
behind. For use in a process of its own (see test_host_launches.py): the stub
stays in it. Buffers are addresses that nothing reads or writes."""

import ctypes
import os
import re
import subprocess
import sys
import types

HERE = os.path.dirname(os.path.abspath(__file__))


class Host:
    def __init__(self, workdir):
        so = os.path.join(workdir, "hip_stub.so")
        if not os.path.exists(so):
            subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-o", so, os.path.join(HERE, "hip_stub.c"), "-ldl"],
                           check=True)
        self.stub = ctypes.CDLL(so, mode=ctypes.RTLD_GLOBAL)
        self.stub.stub_kernel.restype = ctypes.c_char_p
        for f in ("stub_blocks", "stub_threads", "stub_shared"):
            getattr(self.stub, f).restype = ctypes.c_ulonglong
        sys.modules["torch"] = types.ModuleType("torch")  # the binding imports it for its HIP runtime only
        from paper_2505_17284_amd import _lib

        self.L, self.lib = _lib, _lib.lib()
        self.base = 1 << 44

    def plan(self, p, group_size=0, group_size_average=0, rows=0, waves=0, bind=True, probes=None):
        m = self.L.MarshalledProblem(p, probes=probes)
        h = ctypes.c_void_p()
        self.L.check(self.lib.sn_plan_create_shaped(ctypes.byref(m.struct), group_size, group_size_average, rows,
                                                    waves, ctypes.byref(h)), "create")
        if bind:
            self.L.check(self.bind(h), "bind")
            self.L.check(self.lib.sn_plan_init(h, None, None), "init")
        return h

    def info(self, h):
        i = self.L.SnPlanInfo()
        self.L.check(self.lib.sn_plan_get_info(h, ctypes.byref(i)), "info")
        return {f: getattr(i, f) for f, _ in i._fields_}

    def addresses(self, *sizes):
        out = []
        for n in sizes:
            out.append(ctypes.c_void_p(self.base))
            self.base += (n + 4095) // 4096 * 4096
        return out

    def bind(self, h):
        i = self.info(h)
        return self.lib.sn_plan_bind(h, *self.addresses(i["psi_bytes"], i["psi_bytes"], i["scratch_bytes"]))

    def lds(self):
        """Dynamic LDS bytes of the launches that launches() is about to return."""
        return [self.stub.stub_shared(i) for i in range(self.stub.stub_launches())]

    def launches(self):
        """[(kernel, blocks, threads per block)] since the last call of this."""
        out = []
        for i in range(self.stub.stub_launches()):
            name = re.search(r"sn_[a-z_]+?_kernel", self.stub.stub_kernel(i).decode())
            out.append((name.group(0) if name else "?", self.stub.stub_blocks(i), self.stub.stub_threads(i)))
        self.stub.stub_clear()
        return out

    def fail(self, name, k):
        self.stub.stub_fail(name.encode(), k)
