"""The launches that the library makes for a configuration, without a GPU: it is loaded over a
stand-in for the HIP runtime (hip_stub.cpp) that writes launches down instead of making them.
Only for processes that do not use the real runtime: the tests call it through `recorded`, which
runs a piece of code in a process of its own."""
import ctypes
import json
import os
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


def recorded(code):
    """Run `code` (it has B, synth, Context, stub and puts its answer into `out`) over the stand-in."""
    with tempfile.TemporaryDirectory() as tmp:
        lib = os.path.join(tmp, "hip_stub.so")
        subprocess.check_call(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", os.path.join(HERE, "hip_stub.cpp"), "-o", lib])
        head = ("import json\nfrom tests.launches import Context, load\nstub = load(%r)\n"
                "from paper_1907_09356_amd import binding as B, synth\nout = None\n" % lib)
        run = subprocess.run([sys.executable, "-c", head + code + "\nprint('ANSWER' + json.dumps(out))"], cwd=ROOT,
                             capture_output=True, text=True, timeout=120)
    assert run.returncode == 0, run.stderr[-2000:]
    return json.loads(run.stdout.split("ANSWER")[1])


def load(path):
    stub = ctypes.CDLL(path, mode=ctypes.RTLD_GLOBAL)   # before the library, whose calls then find it first
    stub.stub_launches.restype = ctypes.c_char_p
    from paper_1907_09356_amd import binding
    binding.lib()
    global _stub
    _stub = stub
    return stub


class Context:
    """A context on host memory.  `ld` 0: the shortest; x_off: bytes by which X is off a 256-byte boundary; ws: bytes of
    workspace handed over (default: all that are asked for)."""

    def __init__(self, n, d, compressor, topo=None, x_off=0, align=4, ws=None, **kw):
        import numpy as np
        from paper_1907_09356_amd import binding as B
        from paper_1907_09356_amd import synth
        self.B, self.np = B, np
        ld = (d + align - 1) // align * align
        topo = topo if topo is not None else synth.ring_csr(n)
        self.cfg, self.keep = B.make_config(n, d, *topo, 0.1, compressor, ld=ld, **kw)
        self.asked = B.workspace_bytes(self.cfg)
        nbytes = self.asked if ws is None else ws
        self.x, xp = self._buffer(4 * n * ld + x_off)
        self.ws, wp = self._buffer(nbytes)
        self.g, self.gp = self._buffer(4 * n * ld)
        self.m, self.mp = self._buffer(4 * n * ld)
        self.ctx = ctypes.c_void_p()
        self.rc = B.lib().choco_init(ctypes.byref(self.cfg), xp + x_off, wp, nbytes, ctypes.byref(self.ctx))

    def _buffer(self, nbytes):
        a = self.np.zeros(nbytes + 256, dtype=self.np.uint8)
        return a, (a.ctypes.data + 255) // 256 * 256

    def _launches(self, rc):
        assert rc == self.B.OK, rc
        return [line.split() for line in _stub.stub_launches().decode().splitlines()]

    def step(self):
        """[name, grid, block, LDS bytes] of every launch of one fused iteration."""
        _stub.stub_clear()
        return self._launches(self.B.lib().choco_step(self.ctx, self.gp, 0.1))

    def set_step(self, t):
        assert self.B.lib().choco_set_step(self.ctx, t) == self.B.OK

    def step_momentum(self):
        _stub.stub_clear()
        return self._launches(self.B.lib().choco_step_momentum(self.ctx, self.gp, self.mp, 0.1, 0.9, 1e-4))

    def metrics(self):
        _stub.stub_clear()
        a = [ctypes.c_double(-1.0) for _ in range(3)]
        launches = self._launches(self.B.lib().choco_metrics(self.ctx, *map(ctypes.byref, a)))
        self.figures = [v.value for v in a]
        return launches

    def metrics_noalloc(self):
        _stub.stub_clear()
        return self._launches(self.B.lib().choco_metrics_noalloc(self.ctx, self.mp))

    def close(self):
        self.B.lib().choco_destroy(self.ctx)
