"""The library over a stand-in for the HIP runtime (fake_hip.c): its host code runs without a GPU,
every launch is recorded instead of run, and device memory is addresses that nothing backs.  Only in
a process of its own (see run), before anything else loads the HIP runtime."""
import ctypes
import os
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


def run(module, call, timeout=600):
    """Runs `call` of the tests' module `module` in a fresh process; its output on failure."""
    code = "import sys; sys.path[:0] = [%r, %r]; import %s as m; m.%s" % (HERE, ROOT, module, call)
    res = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=timeout, cwd=ROOT)
    assert res.returncode == 0, res.stdout[-4000:] + res.stderr[-4000:]


class Launch:
    """One recorded launch.  arg(i, type) reads argument i while the call runs (in `watch`)."""

    def __init__(self, name, grid, block, lds, args):
        self.name, self.grid, self.block, self.lds, self._args = name, grid, block, lds, args

    def arg(self, i, ctype):
        value = ctypes.cast(self._args[i], ctypes.POINTER(ctype))[0]
        return type(value).from_buffer_copy(value) if isinstance(value, ctypes.Structure) else value


class FakeHip:
    def __init__(self):
        so = os.path.join(tempfile.mkdtemp(prefix="fake_hip"), "libfake_hip.so")
        subprocess.check_call(["gcc", "-O1", "-shared", "-fPIC", "-o", so, os.path.join(HERE, "fake_hip.c")])
        self.c = ctypes.CDLL(so, mode=ctypes.RTLD_GLOBAL)
        u32 = ctypes.c_uint32
        lcb = ctypes.CFUNCTYPE(None, ctypes.c_char_p, u32, u32, u32, u32, u32, u32, ctypes.c_size_t,
                               ctypes.POINTER(ctypes.c_void_p))
        mcb = ctypes.CFUNCTYPE(None, ctypes.c_int, ctypes.c_uint64, ctypes.c_size_t)
        self._cb = (lcb(self._launch), mcb(self._memory))
        self.c.fake_set(*self._cb)
        self.c.fake_fail_malloc.argtypes = self.c.fake_fail_next.argtypes = [ctypes.c_long]
        self.launches = []
        self.live = {}       # address -> bytes of the device memory held
        self.watch = None    # called with every launch
        self._raised = None
        import paper_2512_23569_amd as ht
        self.ht = ht
        self.L = ht.lib()

    def _launch(self, name, gx, gy, gz, bx, by, bz, lds, args):
        n = Launch(name.decode(), (gx, gy, gz), (bx, by, bz), lds, args)
        self.launches.append(n)
        if self.watch and not self._raised:
            try:
                self.watch(n)
            except Exception as e:   # does not pass through the library: raised again by call
                self._raised = e

    def _memory(self, alloc, addr, size):
        if alloc:
            self.live[addr] = size
        else:
            self.live.pop(addr)

    def holds(self, addr):
        """Whether addr lies in device memory that is held."""
        return any(a <= addr < a + n for a, n in self.live.items())

    def context(self, bases=(1, 3)):
        ctx = self.ht.htsvd_create(0)
        for c in bases:
            self.ht.htsvd_set_basis(ctx, 8, c, *self.ht.load_basis_slices(c))
        return ctx

    def params(self, c, **kw):
        return self.ht.htsvd_default_params(c).replace(**kw)

    def call(self, name, *args, expect=0):
        """A call of the C ABI; its launches, or None where it is refused (expect None: either)."""
        self.launches = []
        status = getattr(self.L, name)(*args)
        if self._raised:
            e, self._raised = self._raised, None
            raise e
        if expect is not None:
            assert status == expect, (name, status, self.ht.htsvd_last_error())
        return self.launches if status == 0 else None
