"""The compiled per-call path of the binding, on the CPU.

A child process per test gives it tensors that torch takes for device tensors
(DLPack capsules over host memory, which nothing here reads) and stand-ins
for the library's entry points, so no GPU is needed or touched.
"""
import os
import subprocess
import sys
import textwrap

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PRELUDE = '''
import ctypes, sys, threading, time
import torch
import paper_2605_11478_amd as fq

class Device(ctypes.Structure):
    _fields_ = [("type", ctypes.c_int32), ("index", ctypes.c_int32)]
class Type(ctypes.Structure):
    _fields_ = [("code", ctypes.c_uint8), ("bits", ctypes.c_uint8), ("lanes", ctypes.c_uint16)]
class Tensor(ctypes.Structure):
    _fields_ = [("data", ctypes.c_void_p), ("device", Device), ("ndim", ctypes.c_int32),
                ("dtype", Type), ("shape", ctypes.POINTER(ctypes.c_int64)),
                ("strides", ctypes.POINTER(ctypes.c_int64)), ("offset", ctypes.c_uint64)]
class Managed(ctypes.Structure):
    _fields_ = [("tensor", Tensor), ("ctx", ctypes.c_void_p), ("deleter", ctypes.c_void_p)]
capsule = ctypes.pythonapi.PyCapsule_New
capsule.restype, capsule.argtypes = ctypes.py_object, [ctypes.c_void_p, ctypes.c_char_p, ctypes.c_void_p]
torch.cuda._lazy_init = lambda: None
held = []

def device_tensor(dtype, *shape):
    """A tensor of device type over host memory (kDLROCM = 10)."""
    code = {torch.float32: (2, 32), torch.uint8: (1, 8), torch.int16: (0, 16), torch.bfloat16: (4, 16)}[dtype]
    host = torch.zeros(shape, dtype=dtype)
    sh = (ctypes.c_int64 * len(shape))(*shape)
    st = (ctypes.c_int64 * len(shape))(*host.stride())
    m = Managed(Tensor(host.data_ptr(), Device(10, 0), len(shape), Type(*code, 1), sh, st, 0), None, None)
    held.append((host, sh, st, m))
    t = torch._C._from_dlpack(capsule(ctypes.addressof(m), b"dltensor", None))
    assert t.is_cuda
    return t

fq.payload_bytes(64, 8, 16)
R, C = device_tensor(torch.float32, 64, 64), device_tensor(torch.float32, 16, 8)
x = device_tensor(torch.float32, 5, 64)
payload, norms = device_tensor(torch.uint8, 5, 4), device_tensor(torch.int16, 5)
out = device_tensor(torch.float32, 5, 64)
q, att = device_tensor(torch.float32, 1, 2, 64), device_tensor(torch.float32, 1, 2, 64)
kp, kn = device_tensor(torch.uint8, 1, 5, 4), device_tensor(torch.int16, 1, 5)
ws = device_tensor(torch.uint8, fq.attn_workspace_bytes(1, 2, 5, 64, 8, 16))
fq._raw_stream = fq._stream = lambda: 0
CALLS = {"fibq_encode": lambda: fq.encode(x, 8, 16, R, C, payload, norms),
         "fibq_decode": lambda: fq.decode(payload, norms, 64, 8, 16, R, C, out=out),
         "fibq_attn_decode": lambda: fq.attn_decode(q, kp, kn, kp, kn, 5, 8, 16, R, C, workspace=ws, out=att)}
real = fq.lib()

class Library:
    """The real library with some entry points replaced."""
    def __init__(self, **other):
        self._other = other
    def __getattr__(self, name):
        return self._other[name] if name in self._other else getattr(real, name)
'''


def _child(code, *args):
    r = subprocess.run([sys.executable, "-c", PRELUDE + textwrap.dedent(code), *args], cwd=ROOT,
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr


def test_library_status_is_raised_and_not_retried():
    """A status other than FIBQ_OK raises FibqError with that status, and the
    library is entered once: a HIP error is reported once, so a second entry
    would find it gone and return as if nothing had happened."""
    _child('''
    for name, call in CALLS.items():
        entered = []
        restype, argtypes = getattr(real, name).restype, getattr(real, name).argtypes
        def entry(*a):
            entered.append(len(a))
            return fq.FIBQ_EHIP if len(entered) == 1 else fq.FIBQ_OK
        fn = ctypes.CFUNCTYPE(restype, *argtypes)(entry)
        L = Library(**{name: fn})
        fq._lib = L
        fq._bind(L)
        try:
            call()
        except fq.FibqError as e:
            assert e.status == fq.FIBQ_EHIP and name in str(e), e
        else:
            raise AssertionError(f"{name}: the status was lost")
        assert len(entered) == 1, (name, entered)
        call()
        assert len(entered) == 2, (name, entered)
    ''')


def test_other_threads_run_during_a_library_call(tmp_path):
    """The library is entered without the interpreter lock: each stand-in (C)
    waits until another Python thread has set a flag, 10 s at most, and
    returns an error if none did."""
    src, so = tmp_path / "wait.c", tmp_path / "wait.so"
    src.write_text("""
#include <unistd.h>
volatile int entered, flag;
int wait_for_flag(void) {
  entered = 1;
  for (int i = 0; i < 10000 && !flag; ++i) usleep(1000);
  const int seen = flag;
  entered = flag = 0;
  return seen ? 0 : -3;
}
""")
    subprocess.run(["gcc", "-shared", "-fPIC", "-O1", str(src), "-o", str(so)], check=True)
    _child('''
    W = ctypes.CDLL(sys.argv[1])
    entered, flag = ctypes.c_int.in_dll(W, "entered"), ctypes.c_int.in_dll(W, "flag")
    done = False
    def other():
        while not done:
            if entered.value and not flag.value:
                flag.value = 1
            time.sleep(0.001)
    t = threading.Thread(target=other)
    t.start()
    try:
        for name, call in CALLS.items():
            fq._lib = Library(**{name: W.wait_for_flag})
            fq._bind(fq._lib)
            call()
    finally:
        done = True
        t.join()
    ''', str(so))


def test_host_functions_need_neither_torch_nor_the_compiled_module():
    """Building and loading codes works where torch cannot be imported and the
    compiled module is not there."""
    code = """
import sys
sys.modules["torch"] = None
import paper_2605_11478_amd as fq
fq.BINDING_PATH += ".absent"
assert fq.build_rotation(64, 3).shape == (64, 64) and fq.payload_bytes(64, 8, 16) == 4
assert fq.build_codebook(64, 4, 16, 1, M=2000, restarts=1, iters=1)[0].shape == (16, 4)
try:
    fq.load_codebook("/nowhere/at/all")
except fq.FibqError as e:
    assert e.status == fq.FIBQ_EIO
"""
    r = subprocess.run([sys.executable, "-c", code], cwd=ROOT, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr


def test_missing_compiled_module_raises_on_every_device_call():
    """Never a silent second-best path: without the module every encode,
    decode and attention call on device tensors raises ImportError."""
    _child('''
    path, fq.BINDING_PATH = fq.BINDING_PATH, fq.BINDING_PATH + ".absent"
    for _ in range(2):
        for name, call in CALLS.items():
            try:
                call()
            except ImportError as e:
                assert "missing" in str(e)
            else:
                raise AssertionError(f"{name} went on without the compiled module")
    fq.BINDING_PATH = path
    entered = []
    entry = lambda *a: entered.append(1) or fq.FIBQ_OK
    fq._lib = Library(**{n: ctypes.CFUNCTYPE(getattr(real, n).restype, *getattr(real, n).argtypes)(entry)
                         for n in CALLS})
    for name, call in CALLS.items():
        call()
    assert len(entered) == 3 and fq._fast is not None
    ''')
