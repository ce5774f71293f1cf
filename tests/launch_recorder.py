"""Which kernels a call launches, asked without a GPU: a child process loads libhiermoe.so behind a stand-in for the HIP
runtime that notes every launch (launch_recorder.c)."""
import json
import os
import re
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# In the child: no torch (its HIP runtime would take the calls instead of the stand-in), so no _hmcall either; B is the
# binding, L the library, at(i) a device address aligned to 128 bytes, launched() what has been launched since it was last
# asked, as {name, grid, block, lds, granted}.
_CHILD = r"""
import ctypes, json, sys, types, warnings
recorder = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
torch = types.ModuleType("torch")
torch.Tensor = torch.dtype = object
sys.modules["torch"] = torch
sys.modules["paper_2508_09591_amd._hmcall"] = None
sys.path.insert(0, sys.argv[2])
from paper_2508_09591_amd import binding as B
warnings.simplefilter("ignore")
L = B.lib()
class Launch(ctypes.Structure):
    _fields_ = [("name", ctypes.c_char_p), ("grid", ctypes.c_uint32 * 3), ("block", ctypes.c_uint32 * 3), ("lds", ctypes.c_uint64),
                ("granted", ctypes.c_uint64)]
recorder.recorder_launch.restype = ctypes.POINTER(Launch)
def at(i):
    return ctypes.c_void_p((1 << 40) + (i << 32))
def launched():
    out = []
    for i in range(recorder.recorder_count()):
        r = recorder.recorder_launch(i).contents
        out.append({"name": r.name.decode(), "grid": list(r.grid), "block": list(r.block), "lds": r.lds, "granted": r.granted})
    recorder.recorder_reset()
    return out
result = None
exec(sys.stdin.read())
print("RESULT " + json.dumps(result))
"""


def build(folder):
    """The stand-in, compiled into `folder`."""
    from paper_2508_09591_amd import build as b
    if not os.path.exists(b.LIB):
        b.build_library()
    rocm = os.path.dirname(os.path.dirname(os.path.realpath(b.hipcc_path())))
    include = os.path.join(rocm if os.path.exists(os.path.join(rocm, "include", "hip")) else "/opt/rocm", "include")
    out = os.path.join(str(folder), "liblaunches.so")
    subprocess.check_call(["gcc", "-O1", "-std=c11", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__=1", "-isystem", include, "-o", out,
                           os.path.join(ROOT, "tests", "launch_recorder.c")])
    return out


def run(recorder, body):
    """What `body`, run in the child, leaves in `result`; kernels by their names in the source (template arguments, no parameters)."""
    p = subprocess.run([sys.executable, "-c", _CHILD, recorder, ROOT], input=body, capture_output=True, text=True, timeout=120)
    assert p.returncode == 0, p.stderr
    text = p.stdout[p.stdout.rindex("RESULT ") + 7:]
    mangled = sorted(set(re.findall(r'"(_ZN2hm\w+)"', text)))
    if mangled:
        names = subprocess.run(["c++filt"], input="\n".join(mangled), capture_output=True, text=True, check=True).stdout.splitlines()
        for m, n in zip(mangled, names):
            n = n.replace("hm::", "").replace("void ", "", 1)
            text = text.replace('"%s"' % m, json.dumps(n[:n.index("(")]))
    return json.loads(text)
