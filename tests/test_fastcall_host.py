"""The binding's native calls (csrc/fastcall.cpp) without a GPU: the module built to take CPU tensors, in front of entry points
that do nothing.  What is checked runs in a process of its own."""
import functools
import os
import re
import subprocess
import sys
import tempfile

from paper_2511_19797_amd import build

CSRC = os.path.join(os.path.dirname(build.__file__), "csrc")


@functools.lru_cache(maxsize=None)
def _module_dir():
    tmp = tempfile.mkdtemp(prefix="tvm_fastcall_")
    text = open(os.path.join(CSRC, "fastcall.cpp")).read()
    for real, here in (("!t.is_cuda()", "!t.is_cpu()"), ("(void*)c10::hip::getCurrentHIPStream().stream()", "nullptr"),
                       ('"../../include/tvmattn.h"', f'"{os.path.join(os.path.dirname(build.HERE), "include", "tvmattn.h")}"')):
        assert real in text
        text = text.replace(real, here)
    src = os.path.join(tmp, "fastcall.cpp")
    with open(src, "w") as f:
        f.write(text)
    stubs = os.path.join(tmp, "stubs.cpp")
    with open(stubs, "w") as f:
        for name in sorted(set(re.findall(r"\b(tvmattn_\w+)\b(?=[(,])", text))):
            f.write(f'extern "C" long {name}() {{ return 0; }}\n')
    r = subprocess.run(build.fastcall_command(src, os.path.join(tmp, "_fastcall.so"), [stubs]), capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    return tmp


def python(code):
    """Runs `code` in a Python of its own that finds the module; returns what it printed."""
    r = subprocess.run([sys.executable, "-X", "faulthandler", "-c", code], capture_output=True, text=True, timeout=110,
                       env={**os.environ, "PYTHONPATH": _module_dir()})
    assert r.returncode == 0, (r.returncode, r.stdout[-500:], r.stderr[-3000:])
    return r.stdout


CALLS = """
import torch, _fastcall
r = lambda *s: torch.zeros(*s)
q, g, x, m, x2, w, b, y = r(1, 2, 8, 8), r(8), r(2, 4, 8), r(2, 8), r(6, 32), r(64, 32), r(64), r(6, 64)
rows = r(1, 2, 8)
calls = {
    "jvp_fwd": [q] * 6 + [0.0, True, 0],
    "jvp_bwd": [q] * 8 + [rows] * 2 + [q] * 2 + [0.0, 0],
    "qknorm_fwd": [q] * 4 + [g] * 2 + [1e-6],
    "bwd_qknorm": [q] * 4 + [g] * 2 + [1e-6] + [q] * 8 + [rows] * 2 + [q] * 2 + [0.0] + [q] * 6 + [g] * 2,
    "adaln_fwd": [x] * 2 + [m] * 4 + [1e-6],
    "adaln_bwd": [x] * 2 + [m] * 4 + [1e-6] + [x] * 4,
    "gate_fwd": [x] * 4 + [m] * 2 + [1e-6],
    "gate_bwd": [x] * 2 + [m] * 2 + [1e-6] + [x] * 2,
    "gelu_fwd": [x] * 2,
    "gelu_bwd": [x] * 4,
    "linear_fwd": [x2] * 2 + [w, b],
    "linear_bwd": [x2] * 2 + [w] + [y] * 2 + [True],
}
calls = {n: [t.clone() if isinstance(t, torch.Tensor) else t for t in a] for n, a in calls.items()}
"""


def test_tensors_that_refuse_access_raise():
    """A data pointer that cannot be had, of any argument of any call, raises what torch raises; the interpreter lives on."""
    out = python(CALLS + """
for name, args in calls.items():
    assert getattr(_fastcall, name)(*args) is not None, name
    for i, t in enumerate(args):
        if isinstance(t, torch.Tensor):
            locked = t.clone()
            torch._C._set_throw_on_mutable_data_ptr(locked)
            print(name, i, flush=True)
            try:
                getattr(_fastcall, name)(*args[:i], locked, *args[i + 1:])
            except RuntimeError as e:
                assert "Cannot access data pointer" in str(e)
            else:
                raise AssertionError((name, i))
""")
    assert len({line.split()[0] for line in out.splitlines()}) == 12
